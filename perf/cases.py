"""The work this framework is measured on: exact attention, forward and backward, through its public entry points.

`flash_attention` (the autograd front end) serves the cases that stand for a layer inside a training
program; `attn_fwd` / `attn_bwd` / `attn_blocksparse_*` of the binding, with buffers that the program
keeps, serve the others.  Sizes are those of the repository's own configurations and benchmark
sweep, or generic ragged ones.

A case is a dict of

  entry   "autograd", "binding" or "sparse" (the block-sparse entry points of the binding)
  train   True: forward and backward; False: forward only
  B, H, N, d, dtype ("fp16" | "bf16"), causal, p (dropout)
  layout  "head" ([B,H,N,d] packed) or "token" (a [B,H,N,d] view of [B,N,H,d] memory)
  padded  True: a key-padding mask with lengths between N/2 and N (the autograd entry: no LSE of padded rows among the outputs)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2205_14135_amd import binding
from paper_2205_14135_amd.autograd import flash_attention
from paper_2205_14135_amd.inputs import butterfly_block_mask

BLOCK = 128                 # side of a block of the block-sparse mask
MAX_FLOPS = 14 * 64 * 4096 ** 2 * 128   # the largest listed case: forward and backward, B H = 64, N = 4096, d = 128
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}


def _case(name, entry, train, B, H, N, d, dtype, causal=False, p=0.0, layout="head", padded=False):
    c = dict(entry=entry, train=train, B=B, H=H, N=N, d=d, dtype=dtype, causal=causal, p=p, layout=layout, padded=padded)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one head of 128 tokens, where the launch and the host path are all there is
        _case("single_head_fwd", "binding", False, 1, 1, 128, 64, "fp16"),
        # a small batch of a length that no tile divides, heads interleaved in memory as a projection leaves them
        _case("ragged_N197_train", "autograd", True, 8, 12, 197, 64, "fp16", layout="token"),
        # short end of the sequence-length sweep (16384 tokens, 16 heads): many heads of one tile each
        _case("sweep_N128_d64_train", "autograd", True, 128, 16, 128, 64, "bf16"),
        # the layer of a BERT-large training step: N = 512, dropout
        _case("bert_large_train", "autograd", True, 16, 16, 512, 64, "fp16", p=0.1),
        # the layer of a GPT-2-medium training step: causal, dropout, and the same width as 8 heads of 128
        _case("gpt2_medium_train", "autograd", True, 8, 16, 1024, 64, "bf16", causal=True, p=0.1),
        _case("gpt2_medium_d128_train", "autograd", True, 8, 8, 1024, 128, "bf16", causal=True, p=0.1),
        # narrow heads, padded batch: an encoder over sentences of different lengths
        _case("padded_N700_d32_train", "autograd", True, 16, 8, 700, 32, "bf16", padded=True),
        # middle of the sweep at d = 64
        _case("sweep_N2048_d64_train", "binding", True, 8, 16, 2048, 64, "bf16"),
        # the benchmark's default workload, and the same under the causal mask
        _case("sweep_N4096_d128_train", "binding", True, 4, 16, 4096, 128, "bf16"),
        _case("sweep_N4096_d128_causal_train", "binding", True, 4, 16, 4096, 128, "bf16", causal=True),
        # long end of the sweep, forward alone: reading in a long prompt
        _case("sweep_N16384_d64_causal_fwd", "binding", False, 1, 16, 16384, 64, "bf16", causal=True),
        # the long-range block-sparse workload (butterfly mask of 128 x 128 blocks)
        _case("blocksparse_N16384_train", "sparse", True, 1, 8, 16384, 64, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the kinds of the list, sizes over the logarithm of their range, odd ones among them."""
    while True:
        kind = rng.choice(["autograd", "autograd", "binding", "binding", "forward", "sparse"])
        dtype = rng.choice(["fp16", "bf16", "bf16"])
        causal = rng.random() < 0.4
        if kind == "sparse":
            N = BLOCK * _log_int(rng, 8, 256)
            c = _case(None, "sparse", True, 1, _log_int(rng, 2, 8), N, rng.choice([64, 64, 128]), dtype, causal=causal)
        elif kind == "forward":
            N = _log_int(rng, 100, 16384)
            tokens = _log_int(rng, N, 32768)
            c = _case(None, "binding", False, max(1, tokens // N), _log_int(rng, 1, 16), N, rng.choice([64, 64, 128, 128, 32]),
                      dtype, causal=causal, layout=rng.choice(["head", "token"]))
        else:
            N = _log_int(rng, 100, 8192)
            tokens = _log_int(rng, max(N, 1024), 16384)
            c = _case(None, kind, True, max(1, tokens // N), rng.choice([8, 12, 16]), N, rng.choice([64, 64, 128, 128, 32]),
                      dtype, causal=causal, p=rng.choice([0.0, 0.0, 0.1]), layout=rng.choice(["head", "token"]),
                      padded=kind == "autograd" and not causal and rng.random() < 0.4)
        if work(c)["flops"] <= MAX_FLOPS:
            return c


def _lengths(case):
    """True lengths of a padded batch: from N/2 to N, spread evenly, the longest first (no tensor: part of the case)."""
    B, N = case["B"], case["N"]
    return [N - (b * (N // 2)) // max(1, B - 1) for b in range(B)] if case["padded"] else [N] * B


def _block_mask(case):
    return butterfly_block_mask(case["N"] // BLOCK)


def _pairs(case):
    """(query, key) pairs of one head, summed over the batch."""
    N = case["N"]
    if case["entry"] == "sparse":
        m = _block_mask(case).astype(bool)
        if case["causal"]:
            full, diag = int(np.tril(m, -1).sum()), int(np.trace(m))
            return case["B"] * (full * BLOCK * BLOCK + diag * (BLOCK * (BLOCK + 1) // 2))
        return case["B"] * int(m.sum()) * BLOCK * BLOCK
    return sum(n * (n + 1) // 2 if case["causal"] else n * n for n in _lengths(case))


def _seed(seed):
    return 0x5EED0000 + seed


def _inputs(case, seed):
    """Q, K, V and dO: unit normal values rounded to the tensors' type, as after a normalised projection."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, H, N, d = (case[k] for k in "BHNd")
    ts = []
    for _ in range(4 if case["train"] else 3):
        shape = (B, H, N, d) if case["layout"] == "head" else (B, N, H, d)
        x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(DTYPES[case["dtype"]])
        ts.append(x if case["layout"] == "head" else x.transpose(1, 2))
    return ts


def prepare(case, seed):
    ts = _inputs(case, seed)
    q = ts[0]
    kw = dict(softmax_scale=1.0 / math.sqrt(case["d"]), causal=case["causal"])
    if case["entry"] != "sparse":
        kw.update(dropout_p=case["p"], seed=_seed(seed), offset=0)
        if case["padded"]:
            kw["key_lengths"] = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")
    st = dict(entry=case["entry"], train=case["train"], kw=kw, q=q, k=ts[1], v=ts[2], do=ts[3] if case["train"] else None)
    if case["entry"] == "autograd":
        for x in ts[:3]:
            x.requires_grad_(True)
        return st
    # the buffers that a program calling the binding keeps from step to step
    st["out"] = torch.empty_strided(q.shape, q.stride(), dtype=q.dtype, device=q.device)
    st["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=q.device)
    if case["entry"] == "sparse":
        st["mask"] = torch.from_numpy(_block_mask(case)).cuda()
    if case["train"]:
        p = binding.make_params(q, **kw)
        size = binding.attn_blocksparse_bwd_workspace_bytes if case["entry"] == "sparse" else binding.attn_bwd_workspace_bytes
        st["workspace"] = torch.empty(size(p), dtype=torch.uint8, device=q.device)
        st["grads"] = tuple(torch.empty_strided(q.shape, q.stride(), dtype=q.dtype, device=q.device) for _ in range(3))
    return st


def run(st):
    q, k, v, do, kw = st["q"], st["k"], st["v"], st["do"], st["kw"]
    if st["entry"] == "autograd":
        out = flash_attention(q, k, v, **kw)
        return (out, *torch.autograd.grad(out, (q, k, v), do))
    if st["entry"] == "sparse":
        out, lse = binding.attn_blocksparse_fwd(q, k, v, st["mask"], out=st["out"], lse=st["lse"], **kw)
        if not st["train"]:
            return out, lse
        return (out, lse, *binding.attn_blocksparse_bwd(q, k, v, out, do, lse, st["mask"], grads=st["grads"],
                                                        workspace=st["workspace"], **kw))
    out, lse = binding.attn_fwd(q, k, v, out=st["out"], lse=st["lse"], **kw)
    if not st["train"]:
        return out, lse
    return (out, lse, *binding.attn_bwd(q, k, v, out, do, lse, grads=st["grads"], workspace=st["workspace"], **kw))


def work(case):
    """Two tile products forward and five backward; Q, K, V (and dO) in, O (and three gradients) out."""
    B, H, N, d = (case[k] for k in "BHNd")
    tensor = 2 * B * H * N * d
    flops = (14 if case["train"] else 4) * H * _pairs(case) * d
    return {"bytes": (8 if case["train"] else 4) * tensor + (4 * B * H * N if case["entry"] != "autograd" else 0), "flops": flops}


def tolerance(case):
    """Four to five times the measured error against 64 bits (bf16 2.5e-3, fp16 3.1e-4): the outputs' own rounding (2^-9 in bf16, 2^-12 in fp16) and that of
    the 16-bit probabilities and dS that enter the second products."""
    return {"rel": 1.2e-2 if case["dtype"] == "bf16" else 2e-3}


# ---------------------------------------------------------------------------------------------
# The same results in 64 bits.

def _philox_keep(case, seed, b, heads, rows, n_keys):
    """Keep mask [heads, rows, n_keys] of the dropout contract: Philox-4x32-10, key = seed, counter =
    (key / 16, query, b H + h, 0), an 8-bit field per key, kept iff field >= floor(256 p)."""
    dev, m32 = rows.device, 0xFFFFFFFF
    grp = torch.arange((n_keys + 15) // 16, device=dev, dtype=torch.int64)
    shape = (len(heads), len(rows), len(grp))
    c = [grp.view(1, 1, -1).expand(shape), rows.to(torch.int64).view(1, -1, 1).expand(shape),
         (b * case["H"] + heads.to(torch.int64)).view(-1, 1, 1).expand(shape), torch.zeros(shape, dtype=torch.int64, device=dev)]
    key = _seed(seed)
    k0, k1 = key & m32, (key >> 32) & m32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57      # the low 64 bits of the product are what is used
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    words = torch.stack(c, dim=-1)                          # [heads, rows, groups, 4]
    fields = torch.stack([(words >> (8 * e)) & 0xFF for e in range(4)], dim=-1)
    return (fields.reshape(shape[0], shape[1], -1)[:, :, :n_keys] >= int(case["p"] * 256)).to(torch.float64)


def exact(case, seed):
    ts = [t.to(torch.float64) for t in _inputs(case, seed)]
    B, H, N, d = (case[k] for k in "BHNd")
    q, k, v = ts[:3]
    train, causal, sparse = case["train"], case["causal"], case["entry"] == "sparse"
    tau = 1.0 / math.sqrt(d)
    thr = int(case["p"] * 256)
    keep_scale = 256.0 / (256.0 - thr)
    out, lse = torch.zeros_like(q), torch.full((B, H, N), -math.inf, dtype=torch.float64, device=q.device)
    dq, dk, dv = (torch.zeros_like(q) for _ in range(3)) if train else (None,) * 3
    mask = _block_mask(case) if sparse else None
    lengths = _lengths(case)
    step = BLOCK if sparse else min(N, 2048)
    n_heads = max(1, min(H, (1 << 27) // (step * N)))
    idx = torch.arange(N, device=q.device)
    for b in range(B):
        n = lengths[b]
        for h0 in range(0, H, n_heads):
            hs = slice(h0, min(H, h0 + n_heads))
            heads = idx.new_tensor(range(hs.start, hs.stop))
            for r0 in range(0, n, step):
                r1 = min(n, r0 + step)
                rows = idx[r0:r1]
                if sparse:
                    kept = [j for j in np.flatnonzero(mask[r0 // BLOCK]) if not causal or j <= r0 // BLOCK]
                    cols = torch.cat([idx[BLOCK * j:BLOCK * (j + 1)] for j in kept])
                else:
                    cols = idx[:min(n, r1) if causal else n]
                qs, ks, vs = q[b, hs, r0:r1].contiguous(), k[b, hs][:, cols].contiguous(), v[b, hs][:, cols].contiguous()
                s = torch.matmul(qs, ks.transpose(1, 2).contiguous()) * tau
                if causal:
                    s.masked_fill_(cols.view(1, -1) > rows.view(-1, 1), -math.inf)
                l_row = torch.logsumexp(s, dim=-1)
                prob = torch.exp(s - l_row.unsqueeze(-1))
                z = _philox_keep(case, seed, b, heads, rows, len(cols)) * keep_scale if thr > 0 else None
                dropped = prob if z is None else prob * z
                o = torch.matmul(dropped, vs)
                out[b, hs, r0:r1] = o
                lse[b, hs, r0:r1] = l_row
                if not train:
                    continue
                g = ts[3][b, hs, r0:r1].contiguous()
                dv[b, hs] = dv[b, hs].index_add(1, cols, torch.matmul(dropped.transpose(1, 2).contiguous(), g))
                dp = torch.matmul(g, vs.transpose(1, 2).contiguous())
                if z is not None:
                    dp = dp * z
                ds = prob * (dp - (g * o).sum(-1, keepdim=True))
                dq[b, hs, r0:r1] = torch.matmul(ds, ks) * tau
                dk[b, hs] = dk[b, hs].index_add(1, cols, torch.matmul(ds.transpose(1, 2).contiguous(), qs) * tau)
    if case["entry"] == "autograd":
        return out, dq, dk, dv
    return (out, lse, dq, dk, dv) if train else (out, lse)
