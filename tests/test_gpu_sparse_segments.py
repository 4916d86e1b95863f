"""The division of heavy mask columns of the block-sparse backward: planned by workgroups of the dQ launch, walked in segments, converted by
the last segment.  Against the oracle, and with the workspace as a caller may hand it in: dirty, used before, and replayed from a graph."""
import math

import numpy as np
import pytest
import torch

from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


def _masks(kind, H, T):
    """[H, T, T], another mask for each head: full columns that stand out among thin ones, all blocks, or a random half."""
    rng = np.random.default_rng(1000 + T)
    m = np.zeros((H, T, T), dtype=np.uint8)
    for h in range(H):
        if kind == "columns":
            m[h, np.arange(T), np.arange(T)] = 1
            for col in {0, (5 * h + 3) % T, T - 1}:
                m[h, :, col] = 1
        else:
            m[h] = 1 if kind == "dense" else rng.random((T, T)) < 0.5
    m[0, :, 1] = 0   # a column that nobody attends to
    return m


def _backward(dev, bm, workspace=None, **kw):
    o, lse = binding.attn_blocksparse_fwd(dev["Q"], dev["K"], dev["V"], bm, **kw)
    return lambda: binding.attn_blocksparse_bwd(dev["Q"], dev["K"], dev["V"], o, dev["dO"], lse, bm, workspace=workspace, **kw)


# T at the edges of the planning groups (16 columns), of the rules for a heavy column (14, 24 blocks) and of a wavefront's scan
@pytest.mark.parametrize("T", [14, 15, 16, 17, 25])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("kind", ["columns", "dense"])
@pytest.mark.parametrize("causal,p", [(False, 0.0), (True, 0.2)])
def test_segments_against_oracle(T, d, kind, causal, p):
    H, N, dtype, tau = 2, 128 * T, ("fp16", "bf16")[T % 2], 1 / math.sqrt(d)
    t, dev = hp.make_case(1, H, N, d, dtype, inputs.BASE_SEED + 6500 + T + d)
    hp.assert_backward_ok(hp.check_backward(t, dev, dtype, tau, causal=causal, p=p, seed=inputs.BASE_DROPOUT_SEED + 3, offset=1,
                                            block_mask=_masks(kind, H, T), heads=[(0, T % H)]))


def _reference(dev, lse, o, masks, tau, lengths):
    """dQ, dK, dV in float32 on the device, by columns of the mask."""
    q, k, v, do = (dev[n].float() for n in ("Q", "K", "V", "dO"))
    D = (o.float() * do).sum(-1, keepdim=True)
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    B, H, N, _ = q.shape
    for b in range(B):
        n = N if lengths is None else int(lengths[b])
        for h in range(H):
            keep = torch.from_numpy(masks[h]).cuda().bool().repeat_interleave(128, 0)   # [N, T]
            keep[n:] = False
            for c in range((n + 127) // 128):
                rows, cols = keep[:, c], slice(128 * c, min(n, 128 * c + 128))
                p = torch.exp(tau * q[b, h] @ k[b, h, cols].T - lse[b, h, :, None]).masked_fill(~rows[:, None], 0.0)
                dv[b, h, cols] = p.T @ do[b, h]
                ds = tau * p * (do[b, h] @ v[b, h, cols].T - D[b, h])
                dk[b, h, cols] = ds.T @ q[b, h]
                dq[b, h] += ds @ k[b, h, cols]
    return dq, dk, dv


# one, two and more scans of 64 planning groups, segments of both lengths, more columns than the one-wavefront kernel takes at d = 128
@pytest.mark.parametrize("B,H,T", [(1, 1, 40), (2, 3, 33), (1, 2, 65), (3, 16, 17), (2, 33, 33), (1, 1, 200)])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("kind", ["columns", "dense", "random"])
def test_segments_on_dirty_workspaces(B, H, T, d, kind):
    N, tau = 128 * T, 1 / math.sqrt(d)
    _, dev = hp.make_case(B, H, N, d, "bf16", inputs.BASE_SEED + 6600 + T + d)
    masks = _masks(kind, H, T)
    bm = torch.from_numpy(masks).cuda()
    lengths = [N - 200 * b for b in range(B)] if B > 1 else None
    kw = dict(softmax_scale=tau, key_lengths=None if lengths is None else torch.tensor(lengths, dtype=torch.int32, device="cuda"))
    o, lse = binding.attn_blocksparse_fwd(dev["Q"], dev["K"], dev["V"], bm, **kw)
    params = binding.make_params(dev["Q"], **kw)
    ws = torch.full((binding.attn_blocksparse_bwd_workspace_bytes(params) + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    run = _backward(dev, bm, workspace=ws, **kw)
    first, again = run(), run()
    for x, y, want in zip(first, again, _reference(dev, lse, o, masks, tau, lengths)):
        norm = float(want.norm())
        for got in (x, y):
            assert bool(torch.isfinite(got).all())
            assert float((got.float() - want).norm()) <= hp.GRAD_REL_L2 * norm
        # the same float32 sums, those of heavy columns in another order, rounded once
        assert float((x.float() - y.float()).norm()) <= 2.0 ** -8 * norm


# heavy columns of up to 24 blocks: at most two addends to a sum, which is the same whichever comes first (T = 17: the last column's planning group
# has no idle accumulators)
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("T,causal", [(15, False), (17, False), (20, False), (24, False), (24, True)])
def test_gradients_of_short_columns_repeat(T, causal, d):
    _, dev = hp.make_case(1, 6, 128 * T, d, "fp16", inputs.BASE_SEED + 6800 + T + d)
    run = _backward(dev, torch.from_numpy(_masks("columns", 6, T)).cuda(), softmax_scale=1 / math.sqrt(d), causal=causal)
    first = [g.clone() for g in run()]
    for _ in range(20):
        assert all(torch.equal(x, y) for x, y in zip(first, run()))


# more planning groups than the lanes that look for a segment, and more than they look through in one turn: a few heads that keep heavy columns among
# many that keep nothing
@pytest.mark.parametrize("H,T", [(100, 17), (4200, 15)])
def test_segments_far_apart(H, T):
    d, N, at = 32, 128 * T, [0, 31, 32, 33, H // 2 + 1, H - 3, H - 1]
    _, few = hp.make_case(1, len(at), N, d, "bf16", inputs.BASE_SEED + 6900 + T)
    masks = torch.from_numpy(_masks("columns", len(at), T)).cuda()
    kw = dict(softmax_scale=1 / math.sqrt(d))
    want = _backward(few, masks, **kw)()
    many = {n: torch.zeros(1, H, N, d, dtype=t.dtype, device="cuda") for n, t in few.items()}
    for n, t in many.items():
        t[:, at] = few[n]
    all_masks = torch.zeros(H, T, T, dtype=torch.uint8, device="cuda")
    all_masks[at] = masks
    for x, y in zip(_backward(many, all_masks, **kw)(), want):
        # sums of float32 parts, in other orders, rounded once
        assert float((x[:, at].float() - y.float()).norm()) <= 2.0 ** -8 * float(y.float().norm())
        x[:, at] = 0
        assert not bool(x.any())


@pytest.mark.parametrize("d", [64, 128])
def test_segments_replayed(d):
    H, T = 2, 17
    _, dev = hp.make_case(1, H, 128 * T, d, "fp16", inputs.BASE_SEED + 6700 + d)
    bm = torch.from_numpy(_masks("columns", H, T)).cuda()
    run = _backward(dev, bm, softmax_scale=1 / math.sqrt(d))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        run()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        got = run()
    for replay in range(4):
        dev["dO"].mul_(-1.0)
        eager = run()
        for g in got:
            g.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(got, eager):
            assert float((x.float() - y.float()).norm()) <= 2.0 ** -10 * float(y.float().norm()), replay
