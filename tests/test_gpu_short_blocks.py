"""The one-launch backward of heads of 257 to 512 tokens (d <= 64, two key blocks) against the oracle, and against the two launches that a workspace without
room for its float32 dQ brings back: the same products, summed in another order in dQ."""
import math

import pytest
import torch

from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


# lengths at the edges of the key blocks (256, 512), wavefronts (32), tiles (64) and the rule (384)
# (narrow heads of up to 384 tokens without a mask stay with the two launches)
@pytest.mark.parametrize("N,d,causal,p", [(N, d, causal, p) for causal, p in ((False, 0.0), (True, 0.0), (False, 0.1), (True, 0.37)) for d in (16, 32, 64)
                                          for N in (257, 288, 320, 321, 383, 384, 385, 449, 511, 512) if d == 64 or N > 384 or causal])
def test_two_key_blocks(N, d, causal, p):
    B, H = 14, 16   # enough heads that the one launch is taken
    dtype, tau = ("fp16", "bf16")[N % 2], 1 / math.sqrt(d)
    t, dev = hp.make_case(B, H, N, d, dtype, inputs.BASE_SEED + 8000 + N + d)
    q, k, v, do = (dev[n] for n in ("Q", "K", "V", "dO"))
    opts = dict(causal=causal, seed=inputs.BASE_DROPOUT_SEED + 23, offset=1)
    rows = 128 * ((N + 127) // 128)
    small = torch.empty(2 * 4 * B * H * rows, dtype=torch.uint8, device="cuda")
    params = binding.make_params(q, softmax_scale=tau, dropout_p=p, **opts)
    assert binding.attn_debug_bwd_kernel(params, binding.attn_bwd_workspace_bytes(params)) == "bwd_blocks_kernel"
    assert binding.attn_debug_bwd_kernel(params, small.numel()) == "dkv_fr_kernel"
    hp.assert_backward_ok(hp.check_backward(t, dev, dtype, tau, p=p, heads=[(0, 0), (B - 1, H - 1)], **opts))
    lengths = torch.tensor([max(0, N - 41 * b) for b in range(B)], dtype=torch.int32, device="cuda")
    for kl in (None, lengths):
        kw = dict(softmax_scale=tau, dropout_p=p, key_lengths=kl, **opts)
        size = binding.attn_bwd_workspace_bytes(binding.make_params(q, **kw))
        assert size >= small.numel() + 4 * B * H * N * max(d, 32)
        large = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")   # (NaN throughout)
        o, lse = binding.attn_fwd(q, k, v, **kw)
        got, again, want = (binding.attn_bwd(q, k, v, o, do, lse, grads=tuple(torch.full_like(q, 7.0) for _ in range(3)), workspace=ws, **kw)
                            for ws in (large, large, small))
        for a, a2, b in zip(got, again, want):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, a2)
            # float32 sums of the same terms, rounded once: half a unit of the 16-bit type each, where they differ at all
            assert float((a.float() - b.float()).norm()) <= 2.0 ** -8 * float(b.float().norm())


def test_strides_and_float32_output():
    """Heads interleaved in memory, and O in float32."""
    B, H, N, d = 14, 16, 330, 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, do = (torch.randn(B, N, H, d, generator=gen, device="cuda").bfloat16().transpose(1, 2) for _ in range(4))
    kw = dict(softmax_scale=0.125, causal=True, o_fp32=True)
    o, lse = binding.attn_fwd(q, k, v, **kw)
    assert o.dtype == torch.float32
    got = binding.attn_bwd(q, k, v, o, do, lse, **kw)
    packed = [x.contiguous() for x in (q, k, v, o, do)]
    want = binding.attn_bwd(*packed, lse, **kw)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# O in float32 is read by another branch than O in 16 bits: against the oracle, and against the two launches' reading of it
@pytest.mark.parametrize("N,d,causal,p", [(330, 64, True, 0.0), (500, 64, False, 0.1), (400, 32, True, 0.1), (512, 16, False, 0.0)])
def test_float32_output_against_the_oracle(N, d, causal, p):
    B, H, dtype, tau = 14, 16, ("fp16", "bf16")[causal], 1 / math.sqrt(d)
    t, dev = hp.make_case(B, H, N, d, dtype, inputs.BASE_SEED + 8500 + N)
    opts = dict(causal=causal, seed=inputs.BASE_DROPOUT_SEED + 24, offset=2, o_fp32=True)
    hp.assert_backward_ok(hp.check_backward(t, dev, dtype, tau, p=p, heads=[(0, 1), (B - 1, H - 2)], **opts))
    q, k, v, do = (dev[n] for n in ("Q", "K", "V", "dO"))
    kw = dict(softmax_scale=tau, dropout_p=p, **opts)
    params = binding.make_params(q, **kw)
    assert binding.attn_debug_bwd_kernel(params, binding.attn_bwd_workspace_bytes(params)) == "bwd_blocks_kernel"
    small = torch.empty(2 * 4 * B * H * 128 * ((N + 127) // 128), dtype=torch.uint8, device="cuda")
    o, lse = binding.attn_fwd(q, k, v, **kw)
    for a, b in zip(binding.attn_bwd(q, k, v, o, do, lse, **kw), binding.attn_bwd(q, k, v, o, do, lse, workspace=small, **kw)):
        # float32 sums of the same terms, rounded once: half a unit of the 16-bit type each, where they differ at all
        assert float((a.float() - b.float()).norm()) <= 2.0 ** -8 * float(b.float().norm())


# Head dimension 16: the upper halves of the tile rows are zeros that no copy writes, and the rows of the first key block's gradients go out through the
# same LDS.  What is left of a dK element beyond the range of float16 must not meet the second key block.
@pytest.mark.parametrize("N,causal", [(300, True), (400, True), (400, False), (512, False)])
def test_overflow_in_the_first_key_block(N, causal):
    B, H, d = 14, 16, 16
    gen = torch.Generator(device="cuda").manual_seed(9)
    q, k, v, do = (torch.randn(B, H, N, d, generator=gen, device="cuda").half() for _ in range(4))
    # column 0 of dK overflows for every key of the first block (|dK| > 1.5e5), nothing else does (|dK| < 3e4)
    q[..., 0], k, v = 1000., k / 4, v / 10
    k[..., 0] = 0.
    v[:, :, 0:256:2] += 4.
    v[:, :, 1:256:2] -= 4.
    do = torch.full_like(do, 64.)
    kw = dict(softmax_scale=0.25, causal=causal)
    vectors = 2 * 4 * B * H * 128 * ((N + 127) // 128)
    assert binding.attn_bwd_workspace_bytes(binding.make_params(q, **kw)) > vectors   # the one launch
    o, lse = binding.attn_fwd(q, k, v, **kw)
    got = binding.attn_bwd(q, k, v, o, do, lse, **kw)
    want = binding.attn_bwd(q, k, v, o, do, lse, workspace=torch.empty(vectors, dtype=torch.uint8, device="cuda"), **kw)
    over = torch.zeros_like(q, dtype=torch.bool)
    over[:, :, :256, 0] = True
    for a, b, infinite in zip(got, want, (~over & over, over, ~over & over)):   # dQ, dK, dV
        assert torch.equal(torch.isinf(b), infinite) and not bool(b.isnan().any())
        assert torch.equal(torch.isinf(a), infinite) and not bool(a.isnan().any())
        a, b = a.float().masked_fill(infinite, 0.), b.float().masked_fill(infinite, 0.)
        assert float((a - b).norm()) <= 2.0 ** -8 * float(b.norm())
