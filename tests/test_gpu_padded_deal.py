"""Padded batches: the heads are dealt round the XCDs.  Every head of counts that do and do not divide evenly, over the forms of the kernels
that deal them (short heads, divided and undivided tile kernels, pairs, groups of heads, the two-group forward, 64 keys a wavefront)."""
import math

import pytest
import torch

from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H", [(1, 1), (1, 7), (2, 4), (3, 3), (5, 3), (3, 11)])
@pytest.mark.parametrize("N,d,causal", [(100, 64, False), (197, 32, True), (330, 64, True), (330, 128, False), (330, 128, True)])
def test_every_head(B, H, N, d, causal):
    lengths = [max(1, N - b * (N // B)) for b in range(B)]
    t, dev = hp.make_case(B, H, N, d, "bf16", inputs.BASE_SEED + 7000 + N + d + B * H)
    kw = dict(causal=causal, key_lengths=lengths)
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", 1 / math.sqrt(d), **kw))
    hp.assert_backward_ok(hp.check_backward(t, dev, "bf16", 1 / math.sqrt(d), **kw))


@pytest.mark.parametrize("heads", [8, 13, 67])
@pytest.mark.parametrize("fwd,dkv,d,causal", [("pp", "w64", 128, False), ("pp", "rs", 128, True), ("base", "rs", 64, False), ("base", "fr", 128, True)])
def test_forced_kernels(heads, fwd, dkv, d, causal):
    """Batch entries of one head each: what a head gives does not depend on which others are in the batch."""
    N, tau = 352, 1 / math.sqrt(d)
    gen = torch.Generator(device="cuda").manual_seed(11)
    q, k, v, do = (torch.randn(heads, 1, N, d, generator=gen, device="cuda").bfloat16() for _ in range(4))
    lengths = [1 + (37 * b) % N for b in range(heads)]
    try:
        binding.attn_debug_set_variant(fwd=fwd, dkv=dkv)

        def passes(sel):
            kw = dict(softmax_scale=tau, causal=causal, key_lengths=torch.tensor([lengths[b] for b in sel], dtype=torch.int32, device="cuda"))
            a = [x[sel].contiguous() for x in (q, k, v, do)]
            o, lse = binding.attn_fwd(*a[:3], **kw)
            return (o, lse, *binding.attn_bwd(*a[:3], o, a[3], lse, **kw))

        whole = passes(list(range(heads)))
        for b in sorted({0, 1, heads // 2, heads - 2, heads - 1}):
            for got, want in zip(whole, passes([b])):
                assert torch.equal(got[b], want[0])
    finally:
        binding.attn_debug_set_variant(fwd="auto", dkv="auto")
