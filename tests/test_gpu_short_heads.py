"""The one-launch backward of short heads (d <= 64, N <= 256) against the oracle, and against the two launches that the override hook
brings back: the same products in the same order, but for the sum over the keys in dQ."""
import math

import pytest
import torch

from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


# lengths at the edges of wavefronts (32), tiles (64), the four- and eight-wavefront forms (128) and the rule (192, 208, 256)
@pytest.mark.parametrize("N", [1, 33, 64, 65, 128, 129, 191, 193, 208, 209, 256])
@pytest.mark.parametrize("d", [16, 32, 64])
@pytest.mark.parametrize("causal,p", [(False, 0.0), (True, 0.0), (False, 0.1), (True, 0.37)])
def test_short_heads(N, d, causal, p):
    B, H = (10, 16) if N > 192 else (2, 3)   # enough heads that the one launch is taken
    dtype, tau = ("fp16", "bf16")[N % 2], 1 / math.sqrt(d)
    t, dev = hp.make_case(B, H, N, d, dtype, inputs.BASE_SEED + 6000 + N + d)
    opts = dict(causal=causal, seed=inputs.BASE_DROPOUT_SEED + 21, offset=2)
    if N > 1:   # a single key: the exact dQ, dK vanish (tests/test_gpu_bwd.py)
        hp.assert_backward_ok(hp.check_backward(t, dev, dtype, tau, p=p, heads=[(0, 0), (B - 1, H - 1)], **opts))
    lengths = torch.tensor([max(0, N - 37 * b) for b in range(B)], dtype=torch.int32, device="cuda")
    q, k, v, do = (dev[n] for n in ("Q", "K", "V", "dO"))
    for kl in (None, lengths):
        kw = dict(softmax_scale=tau, dropout_p=p, key_lengths=kl, **opts)
        assert binding.attn_debug_kernel_choice(binding.make_params(q, **kw))[1] == "bwd_short_kernel"
        o, lse = binding.attn_fwd(q, k, v, **kw)
        grads = {}
        try:
            for variant in ("auto", "fr"):
                binding.attn_debug_set_variant(dkv=variant)
                grads[variant] = binding.attn_bwd(q, k, v, o, do, lse, grads=tuple(torch.full_like(q, 7.0) for _ in range(3)), **kw)
        finally:
            binding.attn_debug_set_variant(dkv="auto")
        for a, b in zip(grads["auto"], grads["fr"]):
            # float32 sums of the same terms, rounded once: half a unit of the 16-bit type each, where they differ at all
            assert bool(torch.isfinite(a).all())
            assert float((a.float() - b.float()).norm()) <= 2.0 ** -8 * float(b.float().norm())
