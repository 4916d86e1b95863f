"""The dK/dV kernels' threshold test and flag exchange over the range of the 8-bit threshold: the masks they
regenerate, read back through dO = identity slabs, against the oracle's."""
import numpy as np
import pytest
import torch

from oracle import attention_oracle as orc
from paper_2205_14135_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1 / 256, 0.1, 127 / 256, 0.5, 129 / 256, 0.9, 255 / 256])   # thresholds 1 .. 255, both sides of 128
@pytest.mark.parametrize("d,variant,sparse,causal", [(64, "fr", False, False), (64, "fr", False, True), (64, "fr", True, False),
                                                     (128, "fr", False, False), (128, "rs", False, True), (128, "rs", True, False)])
def test_masks(d, variant, sparse, causal, p):
    H, N, seed, offset = 2, 128, 97, 3
    kw = dict(softmax_scale=1.0, causal=causal, dropout_p=p, seed=seed, offset=offset)
    mask = torch.ones(1, 1, dtype=torch.uint8, device="cuda")
    binding.attn_debug_set_variant(dkv=variant)
    try:
        Q = torch.zeros((1, H, N, d), dtype=torch.bfloat16, device="cuda")
        K, V = torch.zeros_like(Q), torch.zeros_like(Q)
        O, L = binding.attn_fwd(Q, K, V, **kw)
        got = np.zeros((H, N, N), dtype=bool)
        idx = torch.arange(d, device="cuda")
        for slab in range(N // d):
            dO = torch.zeros_like(Q)
            dO[:, :, slab * d + idx, idx] = 1.0
            if sparse:
                dV = binding.attn_blocksparse_bwd(Q, K, V, O, dO, L, mask, **kw)[2]
            else:
                dV = binding.attn_bwd(Q, K, V, O, dO, L, **kw)[2]
            got[:, slab * d:(slab + 1) * d, :] = (dV[0] > 0).cpu().numpy().transpose(0, 2, 1)
    finally:
        binding.attn_debug_set_variant(dkv="auto")
    want = np.stack([orc.dropout_keep_mask(0, h, H, N, p, seed, offset) for h in range(H)])
    if causal:
        want = want & np.tril(np.ones((N, N), dtype=bool))
    assert (got == want).all()
