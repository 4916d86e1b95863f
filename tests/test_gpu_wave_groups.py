"""Few work items: the divided forms of the tile kernels (two or four groups of wavefronts, blocks of 64 rows) against the
oracle, at lengths on either side of their lines and where the groups' shares of the tiles differ or some group has none."""
import math

import numpy as np
import pytest
import torch

from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


# N: three and four 64-wide tiles (the fewest that are divided in the forward and the gradients), 12 and 13 (four groups in the forward and at d = 32), 24, 25 and 32 (four
# groups in the gradients); ragged ends that leave the last group a part of a tile, or nothing
@pytest.mark.parametrize("N", [129, 193, 705, 769, 1473, 1537, 1985])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("causal,p", [(False, 0.0), (True, 0.0), (False, 0.1), (True, 0.1)])
def test_few_heads(N, d, causal, p):
    dtype = "bf16" if (N // 64) % 2 else "fp16"
    tau = 1 / math.sqrt(d)
    t, dev = hp.make_case(1, 2, N, d, dtype, inputs.BASE_SEED + 5000 + N + d)
    kw = dict(causal=causal, p=p, seed=inputs.BASE_DROPOUT_SEED + 3, offset=5, heads=[(0, 1)])
    hp.assert_forward_ok(hp.check_forward(t, dev, dtype, tau, **kw))
    hp.assert_backward_ok(hp.check_backward(t, dev, dtype, tau, **kw))


# lengths that leave all groups but the first without a key (or query) to see, and one without any
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("N", [200, 1600])
def test_groups_without_tiles(N, d):
    lengths = [N, 64, 1, 0, N // 2 + 1]
    t, dev = hp.make_case(5, 1, N, d, "bf16", inputs.BASE_SEED + 5100 + N + d)
    kw = dict(key_lengths=lengths, heads=[(0, 0), (1, 0), (3, 0), (4, 0)])
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", 1 / math.sqrt(d), **kw))
    hp.assert_backward_ok(hp.check_backward(t, dev, "bf16", 1 / math.sqrt(d), **kw))


# as many heads as put the item counts on either side of the lines at 256 and 512 blocks: {2, 2}, {4, 2} and {4, 1} of the same problem
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("heads", [42, 43, 85, 86, 129, 171, 257])
@pytest.mark.parametrize("causal", [False, True])
def test_lines_between_forms(d, heads, causal):
    N, tau = 330, 1 / math.sqrt(d)   # six tiles, three blocks of 128 rows
    t, dev = hp.make_case(1, heads, N, d, "bf16", inputs.BASE_SEED + 5200 + heads)
    kw = dict(causal=causal, heads=[(0, 0), (0, heads - 1)])
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", tau, **kw))
    hp.assert_backward_ok(hp.check_backward(t, dev, "bf16", tau, **kw))
    # the same sums in another order: the undivided kernels' results, but for the rounding of a 16-bit output or two
    q, k, v, do = (dev[n] for n in ("Q", "K", "V", "dO"))
    res = {}
    try:
        for variant in ("auto", "fr"):
            binding.attn_debug_set_variant(dkv=variant)
            o, lse = binding.attn_fwd(q, k, v, softmax_scale=tau, causal=causal)
            res[variant] = (o, *binding.attn_bwd(q, k, v, o, do, lse, softmax_scale=tau, causal=causal), lse)
    finally:
        binding.attn_debug_set_variant(dkv="auto")
    for a, b in zip(res["auto"], res["fr"]):
        assert float((a.float() - b.float()).norm() / b.float().norm()) <= 2.0 ** -8


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T", [(1, 3), (2, 9), (5, 30), (9, 32)])
@pytest.mark.parametrize("causal", [False, True])
def test_block_sparse(d, heads, T, causal):
    N, tau = 128 * T, 1 / math.sqrt(d)
    mask = inputs.butterfly_block_mask(T)
    mask[T // 2] = 0   # rows without a block
    t, dev = hp.make_case(1, heads, N, d, "bf16", inputs.BASE_SEED + 5300 + T)
    kw = dict(causal=causal, block_mask=mask, heads=[(0, heads - 1)])
    if N <= 1200:
        hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", tau, **kw))
        hp.assert_backward_ok(hp.check_backward(t, dev, "bf16", tau, **kw))
        return
    m = torch.from_numpy(mask).cuda()
    q, k, v, do = (dev[n] for n in ("Q", "K", "V", "dO"))
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", tau, rows=np.arange(0, N, 37), **kw))
    res = {}
    try:
        for variant in ("auto", "fr"):
            binding.attn_debug_set_variant(dkv=variant)
            o, lse = binding.attn_blocksparse_fwd(q, k, v, m, softmax_scale=tau, causal=causal)
            res[variant] = (o, *binding.attn_blocksparse_bwd(q, k, v, o, do, lse, m, softmax_scale=tau, causal=causal))
    finally:
        binding.attn_debug_set_variant(dkv="auto")
    for a, b in zip(res["auto"], res["fr"]):
        assert float((a.float() - b.float()).norm() / b.float().norm()) <= 2.0 ** -8
