"""Dense causal kernels, one block of rows or keys per work item: whichever heads are dealt out together and in whatever order, each block of
each head is worked on once.  A head's results do not depend on that order: with nothing divided over groups of wavefronts they are, bit for bit, those
of the head alone."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


# blocks of 128 rows: all heads together (few items; heads that divide over the XCDs, or not; a head alone in its last group of eight), and runs of
# grouped heads (128 heads or a multiple, 224 or more; the last group short), each with a ragged last block
@pytest.mark.parametrize("heads,N,d", [(1, 700, 64), (12, 1000, 64), (130, 600, 64), (1, 300, 128), (9, 700, 128), (16, 1000, 128), (130, 600, 128), (128, 600, 128), (229, 390, 128), (256, 300, 128),
                                       (13, 900, 32), (136, 500, 32),
                                       # one head at a time: one round, one block, two short ones, three (the forward; the backward in runs)
                                       (21, 1400, 128), (300, 100, 128), (240, 142, 128), (150, 300, 128),
                                       # levels padded to the XCDs
                                       (133, 600, 64), (103, 700, 128), (39, 500, 32), (462, 192, 64),
                                       # the forward in whole runs of 32
                                       (512, 450, 64),
                                       # K and V beyond the last-level cache: runs, the last one short
                                       (2900, 460, 64), (167, 8000, 64), (340, 8000, 32)])
def test_every_block_of_every_head_once(heads, N, d):
    from paper_2205_14135_amd import binding
    binding.load()
    binding.attn_debug_set_variant("base", "fr")
    try:
        g = torch.Generator(device="cuda").manual_seed(heads * N)
        q, k, v, do = (torch.randn(1, heads, N, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(4))
        kw = dict(softmax_scale=1 / math.sqrt(d), causal=True)
        out, lse = binding.attn_fwd(q, k, v, out=torch.full_like(q, math.nan), **kw)
        grads = binding.attn_bwd(q, k, v, out, do, lse, grads=tuple(torch.full_like(q, math.nan) for _ in range(3)), **kw)
        for h in sorted({0, 1, heads // 2, heads - 2, heads - 1} & set(range(heads))):
            one = [x[:, h:h + 1].contiguous() for x in (q, k, v, do)]
            o1, l1 = binding.attn_fwd(*one[:3], **kw)
            g1 = binding.attn_bwd(*one[:3], o1, one[3], l1, **kw)
            for got, want in zip((out, lse, *grads), (o1, l1, *g1)):
                assert torch.equal(got[:, h:h + 1], want), f"head {h}"
        assert all(bool(torch.isfinite(x).all()) for x in (out, lse, *grads))
    finally:
        binding.attn_debug_set_variant("auto", "auto")
