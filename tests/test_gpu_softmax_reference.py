"""The forward's softmax reference at the edge where it moves: a lane keeps the reference of its row while the
sum of its 32 probabilities of a 64-key tile stays at or below 1024."""
import math

import numpy as np
import pytest

from tests import helpers as hp
from paper_2205_14135_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _both_kernels(fwd_variant):
    """The free-running and the two-group kernel share the softmax."""


# base-2 logits of the second tile over those of the first: every key 2^4.75 (a lane's sum 861) or 2^5.25 (1218);
# one key at 2^9.75 or 2^10.25, held by the first (keys 0..3 of every eight) or the second lane of a query
@pytest.mark.parametrize("rise,where", [(4.75, None), (5.25, None), (9.75, 2), (10.25, 2), (9.75, 61), (10.25, 61), (40.0, 61)])
@pytest.mark.parametrize("d,dtype", [(16, "fp16"), (64, "fp16"), (128, "bf16")])
def test_sum_at_the_edge(rise, where, d, dtype):
    N, tau = 256, math.log(2.0)
    rng = np.random.default_rng(inputs.BASE_SEED + 1500)
    key = np.zeros(N)
    if where is None:
        key[64:128] = rise
    else:
        key[64 + where] = rise
    key[192:] = 2 * rise                         # and once more, on the moved or kept reference
    q, k = np.zeros((1, 1, N, d)), np.zeros((1, 1, N, d))
    q[..., 0] = np.where(np.arange(N) % 3 == 0, 0.5, 1.0)     # every third row of a wavefront sees half the rise
    k[..., 0] = key
    v = rng.standard_normal((1, 1, N, d))
    t = {n: inputs.round_to(x.astype(np.float32), dtype) for n, x in (("Q", q), ("K", k), ("V", v))}
    dev = {n: inputs.to_torch(x, dtype, "cuda") for n, x in t.items()}
    for causal in (False, True):
        res = hp.check_forward(t, dev, dtype, tau, causal=causal)
        print(rise, where, d, dtype, causal, res)
        hp.assert_forward_ok(res)
