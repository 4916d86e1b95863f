"""A query row whose logits are not finite leaves every other row alone, in both forward kernels: each row of O and L, and of
dQ, depends on its own query only."""
import math

import numpy as np
import pytest
import torch

from oracle import attention_oracle as orc
from tests import helpers as hp
from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu

N = 320
BAD_ROWS = [5, 48, 176, 319]          # both halves of a wavefront's 32 rows, first and last row block


@pytest.fixture(autouse=True)
def _both_kernels(fwd_variant):
    """The free-running and the two-group kernel share the softmax."""


def _spoil(t, dev, name, rows, kind):
    # "huge" is finite (2^127): only its products overflow float32, with both signs
    value = {"nan": math.nan, "inf": math.inf, "huge": 2.0 ** 127}[kind]
    t[name][:, :, rows] = value
    dev[name][:, :, rows] = value


def _case(d, dtype, kind, rows, name="Q", **kw):
    t, dev = hp.make_case(1, 2, N, d, dtype, inputs.BASE_SEED + 1800 + d)
    clean = {n: x.copy() for n, x in t.items()}
    _spoil(t, dev, name, rows, kind)
    return clean, t, dev, 1 / math.sqrt(d)


@pytest.mark.parametrize("d,dtype,kind", [(16, "fp16", "nan"), (32, "bf16", "huge"), (64, "bf16", "huge"), (64, "fp16", "nan"),
                                          (128, "bf16", "huge"), (128, "bf16", "inf")])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("p", [0.0, 0.1])
def test_one_row_does_not_touch_the_others(d, dtype, kind, causal, p):
    clean, t, dev, tau = _case(d, dtype, kind, BAD_ROWS)
    good = [i for i in range(N) if i not in BAD_ROWS]
    kw = dict(causal=causal, p=p, seed=inputs.BASE_DROPOUT_SEED + 80, offset=2)
    hp.assert_forward_ok(hp.check_forward(t, dev, dtype, tau, rows=good, **kw))
    # the rows themselves say that they are not numbers, and the others' gradients hold as well
    kw = dict(softmax_scale=tau, causal=causal, dropout_p=p, seed=inputs.BASE_DROPOUT_SEED + 80, offset=2)
    O, L = binding.attn_fwd(dev["Q"], dev["K"], dev["V"], **kw)
    assert torch.isnan(O[:, :, BAD_ROWS]).all()
    dQ = binding.attn_bwd(dev["Q"], dev["K"], dev["V"], O, dev["dO"], L, **kw)[0]
    for h in range(2):
        keep = orc.dropout_keep_mask(0, h, 2, N, p, kw["seed"], 2) if p > 0 else None
        want = orc.backward_head(clean["Q"][0, h], clean["K"][0, h], clean["V"][0, h], clean["dO"][0, h], tau, causal=causal,
                                 p_drop=p, keep=keep)[0]
        assert hp.rel_l2(hp.to_np(dQ)[0, h][good], want[good]) <= hp.GRAD_REL_L2


@pytest.mark.parametrize("d", [64, 128])
def test_rows_before_a_key_that_is_not_a_number(d):
    """Causal mask: the rows before the key do not see it, the rows from it on do."""
    key = 200
    _, t, dev, tau = _case(d, "bf16", "nan", [key], name="K")
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", tau, causal=True, rows=range(key)))
    O, _ = binding.attn_fwd(dev["Q"], dev["K"], dev["V"], softmax_scale=tau, causal=True)
    assert torch.isnan(O[:, :, key:]).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["nan", "huge"])
def test_padded_queries_do_not_touch_the_valid_rows(d, kind):
    length = 200
    _, t, dev, tau = _case(d, "bf16", kind, list(range(length, N)))
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", tau, key_lengths=[length], rows=range(length)))


@pytest.mark.parametrize("causal", [False, True])
def test_block_sparse(causal):
    M, d = 384, 64
    t, dev = hp.make_case(1, 2, M, d, "bf16", inputs.BASE_SEED + 1850)
    bad = [3, 150, 290]
    _spoil(t, dev, "Q", bad, "huge")
    bm = np.array([[1, 0, 0], [1, 1, 0], [0, 1, 1]], dtype=np.uint8)
    good = [i for i in range(M) if i not in bad]
    hp.assert_forward_ok(hp.check_forward(t, dev, "bf16", 1 / math.sqrt(d), causal=causal, block_mask=bm, rows=good))
