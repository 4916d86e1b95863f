"""The native argument marshalling refuses what it has to refuse, with the binding's own error types.  CPU tensors:
every call below is rejected before anything is launched."""
import os

import pytest
import torch

from paper_2205_14135_amd import binding


@pytest.fixture(autouse=True, scope="module")
def _built():
    if not (os.path.exists(binding.LIB_PATH) and os.path.exists(binding.MARSHAL_PATH)):
        from paper_2205_14135_amd import build
        build.build()


def _t(shape=(1, 2, 128, 64), dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype)


def _status(exc):
    return exc.value.status


CALLS = {
    "fwd": lambda q, k, v, **kw: binding.attn_fwd(q, k, v, **kw),
    "bwd": lambda q, k, v, **kw: binding.attn_bwd(q, k, v, q, q, torch.zeros(q.shape[:3]), **kw),
    "sparse_fwd": lambda q, k, v, **kw: binding.attn_blocksparse_fwd(q, k, v, torch.ones(1, 1, dtype=torch.uint8), **kw),
    "sparse_bwd": lambda q, k, v, **kw: binding.attn_blocksparse_bwd(q, k, v, q, q, torch.zeros(q.shape[:3]),
                                                                     torch.ones(1, 1, dtype=torch.uint8), **kw),
}


@pytest.mark.parametrize("call", CALLS)
def test_refusals(call):
    f, q = CALLS[call], _t()
    with pytest.raises(ValueError):
        f(q, _t((1, 2, 64, 64)), q, softmax_scale=0.1)                                     # shapes differ
    with pytest.raises(ValueError):
        f(q, q, _t((1, 128, 2, 64)).transpose(1, 2), softmax_scale=0.1)                    # strides differ
    with pytest.raises(ValueError):
        bad = _t((1, 2, 64, 128)).transpose(2, 3)
        f(bad, bad, bad, softmax_scale=0.1)                                                # last axis not contiguous
    with pytest.raises(TypeError):
        f(_t(dtype=torch.float32), _t(dtype=torch.float32), _t(dtype=torch.float32), softmax_scale=0.1)
    with pytest.raises(TypeError):
        f(q, q, q, softmax_scale=0.1, key_lengths=torch.zeros(1, dtype=torch.int64))
    with pytest.raises(TypeError):
        f(q, q, q, softmax_scale=0.1, key_lengths=torch.zeros(2, dtype=torch.int32))
    with pytest.raises(TypeError):
        f(q, q, q, softmax_scale="a")
    for kw, status in ((dict(softmax_scale=0.0), -6), (dict(softmax_scale=0.1, dropout_p=1.0), -5)):
        with pytest.raises(binding.AttnError) as e:
            f(q, q, q, **kw)
        assert _status(e) == status
    with pytest.raises(binding.AttnError) as e:
        x = _t((1, 2, 128, 48))
        f(x, x, x, softmax_scale=0.1)
    assert _status(e) == -4


def test_mask_and_buffers():
    q = _t()
    with pytest.raises(TypeError):
        binding.attn_blocksparse_fwd(q, q, q, torch.ones(1, 1), softmax_scale=0.1)
    with pytest.raises(ValueError):
        binding.attn_blocksparse_fwd(q, q, q, torch.ones(3, 1, 1, dtype=torch.uint8), softmax_scale=0.1)
    m = torch.ones(1, 1, dtype=torch.uint8)
    with pytest.raises(binding.AttnError) as e:
        binding.attn_blocksparse_fwd(q, q, q, m, softmax_scale=0.1, mask_block=64)
    assert _status(e) == -8
    with pytest.raises(binding.AttnError) as e:
        binding.attn_bwd(q, q, q, q, q, torch.zeros(1, 2, 128), softmax_scale=0.1, workspace=torch.zeros(16, dtype=torch.uint8))
    assert _status(e) == -7
    with pytest.raises(binding.AttnError) as e:                                            # a misaligned output
        out = torch.zeros(q.numel() + 8, dtype=q.dtype)[1:1 + q.numel()].view(q.shape)
        binding.attn_fwd(q, q, q, softmax_scale=0.1, out=out)
    assert _status(e) == -2


def test_wide_seeds_are_taken_modulo_two_to_the_64th():
    q = _t((1, 2, 128, 48))
    with pytest.raises(binding.AttnError):       # refused for its head dimension, after the seed was read
        binding.attn_fwd(q, q, q, softmax_scale=0.1, seed=(1 << 70) + 5, offset=-1)


def test_missing_extension_is_an_error(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_marshal", None)
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(FileNotFoundError):
        binding.attn_fwd(_t(), _t(), _t(), softmax_scale=0.1)
