"""The native argument marshalling refuses what it has to refuse, with the binding's own error types, and hands the library what the
binding's Python marshalling (which the measurement entry points use) would.  CPU tensors: every call below is rejected
before anything is launched, or goes to recorders in the place of the library's entry points."""
import ctypes
import os

import numpy as np
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
    with pytest.raises(ValueError):
        f(q, q, q, softmax_scale="a")
    with pytest.raises(TypeError):
        f(q, q, q, softmax_scale=None)
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


def test_missing_tensors_are_refused():
    """No input and no gradient buffer is made up: whoever passes None for one gets the library's error."""
    q, l, m = _t(), torch.zeros(1, 2, 128), torch.ones(1, 1, dtype=torch.uint8)
    ws = torch.zeros(1 << 20, dtype=torch.uint8)
    dense = lambda O=q, LSE=l, grads=None: binding.attn_bwd(q, q, q, O, q, LSE, softmax_scale=0.1, grads=grads, workspace=ws)
    sparse = lambda O=q, LSE=l, grads=None: binding.attn_blocksparse_bwd(q, q, q, O, q, LSE, m, softmax_scale=0.1, grads=grads,
                                                                          workspace=ws)
    for call in (dense, sparse):
        for kw in (dict(O=None), dict(LSE=None), dict(grads=(q, None, q)), dict(grads=(None, q, q)), dict(grads=(q, q, None)),
                   dict(grads=(None, None, None))):
            with pytest.raises(binding.AttnError) as e:
                call(**kw)
            assert _status(e) == -1
        with pytest.raises(ValueError):
            call(grads=(q, q))


@pytest.mark.parametrize("bad", [
    dict(K=_t((1, 2, 64, 64))), dict(V=_t((1, 128, 2, 64)).transpose(1, 2)), dict(dO=_t((1, 2, 128, 32))), dict(O=None), dict(LSE=None),
    dict(all=_t((1, 2, 64, 128)).transpose(2, 3)), dict(all=_t(dtype=torch.float32)), dict(all=_t((2, 128, 64))), dict(all=_t((1, 2, 128, 48))),
    dict(key_lengths=torch.zeros(1, dtype=torch.int64)), dict(key_lengths=torch.zeros(2, dtype=torch.int32)),
    dict(softmax_scale="a"), dict(softmax_scale=None), dict(softmax_scale=0.0), dict(softmax_scale="-1"), dict(dropout_p=1.0), dict(dropout_p="x"),
    dict(seed="x"), dict(offset=None), dict(stream="x"), dict(grads=(None, None, None)), dict(grads=())], ids=lambda b: "-".join(map(str, b)))
def test_refusals_are_those_of_the_python_marshalling(bad):
    bad = dict(bad)
    q = bad.pop("all", _t())
    ten = {n: bad.pop(n, q) for n in ("K", "V", "O", "dO")}
    lse = bad.pop("LSE", torch.zeros(q.shape[:3]))
    kw = dict(dict(softmax_scale=0.1, grads=(q, q, q)), **bad)
    raised = []
    for f in (binding.attn_bwd, lambda *a, grads, **k: binding.attn_bwd_static(*a, grads, **k)):
        with pytest.raises(Exception) as e:
            f(q, ten["K"], ten["V"], ten["O"], ten["dO"], lse, **kw)
        raised.append(e.value)
    assert type(raised[0]) is type(raised[1])
    if isinstance(raised[0], binding.AttnError):
        assert raised[0].status == raised[1].status
    else:
        assert str(raised[0]) == str(raised[1])


@pytest.fixture
def recorded():
    """What the native marshalling passes to the library's entry points, in order: (name, copy of the params, other arguments)."""
    calls, P, vp = [], ctypes.POINTER(binding.AttnParams), ctypes.c_void_p

    def recorder(name, result, *types):
        def f(p, *rest):
            calls.append((name, bytes(p.contents), rest))
            return 512 if result is ctypes.c_size_t else 0
        return ctypes.CFUNCTYPE(result, P, *types)(f)

    class Recorders:
        attn_fwd = recorder("fwd", ctypes.c_int, *[vp] * 5)
        attn_bwd = recorder("bwd", ctypes.c_int, *[vp] * 10, ctypes.c_size_t)
        attn_bwd_workspace_bytes = recorder("ws", ctypes.c_size_t)
        mask = [vp, ctypes.c_int32, ctypes.c_int64]
        attn_blocksparse_fwd = recorder("sparse_fwd", ctypes.c_int, *mask, *[vp] * 5)
        attn_blocksparse_bwd = recorder("sparse_bwd", ctypes.c_int, *mask, *[vp] * 10, ctypes.c_size_t)
        attn_blocksparse_bwd_workspace_bytes = recorder("sparse_ws", ctypes.c_size_t)

    lib = binding.load()
    binding._attach(Recorders)
    yield calls
    binding._attach(lib)


def _layouts(dtype):
    base = torch.zeros(3, 130, 4, 80, dtype=dtype)
    yield torch.zeros(3, 4, 130, 64, dtype=dtype)                                    # packed
    yield base[..., :64].transpose(1, 2)                                             # token-major, padded rows
    yield torch.zeros(130, 3, 4, 16, dtype=dtype).permute(1, 2, 0, 3)                # rows outermost
    yield torch.zeros(1, 4, 1, 128, dtype=dtype).as_strided((1, 4, 1, 128), (7, 128, 3, 1))   # axes of size 1, any stride
    yield torch.zeros(3, 4, 0, 64, dtype=dtype)                                      # nothing in it (the library refuses it)


OPTIONS = [
    dict(softmax_scale=0.125), dict(softmax_scale=1, causal=True, dropout_p=0.1, seed=5, offset=3),
    dict(softmax_scale="0.5", dropout_p="0.25"), dict(softmax_scale=np.float32(0.3), causal=np.bool_(True), dropout_p=np.float64(0.1)),
    dict(softmax_scale=torch.tensor(0.7), causal=torch.tensor(1), seed=torch.tensor(9), offset=np.int64(-4)),
    dict(softmax_scale=1e300, causal=[], o_fp32="x"), dict(softmax_scale=0.1, seed=(1 << 70) + 5, offset=-1, stream=(1 << 64) - 16),
    dict(softmax_scale=0.1, seed=-(1 << 63) - 1, offset=(1 << 64) + 3, o_fp32=True, stream=0), dict(softmax_scale=0.1, seed=3.9, offset="12"),
]


@pytest.mark.parametrize("options", OPTIONS, ids=range(len(OPTIONS)))
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_params_are_those_of_the_python_marshalling(recorded, options, dtype):
    for q in _layouts(dtype):
        B, H, N, d = q.shape
        for lengths in (None, torch.zeros(B, dtype=torch.int32)):
            kw = dict(options, key_lengths=lengths)
            want = bytes(binding.make_params(q, **kw))
            k, v, o, do = (torch.empty_strided(q.shape, q.stride(), dtype=dtype) for _ in range(4))
            lse = torch.zeros(B, H, N)
            for m in (torch.ones(2, 2, dtype=torch.uint8), torch.ones(H, 2, 2, dtype=torch.uint8)):
                recorded.clear()
                out, l = binding.attn_fwd(q, k, v, **kw)
                dq, dk, dv = binding.attn_bwd(q, k, v, o, do, lse, **kw)
                sout, sl = binding.attn_blocksparse_fwd(q, k, v, m, mask_block=np.int32(128), out=o, lse=lse, **kw)
                ws = torch.zeros(3, 5)
                sg = binding.attn_blocksparse_bwd(q, k, v, o, do, lse, m, workspace=ws, grads=(out, dk, dv), **kw)
                assert sout is o and sl is lse and sg[0] is out and sg[1] is dk and sg[2] is dv
                for t in (out, dq, dk, dv):
                    assert t.shape == q.shape and t.stride() == q.stride()
                    assert t.dtype == (torch.float32 if t is out and kw.get("o_fp32") else dtype)
                assert l.shape == (B, H, N) and l.dtype == torch.float32 and l.is_contiguous()
                p = lambda *ts: tuple(t.data_ptr() or None for t in ts)
                mask = (m.data_ptr(), 128, m.stride(0) if m.dim() == 3 else 0)
                assert [c[0] for c in recorded] == ["fwd", "ws", "bwd", "sparse_fwd", "sparse_bwd"]
                assert all(c[1] == want for c in recorded)
                args = [c[2] for c in recorded]
                assert args[0] == p(q, k, v, out, l) and args[1] == ()
                assert args[2][:9] == p(q, k, v, o, do, lse, dq, dk, dv) and args[2][9] is not None and args[2][10] == 512
                assert args[3] == mask + p(q, k, v, o, lse)
                assert args[4] == mask + p(q, k, v, o, do, lse, out, dk, dv, ws) + (60,)


def test_missing_extension_is_an_error(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_marshal", None)
    monkeypatch.setattr(binding, "MARSHAL_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(FileNotFoundError):
        binding.attn_fwd(_t(), _t(), _t(), softmax_scale=0.1)
