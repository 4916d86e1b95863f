"""The native autograd node of flash_attention behaves as the node in Python does: same bits, same saved tensors, same refusals;
and what has rules of its own for functions written in Python still goes to that one."""
import math

import pytest
import torch
from torch.autograd import forward_ad
from torch.utils.checkpoint import checkpoint

from paper_2205_14135_amd import autograd, binding, inputs
from paper_2205_14135_amd.autograd import flash_attention

pytestmark = pytest.mark.gpu

B, H, N, D = 2, 2, 256, 64


def _tensors(requires_grad=True, token_major=False, n=N):
    torch.manual_seed(inputs.BASE_SEED + 7000)
    shape = (B, n, H, D) if token_major else (B, H, n, D)
    ts = [torch.randn(shape, device="cuda", dtype=torch.bfloat16) for _ in range(4)]
    ts = [t.transpose(1, 2) if token_major else t for t in ts]
    return [t.requires_grad_(requires_grad) for t in ts[:3]], ts[3]


def _python_node(q, k, v, *, causal=False, dropout_p=0.0, seed=0, offset=0, key_lengths=None, block_mask=None):
    return autograd._FlashAttention.apply(q, k, v, 1 / math.sqrt(D), causal, dropout_p, seed, offset, key_lengths, block_mask)


OPTIONS = {
    "plain": {},
    "dropout": dict(causal=True, dropout_p=0.1, seed=2 ** 63 + 5, offset=2 ** 40 + 3),
    "lengths": dict(key_lengths=[N, 77]),
    "mask": dict(block_mask=True),
    "mask per head": dict(block_mask=True, per_head=True),
}


@pytest.mark.parametrize("options", OPTIONS)
@pytest.mark.parametrize("token_major", [False, True])
def test_same_bits_as_the_python_node(options, token_major):
    kw = dict(OPTIONS[options])
    if "key_lengths" in kw:
        kw["key_lengths"] = torch.tensor(kw["key_lengths"], dtype=torch.int32, device="cuda")
    if kw.pop("block_mask", False):
        m = torch.tensor([[1, 0], [1, 1]], dtype=torch.uint8, device="cuda")
        kw["block_mask"] = torch.stack([m, 1 - m]) if kw.pop("per_head", False) else m
    ts, do = _tensors(token_major=token_major)
    got = [out for f in (flash_attention, _python_node) for out in [f(*ts, **kw)]]
    assert torch.equal(got[0], got[1])
    # dO as the output is laid out, with other strides, and expanded from one number (a sum's gradient)
    for g in (do, do.contiguous(), do.transpose(2, 3).contiguous().transpose(2, 3), torch.ones((), device="cuda", dtype=do.dtype).expand_as(do)):
        a, b = (torch.autograd.grad(out, ts, g, retain_graph=True) for out in got)
        for x, y in zip(a, b):
            assert torch.equal(x, y) and x.stride() == y.stride()


def test_graph_rules():
    ts, do = _tensors()
    out = flash_attention(*ts)
    out.backward(do, retain_graph=True)
    first = [t.grad.clone() for t in ts]
    out.backward(do)
    assert all(torch.equal(t.grad, 2 * g) for t, g in zip(ts, first))
    with pytest.raises(RuntimeError):
        out.backward(do)                               # the saved tensors are gone
    out = flash_attention(*ts)
    with torch.no_grad():
        ts[1].add_(1)
    with pytest.raises(RuntimeError):
        out.backward(do)                               # a saved tensor was changed in place
    with torch.no_grad():
        assert flash_attention(*ts).grad_fn is None
    assert flash_attention(*_tensors(False)[0]).grad_fn is None
    q, k, v = (t.detach() for t in ts)
    v.requires_grad_(True)                             # one input alone
    flash_attention(q, k, v).backward(do)
    assert q.grad is None and v.grad is not None


def test_saved_tensor_hooks_and_checkpoint():
    ts, do = _tensors()
    want = torch.autograd.grad(flash_attention(*ts, dropout_p=0.2, seed=3), ts, do)
    seen = {"pack": 0, "unpack": 0}

    def pack(x):
        seen["pack"] += 1
        return x.cpu()

    def unpack(x):
        seen["unpack"] += 1
        return x.cuda()
    with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
        out = flash_attention(*ts, dropout_p=0.2, seed=3)
    got = torch.autograd.grad(out, ts, do)
    assert seen == {"pack": 5, "unpack": 5} and all(torch.equal(a, b) for a, b in zip(got, want))
    for reentrant in (False, True):
        out = checkpoint(lambda *x: flash_attention(*x, dropout_p=0.2, seed=3), *ts, use_reentrant=reentrant)
        assert all(torch.equal(a, b) for a, b in zip(_grads(out, ts, do), want))


# what comes back from the program's hooks is looked at again: as another layout, another type, or left on the host
@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("change,error", [(lambda x: x.contiguous(), ValueError), (lambda x: x.transpose(2, 3).contiguous().transpose(2, 3), ValueError),
                                          (lambda x: x.float(), TypeError), (lambda x: x.cpu(), ValueError)])
@pytest.mark.parametrize("node", ["native", "python"])
def test_saved_tensors_that_come_back_changed(which, change, error, node):
    if error is TypeError and which > 0:
        pytest.skip("the types of k and v are taken to be that of q")
    ts, do = _tensors(token_major=True)
    count = [-1]

    def pack(x):
        count[0] += 1
        return count[0], x

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: change(p[1]) if p[0] == which else p[1]):
        out = (flash_attention if node == "native" else _python_node)(*ts)
    with pytest.raises(error):
        torch.autograd.grad(out, ts, do)


# and of more batch entries than there are lengths, or other heads than the mask is for (dO is broadcast to them)
@pytest.mark.parametrize("node", ["native", "python"])
@pytest.mark.parametrize("axis,kw,error", [(0, "key_lengths", TypeError), (1, "block_mask", ValueError)])
def test_saved_tensors_of_another_batch(axis, kw, error, node):
    gen = torch.Generator(device="cuda").manual_seed(4)
    ts = [torch.randn(1, 1, 256, 64, generator=gen, device="cuda").bfloat16().requires_grad_(True) for _ in range(3)]
    do = torch.ones_like(ts[0])
    opts = {kw: torch.full((1,), 200, dtype=torch.int32, device="cuda") if kw == "key_lengths" else torch.ones(1, 2, 2, dtype=torch.uint8, device="cuda")}
    with torch.autograd.graph.saved_tensors_hooks(lambda x: x, lambda x: torch.cat([x, x], axis)):
        out = (flash_attention if node == "native" else _python_node)(*ts, **opts)
    with pytest.raises(error, match=kw):
        torch.autograd.grad(out, ts, do)


def _grads(out, ts, do):
    for t in ts:
        t.grad = None
    out.backward(do)
    return [t.grad for t in ts]


def test_refusals():
    ts, do = _tensors()
    with pytest.raises(binding.AttnError) as e:
        flash_attention(*ts, softmax_scale=-1.0)
    assert e.value.status == -6
    with pytest.raises(ValueError):
        flash_attention(ts[0], ts[1], ts[2][:, :, :128])
    with pytest.raises(TypeError):
        flash_attention(*(t.detach().float() for t in ts))
    with pytest.raises(TypeError):
        flash_attention(*ts, key_lengths=torch.zeros(B, dtype=torch.int64, device="cuda"))
    with pytest.raises(TypeError):
        flash_attention(*ts, block_mask=torch.ones(2, 2, device="cuda"))
    # on the engine's thread: a dO whose rows do not start on 16 bytes
    odd = torch.empty(do.numel() + 1, device="cuda", dtype=do.dtype)[1:].view(do.shape)
    odd.copy_(do)
    out = flash_attention(*ts)
    with pytest.raises(binding.AttnError) as e:
        out.backward(odd)
    assert e.value.status == -2


def test_transforms_keep_the_python_node():
    ts, do = _tensors(False)
    for transformed in (lambda: torch.func.vmap(flash_attention)(*(t.unsqueeze(0) for t in ts)),
                        lambda: torch.func.grad(lambda q: flash_attention(q, ts[1], ts[2]).float().sum())(ts[0])):
        with pytest.raises(RuntimeError, match="setup_context"):
            transformed()
    with forward_ad.dual_level():
        with pytest.raises(NotImplementedError):
            flash_attention(forward_ad.make_dual(ts[0], do), ts[1], ts[2])
    traced = torch.jit.trace(lambda q, k, v: flash_attention(q, k, v, causal=True), tuple(ts), check_trace=False)
    other = [t.flip(2).contiguous() for t in ts]
    assert torch.equal(traced(*other), flash_attention(*other, causal=True))


def test_backward_on_the_forward_stream():
    ts, do = _tensors(n=2048)
    want = torch.autograd.grad(flash_attention(*ts, causal=True), ts, do)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        out = flash_attention(*ts, causal=True)
    torch.cuda.current_stream().wait_stream(side)
    got = torch.autograd.grad(out, ts, do)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
