"""When heads of 257 to 512 tokens take the one-launch backward, and what workspace that asks for (no GPU needed)."""
import ctypes

import pytest

from paper_2205_14135_amd import binding
from tests.host_library import compile_shim
from tests.test_host_abi import _params, lib   # noqa: F401  (fixture)

SOURCE = r"""
#include <cstring>
extern "C" int one_launch(int heads, int N, int d, int causal, int dropout, int room) {
  attn::KArgs a;
  std::memset(&a, 0, sizeof(a));
  float part = 0.f;
  a.B = 1; a.H = heads; a.N = N; a.T = (N + 127) / 128; a.Nr = 128 * a.T; a.dvalid = d;
  a.dQpart = room ? &part : nullptr;
  return attn::choose_dkv(a, d, causal, dropout, false, attn::Overrides{0, 0}) == attn::kBwdShort;
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return compile_shim(SOURCE, tmp_path_factory.mktemp("blocks"))


@pytest.mark.parametrize("heads,N,d,causal,expect", [
    (191, 384, 64, 0, 0), (192, 384, 64, 0, 1), (256, 257, 64, 0, 1), (257, 257, 64, 0, 0), (223, 512, 64, 0, 0), (224, 512, 64, 0, 1), (256, 513, 64, 0, 0),
    (256, 384, 32, 0, 0), (256, 385, 32, 0, 1), (191, 384, 64, 1, 0), (192, 384, 64, 1, 1), (4000, 300, 64, 1, 0), (191, 384, 32, 1, 0), (192, 384, 32, 1, 1),
    (223, 400, 64, 1, 0), (224, 400, 64, 1, 1), (257, 400, 64, 1, 0), (256, 400, 128, 1, 0)])
def test_lines(shim, heads, N, d, causal, expect):
    for dropout in (0, 1):
        assert shim.one_launch(heads, N, d, causal, dropout, 1) == expect
        assert shim.one_launch(heads, N, d, causal, dropout, 0) == 0   # no room for dQ between the key blocks


def test_workspace(lib):   # noqa: F811
    size = lambda **kw: lib.attn_bwd_workspace_bytes(ctypes.byref(_params(**kw)))
    vectors = 2 * 4 * 256 * 512
    assert size(B=16, H=16, N=512, d=64) == vectors + 256 * 512 * 64 * 4
    assert size(B=16, H=16, N=500, d=64) == vectors + 256 * 512 * 64 * 4
    assert size(B=16, H=17, N=512, d=64) == 2 * 4 * 272 * 512
    # which kernel runs depends on the room, and on the override, which keeps the two launches
    p = _params(B=16, H=16, N=512, d=64)
    room = vectors + 256 * 512 * 64 * 4
    try:
        assert [binding.attn_debug_bwd_kernel(p, n) for n in (vectors, room - 1, room)] == ["dkv_fr_kernel", "dkv_fr_kernel", "bwd_blocks_kernel"]
        assert binding.attn_debug_bwd_kernel(_params(B=1, H=1, N=128, d=64), 1 << 20) == "bwd_short_kernel"
        assert binding.attn_debug_bwd_kernel(_params(B=4, H=16, N=4096, d=128), 1 << 30) == "dkv_w64_kernel"
        binding.attn_debug_set_variant(dkv="fr")
        assert binding.attn_debug_bwd_kernel(p, room) == "dkv_fr_kernel"
    finally:
        binding.attn_debug_set_variant(dkv="auto")
    k = ctypes.c_int32()
    assert lib.attn_debug_bwd_kernel(ctypes.byref(p), vectors - 1, ctypes.byref(k)) == -7
    assert lib.attn_debug_bwd_kernel(ctypes.byref(p), vectors, None) == -1
    assert lib.attn_debug_bwd_kernel(ctypes.byref(_params(d=7)), vectors, ctypes.byref(k)) == -4
    # with the vectors alone the call is not refused for its workspace (the NULL tensor is what is refused)
    v, z = ctypes.c_void_p(0x1000), ctypes.c_void_p(0)
    p = _params(B=16, H=16, N=512, d=64)
    assert lib.attn_bwd(ctypes.byref(p), *([v] * 9), v, vectors - 1) == -7
    assert lib.attn_bwd(ctypes.byref(p), *([v] * 8 + [z]), v, vectors) == -1
