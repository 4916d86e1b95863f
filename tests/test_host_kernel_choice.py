"""Which backward kernel a problem takes, at the lines of the rules (no GPU needed)."""
import pytest

from tests.host_library import compile_shim

SOURCE = r"""
#include <cstring>
extern "C" int choice(int heads, int N, int d, int causal, int dropout) {
  attn::KArgs a;
  std::memset(&a, 0, sizeof(a));
  a.B = 1; a.H = heads; a.N = N; a.T = (N + 127) / 128; a.Nr = 128 * a.T; a.dvalid = d;
  return attn::choose_dkv(a, d, causal, dropout, false, attn::Overrides{0, 0});
}
extern "C" int role_split() { return attn::kDkvRoleSplit; }
extern "C" int one_wave128() { return attn::kDkvOneWave128; }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return compile_shim(SOURCE, tmp_path_factory.mktemp("choice"))


# the role-split kernel's pairs of key blocks: long heads, in one round over 256 compute units, and more blocks than compute units
@pytest.mark.parametrize("heads,N,expect", [(64, 1024, 0), (42, 1152, 0), (34, 1400, 0), (32, 1536, 0), (29, 1664, 0), (32, 1792, 1), (36, 1792, 1), (37, 1792, 0),
                                            (32, 1920, 1), (33, 1920, 0), (32, 2048, 1), (33, 2048, 0), (16, 2048, 0), (17, 2048, 1), (10, 4096, 1), (8, 8192, 1),
                                            (4, 8192, 0), (9, 8192, 0), (1, 65536, 1)])
def test_role_split_where_its_pairs_are_one_round(shim, heads, N, expect):
    assert shim.choice(heads, N, 128, 1, 1) == (shim.role_split() if expect else shim.one_wave128())
    assert shim.choice(heads, N, 128, 1, 0) == shim.one_wave128()
