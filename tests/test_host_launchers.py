"""What the launchers of the backward refuse before they launch anything (no GPU needed)."""
import pytest

from tests.host_library import compile_shim

SOURCE = r"""
#include <cstring>
// launches the dK/dV kernel that `choice` names for a dense problem of one head of 100 tokens; no pointer of it is valid
extern "C" int launch(int dvalid, int d, int choice) {
  attn::KArgs a;
  std::memset(&a, 0, sizeof(a));
  a.B = a.H = a.T = 1; a.N = 100; a.Nr = 128; a.dvalid = dvalid; a.sn = dvalid; a.sh = a.sb = 100 * dvalid;
  return attn::launch_dkv(a, 1, d, false, false, false, choice, true, nullptr);
}
extern "C" int invalid_value() { return (int)hipErrorInvalidValue; }
extern "C" int role_split() { return attn::kDkvRoleSplit; }
extern "C" int whole_backward() { return attn::kBwdShort; }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return compile_shim(SOURCE, tmp_path_factory.mktemp("launchers"))


@pytest.mark.parametrize("dvalid,d", [(16, 32), (32, 32), (64, 64)])
def test_whole_backward_is_not_a_dkv_kernel(shim, dvalid, d):
    """The choice of the one-launch backward never falls through to the role-split kernel: it can only get here from a caller that has decided twice."""
    assert shim.launch(dvalid, d, shim.whole_backward()) == shim.invalid_value()


def test_role_split_kernel_has_no_head_dimension_16(shim):
    """Its rows are 32 elements there: it would read and write beyond those of the tensors."""
    assert shim.launch(16, 32, shim.role_split()) == shim.invalid_value()
