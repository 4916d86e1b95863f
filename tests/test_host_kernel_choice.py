"""Which kernel, or which division of one, a problem takes, at the lines of the rules (no GPU needed)."""
import pytest

from tests.host_library import compile_shim

SOURCE = r"""
#include <cstring>
static attn::KArgs problem(int heads, int N, int d) {
  attn::KArgs a;
  std::memset(&a, 0, sizeof(a));
  a.B = 1; a.H = heads; a.N = N; a.T = (N + 127) / 128; a.Nr = 128 * a.T; a.dvalid = d;
  return a;
}
extern "C" int choice(int heads, int N, int d, int causal, int dropout) {
  return attn::choose_dkv(problem(heads, N, d), d, causal, dropout, false, attn::Overrides{0, 0});
}
extern "C" int fwd_form(int heads, int N, int d, int causal) {   // wavefronts of rows, groups
  const attn::WaveGroups w = attn::fwd_groups(problem(heads, N, d), d, causal, false, true);
  return 10 * w.waves + w.groups;
}
extern "C" int sparse_fwd_form(int heads, int N, int d, int causal) {
  const attn::WaveGroups w = attn::fwd_groups(problem(heads, N, d), d, causal, true, true);
  return 10 * w.waves + w.groups;
}
extern "C" int dq_form(int heads, int N, int d, int causal) {
  const attn::WaveGroups w = attn::dq_groups(problem(heads, N, d), d, causal, false, true);
  return 10 * w.waves + w.groups;
}
extern "C" int dkv_form(int heads, int N, int d, int causal) {
  const attn::WaveGroups w = attn::dkv_fr_groups(problem(heads, N, d), d, causal, false, true);
  return 10 * w.waves + w.groups;
}
extern "C" int dealt_together(int heads, int N, int d, int rows, int fwd) {
  attn::KArgs a = problem(heads, N, d);
  a.n_items = heads * ((N + rows - 1) / rows);
  return attn::causal_group(a, d, false, fwd != 0, (int64_t)4 * N * d);
}
extern "C" int places_of_a_level(int heads, int N, int d, int fwd) {   // of all heads dealt out together (blocks of 128 rows); 0: not padded
  attn::KArgs a = problem(heads, N, d);
  a.n_items = heads * a.T;
  attn::whole_levels(a, d, fwd != 0, a.T);
  if (a.group == 0) return a.n_items == heads * a.T ? 0 : -1;
  return a.n_items == -a.group * a.T && a.chunk * attn::kXcds == a.n_items ? -a.group : -1;
}
extern "C" int short_heads() { return attn::kBwdShort; }
extern "C" int one_wave128() { return attn::kDkvOneWave128; }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return compile_shim(SOURCE, tmp_path_factory.mktemp("choice"))


# causal mask and dropout at d = 128: the one-wavefront kernel, also where the role-split kernel's pairs of key blocks would be one round over 256 compute units
@pytest.mark.parametrize("heads,N", [(64, 1024), (32, 1792), (36, 1792), (37, 1792), (33, 1920), (16, 2048), (17, 2048), (32, 2048), (10, 4096), (8, 8192), (1, 65536)])
def test_causal_mask_and_dropout_at_128_columns(shim, heads, N):
    assert shim.choice(heads, N, 128, 1, 1) == shim.one_wave128()
    assert shim.choice(heads, N, 128, 1, 0) == shim.one_wave128()


# the one-launch backward: always up to two tiles of 64 tokens, and with three up to a round of 256 heads; with four, where the two launches have two rounds over 256
# compute units and it has one
@pytest.mark.parametrize("heads,N", [(h, n) for h in (1, 64, 256) for n in (1, 128, 129, 192)] + [(h, n) for h in (600, 5000) for n in (1, 128)])
def test_short_heads_up_to_three_tiles(shim, heads, N):
    for d in (32, 64):
        assert all(shim.choice(heads, N, d, c, p) == shim.short_heads() for c in (0, 1) for p in (0, 1))


@pytest.mark.parametrize("heads,N,d,causal,dropout,expect", [
    (64, 197, 64, 0, 0, 0), (65, 197, 64, 0, 0, 1), (65, 197, 64, 0, 1, 0), (96, 209, 64, 0, 0, 0), (96, 197, 32, 0, 0, 0), (128, 256, 64, 0, 1, 0), (129, 256, 64, 0, 1, 1),
    (129, 256, 32, 0, 0, 1), (256, 256, 32, 0, 0, 1), (129, 256, 32, 0, 1, 1), (1, 256, 64, 1, 0, 0), (96, 193, 64, 1, 0, 0), (97, 208, 64, 1, 0, 1), (97, 209, 64, 1, 0, 0), (97, 193, 64, 1, 1, 0), (128, 193, 32, 1, 1, 0), (129, 256, 64, 1, 0, 1),
    (129, 256, 32, 1, 1, 1), (256, 256, 64, 1, 1, 1)])
def test_short_heads_of_four_tiles(shim, heads, N, d, causal, dropout, expect):
    assert (shim.choice(heads, N, d, causal, dropout) == shim.short_heads()) == bool(expect)


# more than a round of 256 heads: the longest heads that take it with the second, the third or a later round up to half full, and beyond
@pytest.mark.parametrize("d,causal,dropout,longest", [
    (64, 0, 0, (192, 224, 192, 224, 176, 192)), (64, 0, 1, (160, 224, 144, 192, 144, 144)), (64, 1, 0, (128, 192, 128, 192, 128, 160)), (64, 1, 1, (128, 192, 128, 144, 128, 128)),
    (32, 0, 0, (128, 192, 128, 144, 128, 128)), (32, 0, 1, (192, 224, 192, 224, 192, 192)), (32, 1, 0, (128, 224, 144, 192, 128, 192)), (32, 1, 1, (128, 224, 176, 224, 176, 192))])
def test_short_heads_of_several_rounds(shim, d, causal, dropout, longest):
    rounds = [(257, 320), (385, 512), (513, 640, 769, 896), (641, 768, 897, 1024), (1025, 1152, 5121), (1153, 1280, 5000)]
    for heads, N in zip(rounds, longest):
        for h in heads:
            assert [shim.choice(h, n, d, causal, dropout) == shim.short_heads() for n in (128, N, N + 1)] == [True, True, False]
    quarter = 192 if causal and (d, dropout) != (64, 1) else longest[0]   # (the second round more than a quarter full)
    for h in (321, 384):
        assert [shim.choice(h, n, d, causal, dropout) == shim.short_heads() for n in (quarter, quarter + 1)] == [True, False]


# heads of up to two tiles have one form, however many there are; three are divided between two groups of wavefronts where there are few
@pytest.mark.parametrize("heads,N,d,causal,form", [(1, 64, 64, 0, 41), (1, 128, 64, 0, 41), (500, 128, 64, 0, 41), (1, 128, 64, 1, 41), (1, 129, 64, 1, 22), (85, 192, 64, 0, 22),
                                                   (86, 192, 64, 0, 41), (1, 128, 32, 1, 41), (1, 129, 32, 1, 22), (1, 320, 128, 0, 41), (1, 321, 128, 0, 22)])
def test_forward_of_few_tiles(shim, heads, N, d, causal, form):
    assert shim.fwd_form(heads, N, d, causal) == form


# causal heads of 64 columns: {2, 2} up to 11/8 half blocks per compute unit from nine tiles on, {4, 2} from twelve tiles on (sixteen
# for more than three halves of 128 rows on four compute units)
@pytest.mark.parametrize("heads,N,form", [(160, 225, 41), (128, 225, 22), (75, 506, 41), (64, 506, 22), (52, 520, 22), (56, 520, 22), (70, 520, 22), (71, 520, 41), (67, 654, 41), (85, 700, 41),
                                          (85, 705, 41), (64, 705, 42), (65, 705, 41), (57, 960, 41), (57, 961, 42), (50, 705, 22), (51, 985, 42), (64, 1024, 42), (65, 1024, 41)])
def test_forward_of_causal_heads_of_64_columns(shim, heads, N, form):
    assert shim.fwd_form(heads, N, 64, 1) == form


# block masks: how many tiles a row keeps is not known on the host, and the causal mask changes nothing in the division
@pytest.mark.parametrize("heads,N,d,form", [(8, 4096, 32, 24), (9, 4096, 32, 24), (10, 4096, 32, 24), (5, 8192, 32, 24), (11, 4096, 32, 42), (16, 4096, 32, 42), (17, 4096, 32, 41),
                                            (4, 4096, 64, 24), (8, 4096, 64, 42), (9, 4096, 64, 41), (4, 4096, 128, 22)])
def test_forward_under_a_block_mask(shim, heads, N, d, form):
    assert shim.sparse_fwd_form(heads, N, d, 0) == form
    assert shim.sparse_fwd_form(heads, N, d, 1) == form


# causal heads: how many of them are dealt out together (0: all), with the rows of a work item
@pytest.mark.parametrize("heads,N,d,rows,fwd,bwd", [
    (35, 677, 128, 128, 1, 1), (13, 993, 128, 64, 1, 1), (64, 512, 128, 128, 1, 1), (61, 194, 128, 64, 1, 1), (65, 512, 128, 128, 0, 0), (12, 8192, 128, 128, 0, 0),   # one round
    (1414, 111, 128, 128, 0, 1), (7, 64, 128, 64, 0, 1),                                                                       # one block
    (224, 142, 128, 128, 0, 0), (225, 142, 128, 128, 1, 8), (256, 250, 128, 128, 1, 8), (257, 250, 128, 128, 8, 8),            # two
    (128, 300, 128, 128, 0, 0), (129, 300, 128, 128, 1, 8), (170, 300, 128, 128, 1, 8), (171, 300, 128, 128, 0, 0), (214, 300, 128, 128, 1, 0), (256, 300, 128, 128, 1, 8),
    (257, 300, 128, 128, 8, 8), (64, 2352, 128, 128, 0, 6), (128, 1110, 128, 128, 8, 8), (136, 1110, 128, 128, 0, 0), (96, 2048, 32, 128, 0, 0), (2, 200, 64, 64, 0, 0),
    (512, 2560, 64, 128, 32, 0), (512, 2561, 64, 128, 12, 12), (1300, 1024, 64, 128, 32, 32), (40, 40000, 64, 128, 1, 1), (80, 32768, 32, 128, 0, 0), (81, 32768, 32, 128, 2, 2),   # beyond the cache
    (100, 10485, 128, 128, 0, 0), (100, 10500, 128, 128, 1, 1),
    (512, 385, 64, 128, 32, 0), (512, 384, 64, 128, 0, 0), (1024, 1024, 64, 128, 32, 0), (1280, 512, 64, 128, 0, 0), (640, 512, 64, 128, 0, 0), (512, 512, 32, 128, 0, 0)])
def test_causal_heads_dealt_together(shim, heads, N, d, rows, fwd, bwd):
    assert (shim.dealt_together(heads, N, d, rows, 1), shim.dealt_together(heads, N, d, rows, 0)) == (fwd, bwd)


# a level of all heads is padded to whole rounds over the XCDs where that is up to 3 %
@pytest.mark.parametrize("heads,N,d,fwd,bwd", [(462, 192, 64, 464, 464), (464, 192, 64, 0, 0), (1, 700, 64, 0, 0), (12, 700, 64, 0, 0), (31, 700, 64, 0, 0), (39, 700, 64, 40, 40), (233, 700, 128, 0, 0), (234, 700, 64, 240, 240),
                                               (232, 700, 64, 0, 0), (201, 700, 64, 0, 0), (203, 700, 32, 0, 208)])
def test_levels_padded_to_the_xcds(shim, heads, N, d, fwd, bwd):
    assert (shim.places_of_a_level(heads, N, d, 1), shim.places_of_a_level(heads, N, d, 0)) == (fwd, bwd)


# long causal sweeps of narrow heads over four groups of wavefronts: 86 tiles and up to four blocks of 64 rows per compute unit
@pytest.mark.parametrize("heads,N,causal,form", [(8, 7975, 1, 24), (11, 5441, 1, 24), (11, 5440, 1, 22), (12, 5441, 1, 22), (8, 7975, 0, 42), (7, 5440, 1, 24)])
def test_forward_of_long_narrow_heads(shim, heads, N, causal, form):
    assert shim.fwd_form(heads, N, 32, causal) == form


# gradients of causal heads of 64 columns: {2, 2} up to 11/8 half blocks per compute unit from 11 tiles on, {4, 2} for longer sweeps in up to one half of 128 rows (three on four compute
# units where they are short)
@pytest.mark.parametrize("heads,N,dq,dkv", [(50, 600, 22, 22), (60, 592, 41, 42), (52, 694, 22, 22), (58, 700, 22, 22), (59, 700, 41, 42), (64, 700, 41, 42), (65, 700, 41, 41), (64, 800, 41, 42), (65, 800, 41, 41),
                                            (90, 408, 41, 41), (128, 512, 41, 41), (44, 1024, 22, 22), (45, 1024, 42, 42), (48, 1024, 42, 42), (49, 1024, 41, 42), (64, 1024, 41, 42), (65, 1024, 41, 41),
                                            (37, 1500, 42, 42), (40, 1500, 42, 42), (43, 1500, 41, 41)])
def test_gradients_of_causal_heads_of_64_columns(shim, heads, N, dq, dkv):
    assert (shim.dq_form(heads, N, 64, 1), shim.dkv_form(heads, N, 64, 1)) == (dq, dkv)


# gradients of causal heads of 32 columns: {2, 2} in dQ up to three blocks of 64 rows per compute unit, four from nine tiles on; in dK/dV up to two halves, fewer where there are few tiles
@pytest.mark.parametrize("heads,N,dq,dkv", [(153, 310, 22, 41), (154, 310, 41, 41), (106, 324, 22, 22), (107, 324, 22, 41), (88, 450, 22, 22), (89, 450, 22, 41), (96, 512, 22, 41), (97, 512, 41, 41),
                                            (102, 576, 22, 22), (103, 576, 22, 41), (113, 576, 22, 41), (114, 576, 41, 41), (128, 256, 22, 22), (160, 205, 22, 22), (161, 205, 22, 41)])
def test_gradients_of_causal_heads_of_32_columns(shim, heads, N, dq, dkv):
    assert (shim.dq_form(heads, N, 32, 1), shim.dkv_form(heads, N, 32, 1)) == (dq, dkv)


# causal heads of 64 columns in nearly a round of half blocks: {2, 2} instead of {2, 4} where the sweeps are short
@pytest.mark.parametrize("heads,N,form", [(20, 1149, 24), (21, 1149, 22), (18, 1280, 24), (19, 1280, 22), (17, 1472, 22), (17, 1473, 24), (14, 1728, 24), (15, 1728, 22), (12, 2240, 24), (13, 2240, 22), (12, 2496, 22), (12, 2497, 24),
                                           (8, 4096, 24)])
def test_forward_of_nearly_a_round_of_causal_heads(shim, heads, N, form):
    assert shim.fwd_form(heads, N, 64, 1) == form
    assert shim.sparse_fwd_form(heads, 1024, 64, 1) == shim.sparse_fwd_form(heads, 1024, 64, 0)
