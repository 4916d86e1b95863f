"""Which mask columns the block-sparse backward cuts into segments (csrc/attn_sparse.h): the rule itself, and the count of kept blocks that it
rests on, against the whole masks (no GPU needed)."""
import ctypes

import numpy as np
import pytest

from paper_2205_14135_amd.inputs import butterfly_block_mask
from tests.host_library import compile_shim

PLACES = 512   # a fair share is taken of two workgroups on each of 256 compute units

SOURCE = r"""
#include <cstring>
#include "attn_sparse.h"
extern "C" int64_t estimate(const uint8_t* mask, int per_head, const int* lengths, int B, int H, int T, int causal, int threads) {
  attn::KArgs a;
  std::memset(&a, 0, sizeof(a));
  a.mask = mask; a.mask_sh = per_head ? (int64_t)T * T : 0; a.klen = lengths; a.B = B; a.H = H; a.T = T; a.N = 128 * T;
  const attn::MaskSample s(a);
  int64_t counted = 0;
  for (int t = 0; t < threads; ++t) counted += s.count(a, causal != 0, t, threads);
  return s.total(a, counted);
}
extern "C" int window(int T, int cg) { return attn::plan_window(T, cg); }
extern "C" int entry(int c, int segs, unsigned light, unsigned three) { return attn::column_entry(c, segs, light, three); }
extern "C" int segs_of(int entry) { return attn::segs_of(entry); }
extern "C" int slot(int item, int entry, int seg) { return attn::slot_of(item, entry, seg); }
extern "C" int segments(int cnt, int near, int n_near, int64_t total) { return attn::column_segments(cnt, near, n_near, total); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    lib = compile_shim(SOURCE, tmp_path_factory.mktemp("plan"))
    lib.estimate.restype = ctypes.c_int64
    lib.estimate.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int] * 5
    lib.segments.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64]
    return lib


def _estimate(shim, mask, B, H, lengths=None, causal=False, threads=256):
    m = np.ascontiguousarray(mask)
    n = None if lengths is None else np.asarray(lengths, dtype=np.int32)
    return shim.estimate(m.ctypes.data, int(m.ndim == 3), None if n is None else n.ctypes.data, B, H, m.shape[-1], int(causal), threads)


def _kept(mask, B, H, lengths=None, causal=False):
    """Kept blocks of the whole problem."""
    T, total = mask.shape[-1], 0
    for b in range(B):
        n = T if lengths is None else (min(max(lengths[b], 0), 128 * T) + 127) // 128
        for m in (mask if mask.ndim == 3 else [mask] * H):
            m = (np.tril(m) if causal else m)[:n, :n]
            total += int((m != 0).sum())
    return total


def _planned(shim, mask, col):
    """Kept blocks of a column, and of the columns that are looked at together with it."""
    T = mask.shape[0]
    c0 = shim.window(T, col // 16)
    counts = (mask != 0).sum(0)
    near = counts[c0:c0 + 16]
    return int(counts[col]), int(near.sum()), len(near)


@pytest.mark.parametrize("T", [15, 16, 17, 33, 63, 64])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("threads", [1, 128, 512])
def test_small_shared_masks_are_counted_whole(shim, T, causal, threads):
    rng = np.random.default_rng(T)
    m = (rng.random((T, T)) < 0.3).astype(np.uint8) * rng.integers(1, 256, (T, T)).astype(np.uint8)   # any value but 0 keeps a block
    assert _estimate(shim, m, 3, 5, causal=causal, threads=threads) == _kept(m, 3, 5, causal=causal)


@pytest.mark.parametrize("T", [65, 128, 200, 256, 512])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["butterfly", "random", "columns", "dense"])
def test_large_masks_are_sampled(shim, T, causal, kind):
    rng = np.random.default_rng(T)
    m = {"butterfly": butterfly_block_mask(T), "dense": np.ones((T, T), np.uint8), "random": (rng.random((T, T)) < 0.2).astype(np.uint8),
         "columns": np.eye(T, dtype=np.uint8)}[kind]
    if kind == "columns":
        m[:, :9] = 1
    # 16 rows at least, one from each sixteenth of the mask or nearly: the causal triangle's rows lie within 1/16 of the mean of theirs
    assert abs(_estimate(shim, m, 1, 16, causal=causal) / _kept(m, 1, 16, causal=causal) - 1) <= 0.2


@pytest.mark.parametrize("B,H,T", [(3, 2, 20), (4, 3, 40), (2, 16, 64), (7, 5, 130)])
def test_lengths_and_masks_per_head(shim, B, H, T):
    rng = np.random.default_rng(B * H * T)
    m = (rng.random((H, T, T)) < np.linspace(0.1, 0.5, H)[:, None, None]).astype(np.uint8)
    lengths = [128 * T, -5, 0, 64 * T, 128 * T + 999, 1, 100 * T][:B]
    for mask, n in ((m, None), (m, lengths), (m[0], lengths)):
        got, want = _estimate(shim, mask, B, H, lengths=n), _kept(mask, B, H, lengths=n)
        rows = (B if n is not None else 1) * (H if mask.ndim == 3 else 1) * T
        assert got == want if rows <= max(16, 4096 // T) else abs(got / want - 1) <= 0.25


def _length_over_share(heads, T):
    m = butterfly_block_mask(T)
    return T / (_kept(m, 1, heads) / PLACES)


# (not where the global column is so near a fair share that a sampled total may decide either way)
@pytest.mark.parametrize("heads,T", [(h, t) for t in (64, 128, 256, 512) for h in (1, 8, 16, 24, 32, 40, 48, 64, 256) if not 0.75 < _length_over_share(h, t) < 1.35])
def test_the_global_column_is_split_while_it_exceeds_a_fair_share(shim, heads, T):
    """The column that every row keeps, in the mask whose other columns keep about ten blocks: it is cut wherever it is longer than half of what a
    compute unit gets, however many heads there are."""
    m = butterfly_block_mask(T)
    assert (shim.segments(*_planned(shim, m, 0), _estimate(shim, m, 1, heads)) > 0) == (_length_over_share(heads, T) > 1)


@pytest.mark.parametrize("heads,T", [(16, 512), (24, 256), (32, 128), (48, 64), (8, 128)])
def test_no_workgroup_outlasts_the_others(shim, heads, T):
    """Blocks dealt longest first to 512 places: the last place ends no more than a quarter and one segment of 12 blocks after the mean."""
    m = butterfly_block_mask(T)
    counts, work = (m != 0).sum(0), []
    total = _estimate(shim, m, 1, heads)
    for col in range(T):
        cnt, near, n_near = _planned(shim, m, col)
        s = shim.segments(cnt, near, n_near, total)
        work += [-(-cnt // s)] * s if s else [cnt]
    places = np.zeros(PLACES)
    for w in sorted(work * heads, reverse=True):
        places[places.argmin()] += w
    assert places.max() <= 1.25 * counts.sum() * heads / PLACES + 12


@pytest.mark.parametrize("T", [17, 18, 31, 33, 34, 47, 49])
def test_the_last_columns_stand_out_too(shim, T):
    """A full column among thin ones is cut, wherever it stands: also where the columns do not divide by the sixteen of a planning workgroup."""
    for col in range(T):
        m = np.eye(T, dtype=np.uint8)
        m[:, col] = 1
        cnt, near, n_near = _planned(shim, m, col)
        assert n_near == 16 and shim.segments(cnt, near, n_near, _estimate(shim, m, 1, 1)) >= 2


def test_standing_out_is_by_the_neighbours(shim):
    """Twice as many blocks as the other columns keep on average, not as all of them do: 15 blocks beside fifteen columns of 7 (106 in all) are more than that."""
    assert shim.segments(15, 15 + 15 * 7, 16, 1000) > 0
    assert shim.segments(15, 15 + 15 * 8, 16, 1000) == 0


def test_short_columns_add_no_more_than_two_parts_into_one_place(shim):
    """Their gradients stay reproducible: float32 sums of two addends do not depend on which comes first.  Columns of up to 24 blocks have three
    segments at most, the third of which goes to the accumulators of a column that does not use its own."""
    assert [shim.segments(cnt, cnt, 16, 100) for cnt in (14, 15, 16, 17, 24, 25)] == [0, 2, 2, 3, 3, 4]
    rng = np.random.default_rng(5)
    for _ in range(2000):
        n_cols = int(rng.integers(1, 17))
        cnt = rng.choice([3, 15, 17, 24, 30, 64], size=n_cols)
        segs = [shim.segments(int(c), int(c), 16, 100) for c in cnt]   # (every column stands out)
        light = sum(1 << c for c in range(n_cols) if segs[c] == 0)
        three = sum(1 << c for c in range(n_cols) if segs[c] == 3 and cnt[c] <= 24)
        item0 = 16 * int(rng.integers(0, 1 << 20))
        added = {}
        for c in range(n_cols):
            entry = shim.entry(c, segs[c], light, three)
            n = shim.segs_of(entry)
            assert n == segs[c] or (n, segs[c]) == (2, 3)
            for seg in range(n):
                slot = shim.slot(item0 + c, entry, seg)
                assert slot == item0 + c or (seg == 2 and light >> (slot - item0) & 1)
                added.setdefault(slot, []).append(c)
        for slot, cs in added.items():
            assert len(set(cs)) == 1
            if cnt[cs[0]] <= 24:
                assert len(cs) <= 2
        given = sum(1 for c in range(n_cols) if three >> c & 1 and shim.segs_of(shim.entry(c, segs[c], light, three)) == 3)
        assert given == min(bin(three).count("1"), bin(light).count("1"))   # as many as there are idle ones
