"""What bench.py reports of the launches of a step, where the backward pass is two launches and where it is one (no GPU needed)."""
import bench


def test_backward_of_one_launch_is_timed_whole():
    for kernel in ("bwd_short_kernel", "bwd_blocks_kernel"):
        names, spans = bench.backward_launches("fwd_kernel", kernel)
        assert names == ["fwd_kernel", kernel]
        assert spans == [(0, 1), (1, 4)]   # events 3 and 4 coincide: nothing lies between them
        assert bench.tile_products(names) == {"fwd_kernel": (2, 2), kernel: (5, 5)}


def test_backward_of_two_launches():
    names, spans = bench.backward_launches("fwd_pp_kernel", "dkv_w64_kernel")
    assert names == ["fwd_pp_kernel", "dq_kernel", "dkv_w64_kernel"] and spans == [(0, 1), (1, 3), (3, 4)]
    assert bench.tile_products(names) == {"fwd_pp_kernel": (2, 2), "dq_kernel": (1, 3), "dkv_w64_kernel": (4, 4)}


def test_every_launch_has_its_bytes():
    cfg = dict(B=2, H=3, N=100, d=64)
    rows, elem = 600, 600 * 64 * 2
    assert bench.kernel_bytes(cfg, 3) == [4 * elem + 4 * rows, 6 * elem + 12 * rows, 6 * elem + 8 * rows]
    assert bench.kernel_bytes(cfg, 2) == [4 * elem + 4 * rows, 8 * elem + 4 * rows]   # reads Q, K, V, O, dO and the statistic, writes dQ, dK, dV
