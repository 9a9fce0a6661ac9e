"""The rules that pick a convolution's kernel and tile, through dat_conv_plan (host code only: runs without a GPU)."""
import sys
import threading

import numpy as np
import pytest

import paper_2206_06257_amd as dat
from paper_2206_06257_amd import binding

OPTIONS = (dat.KOPT_RING_KERNEL, dat.KOPT_TILE_160, dat.KOPT_NARROW_UNDERFILLED)


@pytest.fixture(autouse=True)
def _default_switches():
    yield
    for o in OPTIONS:
        dat.set_kernel_option(o, 1)


def test_slabs_written_are_the_slabs_read_while_a_switch_changes():
    """The switches are read once per convolution: a change from another thread between the slab count and the launch would
    leave the batch-norm sums short of slabs, or with stale ones."""
    shapes = [(256, 14, 14, 256, 256, 3, 1, 1), (512, 16, 16, 320, 320, 3, 1, 1)]   # 256-pixel tiles with a switch on, 128 with it off
    for s, o in zip(shapes, OPTIONS):
        assert dat.conv_plan(s, stats=1)["tile_p"] == 256
        dat.set_kernel_option(o, 0)
        assert dat.conv_plan(s, stats=1)["tile_p"] == 128
        dat.set_kernel_option(o, 1)
    stop, interval, info = threading.Event(), sys.getswitchinterval(), np.zeros(10, np.int32)
    set_option, plan, out = binding._lib.dat_set_kernel_option, binding._lib.dat_conv_plan, info.ctypes.data

    def toggle():
        while not stop.is_set():
            for v in (0, 1):
                set_option(OPTIONS[0], v)
                set_option(OPTIONS[1], v)

    threads = [threading.Thread(target=toggle) for _ in range(3)]
    sys.setswitchinterval(1e-7)
    for t in threads:
        t.start()
    try:
        tiles, bad = set(), 0
        for i in range(80000):
            assert plan(i >> 1 & 1, 1 + (i >> 1 & 1), *shapes[i & 1], out) == 0
            tiles.add(int(info[3]))
            bad += int(info[8]) != int(info[9])
    finally:
        stop.set()
        for t in threads:
            t.join()
        sys.setswitchinterval(interval)
    assert tiles == {128, 256} and bad == 0


@pytest.mark.parametrize("shape,tile_c", [
    ((512, 4, 4, 512, 512, 3, 1, 1), 128), ((256, 8, 8, 256, 256, 3, 1, 1), 128),   # 256 128x128 tiles: one full round
    ((513, 4, 4, 512, 512, 3, 1, 1), 256), ((257, 8, 8, 256, 256, 3, 1, 1), 256),   # one more: 130 and 129 256x128 tiles
])
def test_256_channel_tiles_start_where_128_channel_tiles_need_a_second_round(shape, tile_c):
    for p in (dat.conv_plan(shape), dat.conv_plan(shape, True)):
        assert (p["kernel"], p["tile_c"], p["tile_p"]) == (2, tile_c, 128)


@pytest.mark.parametrize("shape", [(16, 14, 14, 64, 160, 1, 1, 0), (128, 14, 14, 192, 160, 1, 1, 0), (16, 14, 14, 128, 480, 1, 1, 0), (128, 14, 14, 64, 320, 1, 1, 0)])
def test_short_contractions_into_multiples_of_160_go_direct_to_lds(shape):
    p = dat.conv_plan(shape)
    assert (p["kernel"], p["tile_c"], p["tile_p"], p["k_tile"]) == (1, 160, 128, 64)


def test_multi_stage_shapes_of_the_gpu_tests_reach_every_configuration():
    """The list that tests/test_gpu_conv.py runs: each shape gets the tiles it is there for, and together they reach every
    tile of the multi-stage kernel, ordinary launches and launches in parity classes."""
    from tests.test_gpu_conv import RING_SHAPES
    reached = set()
    for shape, forward, backward in RING_SHAPES:
        for p, want in ((dat.conv_plan(shape), forward), (dat.conv_plan(shape, True), backward)):
            assert (p["kernel"], p["tile_c"], p["tile_p"], p["straddle"], p["classes"]) == want, (shape, p)
            if p["kernel"] == 2:
                reached.add(want[1:])
    ordinary = {(32, 128, 0), (64, 128, 0), (128, 128, 0), (256, 128, 0), (256, 256, 0), (160, 128, 0), (160, 256, 0), (160, 128, 1), (160, 256, 1)}
    classes = {(32, 128, 0), (64, 128, 0), (128, 128, 0), (160, 128, 0), (160, 128, 1)}
    assert reached == {t + (0,) for t in ordinary} | {t + (4,) for t in classes}
