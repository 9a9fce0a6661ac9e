"""GPU parity of the three MFMA convolution kernels against the CPU reference's direct
convolution, per layer shape (bf16 operands, fp32 accumulate): the inputs are bf16 values, so
the exact result is the fp64 sum; the kernel may differ from it by fp32 accumulation error
before its single rounding to bf16."""
import contextlib

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

# (B, H, W, Cin, Cout, k, stride, pad): the distinct kinds of layers in the four networks at
# reduced spatial size, with ragged tiles (pixel counts and channel counts off the tile sizes)
SHAPES = [
    (2, 9, 7, 16, 24, 3, 1, 1),        # everything ragged
    (3, 8, 8, 64, 64, 3, 1, 1),        # ResNet 3x3
    (2, 8, 8, 64, 128, 3, 2, 1),       # strided 3x3
    (2, 7, 7, 64, 256, 1, 1, 0),       # bottleneck expand
    (2, 8, 8, 256, 64, 1, 1, 0),       # bottleneck reduce
    (2, 8, 8, 128, 256, 1, 2, 0),      # projection shortcut
    (2, 18, 14, 8, 64, 7, 2, 3),       # ImageNet stem (3 channels padded to 8)
    (2, 8, 8, 8, 16, 3, 1, 1),         # CIFAR stem
    (1, 6, 6, 160, 320, 3, 2, 1),      # wide-ResNet widths
    (5, 12, 12, 32, 40, 3, 1, 1),      # several pixel tiles + ragged channel tile
    (2, 9, 7, 16, 32, 3, 2, 1),        # stride 2 on odd sizes (parity classes of unequal size)
    (2, 15, 13, 8, 64, 7, 2, 3),       # stem on odd sizes
    (2, 7, 9, 64, 128, 1, 2, 0),       # 1x1 stride 2: three parity classes receive zeros
    (3, 16, 16, 128, 128, 3, 1, 1),    # full 128x128 tiles
    (130, 2, 2, 64, 64, 1, 2, 0),      # 1x1 output maps: every pixel of a 64-pixel tile is another image
    (70, 3, 3, 16, 40, 3, 1, 1),       # output rows shorter than a tile: several row and image wraps per tile step
    (32, 64, 64, 8, 128, 1, 1, 0),     # enough pixel tiles for the 128x256 configuration
    (32, 64, 64, 8, 64, 3, 1, 1),      # ... and the 64x256 one
    (33, 63, 65, 16, 136, 3, 1, 1),    # wide tiles with ragged pixel and channel tails
    (5, 7, 7, 128, 128, 3, 1, 1),      # 3x3 on 7x7 images: a pixel tile spans several images, ragged tail
    (3, 14, 14, 256, 72, 3, 1, 1),     # 3x3, four channel chunks, ragged channel tile
    (2, 28, 28, 64, 64, 3, 1, 1),      # 3x3 into 64 channels (narrow tile), several tiles per image
    (1, 56, 56, 64, 128, 3, 1, 1),     # widest image the LDS-resident patch supports at this size
    (3, 10, 10, 160, 160, 3, 1, 1),    # wide-ResNet stage 1: a contraction of 160 channels (register-staged 32-wide k-tiles)
    (2, 12, 12, 64, 160, 3, 1, 1),     # ... and one the direct-to-LDS kernel takes
    (3, 8, 8, 320, 320, 3, 1, 1),      # stage 2 width
    (2, 16, 16, 128, 320, 1, 1, 0),    # ... 1x1
    (2, 16, 16, 160, 320, 1, 2, 0),    # ... strided projection of the wide nets
    (5, 9, 11, 160, 160, 3, 1, 1),     # 160-channel tiles with a ragged pixel tail
    (2, 8, 8, 96, 160, 3, 1, 1),       # k-tiles of 64 over 96-channel taps: a tile ends two thirds into a tap
    (2, 9, 9, 32, 160, 5, 1, 2),       # ... and two taps per k-tile (5x5 window)
    (3, 11, 7, 192, 480, 1, 1, 0),     # 160-channel tiles, a contraction of three 64-wide k-tiles
    (8, 4, 4, 512, 512, 3, 1, 1),      # last stage of the CIFAR ResNets: few tiles, long contraction
    (2, 8, 8, 1024, 256, 1, 1, 0),     # reducing 1x1 layer with a long contraction
]
WIDE_NET_SHAPES = [s for s in SHAPES if s[4] in (160, 320) or s[3] in (160, 320)]


@pytest.fixture(scope="module")
def dat():
    import paper_2206_06257_amd as dat
    return dat


def _bf16_values(rng, shape, scale=1.0):
    t = torch.tensor(rng.standard_normal(shape) * scale, dtype=torch.float32).to(torch.bfloat16)
    return t


def _check(got_bf16, exact64, what):
    got = got_bf16.float().cpu().numpy().astype(np.float64)
    # one rounding to bf16 (2^-9 relative) plus fp32 accumulation noise on the largest terms
    tol = 2.0 ** -8 * np.abs(exact64) + 1e-5 * np.abs(exact64).max()
    bad = np.abs(got - exact64) > tol
    assert not bad.any(), (what, int(bad.sum()), float(np.abs(got - exact64).max()))


@pytest.mark.parametrize("shape", SHAPES)
def test_conv_forward_backward_parity(dat, shape):
    B, H, W, Ci, Co, k, st, pad = shape
    rng = np.random.default_rng(hash(shape) % (2 ** 31))
    x = _bf16_values(rng, (B, H, W, Ci))
    w = _bf16_values(rng, (Co, k, k, Ci), 1.0 / np.sqrt(Ci * k * k))
    x64, w64 = x.double().numpy(), w.double().numpy()
    y64 = oracle.conv_forward(x64, w64, st, pad)
    y = dat.conv_forward(x.cuda(), w.cuda(), st, pad)
    torch.cuda.synchronize()
    assert tuple(y.shape) == y64.shape
    _check(y, y64, "forward")
    dy = _bf16_values(rng, y64.shape)
    dx64, dw64 = oracle.conv_backward(x64, w64, dy.double().numpy(), st, pad)
    dx = dat.conv_backward_data(dy.cuda(), w.cuda(), (H, W), st, pad)
    _check(dx, dx64, "backward_data")
    dw = dat.conv_backward_weight(x.cuda(), dy.cuda(), k, st, pad).cpu().numpy().astype(np.float64)
    err = np.abs(dw - dw64).max() / np.abs(dw64).max()
    assert err < 2e-5, ("backward_weight", err)



@contextlib.contextmanager
def _switches(dat, value):
    """All three kernel switches: with all of them off every layer runs in the single-stage and register-staged kernels, none
    in 160-channel tiles (one off alone leaves the others' tiles)."""
    options = (dat.KOPT_RING_KERNEL, dat.KOPT_TILE_160, dat.KOPT_NARROW_UNDERFILLED)
    try:
        for o in options:
            dat.set_kernel_option(o, value)
        yield
    finally:
        for o in options:
            dat.set_kernel_option(o, 1)


@pytest.mark.parametrize("shape", SHAPES)
def test_single_stage_kernels_parity(dat, shape):
    """The kernels that larger layers of these kinds run in, held to the oracle at the same small sizes (by themselves the
    sizes have few tiles, and most of them choose the multi-stage kernel)."""
    B, H, W, Ci, Co, k, st, pad = shape
    rng = np.random.default_rng(hash(shape) % (2 ** 31) + 2)
    x, w = _bf16_values(rng, (B, H, W, Ci)), _bf16_values(rng, (Co, k, k, Ci), 1.0 / np.sqrt(Ci * k * k))
    x64, w64 = x.double().numpy(), w.double().numpy()
    y64 = oracle.conv_forward(x64, w64, st, pad)
    dy = _bf16_values(rng, y64.shape)
    with _switches(dat, 0):
        for backward in (False, True):
            p = dat.conv_plan(shape, backward)
            assert p["kernel"] < 2 and p["tile_c"] != 160
        _check(dat.conv_forward(x.cuda(), w.cuda(), st, pad), y64, "forward")
        _check(dat.conv_backward_data(dy.cuda(), w.cuda(), (H, W), st, pad), oracle.conv_backward(x64, w64, dy.double().numpy(), st, pad)[0],
               "backward_data")


# long contractions into more than 64 channels: at these sizes they have few tiles and run in 32-channel tiles
FEW_TILE_SHAPES = [s for s in SHAPES if s[3] % 64 == 0 and s[4] > 64 and s[4] % 160 != 0 and s[5] * s[5] * s[3] >= 1024]


def _ab(dat, shape):
    """Forward and backward-data with the switches on and off."""
    B, H, W, Ci, Co, k, st, pad = shape
    g = torch.Generator(device="cuda").manual_seed(B * H + Co)
    Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    x, w, dy = (torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16) for s in ((B, H, W, Ci), (Co, k, k, Ci), (B, Ho, Wo, Co)))
    res = []
    for on in (1, 0):
        with _switches(dat, on):
            res.append((dat.conv_forward(x, w, st, pad), dat.conv_backward_data(dy, w, (H, W), st, pad)))
            torch.cuda.synchronize()
    for a, b in zip(*res):
        assert torch.isfinite(a.float()).all() and a.float().abs().max() > 0
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("shape", WIDE_NET_SHAPES)
def test_160_channel_tiles_give_the_bits_of_128_channel_tiles(dat, shape):
    """Layers 160 or 320 channels wide run in 160-channel tiles (no partly empty last tile).  Every output element is
    the same chain of MFMA accumulations over the same k order under either tiling, so forward and backward-data
    results must not differ by a bit from those of the 128-channel tiles."""
    for backward, width in ((False, shape[4]), (True, shape[3])):
        assert (dat.conv_plan(shape, backward)["tile_c"] == 160) == (width in (160, 320))
    _ab(dat, shape)


@pytest.mark.parametrize("shape", FEW_TILE_SHAPES)
def test_32_channel_tiles_of_underfilled_layers_give_the_bits_of_128_channel_tiles(dat, shape):
    """A long contraction with too few 128x128 tiles to keep the compute units busy runs in 32-channel tiles of the multi-stage
    kernel.  Same k order per accumulator, so the same bits as the 128-channel tiles of the single-stage kernel."""
    assert len(FEW_TILE_SHAPES) >= 5
    p = dat.conv_plan(shape)
    assert (p["kernel"], p["tile_c"]) == (2, 32)
    with _switches(dat, 0):
        p = dat.conv_plan(shape)
        assert (p["kernel"], p["tile_c"]) == (1, 128)
    _ab(dat, shape)


# One shape for every tile configuration of the multi-stage kernel, with ragged pixel and channel tails: the number of tiles
# decides which one a layer gets (256 compute units), so these have as many pixels as that takes.  After the shape: (kernel,
# tile channels, tile pixels, k-tiles straddle taps, classes) of the forward and of the backward-data pass, kernel 2 being
# the multi-stage one.
RING_SHAPES = [
    ((13, 4, 4, 512, 200, 3, 1, 1), (2, 32, 128, 0, 0), (0, 128, 128, 1, 0)),      # few tiles
    ((1, 3, 3, 256, 40, 1, 1, 0), (2, 32, 128, 0, 0), (0, 128, 128, 1, 0)),        # ... fewer k-tiles than stages + 1, one pixel tile
    ((11, 28, 28, 64, 72, 3, 1, 1), (2, 64, 128, 0, 0), (0, 64, 128, 1, 0)),       # 68 128-pixel tiles
    ((11, 28, 28, 128, 128, 3, 1, 1), (2, 64, 128, 0, 0), (2, 64, 128, 0, 0)),
    ((21, 28, 28, 64, 104, 3, 1, 1), (2, 128, 128, 0, 0), (0, 64, 128, 1, 0)),     # 129
    ((11, 28, 28, 136, 128, 3, 1, 1), (0, 128, 128, 1, 0), (2, 128, 128, 0, 0)),   # 68 x 2, the second channel tile almost empty
    ((21, 28, 28, 128, 256, 3, 1, 1), (2, 256, 128, 0, 0), (2, 128, 128, 0, 0)),   # 129
    ((42, 31, 31, 256, 256, 3, 1, 1), (2, 256, 256, 0, 0), (2, 256, 256, 0, 0)),   # 158 256-pixel tiles, the last one two thirds full
    ((3, 29, 29, 72, 64, 3, 2, 1), (0, 64, 128, 1, 0), (2, 32, 128, 0, 4)),        # odd strided layers: parity classes of 225 to 196
    ((11, 29, 29, 72, 64, 3, 2, 1), (0, 64, 128, 1, 0), (2, 64, 128, 0, 4)),       # pixels per image, 21, 75 and 140 tiles
    ((21, 29, 29, 72, 64, 3, 2, 1), (0, 64, 128, 1, 0), (2, 128, 128, 0, 4)),
    ((3, 17, 17, 160, 96, 5, 2, 2), (0, 128, 128, 0, 0), (2, 160, 128, 1, 4)),      # ... with k-tiles that straddle the filter taps
    ((5, 15, 15, 64, 160, 3, 1, 1), (2, 160, 128, 0, 0), (1, 64, 128, 0, 0)),      # one 128-pixel tile per compute unit
    ((5, 30, 30, 64, 640, 3, 1, 1), (2, 160, 128, 0, 0), (2, 32, 128, 0, 0)),
    ((12, 61, 61, 64, 320, 3, 1, 1), (2, 160, 128, 0, 0), (1, 64, 128, 0, 0)),     # three (349 x 2)
    ((5, 61, 61, 64, 320, 3, 1, 1), (2, 160, 256, 0, 0), (1, 64, 128, 0, 0)),      # two (146 x 2)
    ((9, 61, 61, 160, 160, 3, 1, 1), (2, 160, 256, 1, 0), (2, 160, 256, 1, 0)),    # ... with k-tiles that straddle the filter taps
    ((17, 61, 61, 96, 160, 3, 1, 1), (2, 160, 256, 1, 0), (0, 128, 128, 0, 0)),
    ((5, 61, 61, 96, 160, 3, 1, 1), (2, 160, 128, 1, 0), (0, 128, 128, 0, 0)),     # one (146)
    ((7, 30, 30, 320, 640, 1, 2, 0), (2, 64, 128, 0, 0), (2, 160, 128, 0, 4)),     # 640 channels, 13 tiles
]


@pytest.mark.parametrize("shape,forward,backward", RING_SHAPES)
def test_multi_stage_tiles_give_the_bits_of_the_single_stage_kernels(dat, shape, forward, backward):
    """Every output is the same chain of MFMA accumulations in every tile configuration; with the three switches off the same
    layers run in the kernels that test_single_stage_kernels_parity holds to the oracle."""
    for p, want in ((dat.conv_plan(shape), forward), (dat.conv_plan(shape, True), backward)):
        assert (p["kernel"], p["tile_c"], p["tile_p"], p["straddle"], p["classes"]) == want
    _ab(dat, shape)


# pixel ranges of several chains of sums, few (<= 16) and many of them, both tile widths, images smaller than a tile
WGRAD_SHAPES = [
    (60, 14, 14, 256, 256, 3, 1, 1),   # 14 ranges of about 840 pixels, chains of 256
    (60, 20, 20, 128, 136, 3, 1, 1),   # many ranges, ragged channel tile
    (60, 28, 28, 64, 64, 3, 1, 1),     # narrow tiles, three workgroups per compute unit
    (60, 28, 28, 128, 64, 1, 1, 0),    # narrow 1x1
    (999, 3, 3, 256, 256, 3, 2, 1),    # 2x2 outputs: 16 images in a tile, ragged end
    (700, 5, 5, 64, 200, 3, 1, 1),     # a tile ends inside an image of 25 pixels
    (512, 8, 8, 256, 512, 1, 2, 0),    # 4x4 outputs: four whole images per tile
    (130, 7, 9, 64, 72, 3, 1, 1),      # 63 pixels per image: a tile is one image and one pixel
    (350, 2, 3, 64, 136, 3, 1, 1),     # six pixels per image: ten images, one row and one column per tile
    (3, 65, 67, 40, 64, 5, 1, 2),      # rows longer than a tile, 5x5 window, channels that are no power of two
]


@pytest.mark.parametrize("shape", WGRAD_SHAPES)
def test_backward_weight_sums_pixel_ranges(dat, shape):
    """fp32 chains of n <= 320 terms plus the few partial sums: relative error about sqrt(n) 2^-24 = 1.1e-6."""
    B, H, W, Ci, Co, k, st, pad = shape
    g = torch.Generator(device="cuda").manual_seed(B + Co)
    Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    x, dy = (torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16) for s in ((B, H, W, Ci), (B, Ho, Wo, Co)))
    got = dat.conv_backward_weight(x, dy, k, st, pad).cpu().double()
    xp, d64 = torch.nn.functional.pad(x.cpu().double(), (0, 0, pad, pad, pad, pad)), dy.cpu().double().view(-1, Co).t()
    for r in range(k):
        for s in range(k):
            want = d64 @ xp[:, r:r + (Ho - 1) * st + 1:st, s:s + (Wo - 1) * st + 1:st].reshape(-1, Ci)
            assert float((got[:, r, s] - want).norm() / want.norm()) < 1.1e-6, (r, s)
