"""GPU parity of the fp32 convolutions (tiled products with fp64 sums) at sizes off their tiles: whole fp32 models against
the fp64 reference, so every difference is the fp32 rounding of stored tensors (spec bar 1e-4)."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,B,H,W", [
    (0, 1, 2, 2),        # one pixel left after the strided layer; result tiles almost empty
    (0, 3, 17, 13),      # odd sizes: the strided layer's input gradient has rows without taps, pixel tails in every tile
    (0, 33, 8, 9),       # several pixel ranges in backward-weight, the last one short
    (0, 5, 33, 21),      # a pooled map of more than 64 pixels (17 x 11): 32 threads share a vector
    (100, 2, 18, 14),    # 1x1, 3x3, strided projections, channel counts 8 .. 32
])
def test_fp32_model_off_tile_sizes(arch, B, H, W):
    import paper_2206_06257_amd as dat
    ref, gpu = oracle.Model(arch, 0, H, W, 10), dat.Model(arch, dat.F32, B + 1, H, W, 10)
    theta = syn.perturbed_params(12, ref.offsets, ref.fan_in, ref.kind)
    ref.set_params(theta); gpu.set_params(theta)
    x, y = syn.images(12, B, H, W), syn.labels(12, B, 10)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    r = ref.loss_grad(x, y, "sum")
    gx, logits, _ = gpu.input_grad(xd, yd)
    g_ref, _ = ref.step(x, y)
    g = gpu.step(xd, yd).cpu().numpy()
    # batch statistics over few values amplify the fp32 rounding of what they normalise (deeper networks: op by op in test_gpu_replay.py)
    bar = 1e-4 if arch == 0 else 2e-3
    for got, want in ((logits.cpu().numpy(), r["logits"]), (gx.cpu().numpy(), r["gx"]), (g, g_ref)):
        assert np.linalg.norm(got.astype(np.float64) - want) <= bar * np.linalg.norm(want)
    gpu.close()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 2), (1, 5)])
def test_fp32_taps_outside_the_image_are_no_terms(H, W, bad):
    """A weight or an output gradient that is not finite reaches only the outputs whose taps see it (0 * inf is NaN, so a
    zero staged for a pixel outside the image must not be multiplied by it).  On images this small some taps lie outside
    for every pixel: with only those weights infinite everything stays finite, and with an infinite output gradient the
    gradients of exactly those weights stay zero.  (1, 5): rows outside, columns partly inside."""
    import paper_2206_06257_amd as dat
    B = 3
    ref, gpu = oracle.Model(0, 0, H, W, 10), dat.Model(0, dat.F32, B, H, W, 10)
    theta = syn.perturbed_params(31, ref.offsets, ref.fan_in, ref.kind)
    convs, lin = [t for t in range(ref.num_tensors) if ref.kind[t] == 0], [t for t in range(ref.num_tensors) if ref.kind[t] == 4][0]
    x, y = syn.images(31, B, H, W), syn.labels(31, B, 10)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()

    def outside(cin, stride):      # [Cout, 3, 3, cin]: taps that no output pixel has inside the image (padding 1)
        rows, cols = ([all(not 0 <= o + tap - 1 < n for o in range(0, n, stride)) for tap in range(3)] for n in (H, W))
        return np.logical_or.outer(rows, cols)[None, :, :, None].repeat(32 if cin == 16 else 16, 0).repeat(cin, 3).reshape(-1)

    masks = {convs[0]: outside(3, 1), convs[1]: outside(16, 2)}
    assert masks[convs[1]].any()
    spoiled = theta.copy()
    for t, m in masks.items():
        spoiled[int(ref.offsets[t]):int(ref.offsets[t + 1])][m] = bad
    ref.set_params(theta); gpu.set_params(spoiled)
    want = ref.loss_grad(x, y, "sum")
    gx, logits, _ = gpu.input_grad(xd, yd)
    g_ref, _ = ref.step(x, y)
    for got, w in ((logits.cpu().numpy(), want["logits"]), (gx.cpu().numpy(), want["gx"]), (gpu.step(xd, yd).cpu().numpy(), g_ref)):
        assert np.isfinite(got).all() and np.linalg.norm(got.astype(np.float64) - w) <= 1e-4 * np.linalg.norm(w)
    spoiled = theta.copy()
    spoiled[int(ref.offsets[lin]):int(ref.offsets[lin + 1])] = bad
    gpu.set_params(spoiled)
    g = gpu.step(xd, yd).cpu().numpy()
    part = g[int(ref.offsets[convs[1]]):int(ref.offsets[convs[1] + 1])]
    assert (part[masks[convs[1]]] == 0).all() and np.isnan(part[~masks[convs[1]]]).any()
    gpu.close()
