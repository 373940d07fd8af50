"""GPU parity, against the CPU oracle, of the fp32 layers over few channels on both sides of the lines between the kernels: nine taps over
9 to 32 channels on split operands or in few tiles, filters of 25 to 49 taps over 17 to 64 channels in few tiles; channel counts off the
grid of 8 and 16, every stride and dilation, ragged output channels."""
import numpy as np
import pytest
import torch

import paper_2310_05218_amd as sw
from paper_2310_05218_amd import inputs
from parity import assert_f32_parity

pytestmark = pytest.mark.gpu

# (N, C_in, C_out, H, W, R, S, stride, pad, dilation, kernel)
CASES = [
    (1, 9, 16, 50, 50, 3, 3, 1, 1, 1, "quad"),          # 2500 pixels: on the far side of the next line
    (1, 9, 33, 51, 50, 3, 3, 1, 1, 1, "few"),
    (1, 16, 64, 60, 60, 3, 3, 1, 1, 1, "split"),
    (4, 16, 104, 13, 15, 3, 3, 2, 1, 1, None),          # more than 96 output channels
    (2, 24, 96, 40, 41, 3, 3, 1, 2, 2, "split"),
    (6, 31, 72, 45, 29, 3, 3, 2, 1, 1, "split"),
    (2, 17, 8, 12, 13, 3, 3, 1, 1, 1, "few"),
    (5, 32, 200, 19, 23, 3, 3, 1, 0, 1, "split"),
    (2, 24, 40, 29, 29, 1, 9, 1, 4, 1, None),           # a row of nine taps
    (1, 32, 40, 16, 16, 3, 3, 1, 1, 1, "dma"),          # 256 pixels, 40 output channels
    (2, 17, 16, 20, 24, 5, 5, 1, 2, 1, "few"),
    (2, 64, 40, 20, 24, 5, 5, 2, 2, 1, "few"),
    (2, 64, 15, 20, 24, 5, 5, 2, 2, 1, "rows"),         # fewer outputs than a block
    (1, 63, 17, 14, 12, 7, 7, 1, 3, 1, "few"),
    (1, 64, 17, 14, 12, 7, 7, 1, 3, 1, "rows"),
    (1, 20, 30, 24, 28, 5, 7, 1, 3, 1, "few"),
    (1, 20, 30, 30, 32, 5, 5, 1, 4, 2, "few"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c[:10]))
def test_few_channels(oracle, case):
    N, Ci, Co, H, W, R, S, stride, pad, dil, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 9100 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 9200 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    y_ref, d = oracle.conv2d_dilated(x, w, stride, pad, dil)
    guard = torch.full((y_ref.size + 64,), 7.25, device="cuda")
    out = guard[32:-32].view(y_ref.shape)
    sw.sw_conv2d_dilated(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, pad, dil, out=out)
    if kernel:
        assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_kernel"), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, f"few channels {case}")
    g = guard.cpu().numpy()
    assert np.all(g[:32] == 7.25) and np.all(g[-32:] == 7.25), "wrote outside the output"


# (N, C_in, C_out, H, W, kernel): one tap on both sides of the few-tiles lines
TAPS = [
    (2, 48, 40, 36, 36, "few"), (2, 40, 40, 36, 36, "pointwise"), (10, 48, 250, 8, 8, "few"), (11, 48, 250, 8, 8, "pointwise"),
    (18, 64, 130, 10, 14, "few"), (20, 64, 130, 10, 14, "pointwise"), (24, 64, 127, 10, 14, "pointwise"), (3, 456, 17, 20, 22, "few"),
    (1, 456, 33, 20, 26, "pointwise"), (1, 456, 129, 6, 6, "few"),
]


@pytest.mark.parametrize("case", TAPS, ids=lambda c: "x".join(str(v) for v in c[:5]))
def test_one_tap(oracle, case):
    N, Ci, Co, H, W, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 9300 + Ci)
    w = inputs.normal_f32((Co, Ci, 1, 1), 9400 + Co, (2.0 / Ci) ** 0.5)
    b = inputs.normal_f32((Co,), 9500 + Co)
    y_ref, d = oracle.conv2d_bias_relu(x, w, b, 1, 0, True)
    y = sw.sw_conv2d_bias_relu(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda(), 1, 0, True)
    assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_"), sw.sw_last_kernel()
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"one tap {case}")


@pytest.mark.parametrize("case", [(9, 32, 40, 21, 31, 2, "few"), (3, 64, 24, 31, 31, 1, "few"), (2, 30, 100, 30, 33, 3, "few"), (13, 64, 24, 99, 99, 2, "dma")],
                         ids=lambda c: "x".join(str(v) for v in c[:6]))
def test_one_tap_strided(oracle, case):
    N, Ci, Co, H, W, stride, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 9600 + Ci)
    w = inputs.normal_f32((Co, Ci, 1, 1), 9700 + Co, (2.0 / Ci) ** 0.5)
    y_ref, d = oracle.conv2d(x, w, stride, 0)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, 0)
    assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_"), sw.sw_last_kernel()
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"one tap, stride {stride} {case}")


# (N, C_in, C_out, H, W, R, S, stride, pad, dilation, kernel): nine taps whose windows hold many times the cells of a tile, on both sides of the
# line to the direct-to-LDS and the any-shape kernel; 9 and 13 channels on split operands, several tiles a workgroup
WIDE = [
    (40, 24, 174, 87, 55, 9, 1, 1, 1, 1, "dma"), (16, 24, 349, 46, 46, 3, 3, 1, 4, 4, "dma"), (15, 16, 36, 47, 47, 3, 3, 1, 4, 4, "dma"),
    (17, 12, 370, 70, 70, 3, 3, 1, 0, 3, "any"), (23, 20, 303, 53, 53, 9, 1, 1, 0, 1, "any"),
    (16, 24, 349, 46, 46, 3, 3, 1, 2, 2, "split"), (6, 24, 96, 30, 17, 9, 1, 1, 0, 1, "split"), (17, 11, 64, 70, 70, 3, 3, 1, 0, 3, "split"),
    (12, 9, 104, 40, 44, 3, 3, 1, 1, 1, "split"), (9, 13, 200, 37, 29, 3, 3, 1, 0, 2, "split"),
]


@pytest.mark.parametrize("case", WIDE, ids=lambda c: "x".join(str(v) for v in c[:10]))
def test_wide_windows(oracle, case):
    N, Ci, Co, H, W, R, S, stride, pad, dil, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 9800 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 9900 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    y = sw.sw_conv2d_dilated(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, pad, dil)
    assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_kernel"), sw.sw_last_kernel()
    images = sorted({0, N - 1})                              # (the oracle is slow: the first and the last image)
    y_ref, d = oracle.conv2d_dilated(np.ascontiguousarray(x[images]), w, stride, pad, dil)
    assert_f32_parity(y.cpu().numpy()[images], y_ref, d, f"wide windows {case}")


# (N, C_in, C_out, H, W, kernel): one tap into fewer than 16 channels, planes in tiles of four columns and in wider ones
@pytest.mark.parametrize("case", [(6, 344, 9, 16, 90, "pointwise_split"), (4, 128, 12, 70, 35, "pointwise"), (15, 280, 5, 18, 32, "few"), (17, 160, 7, 24, 24, "few"),
                                  (5, 344, 9, 16, 90, "few"), (21, 104, 11, 20, 20, "few")], ids=lambda c: "x".join(str(v) for v in c[:5]))
def test_one_tap_few_outputs(oracle, case):
    N, Ci, Co, H, W, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 9310 + Ci)
    w = inputs.normal_f32((Co, Ci, 1, 1), 9410 + Co, (2.0 / Ci) ** 0.5)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0)
    assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_kernel"), sw.sw_last_kernel()
    y_ref, d = oracle.conv2d(x, w, 1, 0)
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"one tap, few outputs {case}")


# launches of eight wavefronts, two workgroups a CU, below, in and above the range of three turns of half a launch's (405, 672, 605, 688 and 880 workgroups)
@pytest.mark.parametrize("case", [(5, 11, 2, 53, 23, 3, 5, 1, 1, 1), (14, 5, 4, 81, 84, 13, 3, 1, 0, 1), (5, 155, 3, 46, 46, 4, 4, 1, 2, 2),
                                  (43, 440, 8, 32, 32, 1, 1, 2, 0, 1), (5, 324, 4, 132, 132, 1, 2, 3, 0, 1)], ids=lambda c: "x".join(str(v) for v in c))
def test_two_workgroups_a_cu(oracle, case):
    N, Ci, Co, H, W, R, S, stride, pad, dil = case
    x = inputs.normal_f32((N, Ci, H, W), 9950 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 9960 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    y = sw.sw_conv2d_dilated(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, pad, dil)
    assert sw.sw_last_kernel().startswith("mfma_f32_few_kernel<8,"), sw.sw_last_kernel()
    y_ref, d = oracle.conv2d_dilated(x, w, stride, pad, dil)
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"two workgroups a CU {case}")
