"""One filter per plane in bands of output rows: odd widths, every unrolled extent and stride and some that are not, views that
are only element-aligned with NaN on both sides (the loads are 16 bytes wide), fp32 and bf16."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs
from parity import assert_f32_parity, assert_guards_intact, guarded_empty

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    import paper_2310_05218_amd as sw

    return sw


CASES = [
    # N, C, H, W, R, S, stride, pad, kernel
    (2, 40, 75, 75, 5, 5, 2, 2, "plane_bands_kernel<5,2"),       # several bands per plane, the last one short
    (1, 70, 62, 62, 3, 3, 1, 1, "plane_bands_kernel<3,1"),
    (1, 9, 113, 57, 3, 3, 2, 1, "plane_bands_kernel<3,2"),
    (2, 33, 47, 42, 7, 7, 1, 3, "plane_bands_kernel<7,1"),
    (1, 20, 71, 71, 7, 7, 2, 3, "plane_bands_kernel<7,2"),
    (1, 64, 35, 41, 5, 5, 1, 0, "plane_bands_kernel<5,1"),       # no padding
    (1, 30, 57, 57, 9, 9, 2, 4, "plane_bands_kernel<0,0"),       # taps in loops
    (1, 30, 33, 33, 4, 3, 3, 2, "plane_bands_kernel<0,0"),       # rectangular, stride 3, columns of padding only
    (1, 3, 9, 2001, 3, 3, 1, 1, "plane_bands_kernel<3,1"),       # rows of 2001: bands of four output rows
    (1, 5, 7, 7, 7, 7, 1, 0, "plane_bands_kernel<7,1"),          # a single output
    (1, 1, 64, 103, 3, 3, 1, 6, "plane_bands_kernel<3,1"),       # padding wider than a group of columns
]


def _view(torch, a, shift, dtype):
    """a on the GPU, `shift` elements off the 16-byte grid, NaN before and behind it."""
    buf = torch.full((a.size + 24,), float("nan"), dtype=dtype, device="cuda")
    at = 8 + shift
    src = torch.from_numpy(a).cuda() if dtype == torch.float32 else torch.from_numpy(a.view(np.int16)).cuda().view(dtype)
    buf[at:at + a.size] = src.reshape(-1)
    return buf[at:at + a.size].view(a.shape)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:8])))
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_plane_bands(torch, sw, oracle, case, shift):
    N, C, H, W, R, S, st, pad, kernel = case
    x = inputs.normal_f32((N, C, H, W), 6100 + H)
    w = inputs.normal_f32((C, 1, R, S), 6200 + R, 1.0 / R)
    b = inputs.normal_f32((C,), 6300, 0.5)
    y_ref, d = oracle.conv2d_depthwise(x, w, st, pad)
    xd, wd = _view(torch, x, shift, torch.float32), torch.from_numpy(w).cuda()
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_depthwise(xd, wd, st, pad, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_depthwise_bias_relu(xd, wd, torch.from_numpy(b).cuda(), st, pad, True)
    yr, dr = oracle.conv2d_depthwise_bias_relu(x, w, b, st, pad, True)
    assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:8])))
@pytest.mark.parametrize("shift", [0, 1])
def test_plane_bands_bf16(torch, sw, oracle, case, shift):
    N, C, H, W, R, S, st, pad, kernel = case
    x = inputs.normal_bf16((N, C, H, W), 6400 + H)
    w = inputs.normal_f32((C, 1, R, S), 6500 + R, 1.0 / R)
    wide = (x.astype(np.uint32) << 16).view(np.float32)
    y_ref, d = oracle.conv2d_depthwise(wide, w, st, pad)
    xd = _view(torch, x, shift, torch.bfloat16)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.bfloat16, fill=1024)
    sw.sw_conv2d_depthwise_bf16(xd, torch.from_numpy(w).cuda(), st, pad, out=out)
    if y_ref.shape[2] * y_ref.shape[3] * R * S >= 2000:
        assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert np.all(np.abs(out.float().cpu().numpy() - y_ref) <= 2e-5 * d + 2.0 ** -8 * np.abs(y_ref) + 1e-37), str(case)
    assert_guards_intact(buf, front, n, guard)


def test_one_input_channel_many_filters(torch, sw, oracle):
    """One input plane under several filters (a convolution with C_in = 1)."""
    x = inputs.normal_f32((3, 1, 45, 51), 6600)
    w = inputs.normal_f32((37, 1, 5, 5), 6601, 0.2)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 2)
    assert sw.sw_last_kernel().startswith("plane_bands_kernel<5,1"), sw.sw_last_kernel()
    assert_f32_parity(y.cpu().numpy(), *oracle.conv2d(x, w, 1, 2), "one input channel")


@pytest.mark.parametrize("case", [
    # N, filters, H, W, R, S, stride, pad, kernel: one input channel, on both sides of what bands are worth
    (8, 64, 5, 5, 3, 3, 1, 1, "plane_bands_kernel<3,1"), (27, 19, 5, 5, 3, 3, 1, 1, "direct_conv2d_kernel"),          # 512, 513 planes
    (64, 64, 7, 7, 5, 5, 1, 2, "plane_bands_kernel<5,1"), (241, 17, 7, 7, 5, 5, 1, 2, "direct_conv2d_kernel"),        # 4096, 4097
    (100, 64, 11, 11, 3, 3, 1, 1, "plane_bands_kernel<3,1"), (100, 64, 7, 9, 3, 3, 2, 1, "direct_conv2d_kernel"),
    (100, 64, 13, 13, 7, 7, 2, 3, "plane_bands_kernel<7,2"), (100, 64, 9, 9, 7, 7, 2, 3, "direct_conv2d_kernel"),
    (4, 16, 33, 33, 3, 3, 4, 1, "direct_conv2d_kernel"), (4, 16, 33, 33, 9, 9, 4, 4, "plane_bands_kernel<0,0"),       # taps in loops
], ids=lambda c: "x".join(map(str, c[:8])))
def test_many_small_planes(torch, sw, oracle, case):
    N, K, H, W, R, S, st, pad, kernel = case
    x = inputs.normal_f32((N, 1, H, W), 6700 + H)
    w = inputs.normal_f32((K, 1, R, S), 6800 + R, 1.0 / R)
    b = inputs.normal_f32((K,), 6900, 0.5)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y_ref, d = oracle.conv2d(x, w, st, pad)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d(xd, wd, st, pad, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), st, pad, True)
    yr, dr = oracle.conv2d_bias_relu(x, w, b, st, pad, True)
    assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")
