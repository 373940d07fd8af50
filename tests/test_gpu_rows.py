"""The register-only rows kernel at the edges of its strips, bands and lane groups: pooling over rows of any width that begin at any
4-byte address, filters over planes whose rows and columns end inside a band."""
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


def within_nan(torch, a, shift):
    """`a` on the GPU, `shift` floats off the 16-byte grid, between NaN that must not be reached."""
    buf = torch.full((a.size + 12,), float("nan"), device="cuda")
    buf[4 + shift:4 + shift + a.size] = torch.from_numpy(a).cuda().reshape(-1)
    return buf[4 + shift:4 + shift + a.size].view(a.shape)


POOL_CASES = [
    # N, C, H, W, R, stride, pad: lane groups of 8 up to 31 columns, 16 up to 63, 32 up to 127, strips beyond, the second from 257
    (3, 7, 5, 7, 3, 2, 1), (1, 5, 9, 9, 3, 1, 1), (2, 9, 7, 31, 3, 2, 1), (1, 3, 6, 32, 3, 2, 1), (2, 3, 8, 33, 2, 2, 0), (1, 4, 11, 63, 3, 1, 0),
    (1, 2, 13, 65, 3, 2, 0), (2, 2, 10, 79, 3, 2, 1), (1, 3, 9, 127, 3, 1, 1), (1, 2, 4, 129, 3, 2, 1), (1, 2, 7, 254, 3, 1, 1), (1, 2, 6, 255, 3, 2, 0),
    (1, 1, 5, 257, 3, 1, 1), (1, 2, 8, 505, 3, 2, 1), (1, 1, 3, 502, 2, 2, 0), (2, 1, 1, 10, 3, 1, 1), (1, 1, 2, 1001, 3, 2, 1),
]


@pytest.mark.parametrize("shift", [0, 1, 3], ids=["aligned", "4-byte", "12-byte"])
@pytest.mark.parametrize("mode", [0, 1], ids=["avg", "max"])
@pytest.mark.parametrize("case", POOL_CASES, ids=lambda c: "x".join(map(str, c)))
def test_pool_any_width(torch, sw, oracle, case, mode, shift):
    N, C, H, W, R, stride, pad = case
    x = inputs.normal_f32((N, C, H, W), 6100 + W) - np.float32(3.0 * mode)      # (mostly negative: padding must not win)
    y_ref, d = oracle.pool2d(x, R, R, stride, pad, mode)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_pool2d(within_nan(torch, x, shift), R, R, stride, pad, mode, out=out)
    assert sw.sw_last_kernel().startswith(f"sliding_rows_kernel<{R},{R},{pad},"), sw.sw_last_kernel()
    y = out.cpu().numpy()
    if mode == 1:
        assert np.array_equal(y.astype(np.float64), y_ref)
    else:
        assert_f32_parity(y, y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)


@pytest.mark.parametrize("case", [
    # H, W, R, stride, pad
    (1, 8, 3, 1, 1), (2, 260, 3, 1, 1), (5, 256, 5, 1, 0), (6, 252, 7, 1, 3), (9, 508, 5, 2, 2), (7, 64, 7, 2, 3), (3, 32, 3, 2, 0), (8, 28, 3, 1, 0),
], ids=lambda c: "x".join(map(str, c)))
def test_filters_at_the_edges_of_bands(torch, sw, oracle, case):
    """One channel under one and under three filters: rows above and below the image, columns beside it, NaN around the tensor."""
    H, W, R, stride, pad = case
    x = inputs.normal_f32((2, 1, H, W), 6200 + W)
    for K in (1, 3):
        w = inputs.normal_f32((K, 1, R, R), 6300 + R)
        y_ref, d = oracle.conv2d(x, w, stride, pad)
        buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
        sw.sw_conv2d(within_nan(torch, x, 0), torch.from_numpy(w).cuda(), stride, pad, out=out)
        assert sw.sw_last_kernel().startswith("sliding_rows_kernel"), sw.sw_last_kernel()
        assert_f32_parity(out.cpu().numpy(), y_ref, d, f"{case} {K}")
        assert_guards_intact(buf, front, n, guard)


@pytest.mark.parametrize("case", [
    # N, C, H, W, R, stride, pad, kernel: on both sides of the lines between the rows kernel, small planes and whole planes
    (2, 35, 9, 8, 3, 1, 1, "small_planes_kernel<3,3,1>"), (2, 35, 9, 12, 3, 1, 1, "sliding_rows_kernel<3,3,1,"),
    (8, 64, 11, 12, 5, 1, 2, "small_planes_kernel<5,5,1>"), (27, 19, 11, 12, 5, 1, 2, "sliding_rows_kernel<5,5,2,"),        # 512, 513 planes
    (27, 19, 14, 28, 7, 1, 3, "sliding_rows_kernel<7,7,3,"), (2, 50, 4, 4, 3, 2, 1, "sliding_rows_kernel<3,3,1,"),
    (3, 41, 13, 16, 5, 2, 2, "sliding_rows_kernel<5,5,2,"), (3, 41, 8, 8, 7, 2, 3, "sliding_rows_kernel<7,7,3,"),
    (16, 64, 56, 56, 3, 1, 1, "sliding_rows_kernel<3,3,1,"), (25, 41, 56, 56, 3, 1, 1, "sliding_plane_full_kernel<3,3,1,0>"),        # 1024, 1025
    (25, 41, 55, 56, 5, 1, 2, "sliding_rows_kernel<5,5,2,"),
], ids=lambda c: "x".join(map(str, c[:7])))
def test_depthwise_routes(torch, sw, oracle, case):
    N, C, H, W, R, stride, pad, kernel = case
    x, w = inputs.normal_f32((N, C, H, W), 6400 + W), inputs.normal_f32((C, 1, R, R), 6500 + R)
    b = inputs.normal_f32((C,), 6600, 0.5)
    y_ref, d = oracle.conv2d_depthwise(x, w, stride, pad)
    xd, wd, bd = (torch.from_numpy(a).cuda() for a in (x, w, b))
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_depthwise(xd, wd, stride, pad, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_depthwise_bias_relu(xd, wd, bd, stride, pad, True)
    z = torch.clamp(out + bd.view(1, -1, 1, 1), min=0)      # (one rounding on the same sum either way)
    assert torch.equal(y, z)


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "4-byte"])
@pytest.mark.parametrize("W,filt", [
    (W, f) for W in (9, 13, 29, 30, 31, 32, 61, 62, 63, 125, 126, 127, 129, 254, 257)
    for f in ((3, 1, 0), (3, 1, 1), (3, 2, 1), (5, 1, 2), (5, 2, 1), (7, 1, 3), (7, 2, 3), (7, 2, 1)) if W < 200 or f[0] < 7
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_depthwise_any_width(torch, sw, oracle, W, filt, shift):
    """Rows off the 16-byte grid: lane groups whose last columns are the next plane's padding, strips, the tensor's last row."""
    R, stride, pad = filt
    N, C, H = 2, 520, 3 if W > 200 else 7
    x, w = inputs.normal_f32((N, C, H, W), 6700 + W), inputs.normal_f32((C, 1, R, R), 6800 + R)
    y_ref, d = oracle.conv2d_depthwise(x, w, stride, pad)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_depthwise(within_nan(torch, x, shift), torch.from_numpy(w).cuda(), stride, pad, out=out)
    assert sw.sw_last_kernel().startswith(f"sliding_rows_kernel<{R},{R},{pad},"), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, f"{W} {filt}")
    assert_guards_intact(buf, front, n, guard)
