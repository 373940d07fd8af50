"""The fp32 kernel of launches with few tiles: its reduction split over wavefronts, at the edges of its runs of 32 products, pixel
tiles, channel blocks and chunks of channels, against the oracle."""
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
    # N, C_in, C_out, H, W, R, S, stride, pad, dilation
    (1, 256, 256, 14, 14, 3, 3, 1, 1, 1),       # whole runs, rows of 14 pixels
    (2, 67, 19, 9, 11, 3, 3, 1, 1, 1),          # 603 products: 27 beyond the last run, filters off the 16-byte grid, ragged channel block
    (1, 65, 16, 3, 3, 3, 3, 1, 0, 1),           # a single output pixel
    (3, 96, 33, 17, 23, 3, 3, 2, 1, 1),         # stride 2
    (1, 80, 24, 20, 20, 3, 3, 1, 2, 2),         # dilation 2
    (1, 72, 40, 5, 90, 3, 3, 1, 0, 1),          # rows wider than a tile
    (2, 70, 50, 7, 9, 1, 1, 1, 0, 1),           # one tap, several channels a load, 70 products
    (4, 128, 130, 13, 13, 1, 1, 2, 0, 1),       # one tap at stride 2
    (1, 320, 280, 18, 18, 1, 1, 1, 0, 1),       # one tap in place of the pointwise kernel
    (2, 68, 36, 12, 12, 2, 2, 1, 0, 1),         # four taps
    (3, 21, 48, 15, 15, 5, 5, 1, 2, 1),         # 25 taps over few channels
    (1, 130, 24, 21, 18, 5, 5, 2, 2, 1),        # 25 taps at stride 2
    (1, 300, 20, 11, 30, 7, 7, 1, 3, 1),        # 49 taps: two loads a channel, all channels in 138 KB
    (2, 24, 17, 14, 14, 7, 5, 3, 2, 1),         # rectangular, stride 3
    (1, 70, 18, 16, 16, 1, 7, 1, 3, 1),         # a row of seven taps
    (2, 130, 64, 40, 42, 5, 5, 1, 2, 1),        # several workgroups per CU
]


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "4-byte"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_few_tiles_kernel(torch, sw, oracle, case, shift):
    N, Ci, Co, H, W, R, S, st, pad, dil = case
    if shift and R * S == 1 and st == 1 and Ci == 320:
        pytest.skip("the same route as the other single taps")
    x = inputs.normal_f32((N, Ci, H, W), 8100 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 8200 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    b = inputs.normal_f32((Co,), 8300, 0.5)

    def view(a):        # four bytes off the 16-byte grid, NaN around
        buf = torch.full((a.size + 8,), float("nan"), device="cuda")
        buf[shift:shift + a.size] = torch.from_numpy(a).cuda().reshape(-1)
        return buf[shift:shift + a.size].view(a.shape)

    xd, wd = view(x), view(w)
    y_ref, d = oracle.conv2d_dilated(x, w, st, pad, dil)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_dilated(xd, wd, st, pad, dil, out=out)
    assert sw.sw_last_kernel().startswith("mfma_f32_few_kernel"), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    if dil == 1:
        y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), st, pad, True)
        yr, dr = oracle.conv2d_bias_relu(x, w, b, st, pad, True)
        assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


@pytest.mark.parametrize("case,plan", [
    # wavefronts, those that share a tile's products, tiles of 16 pixels, chunks of channels
    ((1, 256, 64, 14, 14, 7, 7, 2, 3, 1), "8,8,1,2"), ((6, 302, 9, 14, 4, 5, 5, 2, 2, 1), "8,8,1,2"),       # whole runs to the end of the last chunk; 30 products over
    ((7, 283, 5, 29, 34, 7, 7, 1, 3, 1), "8,4,2,2"), ((5, 259, 36, 17, 59, 5, 5, 1, 2, 1), "8,2,4,3"), ((7, 176, 48, 35, 35, 5, 5, 1, 2, 1), "8,1,8,2"),
    ((5, 69, 97, 13, 57, 2, 2, 1, 1, 1), "4,1,1,1"), ((4, 82, 76, 22, 59, 2, 2, 1, 1, 1), "4,1,2,1"), ((8, 74, 48, 20, 31, 2, 2, 1, 1, 1), "4,2,2,1"),
    ((3, 80, 12, 28, 60, 2, 2, 1, 1, 1), "4,4,1,1"), ((5, 76, 100, 32, 21, 2, 2, 1, 1, 1), "8,1,1,1"), ((5, 83, 174, 9, 45, 2, 2, 1, 1, 1), "8,1,2,1"),
    ((9, 85, 20, 40, 40, 2, 2, 1, 1, 1), "8,1,4,1"), ((7, 94, 141, 35, 12, 2, 2, 1, 1, 1), "8,1,8,1"), ((4, 67, 96, 38, 13, 2, 2, 1, 1, 1), "8,2,2,1"),
    ((9, 199, 108, 12, 16, 2, 2, 1, 1, 1), "8,2,4,1"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_few_tiles_plans(torch, sw, oracle, case, plan):
    """Every form of a plan: tiles whose products one wavefront adds up, several pixel tiles and channel tiles a workgroup, a window that
    comes in chunks of channels, the last of which ends in a partial run."""
    N, Ci, Co, H, W, R, S, st, pad, dil = case
    x = inputs.normal_f32((N, Ci, H, W), 8400 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 8500 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    y_ref, d = oracle.conv2d_dilated(x, w, st, pad, dil)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_dilated(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), st, pad, dil, out=out)
    assert sw.sw_last_kernel() == f"mfma_f32_few_kernel<{plan}>"
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("shape", [(2, 67, 19, 9, 11, 3), (2, 70, 50, 7, 9, 1), (2, 21, 48, 15, 15, 5)], ids=lambda s: "x".join(map(str, s)))
def test_few_tiles_kernel_keeps_special_values_in_place(torch, sw, shape, value):
    """A value that is not finite in the first weight of the second filter, or in the first channel of the second image: the loads that
    reach over the end of a filter or of an image's channels do not carry it into the sums before it."""
    N, Ci, Co, H, W, R = shape
    rng = np.random.default_rng(83)
    x = rng.uniform(0.5, 1.0, (N, Ci, H, W)).astype(np.float32)
    w = rng.uniform(0.5, 1.0, (Co, Ci, R, R)).astype(np.float32)
    run = lambda x, w: sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    clean = run(x, w)
    assert sw.sw_last_kernel().startswith("mfma_f32_few_kernel"), sw.sw_last_kernel()
    w2 = w.copy()
    w2[1, 0, 0, 0] = value
    y = run(x, w2)
    assert not np.isfinite(y[:, 1]).any() and np.array_equal(np.delete(y, 1, 1), np.delete(clean, 1, 1))
    x2 = x.copy()
    x2[1, 0] = value
    y = run(x2, w)
    assert not np.isfinite(y[1]).any() and np.array_equal(y[0], clean[0])


@pytest.mark.parametrize("case,takes", [
    ((1, 2, 40, 90, 100, 5, 5, 1, 2), True), ((9, 2, 51, 60, 31, 5, 5, 1, 2), False), ((3, 5, 34, 60, 71, 5, 5, 1, 0), True), ((8, 5, 34, 70, 71, 7, 7, 1, 3), False),
    ((2, 2, 24, 91, 171, 6, 6, 1, 0), True), ((2, 2, 24, 198, 329, 6, 6, 1, 0), False), ((2, 2, 16, 198, 229, 6, 6, 1, 0), True), ((8, 9, 34, 70, 71, 7, 7, 1, 3), True),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_large_filters_over_few_channels(torch, sw, oracle, case, takes):
    """Short sums in launches that fill the chip: the any-shape kernel, with the same result."""
    N, Ci, Co, H, W, R, S, st, pad = case
    x = inputs.normal_f32((N, Ci, H, W), 8600 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 8700 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    y_ref, d = oracle.conv2d(x, w, st, pad)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), st, pad)
    assert sw.sw_last_kernel().startswith("mfma_f32_few_kernel" if takes else "mfma_f32_any_kernel"), sw.sw_last_kernel()
    assert_f32_parity(y.cpu().numpy(), y_ref, d, str(case))
