"""The fp32 kernels that take each operand as a sum of three bf16 values: parity against the oracle at the edges of their
tiles, channel chunks and window sizes, and the values that no such sum holds (infinities, NaN, the largest and the smallest)."""
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
    # N, C_in, C_out, H, W, R, S, stride, pad, dilation, kernel
    (1, 48, 32, 9, 9, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<41,1,3>"),      # three chunks, tiles of three rows
    (2, 64, 70, 35, 35, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<21,1,1>"),           # ragged channel block
    (3, 53, 77, 23, 41, 3, 3, 2, 1, 1, "mfma_f32_split_kernel<21,1,1>"),           # five of sixteen channels in the last chunk, stride 2
    (1, 57, 33, 12, 12, 3, 3, 1, 0, 1, "mfma_f32_split_kernel<41,1,3>"),           # nine of sixteen: the second octet holds one channel
    (45, 48, 40, 7, 7, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<41,1,4>"),            # row tiles of small images, the last one short
    (4, 48, 64, 6, 6, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<"),            # several whole images per tile where the planner takes them
    (12, 48, 64, 56, 56, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<12,1,6>"),          # large windows
    (12, 48, 96, 56, 56, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<11,1,4>"),          # more tiles than workgroups
    (1, 48, 40, 30, 31, 3, 3, 1, 2, 2, "mfma_f32_split_kernel<21,1,1>"),           # dilation 2
    (1, 64, 64, 40, 40, 3, 3, 2, 3, 3, "mfma_f32_split_kernel<21,1,1>"),           # dilation 3 with stride 2
    (2, 50, 64, 20, 24, 1, 9, 1, 4, 1, "mfma_f32_split_kernel<41,1,1>"),           # a row of nine taps
    (1, 48, 8, 3, 3, 3, 3, 1, 0, 1, "mfma_f32_split_kernel<41,1,1>"),              # a single output pixel
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:10])))
def test_split_window_kernel(torch, sw, oracle, case):
    N, Ci, Co, H, W, R, S, st, pad, dil, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 5100 + Ci)
    w = inputs.normal_f32((Co, Ci, R, S), 5200 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    b = inputs.normal_f32((Co,), 5300, 0.5)
    y_ref, d = oracle.conv2d_dilated(x, w, st, pad, dil)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_dilated(xd, wd, st, pad, dil, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    if dil == 1:
        y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), st, pad, True)
        assert sw.sw_last_kernel().startswith(kernel)
        yr, dr = oracle.conv2d_bias_relu(x, w, b, st, pad, True)
        assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


def _same_but_finite(y, ref, what):
    """Infinities and NaN where the definition has them, nowhere else."""
    assert np.array_equal(np.isnan(y), np.isnan(ref)), what
    inf = np.isinf(ref)
    assert np.array_equal(y[inf], ref[inf]) and not np.isinf(y[~inf]).any(), what


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4028234e38], ids=str)
@pytest.mark.parametrize("where", ["x", "w"])
def test_split_kernel_special_values(torch, sw, value, where):
    """One operand that is no sum of three bf16 values: what it reaches has the value fp32 arithmetic gives, the rest is
    untouched (positive operands, so that no other infinity or NaN can arise)."""
    rng = np.random.default_rng(7)
    x = rng.uniform(0.5, 1.0, (1, 48, 10, 10)).astype(np.float32)
    w = rng.uniform(0.001, 0.002, (32, 48, 3, 3)).astype(np.float32)
    clean = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    (x if where == "x" else w).flat[1234 if where == "x" else 700] = value
    if where == "w":
        x *= 0.125      # (largest value x products stay finite)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    assert sw.sw_last_kernel().startswith("mfma_f32_split_kernel")
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double()).numpy()
    with np.errstate(all="ignore"):
        _same_but_finite(y, ref.astype(np.float32) if not np.isfinite(value) else ref, f"{value} in {where}")
        ok = np.isfinite(ref)
        assert np.max(np.abs(y[ok] - ref[ok]) / np.abs(ref[ok])) <= 2e-5
    if where == "x":
        reached = np.zeros((10, 10), bool)
        reached[(1234 // 10) % 10, 1234 % 10] = True
        i, j = np.argwhere(reached)[0]
        keep = np.ones((8, 8), bool)
        keep[max(0, i - 2):i + 1, max(0, j - 2):j + 1] = False
        assert np.max(np.abs(y[..., keep] - clean[..., keep]) / clean[..., keep]) <= 2e-5


@pytest.mark.parametrize("exponent", [-100, -110, -120, -126])
def test_split_kernel_small_values(torch, sw, oracle, exponent):
    """Inputs whose low parts would leave the bf16 range, under weights that lift the products back: the fp32 bar holds."""
    x = inputs.normal_f32((1, 48, 9, 9), 71).astype(np.float32)
    x = np.where(np.abs(x) < 1.0, np.copysign(np.float32(1.25), x), x) * np.float32(2.0 ** exponent)
    w = inputs.normal_f32((32, 48, 3, 3), 72) * np.float32(2.0 ** 90)
    y_ref, d = oracle.conv2d(x, w, 1, 1)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 1)
    assert sw.sw_last_kernel().startswith("mfma_f32_split_kernel")
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"2^{exponent}")


STEM_CASES = [
    # N, C_in, C_out, H, W, R, S, stride, pad, kernel (steps of two filter rows, output rows per tile)
    (2, 3, 64, 33, 47, 7, 7, 2, 3, "mfma_f32_stem_kernel<11,"),     # odd plane, rows of 24 outputs
    (1, 3, 32, 32, 32, 7, 7, 2, 3, "mfma_f32_stem_kernel<11,"),     # one block of output channels: every wavefront takes it
    (1, 3, 70, 19, 300, 7, 7, 2, 3, "mfma_f32_stem_kernel<11,"),    # two channel groups, the second with six channels; long rows
    (9, 3, 48, 61, 75, 7, 7, 2, 3, "mfma_f32_stem_kernel<11,"),     # a group of 48 channels; the last row tile short
    (40, 3, 64, 56, 56, 7, 7, 2, 3, "mfma_f32_stem_kernel<11,"),    # several tiles per workgroup
    (1, 3, 48, 20, 20, 3, 3, 2, 1, "mfma_f32_stem_kernel<5,"),      # nine row pairs
    (1, 5, 70, 30, 31, 3, 3, 2, 0, "mfma_f32_stem_kernel<8,"),      # fifteen, no padding
    (2, 2, 64, 40, 41, 5, 5, 4, 2, "mfma_f32_stem_kernel<5,"),      # stride 4
    (1, 4, 64, 24, 26, 4, 2, 2, 1, "mfma_f32_stem_kernel<8,"),      # rectangular, even extents
    (1, 2, 64, 12, 40, 11, 8, 2, 4, "mfma_f32_stem_kernel<11,"),    # rows of eight taps, 22 pairs
    (1, 3, 8, 7, 7, 7, 7, 2, 0, "mfma_f32_stem_kernel<11,"),        # a single output pixel
]


@pytest.mark.parametrize("case", STEM_CASES, ids=lambda c: "x".join(map(str, c[:9])))
@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "4-byte"])
def test_few_channels_kernel(torch, sw, oracle, case, shift):
    """Few input channels at an even stride: K along the filter rows.  The input and the filters also from views that are only
    4-byte aligned (the loads are 16 bytes wide), followed by NaN that must not be reached."""
    N, Ci, Co, H, W, R, S, st, pad, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 5400 + H)
    w = inputs.normal_f32((Co, Ci, R, S), 5500 + Co, (2.0 / (Ci * R * S)) ** 0.5)
    b = inputs.normal_f32((Co,), 5600, 0.5)
    y_ref, d = oracle.conv2d(x, w, st, pad)

    def view(a):
        buf = torch.full((a.size + 8,), float("nan"), device="cuda")
        buf[shift:shift + a.size] = torch.from_numpy(a).cuda().reshape(-1)
        return buf[shift:shift + a.size].view(a.shape)

    xd, wd = view(x), view(w)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d(xd, wd, st, pad, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), st, pad, True)
    yr, dr = oracle.conv2d_bias_relu(x, w, b, st, pad, True)
    assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4028234e38, 2.0 ** -120], ids=str)
@pytest.mark.parametrize("where", ["x", "w"])
def test_few_channels_kernel_special_values(torch, sw, value, where):
    rng = np.random.default_rng(8)
    x = rng.uniform(0.5, 1.0, (1, 3, 20, 22)).astype(np.float32)
    w = rng.uniform(0.001, 0.002, (32, 3, 7, 7)).astype(np.float32)
    if value < 1e-30:       # a value whose parts leave the bf16 range, alone under a weight that lifts it back
        (x if where == "x" else w)[:] = 0.0
        (w if where == "x" else x)[:] *= np.float32(2.0 ** 100)
        value = np.float32(value) * np.float32(1.2345678)
    elif where == "w":
        x *= 0.125
    (x if where == "x" else w).flat[633 if where == "x" else 700] = value
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 2, 0).cpu().numpy()
    assert sw.sw_last_kernel().startswith("mfma_f32_stem_kernel")
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=2).numpy()
    with np.errstate(all="ignore"):
        _same_but_finite(y, ref.astype(np.float32) if not np.isfinite(value) else ref, f"{value} in {where}")
        ok = np.isfinite(ref)
        assert np.all(np.abs(y[ok] - ref[ok]) <= 2e-5 * np.abs(ref[ok]))


# N, C_in, C_out, H, W: 1 x 1 layers whose operands are split, one per (channel blocks, pixels per lane) and remainder
POINTWISE_CASES = [(2, 64, 100, 28, 28), (32, 48, 64, 56, 56), (32, 152, 40, 30, 32), (30, 64, 128, 33, 34), (1, 136, 7, 9, 10),
                   (8, 256, 64, 40, 40), (3, 384, 33, 12, 12), (40, 512, 512, 8, 8)]


@pytest.mark.parametrize("case", POINTWISE_CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_pointwise(torch, sw, oracle, case):
    N, Ci, Co, H, W = case
    x = inputs.normal_f32((N, Ci, H, W), 5700 + Ci)
    w = inputs.normal_f32((Co, Ci, 1, 1), 5800 + Co, (2.0 / Ci) ** 0.5)
    b = inputs.normal_f32((Co,), 5900, 0.5)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y_ref, d = oracle.conv2d(x, w, 1, 0)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d(xd, wd, 1, 0, out=out)
    assert sw.sw_last_kernel().startswith("mfma_f32_pointwise_kernel"), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), 1, 0, True)
    yr, dr = oracle.conv2d_bias_relu(x, w, b, 1, 0, True)
    assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4028234e38, 2.0 ** -120], ids=str)
@pytest.mark.parametrize("where", ["x", "w"])
def test_split_pointwise_special_values(torch, sw, value, where):
    rng = np.random.default_rng(9)
    x = rng.uniform(0.5, 1.0, (1, 136, 9, 10)).astype(np.float32)
    w = rng.uniform(0.001, 0.002, (40, 136, 1, 1)).astype(np.float32)
    if value < 1e-30:
        (x if where == "x" else w)[:] = 0.0
        (w if where == "x" else x)[:] *= np.float32(2.0 ** 100)
        value = np.float32(value) * np.float32(1.2345678)
    elif where == "w":
        x *= 0.125
    (x if where == "x" else w).flat[7777 if where == "x" else 700] = value
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    assert sw.sw_last_kernel().startswith("mfma_f32_pointwise_kernel")
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double()).numpy()
    with np.errstate(all="ignore"):
        _same_but_finite(y, ref.astype(np.float32) if not np.isfinite(value) else ref, f"{value} in {where}")
        ok = np.isfinite(ref)
        assert np.all(np.abs(y[ok] - ref[ok]) <= 2e-5 * np.abs(ref[ok]))
