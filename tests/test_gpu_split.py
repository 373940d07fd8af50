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
    (4, 48, 64, 6, 6, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<41,1,2>"),             # row tiles of small images
    (65, 48, 128, 6, 6, 3, 3, 1, 1, 1, "mfma_f32_split_kernel<21,2,6>"),           # two whole images per tile, the last one single
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


@pytest.mark.parametrize("case", [
    (22, 88, 24, 47, 54, 2, "mfma_f32_split_kernel<12,1,5>"),       # 9 blocks: one wavefront has two; the last tile's two rows leave wavefronts without any
    (24, 64, 64, 33, 40, 1, "mfma_f32_split_kernel<12,1,9>"),       # 12 blocks; 8 in the last tile, one each
    (32, 96, 96, 28, 28, 1, "mfma_f32_split_kernel<12,1,14>"),      # 13 blocks, the last of 8 pixels
], ids=lambda c: "x".join(map(str, c[:6])))
def test_tiles_of_uneven_blocks(torch, sw, oracle, case):
    """Tiles whose wavefronts multiply two pixel blocks, one or none."""
    N, Ci, Co, H, W, dil, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 5150 + Ci)
    w = inputs.normal_f32((Co, Ci, 3, 3), 5250 + Co, (2.0 / (Ci * 9)) ** 0.5)
    y_ref, d = oracle.conv2d_dilated(x, w, 1, dil, dil)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d_dilated(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, dil, dil, out=out)
    assert sw.sw_last_kernel() == kernel, sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)


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


# N, C_in, C_out, H, W: 1 x 1 layers, one per (channel blocks, pixels per lane) and remainder
POINTWISE_CASES = [(2, 64, 100, 28, 28, "mfma_f32_pointwise_kernel<1,2>"), (2, 200, 100, 28, 28, "mfma_f32_pointwise_split_kernel<1,2>"),
                   (32, 48, 64, 56, 56, "mfma_f32_pointwise_split_kernel<2,4>"), (16, 32, 256, 28, 28, "mfma_f32_pointwise_split_kernel<1,4>"),
                   (32, 152, 40, 30, 32, "mfma_f32_pointwise_split_kernel<1,2>"), (30, 64, 128, 33, 34, "mfma_f32_pointwise_split_kernel<2,2>"),
                   (1, 136, 7, 9, 10, "mfma_f32_pointwise_kernel<1,2>"), (1, 200, 7, 9, 10, "mfma_f32_pointwise_split_kernel<1,2>"),
                   (8, 256, 64, 40, 40, "mfma_f32_pointwise_kernel<1,2>"), (3, 384, 33, 12, 12, "mfma_f32_pointwise_split_kernel<1,2>"),
                   (40, 512, 512, 8, 8, "mfma_f32_pointwise_split_kernel<1,2>"),
                   # more tiles of <2,4> than run at once, and more than two rounds of them
                   (16, 64, 192, 56, 56, "mfma_f32_pointwise_kernel<2,4>"), (22, 64, 256, 56, 56, "mfma_f32_pointwise_split_kernel<2,4>")]


@pytest.mark.parametrize("case", POINTWISE_CASES, ids=lambda c: "x".join(map(str, c[:5])))
def test_split_pointwise(torch, sw, oracle, case):
    N, Ci, Co, H, W, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 5700 + Ci)
    w = inputs.normal_f32((Co, Ci, 1, 1), 5800 + Co, (2.0 / Ci) ** 0.5)
    b = inputs.normal_f32((Co,), 5900, 0.5)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y_ref, d = oracle.conv2d(x, w, 1, 0)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d(xd, wd, 1, 0, out=out)
    assert sw.sw_last_kernel() == kernel
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)
    y = sw.sw_conv2d_bias_relu(xd, wd, torch.from_numpy(b).cuda(), 1, 0, True)
    yr, dr = oracle.conv2d_bias_relu(x, w, b, 1, 0, True)
    assert_f32_parity(y.cpu().numpy(), yr, np.maximum(dr, 1e-30), f"{case} bias, rectifier")


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4028234e38, 2.0 ** -120], ids=str)
@pytest.mark.parametrize("where", ["x", "w"])
def test_split_pointwise_special_values(torch, sw, value, where):
    rng = np.random.default_rng(9)
    x = rng.uniform(0.5, 1.0, (1, 200, 9, 10)).astype(np.float32)
    w = rng.uniform(0.001, 0.002, (40, 200, 1, 1)).astype(np.float32)
    if value < 1e-30:
        (x if where == "x" else w)[:] = 0.0
        (w if where == "x" else x)[:] *= np.float32(2.0 ** 100)
        value = np.float32(value) * np.float32(1.2345678)
    elif where == "w":
        x *= 0.125
    (x if where == "x" else w).flat[7777 if where == "x" else 700] = value
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    assert sw.sw_last_kernel().startswith("mfma_f32_pointwise_split_kernel")
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double()).numpy()
    with np.errstate(all="ignore"):
        _same_but_finite(y, ref.astype(np.float32) if not np.isfinite(value) else ref, f"{value} in {where}")
        ok = np.isfinite(ref)
        assert np.all(np.abs(y[ok] - ref[ok]) <= 2e-5 * np.abs(ref[ok]))


# One launch of every variant of the split kernels, most of them with several tiles per workgroup:
# N, C_in, C_out, H, W, R, stride, pad, kernel
LAUNCHES = [
    (12, 48, 96, 56, 56, 3, 1, 1, "mfma_f32_split_kernel<11,1,4>"),     # 504 tiles
    (129, 48, 512, 8, 8, 3, 1, 1, "mfma_f32_split_kernel<12,5,8>"),     # 416 tiles of five images, the last of four
    (130, 48, 512, 6, 6, 3, 1, 1, "mfma_f32_split_kernel<21,3,6>"),     # 704 tiles of three images, the last of one
    (201, 64, 64, 3, 3, 3, 1, 1, "mfma_f32_split_kernel<41,2,3>"),      # 202 tiles of two images, one per workgroup
    (40, 3, 64, 56, 56, 7, 2, 3, "mfma_f32_stem_kernel<11,"),
    (64, 5, 48, 56, 56, 3, 2, 1, "mfma_f32_stem_kernel<8,"),
    (64, 2, 96, 56, 56, 5, 2, 2, "mfma_f32_stem_kernel<5,"),
    (32, 64, 64, 56, 56, 1, 1, 0, "mfma_f32_pointwise_split_kernel<2,4>"),
    (32, 128, 128, 28, 28, 1, 1, 0, "mfma_f32_pointwise_split_kernel<1,4>"),
    (40, 64, 128, 33, 34, 1, 1, 0, "mfma_f32_pointwise_split_kernel<2,2>"),
    (2, 200, 40, 9, 10, 1, 1, 0, "mfma_f32_pointwise_split_kernel<1,2>"),
]
launches = pytest.mark.parametrize("case", LAUNCHES, ids=lambda c: "x".join(map(str, c[:8])))


@launches
def test_several_images_and_tiles(torch, sw, oracle, case):
    N, Ci, Co, H, W, R, st, pad, kernel = case
    x = inputs.normal_f32((N, Ci, H, W), 6700 + Ci)
    w = inputs.normal_f32((Co, Ci, R, R), 6800 + Co, (2.0 / (Ci * R * R)) ** 0.5)
    y_ref, d = oracle.conv2d(x, w, st, pad)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), st, pad, out=out)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, str(case))
    assert_guards_intact(buf, front, n, guard)


@launches
def test_one_small_value_changes_nothing(torch, sw, case):
    """A weight or an input far too small to show in any result (denormal, or just above) in the first filter and in the last
    image: every output has the bits it has with a zero in its place.  (An output computed any other way would not.)"""
    N, Ci, Co, H, W, R, st, pad, kernel = case
    g = torch.Generator(device="cuda").manual_seed(41)
    x = torch.randn(N, Ci, H, W, generator=g, device="cuda")
    w = torch.randn(Co, Ci, R, R, generator=g, device="cuda")
    w[0, Ci - 1, 0, 0] = 0.0
    x[N - 1, Ci - 1, H // 2, W // 2] = 0.0
    clean = sw.sw_conv2d(x, w, st, pad)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    for small in (1e-38, -3e-32, 1e-42):
        w[0, Ci - 1, 0, 0] = small
        assert torch.equal(sw.sw_conv2d(x, w, st, pad), clean), f"weight {small}"
        w[0, Ci - 1, 0, 0] = 0.0
        x[N - 1, Ci - 1, H // 2, W // 2] = small
        assert torch.equal(sw.sw_conv2d(x, w, st, pad), clean), f"input {small}"
        x[N - 1, Ci - 1, H // 2, W // 2] = 0.0


@launches
def test_powers_of_two_pass_through(torch, sw, case):
    """Inputs times 2^-142 (denormal: the last bits of the smallest fp32 values) under weights times 2^100, and the other way
    round: the same bits as without the factors, because a factor of 2 changes no rounding."""
    N, Ci, Co, H, W, R, st, pad, kernel = case
    g = torch.Generator(device="cuda").manual_seed(42)
    a = torch.randint(-1000, 1001, (N, Ci, H, W), generator=g, device="cuda").float() / 128     # whole multiples of 2^-7
    b = torch.randn(Co, Ci, R, R, generator=g, device="cuda").clamp_(-6, 6)
    plain = sw.sw_conv2d(a, b, st, pad)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    small = (a.double() * 2.0 ** -142).float()
    assert torch.equal((small.double() * 2.0 ** 142).float(), a)
    y = sw.sw_conv2d(small, b * 2.0 ** 100, st, pad)
    assert torch.equal(y * 2.0 ** 42, plain)
    a, b = a.clamp_(-6, 6) / 8, (torch.randint(-1000, 1001, b.shape, generator=g, device="cuda").float() / 128)
    plain = sw.sw_conv2d(a, b, st, pad)
    y = sw.sw_conv2d(a * 2.0 ** 100, (b.double() * 2.0 ** -142).float(), st, pad)
    assert torch.equal(y * 2.0 ** 42, plain)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4028234e38, 1e32], ids=str)
@launches
def test_one_special_value(torch, sw, case, value):
    """One operand that the scaled sums do not hold, in the last image or in one filter: what it reaches has the value fp32
    arithmetic gives, everything else the bits it has without it.  Positive operands: no other infinity or NaN can arise."""
    N, Ci, Co, H, W, R, st, pad, kernel = case
    g = torch.Generator(device="cuda").manual_seed(43)
    x = torch.rand(N, Ci, H, W, generator=g, device="cuda") * 0.1 + 0.1
    w = torch.rand(Co, Ci, R, R, generator=g, device="cuda") * 0.001 + 0.001
    clean = sw.sw_conv2d(x, w, st, pad)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()

    def check(xv, wv, reached, images, channels, what):
        y = sw.sw_conv2d(xv, wv, st, pad)
        ref = torch.nn.functional.conv2d(xv[images].double().cpu(), wv[channels].double().cpu(), stride=st, padding=pad)
        got = y[images][:, channels].cpu()
        with np.errstate(all="ignore"):
            _same_but_finite(got.numpy(), ref.float().numpy() if not np.isfinite(value) else ref.numpy(), what)
        ok = torch.isfinite(ref)
        # plain multiply-adds one after the other: a rounding of 2^-24 of a partial sum each, all terms positive
        assert torch.all((got.double() - ref).abs()[ok] <= Ci * R * R * 2.0 ** -24 * ref.abs()[ok]), what
        assert torch.equal(y[~reached], clean[~reached]), f"{what}: outputs that it does not reach"

    i, j = H // 2, W // 2
    xv = x.clone()
    xv[N - 1, Ci - 1, i, j] = value
    reached = torch.zeros_like(clean, dtype=torch.bool)
    for r in range(R):
        for s in range(R):
            p, q = i + pad - r, j + pad - s
            if p % st == 0 and q % st == 0 and 0 <= p // st < clean.shape[2] and 0 <= q // st < clean.shape[3]:
                reached[N - 1, :, p // st, q // st] = True
    # (a window's cells beyond a filter's last tap meet zero weights: outputs beside the reached ones are computed again too)
    if kernel.startswith("mfma_f32_stem"):
        reached[N - 1] = True
    check(xv, w, reached, slice(N - 1, N), slice(0, Co), f"{value} in x")
    wv = w.clone()
    wv[Co // 2, Ci - 1, R // 2, R // 2] = value
    reached = torch.zeros_like(clean, dtype=torch.bool)
    reached[:, Co // 2] = True
    # (a lane's sixteen output channels are computed again together)
    block = Co // 2 // 32 * 32
    reached[:, block:block + 32] = True
    check(x, wv, reached, slice(0, min(N, 2)), slice(Co // 2, Co // 2 + 1), f"{value} in w")


@launches
def test_left_out_products(torch, sw, case):
    """Operands of 1 + 2^-8 - 2^-17 throughout: of a product, what the six bf16 products leave out is 2^-24.01, its largest, and
    has one sign (2^-24 of the result).  The parts are powers of two, their sums whole multiples of 2^-17: what else is rounded is the
    result (2^-24)."""
    N, Ci, Co, H, W, R, st, pad, kernel = case
    v = 1.0 + 2.0 ** -8 - 2.0 ** -17
    x = torch.full((N, Ci, H, W), v, device="cuda")
    w = torch.full((Co, Ci, R, R), v, device="cuda")
    y = sw.sw_conv2d(x, w, st, pad).double().cpu()
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    taps = torch.nn.functional.conv2d(torch.ones(1, Ci, H, W, dtype=torch.float64), torch.ones(1, Ci, R, R, dtype=torch.float64), stride=st, padding=pad)
    ref = taps * (v * v)
    assert torch.all((y - ref).abs() <= 2.0 ** -23 * ref)


@pytest.mark.parametrize("case", [(40, 152, 160, 25, 25, 1, "pointwise_split"), (1648, 40, 442, 3, 3, 1, "pointwise_split"), (12, 9, 104, 40, 44, 3, "split"),
                                  (1, 16, 64, 60, 60, 3, "split"), (5, 32, 200, 19, 23, 3, "split")], ids=lambda c: "x".join(str(v) for v in c[:6]))
def test_sums_of_a_single_product(torch, sw, case):
    """One weight per output channel: every output is one product.  2^-24 of it may be left out, and of the five additions of its six parts three meet
    the full magnitude at most, 2^-24 each."""
    N, C, K, H, W, R, kernel = case
    rng = np.random.default_rng(4100 + C)
    x = inputs.normal_f32((N, C, H, W), 4101) * np.float32(2.0) ** rng.integers(-30, 30, (N, C, 1, 1)).astype(np.float32)
    w = np.zeros((K, C, R, R), np.float32)
    ci, r, s = rng.integers(0, C, K), rng.integers(0, R, K), rng.integers(0, R, K)
    v = inputs.normal_f32((K,), 4102)
    w[np.arange(K), ci, r, s] = v
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, R // 2).cpu().numpy()
    assert sw.sw_last_kernel().startswith(f"mfma_f32_{kernel}_kernel"), sw.sw_last_kernel()
    xp = np.pad(x, ((0, 0), (0, 0), (R // 2, R // 2), (R // 2, R // 2)))
    for k in range(K):
        ref = xp[:, ci[k], r[k]:r[k] + H, s[k]:s[k] + W].astype(np.float64) * np.float64(v[k])
        err = np.abs(y[:, k] - ref)
        assert np.all(err <= 4 * 2.0 ** -24 * np.abs(ref)), (k, float(np.max(err / np.maximum(np.abs(ref), 1e-300))))
