"""The int8 channel-first kernel that turns its operands in registers: bit-exact against the oracle at the edges of its column quads,
pixel tiles, channel groups and units, with int32 sums and requantised."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs
from parity import assert_guards_intact, guarded_empty

pytestmark = pytest.mark.gpu

CASES = [
    # N, C_in, C_out, H, W, R, S, stride, pad
    (2, 352, 208, 10, 10, 3, 3, 1, 1),      # units shared by the wavefronts, the last unit with two groups
    (1, 16, 24, 7, 4, 3, 3, 1, 1),          # rows of one quad, a single channel group
    (3, 48, 17, 9, 5, 3, 3, 1, 0),          # rows of five columns: the second quad overlaps the first; ragged channel block
    (2, 80, 33, 14, 53, 3, 3, 2, 1),        # stride 2 on odd columns
    (1, 64, 16, 3, 6, 3, 3, 1, 0),          # a single output row
    (4, 112, 48, 21, 37, 3, 3, 1, 2),       # wide padding, column tiles that end inside a quad
    (5, 176, 112, 7, 101, 1, 1, 1, 0),      # one tap
    (3, 272, 40, 13, 11, 1, 1, 2, 0),       # one tap at stride 2, five units
    (2, 32, 70, 40, 40, 3, 3, 1, 1),
    (1, 48, 32, 20, 9, 9, 1, 1, 4),         # nine taps in a column
    (9, 128, 160, 30, 30, 3, 3, 2, 1),      # several workgroups per CU, filters shared by pixel tiles
]


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "off the grid"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_s8_tiles(oracle, case, shift):
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, Ci, Co, H, W, R, S, st, pad = case
    x = inputs.uniform_s8((N, Ci, H, W), 9100 + Ci)
    w = inputs.uniform_s8((Co, Ci, R, S), 9200 + Co)

    def view(a, by):        # x one byte, w four bytes off the 16-byte grid
        buf = torch.full((a.size + 32,), 99, dtype=torch.int8, device="cuda")
        buf[by:by + a.size] = torch.from_numpy(a).cuda().reshape(-1)
        return buf[by:by + a.size].view(a.shape)

    xd, wd = view(x, shift), view(w, 4 * shift)
    y_ref = oracle.conv2d_s8(x, w, st, pad)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.int32)
    sw.sw_conv2d_s8(xd, wd, st, pad, out=out)
    assert sw.sw_last_kernel().startswith("mfma_s8_tiles_kernel"), sw.sw_last_kernel()
    assert np.array_equal(out.cpu().numpy(), y_ref)
    assert_guards_intact(buf, front, n, guard)

    rng = np.random.default_rng(9300)
    bias = rng.integers(-20000, 20000, Co).astype(np.int32)
    std = (Ci * R * S) ** 0.5 * 5461.0
    scale = (rng.uniform(0.5, 2.0, Co) * 40.0 / std).astype(np.float32)
    scale[::3] = np.float32(2.0 ** np.round(np.log2(40.0 / std)))      # powers of two produce exact ties
    scale[1::5] *= np.float32(-1.0)
    for b, relu in ((bias, False), (None, True)):
        q_ref = oracle.conv2d_s8_requant(x, w, b, scale, st, pad, relu)
        buf, out, front, n, guard = guarded_empty(torch, q_ref.shape, torch.int8, fill=77)
        sw.sw_conv2d_s8_requant(xd, wd, None if b is None else torch.from_numpy(b).cuda(), torch.from_numpy(scale).cuda(), st, pad, relu, out=out)
        assert sw.sw_last_kernel().startswith("mfma_s8_tiles_kernel"), sw.sw_last_kernel()
        assert np.array_equal(out.cpu().numpy(), q_ref)
        assert_guards_intact(buf, front, n, guard)


@pytest.mark.parametrize("case,plan", [
    # taps, wavefronts that share a tile's units, tiles of 16 channels, tiles of 16 pixels per wavefront; ragged channels, tiles partly beyond
    ((7, 16, 151, 17, 53, 3, 3, 1, 1), "9,1,8,4"), ((5, 16, 153, 38, 34, 3, 3, 1, 1), "9,1,4,4"), ((9, 80, 68, 26, 26, 3, 3, 1, 1), "9,2,4,4"),
    ((9, 80, 24, 39, 43, 3, 3, 1, 1), "9,2,2,4"), ((5, 160, 18, 37, 48, 3, 3, 1, 1), "9,4,2,4"), ((8, 272, 5, 35, 31, 3, 3, 1, 1), "9,8,1,4"),
    ((8, 16, 110, 32, 17, 3, 3, 1, 1), "9,1,8,2"), ((8, 80, 21, 33, 34, 3, 3, 1, 1), "9,2,2,2"), ((2, 144, 17, 34, 60, 3, 3, 1, 1), "9,4,2,2"),
    ((5, 304, 5, 34, 29, 3, 3, 1, 1), "9,8,1,2"), ((4, 48, 158, 29, 55, 1, 1, 1, 0), "1,1,8,4"), ((9, 48, 134, 34, 26, 1, 1, 1, 0), "1,1,4,4"),
    ((6, 96, 132, 31, 59, 1, 1, 1, 0), "1,1,2,4"), ((6, 48, 165, 38, 46, 1, 1, 2, 0), "1,1,8,2"), ((8, 48, 186, 7, 35, 1, 1, 1, 0), "1,1,4,2"),
    ((8, 224, 17, 33, 20, 1, 1, 1, 0), "1,4,2,2"), ((6, 272, 7, 30, 23, 1, 1, 1, 0), "1,8,1,2"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_s8_tiles_plans(oracle, case, plan):
    """Several pixel tiles a wavefront, with and without other wavefronts on the same tiles' units, under one and nine taps."""
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, Ci, Co, H, W, R, S, st, pad = case
    x, w = inputs.uniform_s8((N, Ci, H, W), 9600 + Ci), inputs.uniform_s8((Co, Ci, R, S), 9700 + Co)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y_ref = oracle.conv2d_s8(x, w, st, pad)
    buf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.int32)
    sw.sw_conv2d_s8(xd, wd, st, pad, out=out)
    assert sw.sw_last_kernel() == f"mfma_s8_tiles_kernel<{plan}>"
    assert np.array_equal(out.cpu().numpy(), y_ref)
    assert_guards_intact(buf, front, n, guard)
    rng = np.random.default_rng(9800)
    bias = rng.integers(-20000, 20000, Co).astype(np.int32)
    scale = (rng.uniform(0.5, 2.0, Co) * 40.0 / ((Ci * R * S) ** 0.5 * 5461.0)).astype(np.float32)
    q_ref = oracle.conv2d_s8_requant(x, w, bias, scale, st, pad, False)
    buf, out, front, n, guard = guarded_empty(torch, q_ref.shape, torch.int8, fill=77)
    sw.sw_conv2d_s8_requant(xd, wd, torch.from_numpy(bias).cuda(), torch.from_numpy(scale).cuda(), st, pad, False, out=out)
    assert sw.sw_last_kernel() == f"mfma_s8_tiles_kernel<{plan}>"
    assert np.array_equal(out.cpu().numpy(), q_ref)
    assert_guards_intact(buf, front, n, guard)


@pytest.mark.parametrize("case,takes", [((8, 32, 64, 14, 14, 1, 0), False), ((8, 48, 64, 14, 14, 1, 0), True), ((21, 48, 36, 92, 80, 1, 0), False),
                                        ((5, 48, 36, 92, 80, 1, 0), True), ((21, 48, 36, 92, 81, 1, 0), True), ((21, 80, 36, 92, 80, 1, 0), True), ((2, 40, 64, 14, 14, 3, 1), False),
                                        ((1, 64, 64, 9, 3, 3, 1), False)], ids=str)
def test_s8_tiles_leaves_the_rest(oracle, case, takes):
    """Few channels under one tap (up to 64 in launches that fill the chip, on planes of whole dwords), channel counts off the grid, rows shorter than a quad: the kernels of before, with the same sums."""
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, Ci, Co, H, W, R, pad = case
    x, w = inputs.uniform_s8((N, Ci, H, W), 9400), inputs.uniform_s8((Co, Ci, R, R), 9500)
    y = sw.sw_conv2d_s8(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, pad)
    assert sw.sw_last_kernel().startswith("mfma_s8_tiles_kernel") == takes, sw.sw_last_kernel()
    assert np.array_equal(y.cpu().numpy(), oracle.conv2d_s8(x, w, 1, pad))
