"""GPU parity of the 1 x 1 kernel's form for planes of any size and any 4-byte address against the CPU oracle: the groups that begin
before the end of the one before (every remainder of the plane), planes of fewer pixels than a group, every variant, partial blocks of
output channels, half steps of 16 channels, the store's bias and ReLU, and infinities (the pixel is computed again)."""
import numpy as np
import pytest
import torch

import paper_2310_05218_amd as sw
from paper_2310_05218_amd import inputs
from parity import assert_f32_parity

pytestmark = pytest.mark.gpu

# (N, C_in, C_out, H, W, 4-byte steps off the 16-byte grid, kernel)
CASES = [
    (31, 136, 97, 15, 15, 0, "<1,2,1>"),
    (25, 24, 48, 23, 23, 0, "<1,2,1>"),
    (23, 56, 456, 7, 7, 3, "<1,2,1>"),
    (1500, 56, 64, 1, 3, 0, "<1,2,1>"),         # two groups of two pixels, one of them shared
    (36, 136, 65, 29, 25, 0, "<2,2,1>"),
    (10, 136, 232, 45, 39, 0, "<1,4,1>"),        # HW % 4 == 3
    (40, 152, 160, 25, 25, 1, "<1,4,1>"),       # HW % 4 == 1
    (16, 96, 464, 29, 29, 0, "<2,4,1>"),
    (10, 32, 24, 97, 97, 0, "<2,4,1>"),
    (16, 64, 256, 40, 40, 1, "<2,4,1>"),        # an even plane, off the grid
    (12, 64, 256, 38, 41, 2, None),             # eight bytes off: the aligned form
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c[:6]))
@pytest.mark.parametrize("bias", [False, True])
def test_odd_planes(oracle, case, bias):
    N, Ci, Co, H, W, off, form = case
    x = inputs.normal_f32((N, Ci, H, W), inputs.seed_for(7, 31 * Ci + Co))
    w = inputs.normal_f32((Co, Ci, 1, 1), inputs.seed_for(7, 1000 + Ci), (2.0 / Ci) ** 0.5)
    b = inputs.normal_f32((Co,), inputs.seed_for(7, 2000 + Ci))
    xs = torch.empty(x.size + 8, device="cuda")
    xv = xs[off:off + x.size].view(x.shape)
    xv.copy_(torch.from_numpy(x))
    guard = torch.full((N * Co * H * W + 64,), 7.25, device="cuda")
    out = guard[28 + off:28 + off + N * Co * H * W].view(N, Co, H, W)
    wd, bd = torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda()
    if bias:
        sw.sw_conv2d_bias_relu(xv, wd, bd, 1, 0, True, out=out)
        y_ref, d = oracle.conv2d_bias_relu(x, w, b, 1, 0, True)
    else:
        sw.sw_conv2d(xv, wd, 1, 0, out=out)
        y_ref, d = oracle.conv2d(x, w, 1, 0)
    if form:
        assert sw.sw_last_kernel() == "mfma_f32_pointwise_split_kernel" + form
    assert_f32_parity(out.cpu().numpy(), y_ref, d, f"pointwise, odd planes {case}")
    g = guard.cpu().numpy()
    assert np.all(g[:28 + off] == 7.25) and np.all(g[28 + off + out.numel():] == 7.25), "wrote outside the output"


def test_odd_planes_beyond(oracle):
    """An infinity and a NaN in the pixels that two groups share, and in an ordinary one: the channel sums are those of fp32."""
    N, C, H, W = 20, 152, 25, 25
    x = inputs.normal_f32((N, C, H, W), 3)
    w = inputs.normal_f32((160, C, 1, 1), 4)
    x[3, 7].reshape(-1)[622] = np.inf
    x[19, 0].reshape(-1)[624] = np.nan
    x[0, 151].reshape(-1)[1] = -np.inf
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    ref, _ = oracle.conv2d(x, w, 1, 0)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
    assert np.array_equal(np.sign(y[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))


# small planes, whose last group is a large part: pairs of pixels up to 25 and 192 channels, fours beyond
@pytest.mark.parametrize("case", [(2959, 72, 114, 3, 7, "<2,2,1>"), (1648, 40, 442, 3, 3, "<2,2,1>"), (1600, 192, 65, 5, 5, "<2,2,1>"),
                                  (1800, 200, 65, 5, 5, "<2,4,1>"), (1500, 56, 130, 3, 9, "<2,4,1>")], ids=lambda c: "x".join(str(v) for v in c[:5]))
def test_small_planes(oracle, case):
    N, Ci, Co, H, W, form = case
    x = inputs.normal_f32((N, Ci, H, W), inputs.seed_for(8, 31 * Ci + Co))
    w = inputs.normal_f32((Co, Ci, 1, 1), inputs.seed_for(8, 1000 + Ci), (2.0 / Ci) ** 0.5)
    y = sw.sw_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0)
    assert sw.sw_last_kernel() == "mfma_f32_pointwise_split_kernel" + form
    y_ref, d = oracle.conv2d(x, w, 1, 0)
    assert_f32_parity(y.cpu().numpy(), y_ref, d, f"pointwise, small planes {case}")
