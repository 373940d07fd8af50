"""Requantised results packed four at a time (channel-last int8 kernels): ties, saturation on both sides, and scales that are no numbers
to multiply by in earnest, against the definition clamp(rne(scale * float(sum + bias)), lowest, 127), a NaN being the lowest."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape", [(2, 9, 11, 128, 64, 1, "mfma_s8_pointwise_nhwc_kernel"), (1, 12, 12, 64, 64, 3, "mfma_s8q_nhwc_lds_kernel"),
                                   (1, 12, 12, 32, 36, 3, "mfma_s8q_nhwc_lds_kernel")], ids=lambda s: f"{s[6]} {s[4]}")
def test_packed_requantisation(oracle, shape, relu):
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, H, W, Ci, Co, R, kernel = shape
    x, w = inputs.uniform_s8((N, H, W, Ci), 9600), inputs.uniform_s8((Co, R, R, Ci), 9700)
    acc = oracle.conv2d_s8_nhwc(x, w, 1, R // 2)
    rng = np.random.default_rng(9800)
    bias = rng.integers(-30000, 30000, Co).astype(np.int32)
    scale = (2.0 ** rng.integers(-14, -6, Co)).astype(np.float32)       # powers of two: many exact ties
    scale[1::4] = rng.uniform(1e-4, 1e-2, len(scale[1::4])).astype(np.float32)
    special = np.array([0.0, -0.5, np.inf, -np.inf, np.nan, 3e38, -2.0 ** -9, 1e-40], np.float32)
    scale[:len(special)] = special
    with np.errstate(all="ignore"):
        f = (acc + bias).astype(np.float32) * scale
        low = 0.0 if relu else -128.0
        ref = np.where(np.isnan(f), low, np.clip(np.rint(f), low, 127.0)).astype(np.int8)
    assert np.count_nonzero((f != np.rint(f)) & (2 * f == np.rint(2 * f))) > 20
    y = sw.sw_conv2d_s8_nhwc(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, R // 2, torch.from_numpy(bias).cuda(),
                             torch.from_numpy(scale).cuda(), relu)
    assert sw.sw_last_kernel().startswith(kernel), sw.sw_last_kernel()
    assert np.array_equal(y.cpu().numpy(), ref)
