"""Channel-last window-in-LDS kernel: sums that are no numbers leave it as the definition has them (act(t) = t without the rectifier),
in its three floating-point formats, with and without a bias, by 16-byte and by narrower stores."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
@pytest.mark.parametrize("Co", [64, 20])
@pytest.mark.parametrize("R", [1, 3])
@pytest.mark.parametrize("bias", [False, True])
def test_non_finite_sums(oracle, dtype, Co, R, bias):
    """A NaN and infinities of both signs in x, an infinity in w: the same outputs are NaN, inf and -inf as in 64 bits."""
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, H, W, Ci = 2, 11, 13, 32
    x = inputs.normal_f32((N, H, W, Ci), 8101)
    w = inputs.normal_f32((Co, R, R, Ci), 8102, (2.0 / (Ci * R * R)) ** 0.5)
    b = inputs.normal_f32((Co,), 8103) if bias else None
    x[0, 2, 3, 5], x[0, 7, 9, 0], x[1, 5, 5, 31], x[1, 10, 12, 7] = np.nan, np.inf, -np.inf, np.inf
    w[3, 0, 0, 4] = np.inf
    xd, wd = (torch.from_numpy(a).cuda().to(getattr(torch, dtype)) for a in (x, w))
    y = sw.sw_conv2d_nhwc(xd, wd, 1, 0, 1, None if b is None else torch.from_numpy(b).cuda(), False)
    assert "nhwc_lds_kernel" in sw.sw_last_kernel(), sw.sw_last_kernel()
    ref, _ = oracle.conv2d_nhwc(xd.float().cpu().numpy(), wd.float().cpu().numpy(), 1, 0, 1, b, False)
    v = y.float().cpu().numpy()
    assert np.isnan(ref).any() and np.isposinf(ref).any() and np.isneginf(ref).any()
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(v), kind(ref)), kind.__name__
