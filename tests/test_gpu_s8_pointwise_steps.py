"""int8 pointwise layers, channel last: numbers of 32-channel steps around halves and wholes of a chunk of eight, one tile and several a
wavefront, ragged last tiles."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Co", [64, 256])
@pytest.mark.parametrize("px", [33, 3000, 70001])
@pytest.mark.parametrize("steps", [4, 5, 7, 8, 9, 12, 13, 16])
def test_steps(steps, px, Co):
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    Ci = 32 * steps
    x, w = inputs.uniform_s8((1, 1, px, Ci), 7500 + steps), inputs.uniform_s8((Co, 1, 1, Ci), 7600 + steps)
    rng = np.random.default_rng(7700)
    bias = rng.integers(-50000, 50000, Co).astype(np.int32)
    scale = (rng.uniform(0.5, 2.0, Co) * 2.0 ** -13).astype(np.float32)
    q = sw.sw_conv2d_s8_nhwc(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0, torch.from_numpy(bias).cuda(), torch.from_numpy(scale).cuda(), True)
    # exact sums by float64 products (below 2^53)
    acc = (x.reshape(px, Ci).astype(np.float64) @ w.reshape(Co, Ci).T.astype(np.float64)).astype(np.int64).astype(np.int32)
    ref = np.clip(np.rint((acc + bias).astype(np.float32) * scale), 0, 127).astype(np.int8)
    assert sw.sw_last_kernel().startswith("mfma_s8_pointwise_nhwc_kernel"), sw.sw_last_kernel()
    assert np.array_equal(q.cpu().numpy().reshape(px, Co), ref)


@pytest.mark.parametrize("sign", [1, -1])
def test_biases_at_the_ends_of_int32(sign):
    """The sums start from the biases, and between two channels they pass 2^31 where the finished ones do not: they wrap and come back.  The first
    half of the channels adds `sign` 16129 each, the second takes it back but for the last 32; the bias leaves the finished sum 1000 short of the end."""
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    px, Ci, Co = 100, 512, 64
    x = np.full((1, 1, px, Ci), 127, np.int8)
    w = np.full((Co, 1, 1, Ci), 127 * sign, np.int8)
    w[..., Ci // 2:Ci - 32] = -127 * sign
    w[1::2] = w[1::2, ..., ::-1]                             # (odd channels: down first)
    acc = int(x[0, 0, 0].astype(np.int64) @ w[0, 0, 0].astype(np.int64))
    end = 2 ** 31 - 1 if sign > 0 else -(2 ** 31)
    bias = np.full(Co, end - acc - sign * 1000, np.int64) + sign * np.arange(Co)
    assert abs(int(bias[0])) < 2 ** 31 and abs(int(bias[0]) + sign * 16129 * (Ci // 2)) > 2 ** 31
    scale = np.full(Co, 127.0 / 2 ** 31, np.float32) * np.linspace(0.1, 1.0, Co).astype(np.float32)
    q = sw.sw_conv2d_s8_nhwc(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0, torch.from_numpy(bias.astype(np.int32)).cuda(),
                             torch.from_numpy(scale).cuda(), False)
    assert sw.sw_last_kernel().startswith("mfma_s8_pointwise_nhwc_kernel"), sw.sw_last_kernel()
    ref = np.clip(np.rint((acc + bias).astype(np.float32) * scale), -128, 127).astype(np.int8)
    assert np.abs(ref.astype(int)).min() > 5 and np.array_equal(q.cpu().numpy().reshape(px, Co), np.broadcast_to(ref, (px, Co)))
