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
