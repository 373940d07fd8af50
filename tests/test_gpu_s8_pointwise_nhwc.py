"""The int8 pointwise kernel on channel-last tensors, requantised: bit-exact against the oracle at the edges of its pixel tiles,
channel blocks and channel chunks."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs
from parity import assert_guards_intact, guarded_empty

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, C_in, C_out
    (1, 1, 1, 128, 16),          # one pixel, one chunk of four steps
    (2, 9, 7, 160, 48),          # 126 pixels, five steps; two channel blocks, half of the second used
    (1, 13, 5, 256, 128),        # exactly one chunk
    (1, 8, 8, 288, 176),         # one step into the second chunk; a third group of 48 channels
    (3, 28, 28, 512, 128),       # two chunks
    (40, 28, 28, 128, 512),      # more tiles than wavefronts: the next tile's pixels requested ahead
    (1, 6, 6, 1088, 64),         # filters of 64 channels within LDS, those of 128 not
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_s8_pointwise_nhwc(oracle, case):
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    N, H, W, Ci, Co = case
    x = inputs.uniform_s8((N, H, W, Ci), 7100 + Ci)
    w = inputs.uniform_s8((Co, 1, 1, Ci), 7200 + Co)
    rng = np.random.default_rng(7300)
    bias = rng.integers(-50000, 50000, Co).astype(np.int32)
    scale = (rng.uniform(0.5, 2.0, Co) * 2.0 ** -13).astype(np.float32)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    acc = oracle.conv2d_s8_nhwc(x, w, 1, 0)
    for b, relu in ((bias, False), (None, True)):
        t = (acc + (0 if b is None else b)).astype(np.float32) * scale
        ref = np.clip(np.rint(t), 0 if relu else -128, 127).astype(np.int8)
        buf, out, front, n, guard = guarded_empty(torch, ref.shape, torch.int8, fill=77)
        sw.sw_conv2d_s8_nhwc(xd, wd, 1, 0, None if b is None else torch.from_numpy(b).cuda(), torch.from_numpy(scale).cuda(), relu, out=out)
        assert sw.sw_last_kernel().startswith("mfma_s8_pointwise_nhwc_kernel"), sw.sw_last_kernel()
        assert np.array_equal(out.cpu().numpy(), ref)
        assert_guards_intact(buf, front, n, guard)
