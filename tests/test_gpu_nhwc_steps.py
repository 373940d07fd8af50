"""Channel-last window-in-LDS kernel: numbers of taps around the operand steps that are under way (one tap, fewer taps than steps, whole
and ragged rounds), two and three window stages, ragged output channels and tiles, on its three instruction kinds."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    import paper_2310_05218_amd as _sw
    return _sw


@pytest.fixture(scope="module")
def oracle():
    import oracle as _oracle
    return _oracle


CASES = [
    # N, H, W, C_in, C_out, R, S, stride, pad
    (1, 9, 11, 32, 20, 1, 1, 1, 0),      # one tap, one block
    (3, 16, 17, 96, 72, 1, 1, 1, 0),     # one tap, several chunks, ragged channel block
    (1, 10, 9, 64, 40, 1, 2, 1, 0),      # two taps
    (1, 12, 13, 32, 64, 2, 2, 1, 0),     # four
    (2, 11, 12, 32, 64, 2, 3, 1, 1),     # six
    (1, 9, 9, 160, 16, 1, 7, 1, 3),      # seven taps, five chunks
    (1, 20, 20, 32, 100, 3, 3, 1, 1),    # nine, a ragged second channel block
    (4, 30, 30, 64, 64, 3, 3, 2, 1),     # stride 2
    (1, 21, 17, 32, 32, 4, 5, 1, 2),     # twenty
    (1, 15, 19, 32, 36, 5, 5, 1, 2),     # twenty-five, output channels in pieces of four
    (1, 12, 80, 16, 32, 5, 13, 1, 6),    # sixty-five
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_numbers_of_taps(torch, sw, oracle, case):
    """int8 sums exact; bf16 |y - oracle| <= 2e-5 D (fp32 sums) + 2^-8 |oracle| (one rounding); fp32 |y - oracle| <= 2e-5 D."""
    N, H, W, Ci, Co, R, S, st, pad = case
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    if Ci % 32 == 0:
        x, w = inputs.uniform_s8((N, H, W, Ci), 9101), inputs.uniform_s8((Co, R, S, Ci), 9102)
        y = sw.sw_conv2d_s8_nhwc(dev(x), dev(w), st, pad)
        assert sw.sw_last_kernel().startswith("mfma_s8_nhwc_lds_kernel"), sw.sw_last_kernel()
        assert np.array_equal(y.cpu().numpy(), oracle.conv2d_s8_nhwc(x, w, st, pad))
    b = inputs.normal_f32((Co,), 9105, 0.5)
    xb, wb = inputs.normal_bf16((N, H, W, Ci), 9103), inputs.normal_bf16((Co, R, S, Ci), 9104, (2.0 / (Ci * R * S)) ** 0.5)
    as_bf16 = lambda a: torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    y = sw.sw_conv2d_nhwc(as_bf16(xb), as_bf16(wb), st, pad, 1, dev(b), True)
    assert sw.sw_last_kernel().startswith("mfma_bf16_nhwc_lds_kernel"), sw.sw_last_kernel()
    ref, d = oracle.conv2d_bf16_nhwc(xb, wb, st, pad, 1, b, True)
    v = oracle.bf16_to_f32(y.view(torch.int16).cpu().numpy().view(np.uint16)).astype(np.float64)
    assert np.all(np.abs(v - ref) <= 2e-5 * d + 2.0 ** -8 * np.abs(ref) + 1e-37)
    xf, wf = inputs.normal_f32((N, H, W, Ci), 9106), inputs.normal_f32((Co, R, S, Ci), 9107, (2.0 / (Ci * R * S)) ** 0.5)
    y = sw.sw_conv2d_nhwc(dev(xf), dev(wf), st, pad, 1, dev(b), False)
    ref, d = oracle.conv2d_nhwc(xf, wf, st, pad, 1, b, False)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 2e-5 * np.maximum(d, 1e-30)), sw.sw_last_kernel()
