"""Channel-last window-in-LDS kernel: numbers of taps around the operand steps that are under way (one tap, fewer taps than steps, whole
and ragged rounds), two and three window stages with several tiles a workgroup, ragged output channels and tiles, in its five formats."""
import ctypes

import numpy as np
import pytest

from paper_2310_05218_amd import binding, inputs
from test_plans_host import shape

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
    (1, 12, 80, 16, 32, 5, 13, 1, 6),    # sixty-five (fp32: over eight channels, below)
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
    if R * S < 65:
        assert sw.sw_last_kernel().startswith("mfma_f32_nhwc_lds_kernel"), sw.sw_last_kernel()
    ref, d = oracle.conv2d_nhwc(xf, wf, st, pad, 1, b, False)
    assert np.all(np.abs(y.cpu().numpy() - ref) <= 2e-5 * np.maximum(d, 1e-30)), sw.sw_last_kernel()


FORMATS = {"f32": 0, "bf16": 1, "f16": 2, "s8": 3, "s8q": 4}


def run_and_check(torch, sw, oracle, fmt, case, images=None, seed=9110):
    """One call with a bias (none for int32 sums) on the kernel of this file, against the oracle on some of the images; the pointers of the call.
    int8 exact; fp32 2e-5 D, bf16 and half one rounding more (2^-8, 2^-11 of the value, half of a denormal's step)."""
    N, H, W, Ci, Co, R, S, st, pad = case
    images = images or list(range(N))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    if fmt in ("s8", "s8q"):
        x, w = inputs.uniform_s8((N, H, W, Ci), seed), inputs.uniform_s8((Co, R, S, Ci), seed + 1)
        rng = np.random.default_rng(seed)
        bias = rng.integers(-9000, 9000, Co).astype(np.int32) if fmt == "s8q" else None
        scale = (rng.uniform(0.5, 2.0, Co) * 2.0 ** -11 / (Ci * R * S / 128) ** 0.5).astype(np.float32) if fmt == "s8q" else None
        xd, wd = dev(x), dev(w)
        y = sw.sw_conv2d_s8_nhwc(xd, wd, st, pad, *(() if fmt == "s8" else (dev(bias), dev(scale), True)))
        acc = oracle.conv2d_s8_nhwc(np.ascontiguousarray(x[images]), w, st, pad)
        ref = acc if fmt == "s8" else np.clip(np.rint((acc + bias).astype(np.float32) * scale), 0, 127).astype(np.int8)
        ok = np.array_equal(y.cpu().numpy()[images], ref)
    else:
        x, w = inputs.normal_f32((N, H, W, Ci), seed), inputs.normal_f32((Co, R, S, Ci), seed + 1, (2.0 / (Ci * R * S)) ** 0.5)
        b = inputs.normal_f32((Co,), seed + 2, 0.5)
        xd, wd = (dev(a).to({"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt]) for a in (x, w))
        y = sw.sw_conv2d_nhwc(xd, wd, st, pad, 1, dev(b), True)
        ref, d = oracle.conv2d_nhwc(np.ascontiguousarray(xd.float().cpu().numpy()[images]), wd.float().cpu().numpy(), st, pad, 1, b, True)
        rel, least = {"f32": (0, 0), "bf16": (2.0 ** -8, 1e-37), "f16": (2.0 ** -11, 2.0 ** -25)}[fmt]
        ok = np.all(np.abs(y.float().cpu().numpy().astype(np.float64)[images] - ref) <= 2e-5 * d + rel * np.abs(ref) + least)
    name = {"f32": "mfma_f32", "bf16": "mfma_bf16", "f16": "mfma_f16", "s8": "mfma_s8", "s8q": "mfma_s8q"}[fmt]
    assert sw.sw_last_kernel().startswith(name + "_nhwc_lds_kernel"), sw.sw_last_kernel()
    assert ok, (fmt, case)
    return xd.data_ptr(), wd.data_ptr(), y.data_ptr()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_numbers_of_taps_half_and_requantised(torch, sw, oracle, case):
    run_and_check(torch, sw, oracle, "f16", case)
    if case[3] % 32 == 0:
        run_and_check(torch, sw, oracle, "s8q", case)


def test_sixty_five_taps_f32(torch, sw, oracle):
    run_and_check(torch, sw, oracle, "f32", (1, 12, 80, 8, 32, 5, 13, 1, 6))


@pytest.mark.parametrize("fmt,stages,case", [
    ("f32", 2, (27, 33, 35, 32, 40, 3, 3, 1, 0)), ("f32", 3, (30, 29, 20, 8, 80, 1, 3, 1, 0)), ("f32", 3, (38, 27, 52, 8, 4, 1, 1, 1, 0)),
    ("bf16", 2, (26, 33, 53, 32, 48, 5, 5, 2, 2)), ("bf16", 3, (33, 10, 38, 16, 80, 1, 3, 1, 0)), ("bf16", 2, (38, 38, 51, 64, 4, 3, 3, 1, 0)),
    ("f16", 2, (33, 32, 30, 64, 80, 2, 3, 2, 1)), ("f16", 3, (26, 10, 45, 16, 80, 1, 3, 1, 0)), ("f16", 3, (28, 33, 40, 16, 4, 1, 1, 1, 0)),
    ("s8", 2, (38, 25, 45, 128, 48, 3, 3, 2, 1)), ("s8", 3, (37, 19, 35, 32, 40, 1, 3, 1, 0)),
    ("s8q", 2, (33, 32, 36, 128, 80, 2, 3, 2, 1)), ("s8q", 3, (13, 39, 47, 32, 40, 1, 3, 1, 0)), ("s8q", 3, (22, 23, 44, 32, 4, 1, 1, 1, 0)),
], ids=str)
def test_window_stages(torch, sw, oracle, fmt, stages, case):
    """Two and three window stages, several tiles of a workgroup one behind the other: the plan's own numbers, and the first, second and last image."""
    N, H, W, Ci, Co, R, S, st, pad = case
    x, w, y = run_and_check(torch, sw, oracle, fmt, case, images=[0, 1, N - 1], seed=9130)
    f = getattr(binding.lib(), "_ZN6swconv20mfma_nhwc_lds_stagesEPKvS1_S1_RKNS_11Conv2dShapeEiPi")
    f.restype, tiles = ctypes.c_int, ctypes.c_int(0)
    s = shape(N, Ci, Co, H, W, R, S, st, pad)
    assert f(ctypes.c_void_p(x), ctypes.c_void_p(w), ctypes.c_void_p(y), ctypes.byref(s), FORMATS[fmt], ctypes.byref(tiles)) == stages
    assert tiles.value >= 2
