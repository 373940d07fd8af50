"""Channel-last layers of one to four input channels: parity against the oracle, and the bits of the one-thread-per-output kernel, which
runs for outputs off the 16-byte grid."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs
from parity import TOL_F32, assert_f32_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    import paper_2310_05218_amd as sw

    return sw


CASES = [
    # N, H, W, C_in, C_out, R, S, stride, pad, dilation, pixels per thread (0: one thread per output is faster and runs)
    (3, 37, 41, 3, 64, 3, 3, 2, 1, 1, 1), (3, 30, 199, 3, 64, 3, 3, 2, 1, 1, 4),        # rows of one turn, of more than three
    (10, 33, 35, 3, 40, 7, 7, 2, 3, 1, 4), (2, 29, 27, 1, 48, 5, 5, 1, 2, 1, 1),        # long sums; octets that do not divide the workgroup
    (2, 40, 41, 4, 8, 3, 3, 1, 1, 1, 1), (3, 26, 29, 2, 72, 3, 3, 1, 3, 2, 1),          # one octet; dilation and wide padding
    (5, 9, 250, 3, 256, 3, 3, 1, 0, 1, 4), (16, 50, 3, 3, 256, 2, 5, 1, 2, 1, 1),       # 32 octets; columns of padding only
    (2, 37, 41, 3, 64, 3, 3, 2, 1, 1, 0), (1, 30, 199, 3, 64, 3, 3, 2, 1, 1, 0), (1, 33, 35, 3, 40, 7, 7, 2, 3, 1, 0),      # fewer images
    (1, 40, 41, 4, 8, 3, 3, 1, 1, 1, 0), (1, 26, 29, 2, 72, 3, 3, 1, 3, 2, 0), (3, 9, 250, 3, 256, 3, 3, 1, 0, 1, 0), (1, 50, 3, 3, 256, 2, 5, 1, 2, 1, 0),
]


def both(torch, run, shape, dtype):
    """The call into an aligned output and into one a single element off the 16-byte grid."""
    n = int(np.prod(shape))
    outs = []
    for shift in (0, 1):
        buf = torch.full((n + 24,), 7.0, dtype=dtype, device="cuda")
        out = buf[8 + shift:8 + shift + n].view(shape)
        run(out)
        assert bool((buf[:8 + shift] == 7).all()) and bool((buf[8 + shift + n:] == 7).all()), "written beside the output"
        outs.append(out)
    return outs


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:10])))
@pytest.mark.parametrize("ek", [0, 1, 2], ids=["f32", "bf16", "f16"])
def test_few_channels(torch, sw, oracle, ek, case):
    N, H, W, Ci, Co, R, S, stride, pad, dil, px = case
    dtype = (torch.float32, torch.bfloat16, torch.float16)[ek]
    f = (sw.sw_conv2d_nhwc, sw.sw_conv2d_bf16_nhwc, sw.sw_conv2d_f16_nhwc)[ek]
    x = torch.from_numpy(inputs.normal_f32((N, H, W, Ci), 7100 + W)).cuda().to(dtype)
    w = torch.from_numpy(inputs.normal_f32((Co, R, S, Ci), 7200 + Co, (2.0 / (Ci * R * S)) ** 0.5)).cuda().to(dtype)
    b = torch.from_numpy(inputs.normal_f32((Co,), 7300, 0.5)).cuda()
    xn, wn = (np.ascontiguousarray(t.float().cpu().numpy().transpose(0, 3, 1, 2)) for t in (x, w))
    y_ref, d = oracle.conv2d_dilated(xn, wn, stride, pad, dil)
    shape = (y_ref.shape[0], y_ref.shape[2], y_ref.shape[3], y_ref.shape[1])
    names = []

    def run(out, bias=None, relu=False):
        f(x, w, stride, pad, dil, bias, relu, out=out)
        names.append(sw.sw_last_kernel())

    y, z = both(torch, run, shape, dtype)
    assert names == [f"few_channels_nhwc_kernel<{ek},{Ci},{px}>" if px else f"direct_nhwc_kernel<{ek}>", f"direct_nhwc_kernel<{ek}>"], names
    assert torch.equal(y, z)
    got = np.ascontiguousarray(y.float().cpu().numpy().transpose(0, 3, 1, 2))
    if ek == 0:
        assert_f32_parity(got, y_ref, d, str(case))
    else:           # fp32 sums, rounded once to 8 (11) bits, in half to no less than 2^-24
        u = 2.0 ** (-8 if ek == 1 else -11)
        assert np.all(np.abs(got - y_ref) <= u * np.abs(y_ref) + (1 + u) * TOL_F32 * d + 2.0 ** -25), str(case)
    y, z = both(torch, lambda out: run(out, b, True), shape, dtype)
    assert torch.equal(y, z)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan], ids=str)
@pytest.mark.parametrize("where", ["x", "w"])
@pytest.mark.parametrize("N,kernel", [(2, "direct_nhwc_kernel<0>"), (4, "few_channels_nhwc_kernel<0,3,1>")], ids=["2 images", "4 images"])
def test_few_channels_special_values(torch, sw, value, where, N, kernel):
    """Taps in the padding are left out: an infinite filter value reaches no output over padding alone."""
    x, w = inputs.normal_f32((N, 33, 41, 3), 7400), inputs.normal_f32((64, 3, 3, 3), 7500)
    (x if where == "x" else w).flat[700] = value
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    names = []
    y, z = both(torch, lambda out: (sw.sw_conv2d_nhwc(xd, wd, 2, 1, out=out), names.append(sw.sw_last_kernel())), (N, 17, 21, 64), torch.float32)
    assert names == [kernel, "direct_nhwc_kernel<0>"], names
    assert torch.equal(y.isnan(), z.isnan()) and torch.equal(torch.nan_to_num(y), torch.nan_to_num(z))
    assert not bool(torch.isfinite(y).all()) and bool(torch.isfinite(y).any())


@pytest.mark.parametrize("W,takes", [(16372, True), (16373, False)])
@pytest.mark.parametrize("ek", [0, 1, 2], ids=["f32", "bf16", "f16"])
def test_few_channels_fill_the_lds(torch, sw, oracle, ek, W, takes):
    """Filters (a row of eight floats and four to pad it) and an input row to the last float of 64 KB, and one more: one thread per output."""
    dtype = (torch.float32, torch.bfloat16, torch.float16)[ek]
    x = torch.from_numpy(inputs.normal_f32((32, 2, W, 1), 7600)).cuda().to(dtype)
    w = torch.from_numpy(inputs.normal_f32((8, 1, 1, 1), 7700)).cuda().to(dtype)
    y = (sw.sw_conv2d_nhwc, sw.sw_conv2d_bf16_nhwc, sw.sw_conv2d_f16_nhwc)[ek](x, w)
    assert sw.sw_last_kernel() == (f"few_channels_nhwc_kernel<{ek},1,4>" if takes else f"direct_nhwc_kernel<{ek}>")
    assert torch.equal(y, (x.float() * w.float().view(8)).to(dtype))       # (a sum of one product is that product, rounded once)
