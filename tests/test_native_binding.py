"""The native short way of the binding gives what the long way gives: the same bits, the same exceptions."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2310_05218_amd as sw  # noqa: E402
from paper_2310_05218_amd import binding  # noqa: E402


def calls(dev):
    g = torch.Generator().manual_seed(5)
    f = lambda *s: torch.randn(s, generator=g).to(dev)
    q = lambda *s: torch.randint(-128, 128, s, generator=g, dtype=torch.int8).to(dev)
    i = lambda n: torch.randint(-9999, 9999, (n,), generator=g, dtype=torch.int32).to(dev)
    x, w, b = f(2, 8, 12, 14), f(16, 8, 3, 3), f(16)
    xl, wl = f(2, 12, 14, 16), f(32, 3, 3, 16)
    dw, db = f(8, 1, 3, 3), f(8)
    xq, wq, sc = q(2, 32, 12, 14), q(16, 32, 3, 3), torch.rand(16, generator=g).to(dev) * 1e-3
    xql, wql = q(2, 12, 14, 32), q(16, 3, 3, 32)
    s1, t1 = f(3, 500), f(9)
    P = torch.nn.Parameter
    return {
        "conv1d": lambda: sw.sw_conv1d(s1, t1, 2, 3), "conv1d empty": lambda: sw.sw_conv1d(s1[:, :4].contiguous(), t1),
        "conv1d pad": lambda: sw.sw_conv1d(s1, t1, 1, 9), "pool1d": lambda: sw.sw_pool1d(s1, 8, 1, sw.SW_POOL_MAX), "pool1d mode": lambda: sw.sw_pool1d(s1, 8, 1, 7),
        "pool2d": lambda: sw.sw_pool2d(x, 3, 3, 2, 1), "pool2d pad": lambda: sw.sw_pool2d(x, 3, 3, 2, 2),
        "conv2d": lambda: sw.sw_conv2d(x, w, 1, 1), "conv2d keywords": lambda: sw.sw_conv2d(x, w, pad=1, stride=2), "conv2d parameter": lambda: sw.sw_conv2d(x, P(w), 1, 1),
        "conv2d numpy": lambda: sw.sw_conv2d(x, w, np.int64(2), np.int32(1)), "conv2d bool": lambda: sw.sw_conv2d(x, w, True, False),
        "conv2d float": lambda: sw.sw_conv2d(x, w, 1.0, 1), "conv2d zero stride": lambda: sw.sw_conv2d(x, w, 0, 1), "conv2d negative": lambda: sw.sw_conv2d(x, w, 1, -1),
        "conv2d huge": lambda: sw.sw_conv2d(x, w, 2 ** 40, 1), "conv2d channels": lambda: sw.sw_conv2d(x, f(16, 4, 3, 3)), "conv2d small": lambda: sw.sw_conv2d(x[:, :, :2].contiguous(), w),
        "conv2d strided": lambda: sw.sw_conv2d(x.transpose(2, 3), w, 1, 1), "conv2d double": lambda: sw.sw_conv2d(x.double(), w), "conv2d 3-d": lambda: sw.sw_conv2d(x[0], w),
        "conv2d list": lambda: sw.sw_conv2d(x.tolist(), w), "conv2d none": lambda: sw.sw_conv2d(x, None), "conv2d empty": lambda: sw.sw_conv2d(x[:0], w),
        "conv2d channels last": lambda: sw.sw_conv2d(x.contiguous(memory_format=torch.channels_last), w), "conv2d cpu filter": lambda: sw.sw_conv2d(x, w.cpu()),
        "bias_relu": lambda: sw.sw_conv2d_bias_relu(x, w, b, 1, 1, True), "bias_relu none": lambda: sw.sw_conv2d_bias_relu(x, w, None, 1, 1, 1),
        "bias_relu short": lambda: sw.sw_conv2d_bias_relu(x, w, b[:4], 1, 1), "bias_relu double": lambda: sw.sw_conv2d_bias_relu(x, w, b.double(), 1, 1),
        "dilated": lambda: sw.sw_conv2d_dilated(x, w, 1, 2, 2), "dilated zero": lambda: sw.sw_conv2d_dilated(x, w, 1, 2, 0),
        "depthwise": lambda: sw.sw_conv2d_depthwise(x, dw, 2, 1), "depthwise filters": lambda: sw.sw_conv2d_depthwise(x, w, 2, 1),
        "depthwise bias": lambda: sw.sw_conv2d_depthwise_bias_relu(x, dw, db, 1, 1, True), "depthwise bf16": lambda: sw.sw_conv2d_depthwise_bf16(x.bfloat16(), dw, 1, 1),
        "depthwise bf16 of fp32": lambda: sw.sw_conv2d_depthwise_bf16(x, dw, 1, 1),
        "s8": lambda: sw.sw_conv2d_s8(xq, wq, 1, 1), "s8 requant": lambda: sw.sw_conv2d_s8_requant(xq, wq, i(16), sc, 1, 1, True),
        "s8 requant none": lambda: sw.sw_conv2d_s8_requant(xq, wq, None, sc, 1, 1), "s8 requant no scale": lambda: sw.sw_conv2d_s8_requant(xq, wq, None, None),
        "s8 nhwc": lambda: sw.sw_conv2d_s8_nhwc(xql, wql, 1, 1), "s8 nhwc requant": lambda: sw.sw_conv2d_s8_nhwc(xql, wql, 1, 1, i(16), sc, True),
        "nhwc": lambda: sw.sw_conv2d_nhwc(xl, wl, 1, 1, 1, f(32), True), "nhwc bf16": lambda: sw.sw_conv2d_nhwc(xl.bfloat16(), wl.bfloat16(), 2, 1),
        "nhwc f16": lambda: sw.sw_conv2d_f16_nhwc(xl.half(), wl.half(), 1, 2, 2, f(32)), "nhwc mixed": lambda: sw.sw_conv2d_nhwc(xl.half(), wl, 1, 1),
        "nhwc bf16 zero dilation": lambda: sw.sw_conv2d_nhwc(xl.bfloat16(), wl.bfloat16(), 1, 1, 0),
    }


def outcome(f):
    try:
        y = f()
        return y.dtype, tuple(y.shape), y.requires_grad, y.is_contiguous(), y.cpu()
    except Exception as e:
        return type(e), str(e)


def both_ways(monkeypatch, dev):
    binding._native(-1)         # (bound)
    assert binding._native.__name__ == "run", "the native module is not built"
    for name in calls(dev):
        short = outcome(calls(dev)[name])
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", lambda *a: None)
            long = outcome(calls(dev)[name])
        assert len(short) == len(long), f"{name}: {short} / {long}"
        for a, b in zip(short, long):
            assert torch.equal(a, b) if torch.is_tensor(a) else a == b, f"{name}: {short} / {long}"


def test_off_the_gpu(monkeypatch):
    both_ways(monkeypatch, "cpu")


@pytest.mark.gpu
def test_on_the_gpu(monkeypatch):
    both_ways(monkeypatch, "cuda")


@pytest.mark.gpu
def test_transformed_tensors_raise():
    """A tensor without memory of its own is no argument of a kernel: what torch says of it, and the next call is an ordinary one."""
    x, w = torch.randn(2, 8, 12, 14, device="cuda"), torch.randn(16, 8, 3, 3, device="cuda")
    for _ in range(2):
        with pytest.raises(RuntimeError, match="storage"):
            torch.vmap(lambda a: sw.sw_conv2d(a, w, 1, 1))(x[None])
    assert sw.sw_conv2d(x, w, 1, 1).shape == (2, 16, 12, 14)


@pytest.mark.gpu
def test_current_stream_and_threads():
    """The call goes to the current stream of its thread; several threads call at once."""
    import threading

    x, w = torch.randn(1, 4, 64, 64, device="cuda"), torch.randn(8, 4, 3, 3, device="cuda")
    want = sw.sw_conv2d(x, w, 1, 1)
    torch.cuda.synchronize()
    bad = []

    def work():
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(50):
                a = x * 1.0                     # on this stream: the call after it reads what it wrote
                y = sw.sw_conv2d(a, w, 1, 1)
                a.zero_()
            s.synchronize()
            if not torch.equal(y, want):
                bad.append(1)

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
