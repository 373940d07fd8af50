"""The launch plans of kernels that a shape selects, asked on the host (a plan touches no device): limits of a launch, and which
shapes the one-filter-per-plane bands take."""
import ctypes
import time

import pytest

from paper_2310_05218_amd import binding


class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("N", "C_in", "C_out", "H", "W", "R", "S", "stride", "pad", "Ho", "Wo", "dil")]


def shape(N, C_in, C_out, H, W, R, S, stride, pad):
    return Shape(N, C_in, C_out, H, W, R, S, stride, pad, (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1, 1)


def bands(planes, planes_per_x, s, bf16=False):
    f = getattr(binding.lib(), "_ZN6swconv21plane_bands_supportedEPKvliiRKNS_11Conv2dShapeEb")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.POINTER(Shape), ctypes.c_bool]
    return f(4096, planes, planes_per_x, planes_per_x, ctypes.byref(s), bf16)


def test_bands_stay_below_the_work_items_of_a_launch():
    """One workgroup of at least 128 threads per plane: 2^25 planes would be 2^32 work items, one more than a launch has."""
    s = shape(32767, 1, 1024, 70, 64, 64, 64, 2, 0)          # four outputs a plane, 64 x 64 taps
    assert bands(32767 * 1024, 1024, s)
    s.N = 32768
    assert not bands(32768 * 1024, 1024, s)


@pytest.mark.parametrize("planes,size,R,stride,takes", [
    (512, 5, 3, 1, True), (513, 5, 3, 1, False),              # few planes whatever they hold; many that hold little
    (131072, 10, 3, 1, False), (131072, 11, 3, 1, True),      # 100 and 121 outputs of nine taps
    (4096, 7, 5, 1, True), (4097, 7, 5, 1, False), (131072, 8, 5, 1, True),
    (131072, 10, 7, 2, False), (131072, 11, 7, 2, True),      # 25 and 36 outputs of 49 taps
    (512, 113, 2, 4, False), (512, 113, 3, 4, False), (512, 113, 9, 4, True), (512, 113, 51, 3, True),     # taps in loops
    (2574, 12, 33, 9, False),                                 # mostly over the padding
])
def test_bands_take_what_they_are_faster_at(planes, size, R, stride, takes):
    assert bands(planes, planes, shape(1, 1, planes, size, size, R, R, stride, R // 2)) == takes


def split_supported(name, s):
    f = getattr(binding.lib(), f"_ZN6swconv{19 + len(name)}mfma_f32_{name}_supportedERKNS_11Conv2dShapeE")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(Shape)]
    return f(ctypes.byref(s))


def test_few_channels_kernel_stays_below_a_launch_s_second_dimension():
    assert split_supported("stem", shape(1, 3, 64 * 65535, 9, 9, 3, 3, 2, 1))
    assert not split_supported("stem", shape(1, 3, 64 * 65535 + 1, 9, 9, 3, 3, 2, 1))


@pytest.mark.parametrize("name,s", [("split", (1, 33, 8, 15_000_000, 1, 9, 1, 1, 4)), ("stem", (1, 3, 8, 40_000_000, 1, 7, 7, 2, 3))])
def test_plans_of_tall_images_take_no_longer(name, s):
    """The search goes over the tiles that can be, not over all row counts of the image (65 and 85 ms here)."""
    s = shape(*s)
    binding.lib()
    start = time.perf_counter()
    split_supported(name, s)
    assert time.perf_counter() - start < 0.01


@pytest.mark.parametrize("C,R,S,stride,size,takes", [
    (3, 7, 7, 2, 224, True), (3, 3, 3, 2, 224, True), (7, 2, 2, 2, 224, True),
    (2, 1, 1, 2, 224, False), (3, 2, 2, 2, 224, False), (2, 3, 3, 2, 224, False), (2, 5, 4, 2, 224, True),     # 0.07, 0.53, 0.6, 1.33
    (2, 2, 2, 4, 50, True), (2, 2, 2, 4, 20, False), (4, 1, 1, 4, 50, False),                                 # strides from 4 up
])
def test_few_channels_kernel_takes_what_it_is_faster_at(C, R, S, stride, size, takes):
    assert split_supported("stem", shape(8, C, 64, size, size, R, S, stride, 0)) == takes


def pointwise_supported(N, C_in, C_out, H, W, x=4096, w=4096, y=4096):
    f = getattr(binding.lib(), "_ZN6swconv28mfma_f32_pointwise_supportedERKNS_11Conv2dShapeEPKfS4_S4_")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(Shape)] + [ctypes.c_void_p] * 3
    return f(ctypes.byref(shape(N, C_in, C_out, H, W, 1, 1, 1, 0)), x, w, y)


def test_pointwise_plan_refuses_what_no_variant_takes():
    """Odd planes, pointers off the 8-byte loads and filters beyond LDS leave no variant (and no divisor for what follows)."""
    assert pointwise_supported(32, 64, 256, 56, 56)
    assert not pointwise_supported(32, 512, 512, 7, 7)
    assert not pointwise_supported(1, 64, 64, 8, 8, x=4100) and not pointwise_supported(1, 64, 64, 8, 8, y=4100)
    assert not pointwise_supported(1, 2048, 64, 8, 8)


@pytest.mark.parametrize("N,H,W,C,K,R,S,stride,pad,takes", [
    (32, 224, 224, 3, 64, 3, 3, 2, 1, True), (1, 224, 224, 3, 64, 7, 7, 2, 3, True), (1, 224, 224, 3, 96, 4, 4, 4, 0, True),
    (2, 4, 1436, 1, 120, 5, 5, 2, 1, False), (1, 1, 2158, 1, 152, 5, 5, 1, 2, False),      # one long row: 7.4 us and 51.2, 5.3 and 161.6
    (2, 52, 81, 2, 192, 3, 3, 4, 1, False), (21, 4, 399, 4, 216, 1, 1, 8, 0, False),       # few outputs a workgroup: 5.6 and 8.9, 4.1 and 7.3
    (17, 19, 28, 3, 40, 5, 5, 8, 2, False), (30, 17, 20, 4, 104, 3, 8, 16, 0, False),      # ... and many filters: 15.0 and 22.8
])
def test_few_channels_channel_last_kernel_takes_what_it_is_faster_at(N, H, W, C, K, R, S, stride, pad, takes):
    f = getattr(binding.lib(), "_ZN6swconv27few_channels_nhwc_supportedEPKvRKNS_11Conv2dShapeE")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.POINTER(Shape)]
    assert f(4096, ctypes.byref(shape(N, C, K, H, W, R, S, stride, pad))) == takes


@pytest.mark.parametrize("planes,H,W,R,stride,pad,off,takes", [
    (16384, 14, 14, 3, 1, 1, True, True), (8192, 28, 28, 5, 1, 2, False, True), (16384, 16, 16, 7, 1, 3, False, True), (16384, 16, 16, 7, 2, 3, False, True),
    (15200, 78, 4, 5, 2, 2, False, False), (28188, 64, 4, 3, 2, 0, False, False), (19800, 120, 4, 7, 2, 3, False, False),      # tall and narrow: 11.1 us and
    (4797, 95, 9, 5, 1, 0, True, False), (42224, 17, 9, 7, 1, 3, True, False), (32940, 45, 11, 3, 1, 1, True, False),          # 16.9, 10.4 and 14.2, ...
    (1524, 9, 11, 5, 1, 0, True, False), (800, 5, 9, 3, 1, 0, True, False),                                                    # small: 4.4 and 6.0
])
def test_rows_kernel_takes_the_planes_that_it_is_faster_at(planes, H, W, R, stride, pad, off, takes):
    f = getattr(binding.lib(), "_ZN6swconv24rows_before_small_planesElRKNS_11Conv2dShapeEb")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_long, ctypes.POINTER(Shape), ctypes.c_bool]
    assert f(planes, ctypes.byref(shape(1, 1, 1, H, W, R, R, stride, pad)), off) == takes


@pytest.mark.parametrize("planes,H,W,R,stride,pad,x,takes", [
    (16384, 28, 7, 2, 2, 0, 4096, False), (60, 28, 8, 2, 2, 0, 4100, True), (60, 28, 8, 2, 2, 0, 4096, True),       # seven columns under 2x2
    (168, 7, 7, 3, 1, 0, 4096, False), (2621, 7, 7, 3, 1, 0, 4096, False), (2622, 7, 7, 3, 1, 0, 4096, True),       # ... and 3x3, 25 outputs a plane
    (168, 7, 7, 3, 2, 1, 4096, True), (60, 28, 6, 3, 2, 1, 4096, False), (60, 28, 4, 3, 2, 1, 4096, True), (60, 28, 4, 3, 2, 1, 4100, False),
])
def test_pooling_rows_take_what_they_are_faster_at(planes, H, W, R, stride, pad, x, takes):
    f = getattr(binding.lib(), "_ZN6swconv19pool_rows_supportedEPKfliiiiiii")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_long] + [ctypes.c_int] * 7
    assert f(x, planes, W, R, R, stride, pad, (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1) == takes


def s8_tiles_supported(s):
    f = getattr(binding.lib(), "_ZN6swconv23mfma_s8_tiles_supportedEPKabRKNS_11Conv2dShapeE")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_bool, ctypes.POINTER(Shape)]
    return f(4096, True, ctypes.byref(s))


@pytest.mark.parametrize("supported,shapes", [
    (s8_tiles_supported, [(4, 64, 16 * n, 56, 56, 3, 3, 1, 1) for n in range(1, 101)]),
    (lambda s: split_supported("few", s), [(1, 40, 16 * n, 97, 101, 5, 5, 1, 2) for n in range(1, 101)]),
], ids=["s8_tiles", "few"])
def test_plans_of_a_network_s_layers_are_found_once(supported, shapes):
    """A hundred shapes in turn: none is searched for again (7 to 12 us a shape when they are, of which the call from here is 1)."""
    shapes = [shape(*s) for s in shapes]

    def once():
        start = time.perf_counter()
        took = [supported(s) for s in shapes]
        assert all(took)
        return time.perf_counter() - start

    first = once()
    assert min(once() for _ in range(20)) < first / 2.5


@pytest.mark.parametrize("supported,s", [
    (s8_tiles_supported, (1, 16, 1, 1, 100_000_000, 1, 1, 1, 0)), (s8_tiles_supported, (1, 16, 1, 1, 60_000_000, 1, 9, 1, 4)),
    (lambda s: split_supported("few", s), (1, 2, 1, 1, 100_000_000, 1, 7, 1, 3)),
], ids=["s8_tiles", "s8_tiles-9", "few"])
def test_plans_of_wide_images_take_no_longer(supported, s):
    """The search goes over the tile widths that there are, not over all numbers of parts of a row."""
    s = shape(*s)
    binding.lib()
    start = time.perf_counter()
    supported(s)
    assert time.perf_counter() - start < 0.01
