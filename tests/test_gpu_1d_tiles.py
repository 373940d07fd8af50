"""1-D rows at any 4-byte address and of any length, on both sides of the lengths at which the tiles change."""
import numpy as np
import pytest

from paper_2310_05218_amd import inputs
from parity import assert_f32_parity, assert_guards_intact, guarded_empty

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    import paper_2310_05218_amd as sw

    return sw


@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("k", [2, 9, 22, 64])
@pytest.mark.parametrize("rows,length", [(1, 64), (3, 1023), (2, 1025), (5, 4097), (7, 4098), (256, 2111), (300, 2050), (520, 1027), (511, 1021), (130, 8191)])
def test_rows_of_any_length(torch, sw, oracle, rows, length, k, shift):
    """One, two and four passes a tile; NaN around the input must not be reached."""
    x, w = inputs.normal_f32((rows, length), 7600 + length), inputs.normal_f32((k,), 7700 + k)
    buf = torch.full((x.size + 12,), float("nan"), device="cuda")
    xd = buf[4 + shift:4 + shift + x.size].view(rows, length)
    xd.copy_(torch.from_numpy(x))
    y_ref, d = oracle.conv1d(x, w, 1, k // 2)
    ybuf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
    sw.sw_conv1d(xd, torch.from_numpy(w).cuda(), 1, k // 2, out=out)
    assert sw.sw_last_kernel().startswith("sliding_1d_kernel"), sw.sw_last_kernel()
    assert_f32_parity(out.cpu().numpy(), y_ref, d, f"{rows} {length} {k}")
    assert_guards_intact(ybuf, front, n, guard)
    y_ref, d = oracle.pool1d(x, k, 1, 1)
    y = sw.sw_pool1d(xd, k, 1, 1)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("rows,length,k", [
    (3, 1, 2), (5, 2, 2), (4, 3, 3), (7, 5, 4), (2, 17, 16), (9, 63, 64), (600, 58, 6), (9001, 13, 5),      # rows of a few values; more than the workgroups of a launch
    (11, 235, 9), (11, 236, 9), (11, 237, 9), (3, 241, 2), (3, 242, 2), (5, 179, 64), (5, 180, 64), (5, 181, 64),      # on both sides of a value per thread
])
def test_short_rows(torch, sw, oracle, rows, length, k, shift):
    x, w = inputs.normal_f32((rows, length), 7800 + length), inputs.normal_f32((k,), 7900 + k)
    buf = torch.full((x.size + 12,), float("nan"), device="cuda")
    xd = buf[4 + shift:4 + shift + x.size].view(rows, length)
    xd.copy_(torch.from_numpy(x))
    for pad in {0, k // 2, k - 1}:
        if length + 2 * pad < k:
            continue
        y_ref, d = oracle.conv1d(x, w, 1, pad)
        ybuf, out, front, n, guard = guarded_empty(torch, y_ref.shape, torch.float32)
        sw.sw_conv1d(xd, torch.from_numpy(w).cuda(), 1, pad, out=out)
        assert sw.sw_last_kernel().startswith("sliding_1d_kernel"), sw.sw_last_kernel()
        assert_f32_parity(out.cpu().numpy(), y_ref, d, f"{rows} {length} {k} {pad}")
        assert_guards_intact(ybuf, front, n, guard)
    if length >= k:
        for mode in (0, 1):
            y_ref, d = oracle.pool1d(x, k, 1, mode)
            y = sw.sw_pool1d(xd, k, 1, mode).cpu().numpy()
            if mode == 1:
                assert np.array_equal(y.astype(np.float64), y_ref)
            else:
                assert_f32_parity(y, y_ref, d, f"average {rows} {length} {k}")
