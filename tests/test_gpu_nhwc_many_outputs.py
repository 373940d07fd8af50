"""Channel-last window-in-LDS kernel: output channels by the million, so that a tile's bytes of y pass 2^30 and 2^31 (its stores go by
32-bit offsets from the tile)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pixels,C_out", [(8, (1 << 20) + 4), (256, 2_200_004)])
@pytest.mark.parametrize("dtype", ["float32", "int8"])
def test_many_output_channels(dtype, pixels, C_out):
    """Every output against a matrix product: int8 sums exact, fp32 |y - ref| <= 2e-6 sum |x w| (eight products, 2^-24 each and for each
    of their sums, twice over for both sides)."""
    torch = pytest.importorskip("torch")
    import paper_2310_05218_amd as sw

    g = torch.Generator(device="cuda").manual_seed(77)
    if dtype == "int8":
        C, call = 32, sw.sw_conv2d_s8_nhwc
        x = torch.randint(-128, 128, (1, 1, pixels, C), dtype=torch.int8, device="cuda", generator=g)
        w = torch.randint(-128, 128, (C_out, 1, 1, C), dtype=torch.int8, device="cuda", generator=g)
    else:
        C, call = 8, sw.sw_conv2d_nhwc
        x = torch.randn((1, 1, pixels, C), device="cuda", generator=g)
        w = torch.randn((C_out, 1, 1, C), device="cuda", generator=g)
    y = call(x, w, 1, 0).view(pixels, C_out)
    assert "nhwc_lds_kernel" in sw.sw_last_kernel(), sw.sw_last_kernel()
    xf, wf = x.view(pixels, C).float(), w.view(C_out, C).float()
    for p in range(0, pixels, 8):
        ref = xf[p:p + 8] @ wf.T                            # (int8: below 2^24, exact in fp32)
        if dtype == "int8":
            assert torch.equal(y[p:p + 8], ref.int())
        else:
            bound = 2e-6 * (xf[p:p + 8].abs() @ wf.abs().T)
            assert bool(((y[p:p + 8] - ref).abs() <= bound).all())
