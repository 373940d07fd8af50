"""The binding's own output extents agree with the library's over valid and invalid arguments."""
import itertools

from paper_2310_05218_amd import binding


def test_dim_matches_the_library():
    L = binding.lib()
    for n, k, st, pad, dil in itertools.product((-1, 0, 1, 2, 7, 8, 223, 65536), (0, 1, 2, 3, 7, 64), (0, 1, 2, 3, 9), (-1, 0, 1, 3, 40), (0, 1, 2, 6)):
        assert max(0, binding._dim(n, k, st, pad, dil)) == max(0, L.sw_out_dim_dilated(n, k, st, pad, dil)), (n, k, st, pad, dil)
        if dil == 1:
            assert binding._dim(n, k, st, pad) == L.sw_out_dim(n, k, st, pad), (n, k, st, pad)
