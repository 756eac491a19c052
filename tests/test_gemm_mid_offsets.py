"""Addresses of the split-input GEMM, evaluated on the host: the 32-bit offsets within a token tile must be
those of 64-bit arithmetic at every accepted size, also where the tokens after the tile span more than
2^32 bytes. (n * d_in is accepted up to 2^32 elements, 2^33 bytes.)"""
import ctypes

import pytest

A = pytest.importorskip("paper_2606_12876_amd", reason="libaqmb.so not built")

A.lib.aqmb_test_gemm_mid_offset.restype = ctypes.c_uint32
A.lib.aqmb_test_gemm_mid_offset.argtypes = [ctypes.c_int] * 6


@pytest.mark.parametrize("d_in", [8, 136, 8192, 32768, 65536, 1 << 20])
@pytest.mark.parametrize("nb", [1, 2, 5, 8, 12])
def test_offsets_do_not_wrap(d_in, nb):
    tile = 16 * nb
    most = ((1 << 32) - 1) // d_in                               # the most tokens a call may have
    for n in sorted({17, 100, most // 2 - 1, most // 2 + 3, most - 1, most}):
        n = min(n, (1 << 31) - 1)
        assert A.validate(A.make_desc(8, d_in, 4), 1, 1, n, A.DType.BF16, A.DType.BF16, 16, 16) == A.Status.OK
        tiles = (n + tile - 1) // tile
        wrap = max(0, n - (1 << 31) // d_in)                     # first token with 2^32 bytes of X after it
        for t in sorted({0, 1, wrap // tile, wrap // tile + 1, tiles // 2, tiles - 1} & set(range(tiles))):
            t0 = t * tile
            last = n - 1 - t0
            for row in sorted({0, 1, tile // 2, tile - 2, tile - 1, last - 1, last, last + 1} & set(range(tile))):
                want = min(row, n - 1 - t0) * d_in * 2
                for piece in (0, 7):
                    got = A.lib.aqmb_test_gemm_mid_offset(n, t0, nb, d_in, row, piece)
                    assert got == want + piece * 16, (n, t0, row, piece)
