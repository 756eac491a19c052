"""The split-input GEMM (17 tokens and more, k <= 4) against the oracle's GEMM reference. test_named_tiles
runs every tile shape, named by a call that the tests alone use, whatever the library's rule would choose:
last tiles with one row or one token, inputs that end inside a 64-input chunk or a 16-group run, fewer
runs than waves, both code widths, rows that are not a multiple of four (scalar stores), numbers of token
tiles with and without the contiguous ranges per XCD. test_tile_edges calls aqmb_gemm at such sizes: which
kernel serves them is the rule's choice."""
from __future__ import annotations

import ctypes

import pytest
import torch

import oracle
from workloads import LayerSpec, make_layer, make_activations

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is marked gpu
    pytest.skip("no GPU", allow_module_level=True)

import paper_2606_12876_amd as A  # noqa: E402
from gpu_helpers import GpuLayer, out_values, check_close, to_dev, TORCH_DT, A_DT, act_values  # noqa: E402


@pytest.mark.parametrize("d_out,d_in,n,B,ks", [
    (16, 8, 17, 8, (1, 4)),            # one group
    (17, 72, 33, 8, (2,)),             # one row past a tile; 9 groups
    (33, 1000, 64, 8, (1, 2, 3, 4)),   # 125 groups: the last chunk holds 5
    (40, 2184, 65, 4, (1, 4)),         # nibble codes, the last run starts in the second half of a slice
    (4100, 256, 127, 8, (3,)),         # one token short of 8 blocks
    (4090, 520, 200, 8, (2, 4)),       # scalar stores
    (8200, 136, 250, 8, (1,)),         # tall, few inputs
    (12300, 64, 130, 4, (3,)),
    (2050, 1160, 700, 8, (4,)),        # several token tiles of uneven size
    (4090, 264, 50, 8, (1, 2)),        # a last tile with two tokens
    (11000, 200, 61, 8, (1, 3)),
    (11010, 328, 185, 4, (2, 4)),
])
def test_tile_edges(d_out, d_in, n, B, ks):
    L = make_layer(LayerSpec("mid", d_out, d_in, M=max(ks), B=B, seed=700 + n))
    Xbits = make_activations(L, n, "bf16", heavy_tail=True)
    X, Xv = to_dev(Xbits).view(torch.bfloat16), act_values(Xbits, "bf16")
    with GpuLayer(L.codes, L.codebooks, L.scales) as gl:
        for k in ks:
            ref = oracle.gemm_reference(Xv, L.codes, L.codebooks, L.scales, k)
            for ydt in ("bf16", "f32"):
                Y = torch.full((n + 1, d_out), 3.0, dtype=TORCH_DT[ydt], device="cuda")
                A.gemm(gl.handle, k, X, n, Y, A_DT[ydt])
                torch.cuda.synchronize()
                check_close(out_values(Y[:n]), ref, ydt, f"{d_out}x{d_in} n={n} B={B} k={k} {ydt}")
                assert torch.all(Y[n] == 3.0), "wrote past the last token"


SHAPES = [(1, 2), (1, 4), (2, 2), (2, 4), (2, 8), (3, 4), (3, 8), (3, 12), (4, 8)]


@pytest.mark.parametrize("B", [8, 4])
@pytest.mark.parametrize("rb,nb", SHAPES)
def test_named_tiles(rb, nb, B):
    # (row tiles, rows over, token tiles, tokens over, d_in): 1, 2 and multiples of 4 token tiles in the plain order, 3, 5 and 11 per XCD
    for rt, ro, tt, to, d_in in ((1, 1, 1, 1, 72), (2, 4, 3, -15, 1096), (1, 5, 5, -1, 328), (3, -12, 4, -7, 2184), (1, 0, 11, 0, 136)):
        d_out, n = 16 * rb * rt + ro, 16 * nb * tt + to
        L = make_layer(LayerSpec("named", d_out, d_in, M=4, B=B, seed=720 + n))
        Xbits = make_activations(L, n, "bf16", heavy_tail=True)
        X, Xv = to_dev(Xbits).view(torch.bfloat16), act_values(Xbits, "bf16")
        with GpuLayer(L.codes, L.codebooks, L.scales) as gl:
            for k, ydt in ((1, "f32"), (2, "bf16"), (3, "f32"), (4, "bf16"), (4, "f32")):
                Y = torch.full((n + 1, d_out), 3.0, dtype=TORCH_DT[ydt], device="cuda")
                st = A.lib.aqmb_test_gemm_mid(ctypes.c_void_p(gl.handle), k, ctypes.c_void_p(X.data_ptr()), n,
                                              ctypes.c_void_p(Y.data_ptr()), int(A_DT[ydt]), rb, nb,
                                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
                assert st == A.Status.OK, A.last_error()
                torch.cuda.synchronize()
                ref = oracle.gemm_reference(Xv, L.codes, L.codebooks, L.scales, k)
                check_close(out_values(Y[:n]), ref, ydt, f"{rb}x{nb} {d_out}x{d_in} n={n} B={B} k={k} {ydt}")
                assert torch.all(Y[n] == 3.0), "wrote past the last token"
