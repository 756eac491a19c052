"""The split-input GEMM where codeword 0 of a codebook is not finite and no group of the layer names it:
the padding groups of the last code slice hold code 0, and their weights must not reach the sums."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
from workloads import LayerSpec, make_layer, make_activations

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is marked gpu
    pytest.skip("no GPU", allow_module_level=True)

import paper_2606_12876_amd as A  # noqa: E402
from gpu_helpers import GpuLayer, out_values, check_close, to_dev, act_values  # noqa: E402


@pytest.mark.parametrize("bits", [0x7C00, 0xFC00, 0x7E00], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("d_in,B,rb,nb", [(8, 8, 1, 2), (72, 8, 2, 8), (200, 8, 4, 8), (1016, 8, 3, 12), (264, 4, 1, 4),
                                          (136, 4, 3, 8)])
def test_unused_codeword_zero(d_in, B, rb, nb, bits):
    L = make_layer(LayerSpec("pad", 70, d_in, M=2, B=B, seed=50 + d_in))
    codes, books = np.maximum(L.codes, 1), L.codebooks.copy()
    ref_books = books.copy()
    books[:, 0] = bits
    Xbits = make_activations(L, 150, "bf16")
    Y = torch.empty((150, 70), dtype=torch.float32, device="cuda")
    X = to_dev(Xbits)
    with GpuLayer(codes, books, L.scales) as gl:
        for k in (1, 2):
            st = A.lib.aqmb_test_gemm_mid(ctypes.c_void_p(gl.handle), k, ctypes.c_void_p(X.data_ptr()), 150,
                                          ctypes.c_void_p(Y.data_ptr()), int(A.DType.F32), rb, nb,
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            assert st == A.Status.OK, A.last_error()
            torch.cuda.synchronize()
            ref = oracle.gemm_reference(act_values(Xbits, "bf16"), codes, ref_books, L.scales, k)   # codeword 0 unused
            check_close(out_values(Y), ref, "f32", f"d_in={d_in} B={B} k={k}")
