"""The split-input GEMM on inputs of more than 4 GiB (accepted: n * d_in below 2^32 elements): the tokens
of the tiles from whose start X ends just below and above a multiple of 2^32 bytes, and of the first and
last tile, against the oracle's GEMM reference."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
from workloads import LayerSpec, make_layer

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is marked gpu
    pytest.skip("no GPU", allow_module_level=True)

import paper_2606_12876_amd as A  # noqa: E402
from gpu_helpers import GpuLayer, out_values, check_close  # noqa: E402


@pytest.mark.parametrize("d_out,d_in,n,k,rb,nb", [
    (64, 8192, 263141, 1, 4, 8),       # X a little above 4 GiB
    (40, 65536, 32772, 2, 3, 12),
    (24, 32768, 131071, 1, 1, 4),      # just below 8 GiB, the most that is accepted
])
def test_tokens_around_the_wrap(d_out, d_in, n, k, rb, nb):
    L = make_layer(LayerSpec("big", d_out, d_in, M=k, seed=41))
    X = torch.empty((n, d_in), dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    for r in range(0, n, 16384):
        X[r:r + 16384] = torch.randn((min(16384, n - r), d_in), device="cuda", generator=g)
    Y = torch.full((n + 1, d_out), 3.0, dtype=torch.float32, device="cuda")
    tile, left = 16 * nb, {0, n}
    left |= {n - m * ((1 << 31) // d_in) for m in (1, 2) if n > m * ((1 << 31) // d_in)}   # 2^32 m bytes of X are left
    rows = sorted({r for c in left for r in range(c // tile * tile - tile, c // tile * tile + 2 * tile) if 0 <= r < n})
    with GpuLayer(L.codes, L.codebooks, L.scales) as gl:
        st = A.lib.aqmb_test_gemm_mid(ctypes.c_void_p(gl.handle), k, ctypes.c_void_p(X.data_ptr()), n,
                                      ctypes.c_void_p(Y.data_ptr()), int(A.DType.F32), rb, nb,
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == A.Status.OK, A.last_error()
        torch.cuda.synchronize()
    assert torch.all(Y[n] == 3.0), "wrote past the last token"
    xv = X[torch.tensor(rows, device="cuda")].float().cpu().numpy().astype(np.float64)
    ref = oracle.gemm_reference(xv, L.codes, L.codebooks, L.scales, k)
    check_close(out_values(Y[torch.tensor(rows, device="cuda")]), ref, "f32", f"{d_out}x{d_in} n={n} k={k}")
