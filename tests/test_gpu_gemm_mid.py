"""The split-input GEMM (17 tokens and more, k <= 4) at the edges of its tiles, against the oracle's
GEMM reference: every tile shape that its rule picks (16 to 64 weight rows, 2 to 8 token blocks),
last tiles with one row or one token, inputs that end inside a 64-input chunk or a 16-group run,
fewer runs than waves, 4-bit codes, rows that are not a multiple of four (scalar stores)."""
from __future__ import annotations

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
    (4100, 256, 127, 8, (3,)),         # 32-row tiles, 8 token blocks
    (4090, 520, 200, 8, (2, 4)),       # scalar stores
    (8200, 136, 250, 8, (1,)),         # 48- and 64-row tiles
    (12300, 64, 130, 4, (3,)),
    (2050, 1160, 700, 8, (4,)),        # several token tiles of uneven size
    (4090, 264, 50, 8, (1, 2)),        # 32 x 32 tiles, the last with two tokens
    (11000, 200, 61, 8, (1, 3)),       # 48 x 64 tiles
    (11010, 328, 185, 4, (2, 4)),      # 48 x 192 tiles
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
