"""Dequantization, each of its kernels, bit for bit against the oracle's stated order.

Every code width, output type and plane count. Small layers (a thread per group): few rows, 63, 64 and 65
groups, one group. Layers on units of 2, 4 and 8 rows x 64 groups and on output tiles: ragged in rows and
groups, and more units than waves run at once, so that a wave walks several. A layer past 148 MiB of
codes and output (tiles of 32 rows x 64 groups), ragged in both.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from workloads import LayerSpec, make_layer

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is marked gpu
    pytest.skip("no GPU", allow_module_level=True)

import paper_2606_12876_amd as A  # noqa: E402
from gpu_helpers import GpuLayer, TORCH_DT, A_DT  # noqa: E402

SMALL = [(1, 8), (3, 504), (4, 512), (5, 520), (8, 1024), (9, 1032), (70, 776)]


def _check(shape, M, B, ks, dts):
    d_out, d_in = shape
    L = make_layer(LayerSpec("dequant_units", d_out, d_in, M=M, B=B, seed=700 + d_out + d_in + B))
    with GpuLayer(L.codes, L.codebooks, L.scales) as gl:
        for k in ks:
            for dt in dts:
                # rows behind the matrix stay as they are
                W = torch.full((d_out + 1, d_in), 3.0, dtype=TORCH_DT[dt], device="cuda")
                A.dequant(gl.handle, k, W[:d_out], A_DT[dt])
                torch.cuda.synchronize()
                assert bool((W[d_out] == 3.0).all()), f"{shape} B={B} k={k} {dt}: wrote past the matrix"
                ref = oracle.dequant_canonical(L.codes, L.codebooks, L.scales, k, dt)
                got = W[:d_out].cpu()
                if dt == "f32":                              # binary32 values: compare their bits
                    got, ref = got.numpy().view(np.uint32), np.asarray(ref, dtype=np.float32).view(np.uint32)
                else:
                    got = got.view(torch.int16).numpy().view(np.uint16)
                assert np.array_equal(got, ref), f"{shape} B={B} k={k} {dt}"


@pytest.mark.parametrize("M,B", [(8, 8), (8, 4), (3, 16)])
@pytest.mark.parametrize("shape", SMALL)
def test_small_units(shape, M, B):
    _check(shape, M, B, range(1, M + 1), ("bf16", "f16", "f32"))


@pytest.mark.parametrize("shape,M,B,ks,dts", [
    ((1501, 1032), 4, 8, (1, 4), ("f32",)),                  # 2 rows, 4 waves
    ((1501, 1032), 2, 4, (2,), ("f32",)),
    ((1499, 3000), 8, 8, (1, 5, 8), ("bf16", "f32")),        # 4 rows, 4 waves
    ((1499, 3000), 2, 4, (1,), ("f16", "f32")),
    ((1499, 3000), 2, 16, (1, 2), ("bf16", "f32")),          # 16-bit codes: 8 rows at k = 1 to f32
    ((2047, 2048), 2, 8, (2,), ("f32",)),                    # 8 rows, 4 waves
    ((8237, 520), 8, 8, (2, 3, 8), ("bf16", "f32")),         # 65 groups: tiles (bf16); 8 waves from k = 3 (f32)
    ((8237, 520), 8, 4, (3, 8), ("f16", "f32")),             # 8 rows, 8 waves
    ((4100, 1720), 2, 8, (1, 2), ("f16",)),                  # 215 groups: tiles
    ((4097, 6000), 4, 8, (1, 4), ("bf16",)),                 # more than two tiles per compute unit: 8 rows
    ((32797, 16), 2, 4, (1, 2), ("bf16", "f32")),
    ((16397, 520), 2, 16, (1, 2), ("f16", "f32")),           # 16-bit codes: 8 rows, 8 waves at k = 1 to f32
    ((9473, 8232), 1, 8, (1,), ("bf16",)),                   # 159 MiB: output tiles
    ((4099, 4104), 5, 8, (3, 5), ("f16",)),                  # output tiles: units that leave compute units idle, k >= 5
])
def test_layers_of_many_units(shape, M, B, ks, dts):
    _check(shape, M, B, ks, dts)
