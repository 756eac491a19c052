"""The code search's matrix-core filter (8-bit codes, beams of at most 8) at its edges, against the
oracle's binary32 searches, codes and errors bit for bit.

The filter discards candidates by an error bound and hands a group to an exhaustive search where the
bound cannot serve, so what can go wrong is a candidate wrongly discarded: partly filled waves (32
groups or rows each), every padded beam width, ties in number (more near-equal candidates than a
list holds), scales that are negative or zero, and magnitudes at both ends of fp16 (codewords in
fp16's subnormal range, codewords and weights near its largest values, ranges of 10^5 within one
codebook)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from oracle import formats
from workloads import LayerSpec, make_layer, make_weights

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts too; every test here is marked gpu
    pytest.skip("no GPU", allow_module_level=True)

import paper_2606_12876_amd as A  # noqa: E402
from gpu_helpers import to_dev  # noqa: E402


def _vary(kind, L, W, rng):
    """fp16 bit patterns of the codebooks, scales and weights of one kind of input."""
    f = formats.f16_bits_to_f64
    C, s, w = f(L.codebooks), f(L.scales), f(W)
    if kind == "ties":                       # half of every codebook twice, 30 codewords the same
        C[:, 128:] = C[:, :128]
        C[:, 10:40] = C[:, 10:11]
    elif kind == "signs":
        s = np.where(np.arange(len(s)) % 2 == 0, -s, s)
        s[0] = 0.0
    elif kind == "small":                    # codewords of 1e-6: subnormal in fp16
        C, w = C * 1e-4, w * 1e-3
    elif kind == "large":
        C, w = C * 3e5, w * 1e5
    elif kind == "spread":
        C = C * 10.0 ** rng.uniform(-4, 1, size=C.shape[:2] + (1,))
        w = w * 10.0 ** rng.uniform(-2, 2, size=(w.shape[0], 1))
    to = lambda a: np.asarray(a, dtype=np.float64).astype(np.float16).view(np.uint16)
    return to(C), to(s), to(w)


CASES = [("plain", 1, 8, 1, 1), ("plain", 3, 80, 2, 2), ("plain", 5, 264, 3, 3), ("plain", 33, 80, 3, 4),
         ("plain", 31, 256, 2, 5), ("plain", 65, 40, 3, 7), ("plain", 7, 104, 8, 8), ("ties", 9, 136, 3, 8),
         ("ties", 4, 64, 2, 1), ("signs", 6, 96, 3, 6), ("small", 5, 128, 3, 8), ("large", 5, 128, 3, 8),
         ("spread", 12, 128, 4, 4)]


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("kind,d_out,d_in,k,beam", CASES)
def test_filter_edges(kind, d_out, d_in, k, beam, weighted):
    L = make_layer(LayerSpec("f", d_out, d_in, M=k, seed=900 + d_out + beam))
    rng = np.random.default_rng(beam)
    Cb, sb, Wb = _vary(kind, L, make_weights(L), rng)
    f, G = formats.f16_bits_to_f64, d_in // 8
    desc = A.make_desc(d_out, d_in, k, 8)
    codes = torch.full((k, d_out, G), 0xAB, dtype=torch.uint8, device="cuda")
    errs = torch.full((d_out, G), -1.0, dtype=torch.float32, device="cuda")
    Wd, Cd, sd = to_dev(Wb).view(torch.float16), to_dev(Cb), to_dev(sb)
    if weighted:
        X = rng.normal(size=(G, 8, 40)) * np.exp(rng.normal(size=(G, 8, 1)))
        H = np.einsum("gin,gjn->gij", X, X) / 40
        H = np.ascontiguousarray((H + H.transpose(0, 2, 1)) / 2).astype(np.float32)
        A.beam_search_weighted(desc, k, beam, Wd, Cd, sd, to_dev(H), codes, errs)
        ref_c, ref_e = oracle.beam_search_codes_weighted_f32(f(Wb), f(Cb), f(sb), H.astype(np.float64), k, beam)
    else:
        A.beam_search(desc, k, beam, Wd, Cd, sd, codes, errs)
        ref_c, ref_e = oracle.beam_search_codes_f32(f(Wb), f(Cb), f(sb), k, beam)
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy().astype(np.int64), ref_c)
    assert np.array_equal(errs.cpu().numpy(), ref_e)
