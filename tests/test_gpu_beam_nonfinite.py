"""The code search on inputs that are not finite, on zero scales and on codebooks that are all ties, for every
beam that the matrix-core filter serves: codes and errors bit for bit against the decisions stated in
k_beam.hip, written out below in binary32. (The oracle's searches define the same order where every
candidate has an error; what is kept where candidates have none is stated here alone: a missing entry,
error inf, code 255 after codes 0, ranked behind all others.)"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from oracle import formats
from workloads import LayerSpec, make_layer, make_weights

F32 = np.float32


def _dot(a, b):
    acc = (a[..., 0] * b[..., 0]).astype(F32)
    for t in range(1, 8):
        acc = (acc + (a[..., t] * b[..., t]).astype(F32)).astype(F32)
    return acc


def stated_search(W, C, s, k, beam, H=None):
    """(codes [k][d_out][G], errors [d_out][G]) of the stated order; W, C, s, H as float32."""
    d_out, G = W.shape[0], W.shape[1] // 8
    codes, errors = np.zeros((k, d_out, G), dtype=np.int64), np.zeros((d_out, G), dtype=F32)
    missing_key = 0xFFFFFFFF
    with np.errstate(all="ignore"):
        for i in range(d_out):
            for j in range(G):
                w = W[i, 8 * j:8 * j + 8]
                kept, keys = [()], [0]                       # tuples and their keys
                for m in range(k):
                    ranks = [sum(q < key for q in keys) for key in keys]
                    cand = []
                    for p, tup in enumerate(kept):
                        r = w.copy()
                        for mm, c in enumerate(tup):
                            r = (r - (s[i] * C[mm, c]).astype(F32)).astype(F32)
                        if H is None:
                            d = (r - (s[i] * C[m]).astype(F32)).astype(F32)
                            e = _dot(d, d)
                        else:
                            b = _dot(H[j], r[None, :])
                            Q = _dot(C[m], np.stack([_dot(H[j][t][None, :], C[m]) for t in range(8)], axis=1))
                            e = (_dot(r, b) - (F32(2) * s[i] * _dot(C[m], b[None, :])).astype(F32)).astype(F32)
                            e = (e + (F32(s[i] * s[i]) * Q).astype(F32)).astype(F32)
                        cand += [(e[c], (ranks[p] << 8) | c, p) for c in np.flatnonzero(e == e)]
                    cand.sort()
                    keep = beam if m < k - 1 else 1
                    cand = cand[:keep]
                    err = cand[0][0] if cand else F32(np.inf)
                    new = [kept[p] + (key & 255,) for _, key, p in cand]
                    kept = new + [(0,) * m + (255,)] * (keep - len(new))
                    keys = [key for _, key, _ in cand] + [missing_key] * (keep - len(new))
                codes[:, i, j] = kept[0]
                errors[i, j] = err
    return codes, errors


def _inputs(kind, d_out, d_in, k, beam):
    L = make_layer(LayerSpec("nf", d_out, d_in, M=k, seed=700 + d_out + beam))
    f = formats.f16_bits_to_f64
    C, s, W = f(L.codebooks), f(L.scales), f(make_weights(L))
    H = None
    if kind == "codeword":                       # single codewords, the last stage's too
        C[0, 9, 3], C[k - 1, 200, 0], C[k - 1, 17, 7] = np.inf, np.nan, -np.inf
    elif kind == "few":                          # fewer finite codewords than tuples to keep
        C[0, 3:] = np.nan
        C[k - 1, :, 2] = np.nan
        C[k - 1, 77] = 0.01
    elif kind == "inf_book":                     # every error of a stage is inf
        C[0, :, 4] = np.inf
    elif kind == "nan_book":                     # no candidate of a stage has an error
        C[k - 1, :, 1] = np.nan
    elif kind == "weights":                      # some groups of a wave's 32
        W[::3, 5], W[1, 11], W[-1, -1] = np.nan, np.inf, -np.inf
    elif kind == "scales":
        s[::4], s[1], s[3], s[-1] = 0.0, np.nan, np.inf, -0.0
    elif kind == "zero":
        s[:] = 0.0
    elif kind == "zero_inf":                     # zero scales that an inf codeword does not let tie
        s[::2], C[0, 0, 2], C[k - 1, 3, 6] = 0.0, np.inf, -np.inf
    elif kind == "one_codeword":                 # every candidate of a stage ties
        C[:] = C[:, :1]
    to = lambda a: a.astype(np.float16)
    return to(C), to(s), to(W)


def _h(kind, G, rng):
    X = rng.normal(size=(G, 8, 40)) * np.exp(rng.normal(size=(G, 8, 1)))
    H = np.einsum("gin,gjn->gij", X, X) / 40
    H = np.ascontiguousarray((H + H.transpose(0, 2, 1)) / 2).astype(F32)
    if kind == "blocks":
        H[1], H[2, 3, 3], H[-1, 0, 1], H[-1, 1, 0] = 0.0, np.nan, np.inf, np.inf
    return H


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("kind,beam", [("plain", 5), ("one_codeword", 8), ("zero", 3)])
def test_stated_order_is_the_oracles(kind, beam, weighted):
    C, s, W = _inputs(kind, 3, 24, 3, beam)
    H = _h(kind, 3, np.random.default_rng(1)) if weighted else None
    got = stated_search(W.astype(F32), C.astype(F32), s.astype(F32), 3, beam, H)
    a = [x.astype(np.float64) for x in (W, C, s)]
    ref = (oracle.beam_search_codes_weighted_f32(*a, H.astype(np.float64), 3, beam) if weighted
           else oracle.beam_search_codes_f32(*a, 3, beam))
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


KINDS = ["codeword", "few", "inf_book", "nan_book", "weights", "scales", "zero", "zero_inf", "one_codeword"]
CASES = [(kind, k, beam, False) for kind in KINDS for k, beam in ((3, 8), (2, 3))]
CASES += [(kind, 3, beam, True) for kind in KINDS + ["blocks"] for beam in (5, 8)]
CASES += [("few", 3, 1, False), ("few", 2, 2, True), ("codeword", 1, 4, False), ("scales", 5, 6, True), ("few", 6, 4, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,k,beam,weighted", CASES)
def test_not_finite(kind, k, beam, weighted):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_12876_amd as A
    from gpu_helpers import to_dev
    d_out, d_in = 37, 40                         # 185 groups, 37 rows: ragged waves of either search
    C, s, W = _inputs(kind, d_out, d_in, k, beam)
    H = _h(kind, d_in // 8, np.random.default_rng(beam)) if weighted else None
    ref_c, ref_e = stated_search(W.astype(F32), C.astype(F32), s.astype(F32), k, beam, H)
    desc = A.make_desc(d_out, d_in, k, 8)
    codes = torch.full((k, d_out, d_in // 8), 0xAB, dtype=torch.uint8, device="cuda")
    errs = torch.full((d_out, d_in // 8), -1.0, dtype=torch.float32, device="cuda")
    dev = [to_dev(a.view(np.uint16)) for a in (W, C, s)]
    if weighted:
        A.beam_search_weighted(desc, k, beam, *dev, to_dev(H), codes, errs)
    else:
        A.beam_search(desc, k, beam, *dev, codes, errs)
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy().astype(np.int64), ref_c)
    assert np.array_equal(errs.cpu().numpy(), ref_e)
