"""Scores are summed in 32-bit fixed point with a step of 2^-s that depends on
the number of samples N.  A table of R rows looks up 3 R <= 243 entries, each
rounded to half a step, and the sum is rounded to FP32 once, so every score is
within 243 / 2 steps + 2^-24 K2 of the FP64 value; the shift changes with N,
and tables above 80 KB are read from global memory."""
import math

import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


def shift(N):
    most = N * math.log(2.0) + 81.0 * math.log(N / 81.0 + 1.0)
    s = 28
    while s > 0 and most * 2.0 ** s + 256.0 >= 2.0 ** 32:
        s -= 1
    return s


def tolerance(N, k2):
    return 122.0 * 2.0 ** -shift(N) + 2.0 ** -24 * np.abs(k2)


def k2_of(counts):
    n = counts.astype(np.int64)
    L = np.concatenate([[0.0], np.cumsum(np.log(np.arange(1, n.sum(axis=(1, 2)).max() + 2)))])
    return (L[n[:, 0] + n[:, 1] + 1] - (L[n[:, 0]] + L[n[:, 1]])).sum(axis=1)


def encoded(M, N, seed, frac=0.45, **kw):
    d = make_dataset(M, N, frac, 0.05, seed)
    return epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno, **kw)


@pytest.mark.parametrize("variant", ["valu", "mfma", "mfma_fp4"])
@pytest.mark.parametrize("N", [1, 2, 3, 95, 1000, 16384, 20478, 20479, 70000])
def test_triplet_scores_within_the_fixed_point_bound(N, variant):
    ds = encoded(19, N, 7 + N)
    counts, k2 = epi3.scan_tables(ds, variant)
    want = k2_of(counts.cpu().numpy())
    assert (np.abs(k2.cpu().numpy().astype(np.float64) - want) <= tolerance(N, want)).all()


@pytest.mark.parametrize("N", [1, 95, 16384, 20479])
@pytest.mark.parametrize("scan,values", [(epi3.scan_pairs, True), (epi3.scan_quads, True),
                                         (epi3.scan_quads, False)])
def test_pair_and_quad_scores_within_the_fixed_point_bound(N, scan, values):
    h = scan(encoded(17, N, 11 + N, values=values), 100)
    assert (np.abs(h["k2_f32"].astype(np.float64) - h["k2"]) <= tolerance(N, h["k2"])).all()


@pytest.mark.parametrize("variant", ["valu", "mfma_fp4"])
def test_batched_data_sets_keep_their_own_step(variant):
    """One launch over data sets whose tables differ in step and length: each
    score plane equals its plain scan's bit for bit."""
    shapes = [(40, 9000), (3, 5), (33, 64), (70, 700), (41, 30000), (18, 2100)]
    for some in (shapes[:4] + shapes[5:], shapes, shapes[3:4]):
        sets = [encoded(M, N, 31 * M + N) for M, N in some]
        b = epi3.BatchScanner(sets, 3, variant=variant)
        b.run()
        for x, ds in enumerate(sets):
            s = epi3.Scanner(ds, 3, variant)
            s.run()
            assert torch.equal(b.score_plane(x), s.score_plane()), (some[x], variant)
