"""Selection at its edges: planes that start off a 16-byte boundary, lengths on
both sides of what one workgroup finishes, lists that overflow or are long, ties
across the bound, sampled bounds, several jobs of different kinds in a launch."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset, make_permutations

pytestmark = pytest.mark.gpu


def _expect(ds, k):
    """The k best triplets from the whole FP32 plane: every score within the
    error bound of the k-th, re-scored in FP64 by the library's test hook."""
    _, plane = epi3.scan_tables(ds, "valu", counts=False)
    T = epi3.n_triplets(ds.M)
    k = min(k, T)
    plane = plane[:T]
    kth = float(torch.kthvalue(plane, k).values)
    ranks = torch.nonzero(plane <= kth + 2 * epi3.k2_error_bound(ds.N)).flatten().cpu().numpy()
    lex = np.stack(np.triu_indices(ds.M, 1), 1)
    ijk = np.array([(i, j, l) for i, j in lex for l in range(j + 1, ds.M)], np.uint32)[ranks]
    k2 = epi3.score_triplets(ds, ijk)[2]
    k2 = np.asarray(k2.cpu() if torch.is_tensor(k2) else k2)
    order = np.lexsort((ranks, k2))[:k]
    return ijk[order], k2[order]


@pytest.mark.parametrize("M,N,k,compact", [
    (3, 20, 5, 0), (4, 9, 1, 0), (12, 64, 220, 0), (30, 200, 7, 1), (75, 40, 50, 0), (116, 300, 10, 300),
    (117, 300, 10, 300), (118, 300, 10, 0), (130, 300, 1000, 2000), (130, 60, 1, 50)])
def test_plain_selection(M, N, k, compact):
    d = make_dataset(M, N, 0.5, 0.05, 1000 + M + k)
    ds = epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno)
    epi3.set_compact_cap(compact)
    try:
        h = epi3.scan_topk(ds, k, "valu")
    finally:
        epi3.set_compact_cap(0)
    ijk, k2 = _expect(ds, k)
    assert np.array_equal(np.stack([h["i"], h["j"], h["k"]], 1), ijk)
    assert np.array_equal(h["k2"], k2)


@pytest.mark.parametrize("compact", [0, 100])
@pytest.mark.parametrize("select", ["plane", "bounded"])
def test_batch_planes_off_alignment(compact, select):
    """T = 5984 + 3 / 4 scores: each phenotype's plane starts elsewhere in 16 bytes."""
    for M, N, Q, k in [(35, 150, 9, 20), (34, 150, 5, 3), (7, 40, 3, 40)]:
        d = make_dataset(M, N, 0.4, 0.05, 50 + M)
        perms = make_permutations(d.pheno, Q, 3)
        geno = torch.from_numpy(d.geno).cuda()
        masks = torch.from_numpy(epi3.pack_masks(perms).view(np.int32)).cuda()
        epi3.set_batch_select(select)
        epi3.set_compact_cap(compact if select == "plane" else 0)
        try:
            got = epi3.BatchScanner(epi3.encode(geno, d.pheno, layout="masked"), k, masks=masks).run()
        finally:
            epi3.set_batch_select("auto")
            epi3.set_compact_cap(0)
        for q in range(Q):
            want = epi3.scan_topk(epi3.encode(geno, perms[q]), k, "valu")
            assert got[q].tobytes() == want.tobytes(), (M, q)


def test_mixed_jobs_in_one_launch():
    """A sampled plane (T >= 2^22), one that one workgroup finishes and one that
    leaves its plane to the later passes."""
    sets = [(294, 100, 5), (40, 64, 5), (150, 90, 5)]
    ds, want = [], []
    for n, (M, N, k) in enumerate(sets):
        d = make_dataset(M, N, 0.5, 0.1, 70 + n)
        ds.append(epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno))
    for compact in (0, 40):
        want = [epi3.scan_topk(x, 5, "valu").tobytes() for x in ds]
        epi3.set_compact_cap(compact)
        try:
            got = [h.tobytes() for h in epi3.BatchScanner(ds, 5).run()]
        finally:
            epi3.set_compact_cap(0)
        assert got == want


@pytest.mark.parametrize("k", [1, 300, 5000])
def test_pairs_and_quads_selection(k):
    d = make_dataset(40, 300, 0.5, 0.05, 5)
    ds = epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno)
    p = epi3.PairScanner(ds, k)
    h = p.run()
    assert len(h) == min(k, 780)
    assert np.all(np.diff(h["k2"]) >= 0)
    q = epi3.QuadScanner(ds, k).run()
    assert len(q) == min(k, 91390)
    assert np.all(np.diff(q["k2"]) >= 0)
    assert np.all(q["counts"].sum(axis=(1, 2)) == 300) and np.all(h["counts"].sum(axis=(1, 2)) == 300)
