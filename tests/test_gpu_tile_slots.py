"""Tiles handed out by the persistent matrix-core kernels: each workgroup starts with a
slot of its own and counters hand out the rest, so every slot is counted once
whatever the number of tiles is beside the workgroups (two per compute unit):
fewer than the eight parts, a remainder over the parts, about one, two and three
tiles per workgroup.  A missed slot leaves the score plane's fill."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset, make_permutations

pytestmark = pytest.mark.gpu


def tiles(M, JB=8):
    n = 0
    for j0 in range(0, M - 1, JB):
        last = min(j0 + JB - 1, M - 2)
        if last >= 1:
            n += -(-last // 16) * -(-(M - 1 - j0) // (256 // JB))
    return n


@pytest.fixture(autouse=True)
def eight_pivots():
    epi3.tile_rules_clear()
    epi3.tile_rule("mfma_fp4", 0, 0, 8)
    yield
    epi3.tile_rules_clear()
    epi3.load_tiles()


@pytest.mark.parametrize("M", [9, 17, 40, 49, 57, 64, 157, 158, 199, 205, 231, 259])
def test_every_slot_once(M):
    assert 1 <= tiles(M) <= 1024
    d = make_dataset(M, 97, 0.4, 0.05, M)
    ds = epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno)
    want = epi3.scan_tables(ds, "valu", counts=False)[1]
    for _ in range(3):
        assert torch.equal(epi3.scan_tables(ds, "mfma_fp4", counts=False)[1], want)


def test_jobs_of_one_launch():
    """The joint tile order of several data sets, some of one tile."""
    sets = []
    for x, M in enumerate([5, 40, 64, 9, 157, 33]):
        d = make_dataset(M, 97 + 31 * x, 0.4, 0.05, x)
        sets.append(epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno))
    got = epi3.BatchScanner(sets, 5, variant="mfma_fp4").run()
    for ds, h in zip(sets, got):
        assert h.tobytes() == epi3.scan_topk(ds, 5, variant="valu").tobytes()


@pytest.mark.parametrize("Q", [3, 33])
@pytest.mark.parametrize("M", [4, 12, 20, 37, 64, 75])
def test_phenotype_batches(M, Q):
    """Tiles of 64 triplets: from one to beyond three per compute unit."""
    d = make_dataset(M, 131, 0.4, 0.05, M)
    perms = make_permutations(d.pheno, Q, 5)
    g = torch.from_numpy(d.geno).cuda()
    masks = torch.from_numpy(epi3.pack_masks(perms).view(np.int32)).cuda()
    got = epi3.BatchScanner(epi3.encode(g, d.pheno, layout="masked"), 5, masks=masks).run()
    for q in (0, Q // 2, Q - 1):
        want = epi3.scan_topk(epi3.encode(g, perms[q]), 5, variant="valu")
        assert got[q].tobytes() == want.tobytes()


@pytest.mark.parametrize("M", [4, 9, 21, 34, 50])
def test_quads(M):
    d = make_dataset(M, 97, 0.4, 0.05, M)
    g = torch.from_numpy(d.geno).cuda()
    want = epi3.scan_quads(epi3.encode(g, d.pheno, values=False), 20)  # counted on the vector ALUs
    assert epi3.scan_quads(epi3.encode(g, d.pheno), 20).tobytes() == want.tobytes()
