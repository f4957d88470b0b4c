"""Phenotype batches counted and scored in one kernel (FP4, up to about 11400
samples; two kernels beyond): score planes at the edges of its tiles."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset, make_permutations

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,Q", [(3, 1, 1), (5, 300, 64), (17, 129, 3), (18, 256, 32), (33, 513, 33),
                                   (50, 11000, 8), (20, 11400, 5), (20, 11600, 5)])
def test_planes_equal_popcount_scans(M, N, Q):
    """Every score equals the phenotype's popcount scan bit for bit,
    phenotypes without cases or without controls among them."""
    d = make_dataset(M, N, 0.4, 0.05, 77 + M)
    perms = make_permutations(d.pheno, Q, 5)
    perms[0] = 0
    perms[-1] = 1
    geno = torch.from_numpy(d.geno).cuda()
    masks = torch.from_numpy(epi3.pack_masks(perms).view(np.int32)).cuda()
    epi3.set_batch_select("plane")
    try:
        b = epi3.BatchScanner(epi3.encode(geno, d.pheno, layout="masked"), 2, masks=masks)
        b.run()
        planes = [b.score_plane(q).clone() for q in range(Q)]
    finally:
        epi3.set_batch_select("auto")
    for q in range(Q):
        _, want = epi3.scan_tables(epi3.encode(geno, perms[q]), "valu", counts=False)
        assert torch.equal(planes[q], want), q
