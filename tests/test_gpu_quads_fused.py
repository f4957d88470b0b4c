"""Quads counted and scored in one kernel (tables of up to about 12000 entries,
two kernels beyond): tile edges in every SNP, classes without samples, planes
against the vector-ALU scan of the same data set encoded without value planes."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,cases", [(4, 1, 1), (5, 40, 0), (17, 129, 128), (18, 300, 300), (33, 257, 100),
                                       (34, 1000, 1), (50, 513, 250), (64, 700, 300), (20, 11900, 6000),
                                       (20, 12300, 6000), (14, 65536, 30000)])
def test_planes_equal_popcount(M, N, cases):
    gen = torch.Generator(device="cuda").manual_seed(M * 11 + N)
    geno = torch.randint(0, 3, (M, N), dtype=torch.uint8, device="cuda", generator=gen)
    pheno = np.zeros(N, np.uint8)
    pheno[np.random.default_rng(M).permutation(N)[:cases]] = 1
    a = epi3.QuadScanner(epi3.encode(geno, pheno), 10)
    b = epi3.QuadScanner(epi3.encode(geno, pheno, values=False), 10)
    ha, hb = a.run(), b.run()
    assert ha.tobytes() == hb.tobytes()
    assert torch.equal(a.score_plane(), b.score_plane())
