"""The kernel that counts and scores a plain scan's tiles at once (FP4): its
scores equal the popcount kernel's bit for bit at the edges of its tiles, of
the log-factorial table that it keeps in LDS (whole up to 12346 samples with 8
pivots j per tile and 8314 with 4, then cut, then the two-kernel path) and for
empty classes; SNPs of a single genotype put all samples in one row, whose
lookups lie past the cut table."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.fixture
def tile():
    def use(jb):
        epi3.tile_rules_clear()
        epi3.tile_rule("mfma_fp4", 0, 0, jb)
    yield use
    epi3.tile_rules_clear()
    epi3.load_tiles()


def encoded(M, N, frac, seed, uniform=()):
    d = make_dataset(M, N, frac, 0.05, seed)
    for snp, g in uniform:
        d.geno[snp] = g
    return epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno)


def same(ds):
    _, a = epi3.scan_tables(ds, "mfma_fp4", counts=False)
    _, b = epi3.scan_tables(ds, "valu", counts=False)
    assert torch.equal(a, b)


@pytest.mark.parametrize("jb", [8, 4, 2])
@pytest.mark.parametrize("M", [3, 4, 9, 16, 17, 18, 33, 34, 66, 131])
def test_tile_edges(tile, M, jb):
    tile(jb)
    same(encoded(M, 301, 0.4, M))


@pytest.mark.parametrize("N,frac", [(1, 0.0), (1, 1.0), (256, 0.5), (257, 0.0), (257, 1.0), (513, 0.02)])
def test_short_and_empty_classes(tile, N, frac):
    tile(8)
    same(encoded(21, N, frac, N))


@pytest.mark.parametrize("jb,N", [(8, 12346), (8, 12347), (8, 16384), (8, 17638), (8, 17639),
                                  (4, 8314), (4, 8315), (4, 11878), (4, 11879)])
@pytest.mark.parametrize("frac", [0.5, 0.05])
def test_table_limits(tile, jb, N, frac):
    tile(jb)
    same(encoded(26, N, frac, N, uniform=[(0, 0), (5, 0), (9, 1), (11, 2), (17, 0), (18, 2), (25, 1)]))


def test_few_workgroups(tile):
    """A workspace for one tile per pass leaves room for four workgroups."""
    tile(8)
    ds = encoded(90, 700, 0.5, 3)
    want = epi3.scan_tables(ds, "mfma_fp4", counts=False)[1]
    epi3.set_pass_bytes(1)
    try:
        got = epi3.scan_tables(ds, "mfma_fp4", counts=False)[1]
    finally:
        epi3.set_pass_bytes(0)
    assert torch.equal(got, want)
    assert np.isfinite(got.cpu().numpy()).all()
