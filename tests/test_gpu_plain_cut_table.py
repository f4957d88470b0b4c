"""Count-and-score scans whose log-factorial table is cut to what fits in LDS
(12348 entries with 8 pivots j per tile, 8316 with 4): the lookups of a row of
more samples run past the table, into the staging buffers, whose last 4 KB every
wave rewrites in its own time while the others score.  SNPs with one common
genotype (0, 1 or 2) put one row of most triplets at every count from just
inside the table to past the 1024 entries that follow it; scores, hits and
bounds equal the popcount kernel's bit for bit."""
import pytest
import torch

from paper_2201_10956_amd import epi3

pytestmark = pytest.mark.gpu
ENTRIES = {8: 12348, 4: 8316}


@pytest.fixture
def tile():
    def use(jb):
        epi3.tile_rules_clear()
        epi3.tile_rule("mfma_fp4", 0, 0, jb)
    yield use
    epi3.tile_rules_clear()
    epi3.load_tiles()
    epi3.set_scan_select("auto")


def study(M, N, entries, frac, seed):
    """Genotypes (uint8 [M][N] on the GPU) and phenotype.  A SNP's share of samples
    with another than its common genotype is drawn so that a triplet's largest row
    holds about entries - 150 to entries + 1200 samples."""
    g = torch.Generator().manual_seed(seed)
    lo, hi = (1 - ((entries + d) / N) ** (1 / 3) for d in (1200, -150))
    p = lo + (hi - lo) * torch.rand(M, 1, generator=g)
    common = torch.randint(0, 3, (M, 1), generator=g)
    other = (common + 1 + torch.randint(0, 2, (M, N), generator=g)) % 3
    geno = torch.where(torch.rand(M, N, generator=g) < p, other, common).to(torch.uint8)
    pheno = (torch.rand(N, generator=g) < frac).to(torch.uint8)
    top = (geno == common).float().cuda()
    seen = torch.zeros(N + 2, dtype=torch.bool, device="cuda")
    for i in range(M - 2):
        n = ((top[i] * top[i + 1:]) @ top[i + 2:].T).long()  # rows j > i, columns k > i + 1
        j = torch.arange(M - 1 - i, device="cuda")[:, None]
        seen[n[torch.arange(M - 2 - i, device="cuda")[None, :] >= j] + 1] = True
    return geno.cuda(), pheno.numpy(), seen


@pytest.mark.parametrize("frac", [0.5, 0.06, 0.9])
@pytest.mark.parametrize("jb,N", [(8, 16384), (8, 17638), (4, 11878)])
def test_rows_around_the_cut(tile, jb, N, frac):
    tile(jb)
    e = ENTRIES[jb]
    geno, pheno, seen = study(300, N, e, frac, N + jb)
    assert seen[e - 2: e + 1026].all(), "a row of every count"
    ds = epi3.encode(geno, pheno)
    want = epi3.scan_tables(ds, "valu", counts=False)[1]
    for _ in range(3):
        assert torch.equal(epi3.scan_tables(ds, "mfma_fp4", counts=False)[1], want)


@pytest.mark.parametrize("jb,N", [(8, 16384), (4, 11878)])
def test_selected_by_bound(tile, jb, N):
    tile(jb)
    geno, pheno, _ = study(220, N, ENTRIES[jb], 0.5, 7 * jb)
    ds = epi3.encode(geno, pheno)
    want = epi3.scan_topk(ds, 200, variant="valu")
    epi3.set_scan_select("bounded")
    assert epi3.scan_topk(ds, 200, variant="mfma_fp4").tobytes() == want.tobytes()


def test_tables_of_one_launch(tile):
    """Tables shorter than the cut, of its length, and longer."""
    tile(8)
    sets = []
    for x, (M, N) in enumerate([(150, 16384), (70, 3000), (120, 12346), (90, 12347), (60, 17638)]):
        geno, pheno, _ = study(M, N, min(ENTRIES[8], N - 1300), 0.4, x)
        sets.append(epi3.encode(geno, pheno))
    for ds, h in zip(sets, epi3.BatchScanner(sets, 20, variant="mfma_fp4").run()):
        assert h.tobytes() == epi3.scan_topk(ds, 20, variant="valu").tobytes()
