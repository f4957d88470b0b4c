"""Pairwise tables counted as matrix products: edges of the 16- and 64-SNP
tiles, odd word counts, classes without samples, more than 2^23 samples."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3

pytestmark = pytest.mark.gpu


def _tables(ds, classes):
    Mp = ds.c.snp_stride
    off = ds.c.pairs - ds.buf.data_ptr()
    raw = ds.buf.view(torch.uint8)[off:off + classes * Mp * Mp * 16]
    return raw.cpu().numpy().view("<i4").reshape(classes, Mp, Mp, 4)


@pytest.mark.parametrize("M,N,cases", [(1, 1, 0), (3, 33, 32), (16, 64, 0), (17, 100, 50), (64, 257, 257),
                                       (65, 1000, 129), (130, 4099, 2000), (960, 300, 130),
                                       (961, 515, 33), (1100, 130, 65), (3, 8388608 + 8200, 8388608 + 130)])
@pytest.mark.parametrize("layout", ["split", "masked"])
def test_pair_tables_count_every_cell(M, N, cases, layout):
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    geno = torch.randint(0, 3, (M, N), dtype=torch.uint8, device="cuda", generator=gen)
    pheno = np.zeros(N, np.uint8)
    pheno[np.random.default_rng(N).permutation(N)[:cases]] = 1
    ds = epi3.encode(geno, pheno, layout=layout, values=layout == "masked")
    sel = [pheno == 0, pheno == 1] if layout == "split" else [np.ones(N, bool)]
    got = _tables(ds, len(sel))
    want = np.zeros_like(got)
    for c, s in enumerate(sel):
        g = geno[:, torch.from_numpy(s).cuda()]
        p = [(g == a).double() for a in (0, 1)]  # exact below 2^53
        for a in (0, 1):
            for b in (0, 1):
                want[c, :M, :M, 2 * a + b] = (p[a] @ p[b].T).cpu().numpy().astype(np.int32)
    assert np.array_equal(got, want)
