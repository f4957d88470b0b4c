"""AUTO's choice on both sides of its lines at 64 and 80 SNPs and 2048 samples:
the hits and the whole score plane equal the vector-ALU scan's."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,cases", [(3, 2, 1), (63, 2048, 700), (64, 2047, 1000), (64, 2048, 1),
                                       (79, 1500, 700), (80, 1, 0), (80, 2, 1), (81, 33, 33),
                                       (95, 1023, 500), (130, 130, 0), (255, 97, 40), (300, 1000, 990)])
def test_auto_equals_valu(M, N, cases):
    epi3.load_tiles()
    d = make_dataset(M, N, 0.5, 0.05, 900 + M)
    pheno = np.zeros(N, np.uint8)
    pheno[np.random.default_rng(M).permutation(N)[:cases]] = 1
    ds = epi3.encode(torch.from_numpy(d.geno).cuda(), pheno)
    matrix = M >= 80 or (M >= 64 and N >= 2048)
    assert epi3.tile_for(ds, "auto") == ("mfma_fp4" if matrix else "valu")
    k = 20
    sc = epi3.Scanner(ds, k)
    want = epi3.Scanner(ds, k, variant="valu").run()
    assert sc.run().tobytes() == want.tobytes()
    _, plane = epi3.scan_tables(ds, "auto", counts=False)
    _, ref = epi3.scan_tables(ds, "valu", counts=False)
    assert torch.equal(plane, ref)
