"""The allocation-free scan on both sides of where it counts on the matrix
cores: 80 SNPs, room in the static array (about 550 SNPs), tables that do not
fit, with and without the data set's own value planes."""
import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("values", [False, True])
@pytest.mark.parametrize("M,N,cases,k", [(3, 1, 0, 5), (79, 700, 300, 9), (80, 1, 1, 3), (80, 129, 0, 20),
                                         (97, 4097, 4096, 20), (130, 257, 100, 100), (300, 3000, 1400, 20),
                                         (120, 18000, 9000, 5), (520, 600, 300, 10), (545, 300, 100, 10),
                                         (560, 300, 150, 10), (575, 200, 60, 10)])
def test_static_equals_valu(M, N, cases, k, values):
    gen = torch.Generator(device="cuda").manual_seed(M * 7 + N)
    geno = torch.randint(0, 3, (M, N), dtype=torch.uint8, device="cuda", generator=gen)
    pheno = np.zeros(N, np.uint8)
    pheno[np.random.default_rng(M).permutation(N)[:cases]] = 1
    ds = epi3.encode(geno, pheno, values=values)
    sc = epi3.Scanner(ds, k, variant="valu")
    want = sc.run()
    if sc.cand_cap:  # more ties than the default capacity holds: refused as before
        with pytest.raises(epi3.Epi3Error) as e:
            epi3.scan_topk_static(ds, k)
        assert e.value.code == epi3.E_CAPACITY
        return
    assert epi3.scan_topk_static(ds, k).tobytes() == want.tobytes()
