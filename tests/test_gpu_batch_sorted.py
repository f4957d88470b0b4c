"""Uneven batches whose candidates are ordered by the sort (capacities above 16384):
data sets of fewer triplets than the capacity have shorter sort buffers than the
largest, each a power of two of its own.  Nine samples give thousands of exact ties,
so the order is by (K2, i, j, k) over whole lists; hits equal the single scans'."""
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["valu", "mfma_fp4"])
@pytest.mark.parametrize("sizes", [[98, 70, 55, 20], [55, 98], [50, 98, 3, 76, 1, 2, 61], [98, 97]])
@pytest.mark.parametrize("cap", [160000, 0])  # 0: default capacity, the overflow's retry
def test_hits_equal_single_scans(sizes, variant, cap):
    sets = []
    for M in sizes:
        d = make_dataset(M, 9, 0.4, 0.05, M)
        sets.append(epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno))
    got = epi3.BatchScanner(sets, 300, variant=variant, cand_cap=cap).run()
    for ds, h in zip(sets, got):
        assert h.tobytes() == epi3.scan_topk(ds, 300, variant=variant, cand_cap=cap).tobytes()
