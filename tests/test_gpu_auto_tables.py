"""AUTO's choice for scans that write their tables, on both sides of its lines (128
SNPs and 4000 samples, 256 and 1024, 16384 samples): tables and scores equal the
vector-ALU kernel's, and only matrix-core counts need a second kernel."""
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,matrix", [(64, 2048, False), (80, 33, False), (127, 4000, False), (128, 3999, False),
                                        (128, 4000, True), (255, 1024, False), (256, 1023, False),
                                        (256, 1024, True), (64, 16383, False), (64, 16384, True)])
def test_route_and_tables(M, N, matrix):
    epi3.load_tiles()
    d = make_dataset(M, N, 0.4, 0.05, M + N)
    ds = epi3.encode(torch.from_numpy(d.geno).cuda(), d.pheno)
    want = epi3.scan_tables(ds, "valu")
    epi3.timing_enable(True)
    try:
        epi3.timing_reset()
        got = epi3.scan_tables(ds, "auto")
        finished = epi3.timing_query(3)[1]
    finally:
        epi3.timing_enable(False)
        epi3.timing_reset()
    assert (finished > 0) == matrix
    for a, b in zip(got, want):
        assert torch.equal(a, b)
