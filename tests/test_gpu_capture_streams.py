"""Batches that are captured while other threads scan: both fork to the library's
second streams (two-kernel paths), and neither's work ends up in the other's."""
import threading

import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset, make_permutations

pytestmark = pytest.mark.gpu


def test_captures_beside_eager_scans():
    d = make_dataset(60, 700, 0.4, 0.05, 8)
    geno = torch.from_numpy(d.geno).cuda()
    ds = epi3.encode(geno, d.pheno)
    md = epi3.encode(geno, d.pheno, layout="masked")
    perms = make_permutations(d.pheno, 3, 5)
    masks = torch.from_numpy(epi3.pack_masks(perms).view(np.int32)).cuda()
    want = epi3.scan_topk(ds, 40, variant="valu")
    pwant = [epi3.scan_topk(epi3.encode(geno, p), 40, variant="valu") for p in perms]
    torch.cuda.synchronize()
    bad = []

    def guarded(work):
        def run():
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    work()
            except Exception as e:
                bad.append(repr(e))
        return run

    def eager():
        for _ in range(60):
            if epi3.scan_topk(ds, 40, variant="mfma").tobytes() != want.tobytes():
                bad.append("scan")

    def plain_batches():
        for k in range(1, 31):  # a capture of its own for each k
            for h in epi3.BatchScanner([ds, ds], k, variant="mfma").run():
                if h.tobytes() != want[:k].tobytes():
                    bad.append(("batch", k))

    def phenotype_batches():
        for k in range(1, 31):
            for h, w in zip(epi3.BatchScanner(md, k, masks=masks, variant="mfma").run(), pwant):
                if h.tobytes() != w[:k].tobytes():
                    bad.append(("phenotypes", k))

    threads = [threading.Thread(target=guarded(w)) for w in (eager, plain_batches, eager, phenotype_batches)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
