"""Results and encode inputs through pinned memory: with and without an idle
block, above a block's size, and from several threads with streams of their own."""
import threading

import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu


def _sets(n, M=60, N=400):
    out = []
    for x in range(n):
        d = make_dataset(M + x, N + 31 * x, 0.5, 0.05, 300 + x)
        out.append((torch.from_numpy(d.geno).cuda(), d.pheno))
    return out


@pytest.mark.parametrize("k", [1, 4300, 4400])  # 240 bytes a hit: below and above 1 MB
def test_same_hits_without_an_idle_block(k):
    (geno, pheno), = _sets(1)
    ds = epi3.encode(geno, pheno)
    sc = epi3.Scanner(ds, k)
    want = sc.run().tobytes()
    epi3.release()
    assert sc.run().tobytes() == want
    epi3.release()
    assert epi3.BatchScanner([ds, ds], k).run()[1].tobytes() == want
    again = epi3.encode(geno, pheno)
    assert epi3.scan_topk(again, k).tobytes() == want


def test_encode_on_both_sides_of_a_block():
    """87300 and 87500 samples: tables and list just fit a block, or do not."""
    for N in (87300, 87500):
        gen = torch.Generator(device="cuda").manual_seed(N)
        geno = torch.randint(0, 3, (5, N), dtype=torch.uint8, device="cuda", generator=gen)
        pheno = (np.arange(N) % 3 == 0).astype(np.uint8)
        ds = epi3.encode(geno, pheno)
        h = epi3.scan_topk(ds, 10, "valu")
        g = geno.cpu().numpy().astype(np.int64)
        for r in h:
            code = 9 * g[r["i"]] + 3 * g[r["j"]] + g[r["k"]]
            want = np.stack([np.bincount(code[pheno == c], minlength=27) for c in (0, 1)])
            assert np.array_equal(r["counts"].reshape(2, 27), want)


def test_threads_with_streams_of_their_own():
    sets = _sets(6)
    want = [epi3.scan_topk(epi3.encode(g, p), 15).tobytes() for g, p in sets]
    torch.cuda.synchronize()
    bad = []

    def work(x):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            g, p = sets[x]
            ds = epi3.encode(g, p)
            for _ in range(10):
                epi3.encode(g, p, into=ds)
                if epi3.scan_topk(ds, 15).tobytes() != want[x]:
                    bad.append(x)

    threads = [threading.Thread(target=work, args=(x,)) for x in range(len(sets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
