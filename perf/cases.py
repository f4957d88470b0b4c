"""Workloads that the library's speed is followed on: whole scans through the
Python entry points, over the sizes that the library is used at.

listed()      the named workloads
draw(rng)     one more workload of the same ranges
prepare(...)  what a program holds before the call: genotypes on the GPU, the
              phenotype on the host, the encoded data set's buffer, the scanner
run(state)    one pass, as a program makes it; returns every hit whole
work(case)    bytes and operations that the pass cannot do without
exact(...)    the hits' scores in 64 bits by plain torch, for the sizes where
              that takes seconds

A pass of a plain, pair, quad or batched scan starts from genotype bytes: the
data set is encoded into the buffer that the program keeps and then scanned.
A pass of a phenotype batch starts from an encoded genotype set, which
permutation tests scan again and again with new case masks.
"""
from math import comb, exp, log
import random

import numpy as np
import torch

from paper_2201_10956_amd import epi3


def listed():
    return [
        # a candidate-gene panel: the smallest call, where latency counts
        dict(name="plain_64x1024", kind="plain", M=64, N=1024, k=10, frac=0.5, maf_lo=0.05),
        # a small panel of odd sizes with fewer cases than controls
        dict(name="plain_157x2311", kind="plain", M=157, N=2311, k=25, frac=0.37, maf_lo=0.05),
        # one chromosome region in a mid-sized study (benchmark workload)
        dict(name="plain_512x4096", kind="plain", M=512, N=4096, k=100, frac=0.5, maf_lo=0.05),
        # the same of odd sizes, 30% cases
        dict(name="plain_1003x6007", kind="plain", M=1003, N=6007, k=50, frac=0.3, maf_lo=0.05),
        # the paper's smaller synthetic GPU shape (benchmark workload)
        dict(name="plain_2048x16384", kind="plain", M=2048, N=16384, k=1000, frac=0.5, maf_lo=0.01),
        # many SNPs, few samples: too many triplets for a score plane
        dict(name="plain_3100x2500", kind="plain", M=3100, N=2500, k=100, frac=0.45, maf_lo=0.05),
        # a serving loop that may not allocate: popcount scan in the static workspace
        dict(name="static_300x3000", kind="static", M=300, N=3000, k=20, frac=0.5, maf_lo=0.05),
        # second order (benchmark workload)
        dict(name="pairs_2048x16384", kind="pairs", M=2048, N=16384, k=1000, frac=0.5, maf_lo=0.01),
        # fourth order (benchmark workload)
        dict(name="quads_256x4096", kind="quads", M=256, N=4096, k=100, frac=0.5, maf_lo=0.05),
        # a permutation test: 64 phenotypes over one genotype set (default benchmark workload)
        dict(name="perm_1024x8192x64", kind="perm", M=1024, N=8192, Q=64, k=10, frac=0.4, maf_lo=0.05),
        # a permutation test of a small panel, odd sizes, a part-filled group of phenotypes
        dict(name="perm_203x1501x20", kind="perm", M=203, N=1501, Q=20, k=5, frac=0.4, maf_lo=0.05),
        # many studies of uneven shapes in one launch (benchmark workload)
        dict(name="batch_32", kind="batch", sets=32, m_lo=128, m_hi=1024, n_lo=1024, n_hi=16384,
             k=10, shapes=3000, maf_lo=0.05),
    ]


MOST_QUAD = comb(256, 4) * 4096  # sample-quads of the listed fourth-order scan


def _log_int(rng, lo, hi):
    return int(round(exp(rng.uniform(log(lo), log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "static", "pairs", "quads", "perm", "perm", "batch"])
    frac = round(rng.uniform(0.3, 0.7), 3)
    maf_lo = rng.choice([0.01, 0.05])
    if kind == "plain":
        if rng.random() < 0.15:  # beyond the score plane
            return dict(kind=kind, M=rng.randint(2950, 3100), N=_log_int(rng, 1100, 2500),
                        k=rng.choice([10, 50, 100]), frac=frac, maf_lo=maf_lo)
        M, N = _log_int(rng, 48, 2048), _log_int(rng, 500, 16384)
        return dict(kind=kind, M=M, N=N, k=_log_int(rng, 1, 1000), frac=frac, maf_lo=maf_lo)
    if kind == "static":
        return dict(kind=kind, M=_log_int(rng, 32, 570), N=_log_int(rng, 500, 8192),
                    k=_log_int(rng, 1, 100), frac=frac, maf_lo=maf_lo)
    if kind == "pairs":
        return dict(kind=kind, M=_log_int(rng, 100, 4096), N=_log_int(rng, 500, 16384),
                    k=_log_int(rng, 1, 1000), frac=frac, maf_lo=maf_lo)
    if kind == "quads":
        M, N = _log_int(rng, 24, 256), _log_int(rng, 500, 8192)
        while comb(M, 4) * N > MOST_QUAD:
            M = M * 7 // 8
        return dict(kind=kind, M=M, N=N, k=_log_int(rng, 1, 100), frac=frac, maf_lo=maf_lo)
    if kind == "perm":
        M, N, Q = _log_int(rng, 64, 1024), _log_int(rng, 800, 8192), rng.randint(8, 64)
        return dict(kind=kind, M=M, N=N, Q=Q, k=_log_int(rng, 1, 20), frac=frac, maf_lo=maf_lo)
    m_lo, n_lo = rng.randint(40, 128), rng.randint(500, 1024)
    return dict(kind=kind, sets=rng.randint(4, 32), m_lo=m_lo, m_hi=_log_int(rng, 2 * m_lo, 1024),
                n_lo=n_lo, n_hi=_log_int(rng, 2 * n_lo, 16384), k=_log_int(rng, 1, 20),
                shapes=rng.randrange(1 << 20), maf_lo=maf_lo)


# ---------------------------------------------------------------- inputs ----
def _generator(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed & 0x7fffffff)
    return g


def _study(M, N, frac, maf_lo, seed):
    """Genotypes (uint8 [M][N] on the GPU) in Hardy-Weinberg proportions with
    minor allele frequencies U(maf_lo, 0.5), and a phenotype (uint8 [N] on the
    host) of round(frac N) cases, drawn with twice the weight where all three
    genotypes of one planted triplet carry the minor allele."""
    g = _generator(seed)
    q = maf_lo + (0.5 - maf_lo) * torch.rand(M, 1, generator=g, device="cuda")
    geno = torch.empty(M, N, dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 25) // N)
    for m in range(0, M, step):
        u = torch.rand(min(step, M - m), N, generator=g, device="cuda")
        qq = q[m: m + step]
        geno[m: m + step] = (u >= (1 - qq) ** 2).to(torch.uint8) + (u >= 1 - qq * qq).to(torch.uint8)
    at = torch.randperm(M, generator=g, device="cuda")[:3]
    w = 1.0 + (geno[at] >= 1).all(0).to(torch.float32)
    key = -torch.log(1 - torch.rand(N, generator=g, device="cuda")) / w
    pheno = torch.zeros(N, dtype=torch.uint8, device="cuda")
    pheno[torch.argsort(key)[: int(round(frac * N))]] = 1
    return geno, pheno.cpu().numpy()


def _permutations(pheno, Q, seed):
    g = _generator(seed ^ 0x5bd1e995)
    order = torch.argsort(torch.rand(Q, pheno.size, generator=g, device="cuda"), dim=1)
    return torch.from_numpy(pheno).cuda()[order].cpu().numpy()


def _shapes(case):
    """(M, N, case fraction) of each data set of an uneven batch."""
    r = random.Random(case["shapes"])
    return [(r.randint(case["m_lo"], case["m_hi"]), r.randint(case["n_lo"], case["n_hi"]),
             r.uniform(0.3, 0.7)) for _ in range(case["sets"])]


def _inputs(case, seed):
    if case["kind"] == "batch":
        return [_study(M, N, f, case["maf_lo"], seed * 1009 + x)
                for x, (M, N, f) in enumerate(_shapes(case))]
    geno, pheno = _study(case["M"], case["N"], case["frac"], case["maf_lo"], seed)
    if case["kind"] == "perm":
        return geno, pheno, _permutations(pheno, case["Q"], seed)
    return geno, pheno


def prepare(case, seed):
    kind, k = case["kind"], case["k"]
    s = dict(kind=kind, k=k)
    if kind == "batch":
        s["studies"] = _inputs(case, seed)
        s["ds"] = [epi3.encode(g, p) for g, p in s["studies"]]
        s["scanner"] = epi3.BatchScanner(s["ds"], k)
        return s
    if kind == "perm":
        geno, pheno, perms = _inputs(case, seed)
        s["ds"] = epi3.encode(geno, pheno, layout="masked")
        masks = torch.from_numpy(epi3.pack_masks(perms).view(np.int32)).cuda()
        s["scanner"] = epi3.BatchScanner(s["ds"], k, masks=masks)
        return s
    s["geno"], s["pheno"] = _inputs(case, seed)
    if kind in ("static", "pairs"):  # bit planes are all that these scans read
        s["ds"] = epi3.encode(s["geno"], s["pheno"], values=False)
    else:
        s["ds"] = epi3.encode(s["geno"], s["pheno"])
    if kind == "plain":
        s["scanner"] = epi3.Scanner(s["ds"], k)
    elif kind == "pairs":
        s["scanner"] = epi3.PairScanner(s["ds"], k)
    elif kind == "quads":
        s["scanner"] = epi3.QuadScanner(s["ds"], k)
    return s


# ------------------------------------------------------------------ pass ----
_INDEX = {"pairs": ("i", "j"), "quads": ("i", "j", "k", "l")}


def _hits(kind, h):
    return {f: h[f] for f in _INDEX.get(kind, ("i", "j", "k")) + ("k2_f32", "k2", "counts")}


def run(s):
    kind = s["kind"]
    if kind == "perm":
        return _hits(kind, np.concatenate(s["scanner"].run()))
    if kind == "batch":
        for ds, (geno, pheno) in zip(s["ds"], s["studies"]):
            epi3.encode(geno, pheno, into=ds)
        return _hits(kind, np.concatenate(s["scanner"].run()))
    if kind == "static":
        epi3.encode(s["geno"], s["pheno"], into=s["ds"], values=False)
        return _hits(kind, epi3.scan_topk_static(s["ds"], s["k"]))
    epi3.encode(s["geno"], s["pheno"], into=s["ds"], values=kind != "pairs")
    return _hits(kind, s["scanner"].run())


def work(case):
    """Each genotype byte and phenotype read once, each hit written once (a
    phenotype batch: its case masks in place of the phenotype); a multiplication
    and an addition per sample and counted cell: 4 cells of a pair, 8 of a
    triplet, 16 of a quad (the other cells follow from lower-order counts)."""
    kind = case["kind"]
    if kind == "batch":
        sh = _shapes(case)
        return dict(bytes=float(sum(M * N + N + 240 * case["k"] for M, N, _ in sh)),
                    flops=float(sum(16 * comb(M, 3) * N for M, N, _ in sh)))
    M, N, k = case["M"], case["N"], case["k"]
    if kind == "pairs":
        return dict(bytes=float(M * N + N + 96 * k), flops=float(8 * comb(M, 2) * N))
    if kind == "quads":
        return dict(bytes=float(M * N + N + 680 * k), flops=float(32 * comb(M, 4) * N))
    if kind == "perm":
        Q = case["Q"]
        return dict(bytes=float(M * N + Q * N / 8 + 240 * k * Q), flops=float(16 * comb(M, 3) * N * Q))
    return dict(bytes=float(M * N + N + 240 * k), flops=float(16 * comb(M, 3) * N))


# ----------------------------------------------------- scores in 64 bits ----
def _planes(geno, sel):
    """0/1 planes [M][3][n] float32 of the samples in sel."""
    g = geno[:, sel]
    return torch.stack([(g == v).to(torch.float32) for v in range(3)], 1)


def _logs(N):
    n = torch.arange(1, N + 2, dtype=torch.float64, device="cuda")
    return torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"), torch.log(n).cumsum(0)])


def _k2(n0, n1, L):
    """Sum over the last axis (table rows) of L[r + 1] - L[r0] - L[r1]."""
    a, b = n0.to(torch.int64), n1.to(torch.int64)
    return (L[a + b + 1] - (L[a] + L[b])).sum(-1)


def _lowest(best, new, k):
    v = torch.cat([best, new])
    return v if v.numel() <= k else torch.topk(v, k, largest=False).values


def _pairs_exact(geno, pheno, k):
    case = torch.from_numpy(pheno).cuda().bool()
    M, L = geno.shape[0], _logs(pheno.size)
    P = [_planes(geno, ~case), _planes(geno, case)]
    best = torch.empty(0, dtype=torch.float64, device="cuda")
    for i in range(M - 1):
        n = [p[i] @ p[i + 1:].reshape(3 * (M - 1 - i), -1).T for p in P]  # [3][3 j]
        n = [x.reshape(3, M - 1 - i, 3).permute(1, 0, 2).reshape(-1, 9) for x in n]
        best = _lowest(best, _k2(n[0], n[1], L), k)
    return best.sort().values


def _triplets_exact(geno, pheno, k):
    case = torch.from_numpy(pheno).cuda().bool()
    M, L = geno.shape[0], _logs(pheno.size)
    P = [_planes(geno, ~case), _planes(geno, case)]
    best = torch.empty(0, dtype=torch.float64, device="cuda")
    for i in range(M - 2):
        m = M - 1 - i
        at = torch.triu_indices(m, m, 1, device="cuda")
        n = []
        for p in P:
            rest = p[i + 1:].reshape(3 * m, -1)
            t = torch.stack([(p[i, a] * rest) @ rest.T for a in range(3)])  # [a][3 j][3 k]
            t = t.reshape(3, m, 3, m, 3).permute(1, 3, 0, 2, 4).reshape(m, m, 27)
            n.append(t[at[0], at[1]])
        for x in range(0, n[0].shape[0], 1 << 18):
            best = _lowest(best, _k2(n[0][x: x + (1 << 18)], n[1][x: x + (1 << 18)], L), k)
    return best.sort().values


def _quads_exact(geno, pheno, k):
    case = torch.from_numpy(pheno).cuda().bool()
    M, L = geno.shape[0], _logs(pheno.size)
    P = [_planes(geno, ~case), _planes(geno, case)]
    best = torch.empty(0, dtype=torch.float64, device="cuda")
    for i in range(M - 3):
        for j in range(i + 1, M - 2):
            m = M - 1 - j
            at = torch.triu_indices(m, m, 1, device="cuda")
            n = []
            for p in P:
                rest = p[j + 1:].reshape(3 * m, -1)
                t = torch.stack([(p[i, a] * p[j, b] * rest) @ rest.T for a in range(3) for b in range(3)])
                t = t.reshape(9, m, 3, m, 3).permute(1, 3, 0, 2, 4).reshape(m, m, 81)
                n.append(t[at[0], at[1]])
            best = _lowest(best, _k2(n[0], n[1], L), k)
    return best.sort().values


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if sum(comb(M, 3) for M, _, _ in _shapes(case)) > 3e7:
            return None
        v = torch.cat([_triplets_exact(g, p, case["k"]) for g, p in _inputs(case, seed)])
    elif kind == "perm":
        if comb(case["M"], 3) * case["Q"] > 3e7:
            return None
        geno, _, perms = _inputs(case, seed)
        v = torch.cat([_triplets_exact(geno, p, case["k"]) for p in perms])
    elif kind == "pairs":
        v = _pairs_exact(*_inputs(case, seed), case["k"])
    elif kind == "quads":
        if comb(case["M"], 2) > 4000:
            return None
        v = _quads_exact(*_inputs(case, seed), case["k"])
    else:
        if comb(case["M"], 3) > 3e7:
            return None
        v = _triplets_exact(*_inputs(case, seed), case["k"])
    v = v.cpu().numpy()
    none = {f: None for f in _INDEX.get(kind, ("i", "j", "k")) + ("counts",)}
    return dict(none, k2=v, k2_f32=v)
