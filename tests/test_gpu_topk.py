"""The k closest centroids where the first pass cannot tell rows apart: queries without a length in single precision
(against what the contract promises: similarity 0 to every centroid, the lower index first)."""

import numpy as np
import pytest
import torch

from gpu_util import DEV

pytestmark = pytest.mark.gpu
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.bfloat16}


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


def kind(siso, dtype):
    return {"f32": siso.F32, "bf16": siso.BF16, "fp8": siso.FP8}[dtype]


def directions(n, d, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(n, d, device=DEV, generator=g)


@pytest.mark.parametrize("dtype,K,k", [(t, K, 5) for t in ("f32", "bf16", "fp8") for K in (100, 1000, 2100, 8192)]
                         + [("fp8", 8192, 32), ("f32", 8200, 32), ("bf16", 513, 32)])
def test_topk_of_queries_without_length(siso, dtype, K, k):
    """From fewer groups of rows than k to more than a list holds, through every kernel; zero queries, and queries whose
    squared length underflows (the codes of an 8-bit cache have a length whatever the scale: zero queries only).
    The lowest rows that can be chosen are the answer: one of a group holds a NaN, one has no length itself."""
    d = 256
    print(f"case: topk without length {dtype} K={K} k={k}", flush=True)
    rows = directions(K, d, K)
    rows[1, 7] = float("nan")
    rows[2] = 0
    rows[15, 0] = float("nan")
    q = directions(6, d, 5)
    q[0] = 0
    q[3] = 0
    short = [0, 3]
    if dtype != "fp8":
        q[4] = 1e-25 * torch.sign(q[4])     # elements whose squares are below the smallest number
        q[5] *= 1e-30
        short += [4, 5]
    cache = siso.SisoCache(d, K, kind(siso, dtype))
    cache.load(rows.to(TORCH[dtype]))
    idx, sim = cache.lookup_topk(q.to(TORCH[dtype]), k)
    want = [i for i in range(K) if i not in (1, 15)][:k]
    for s in short:
        assert idx[s].tolist() == want, s
        assert (sim[s] == 0).all(), s
    # the queries beside them
    assert (sim[1] > 0).all() and (sim[2] > 0).all() and (np.diff(sim[1].cpu().numpy()) <= 0).all()


@pytest.mark.parametrize("dtype,d", [("f32", 384), ("bf16", 768)])
def test_topk_of_very_short_queries(siso, dtype, d):
    """The same directions at lengths from 1e18 to 1e-18: the same rows."""
    print(f"case: topk lengths {dtype} d={d}", flush=True)
    K, n, k = 3000, 40, 10
    rows = directions(K, d, 11).to(TORCH[dtype])
    q = torch.nn.functional.normalize(directions(n, d, 12)).to(TORCH[dtype])
    cache = siso.SisoCache(d, K, kind(siso, dtype))
    cache.load(rows)
    base = cache.lookup_topk(q, k)
    for e in (59, 20, -20, -45, -49, -51, -59):   # (powers of two: the elements stay what they are)
        got = cache.lookup_topk((q.float() * 2.0 ** e).to(q.dtype), k)
        assert torch.equal(got[0], base[0]), e
        assert (got[1] - base[1]).abs().max() < 1e-5, e
