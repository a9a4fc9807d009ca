"""The k closest centroids where the first pass cannot tell rows apart: queries without a length in single precision
(against what the contract promises: similarity 0 to every centroid, the lower index first)."""

import numpy as np
import pytest
import torch

from gpu_util import DEV, check_topk, to_host

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


# ---- the first pass sums every product in an order of its own: how far it may be off is bounded by the dimension
def spread_rows(K, many):
    """`many` rows of a cache of K that all lie in different groups of 16, in a mixed order."""
    assert K // many >= 33
    return (torch.arange(many) * (K // many) // 33 * 33 + 5)[torch.randperm(many, generator=torch.Generator().manual_seed(many))]


LONG = [("f32", 768, 6000, 9), ("f32", 1536, 6000, 30), ("f32", 3072, 6000, 60), ("f32", 4096, 8200, 1000), ("f32", 4096, 6000, 3),
        ("f32", 2047, 6000, 20), ("bf16", 4096, 6000, 40), ("bf16", 4096, 66000, 300), ("bf16", 4090, 6000, 90), ("bf16", 1536, 6000, 300)]


@pytest.mark.parametrize("dtype,d,K,n", LONG)
def test_topk_of_long_rows_with_equal_elements(siso, dtype, d, K, n):
    """Rows +-c, where every addition of a long sum rounds the same way, so that the sums of the first pass are off by up
    to d / 4 * 2^-24 (measured; every query and row by another share of that) and the cosines formed from them by
    hardly anything.  Query j has 40 rows: 30 that are multiples of it, of which ten are equal to it, and ten at cosines
    1 - 2e-5 i.  The answer: the multiples (equal up to rounding, in any order), then the ten by i."""
    print(f"case: topk of long rows {dtype} d={d} K={K} n={n}", flush=True)
    used = 4
    g = torch.Generator(device=DEV)
    g.manual_seed(d + n)
    rows = directions(K, d, 21).to(TORCH[dtype])
    q = directions(n, d, 22).to(TORCH[dtype])
    places = spread_rows(K, 40 * used).view(used, 40).to(DEV)
    for j in range(min(used, n)):
        s = (torch.randint(0, 2, (d,), device=DEV, generator=g) * 2 - 1).float()
        q[j] = ((0.1 + 0.2 * j) * s).to(TORCH[dtype])
        c = torch.rand(40, device=DEV, generator=g) + 0.1
        c[:10] = 0.1 + 0.2 * j
        r = c[:, None] * s[None]
        r = r.to(TORCH[dtype])
        for i in range(1, 11):      # eight elements shorter by b: cosine 1 - 8 b^2 / 2 d to second order
            b = (2 * d * i * 2e-5 / 8) ** 0.5
            r[29 + i, d - 8:] = (r[29 + i, d - 8:].float() * (1 - b)).to(TORCH[dtype])
        rows[places[j]] = r
    cache = siso.SisoCache(d, K, kind(siso, dtype))
    cache.load(rows)
    for k in (8, 32):
        idx, sim = cache.lookup_topk(q, k)
        for j in range(min(used, n)):
            r = rows[places[j]].double()
            exact = torch.nn.functional.cosine_similarity(r, q[j].double()[None])
            want = torch.sort(exact, descending=True)[0][:k]
            # single precision, a sum per lane and then over the lanes: d / 64 + 8 additions in a row at most
            assert (sim[j].double() - want).abs().max() < (d / 64 + 16) * 2.0 ** -24, (k, j)
            assert set(idx[j].tolist()) <= set(places[j].tolist()), (k, j)
            same = places[j][:10].sort()[0].tolist()
            assert [i for i in idx[j].tolist() if i in same] == same[:len([i for i in idx[j].tolist() if i in same])]
            if k == 32:
                order = torch.argsort(exact[30:], descending=True)[:2]
                assert idx[j, 30:].tolist() == places[j][30:][order].tolist(), j


@pytest.mark.parametrize("d,K,n,k", [(256, 4000, 6, 8), (768, 4000, 100, 8), (768, 4000, 1300, 8), (4096, 2500, 5, 5), (384, 16000, 500, 32)])
def test_topk_of_codes_beside_a_large_one(siso, oracle, d, K, n, k):
    """Eight products that are formed together are cut at 2^-13 of the largest of them: seven of 7.6 beside one of 200,704
    are lost in the first pass (2.6e-4 of the sum).  Three rows are the query itself; forty lack the seven elements, which
    costs them 1.3e-4 in truth and nothing in the first pass."""
    print(f"case: topk of codes d={d} K={K} n={n} k={k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    rows, q = directions(K, d, 31).bfloat16(), directions(n, d, 32).bfloat16()
    places = spread_rows(K, 48).to(DEV)
    base = 0.25 * (torch.randint(0, 2, (d,), device=DEV, generator=g) * 2 - 1).float()
    base[:8] = 2.75
    base[0] = 448
    less = base.clone()
    less[1:8] = 0
    q[2] = base.bfloat16()
    rows[places[:3]] = base.bfloat16()
    rows[places[3:43]] = less.bfloat16()
    cache = siso.SisoCache(d, K, siso.FP8)
    cache.load(rows)
    idx, sim = cache.lookup_topk(q, k)
    want = places[:3].sort()[0].tolist() + places[3:43].sort()[0].tolist()[:k - 3]
    assert idx[2].tolist() == want
    assert (sim[2, :3] - 1).abs().max() < 1e-6
    codes, scales = cache.export_fp8()[:2]
    ora = oracle.fp8_lookup_topk_rows(codes.cpu().numpy(), scales.cpu().numpy(), to_host(q[:5].contiguous(), "bf16"), k + 1)
    check_topk((idx[:5], sim[:5]), ora, "bf16", "codes")


# ---- the workspace of the first pass: less than it asks for, or none
@pytest.mark.parametrize("dtype,d,K,n", [("f32", 300, 5000, 70), ("bf16", 768, 33000, 300), ("bf16", 300, 2000, 41), ("fp8", 384, 4000, 600)])
def test_topk_with_little_room(siso, dtype, d, K, n):
    """The answers do not depend on the room: all of it, room for some queries (the last piece is smaller), none."""
    print(f"case: topk room {dtype} d={d} K={K} n={n}", flush=True)
    k = 8
    rows, q = directions(K, d, 41).to(TORCH[dtype]), directions(n, d, 42).to(TORCH[dtype])
    per_query = 2 * ((K + 31) // 32) * 8
    cache = siso.SisoCache(d, K, kind(siso, dtype))
    cache.load(rows)
    want = cache.lookup_topk(q, k)
    for kib in (max(1, 17 * per_query // 1024 + 1), max(1, n * per_query // 3 // 1024), per_query // 1024 if per_query > 1024 else 0):
        if kib == 0:
            continue
        small = siso.SisoCache(d, K, kind(siso, dtype))
        small.load(rows)
        small.set_option("topk_room", kib)
        got = small.lookup_topk(q, k)
        # (a smaller piece may run on another kernel of the first pass; what is ranked is formed the same way)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), kib


@pytest.mark.parametrize("dtype,d,K,n,before", [("f32", 300, 5000, 70, 0), ("bf16", 300, 2000, 41, 0), ("bf16", 768, 9000, 200, 0),
                                                ("f32", 384, 3000, 100, 30)])
def test_topk_captured_before_its_workspace_exists(siso, dtype, d, K, n, before):
    """The first call of a cache, or the first of a larger batch, under capture: nothing is allocated, the graph replays."""
    print(f"case: topk captured {dtype} d={d} K={K} n={n} before={before}", flush=True)
    k = 8
    rows = directions(K, d, 51).to(TORCH[dtype])
    batches = [directions(n, d, 52 + b).to(TORCH[dtype]) for b in range(3)]
    eager = siso.SisoCache(d, K, kind(siso, dtype))
    eager.load(rows)
    want = [eager.lookup_topk(q, k) for q in batches]
    side = torch.cuda.Stream()
    warm = siso.SisoCache(d, K, kind(siso, dtype))   # (kernels are loaded by an earlier use)
    cache = siso.SisoCache(d, K, kind(siso, dtype))
    q_in = batches[0].clone()
    torch.cuda.synchronize()
    warm.set_stream(side)
    cache.set_stream(side)
    with torch.cuda.stream(side):
        warm.load(rows)
        warm.set_option("topk_room", 1)
        warm.lookup_topk(q_in, k)
        cache.load(rows)
        if before:
            cache.lookup_topk(q_in[:before], k)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        idx, sim = cache.lookup_topk(q_in, k)
    for b, q in enumerate(batches):
        q_in.copy_(q)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(idx, want[b][0]) and torch.equal(sim, want[b][1]), b
    for c in (warm, cache):
        c.set_stream(torch.cuda.current_stream())
    got = cache.lookup_topk(batches[0], k)
    assert torch.equal(got[0], want[0][0]) and torch.equal(got[1], want[0][1])
