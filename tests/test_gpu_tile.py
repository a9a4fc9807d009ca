"""The tiled kernels for single precision and for dimensions and alignments the pipelined bf16 kernels do not take,
at the edges of their tiles: rows and queries one short of, at and one past a tile, dimensions that end inside a
slab (128 bytes of a row), a 16-byte chunk or an 8-byte half of it, rows and queries that are misaligned."""

import numpy as np
import pytest
import torch

from gpu_util import DEV, check_lookup, check_topk, siso_dtype, to_dev
from paper_2508_18736_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


@pytest.fixture(scope="module")
def oracle():
    import oracle as m
    m.build()
    return m


def shifted(t, elements):
    """The same rows at an address that is `elements` elements behind an aligned one."""
    room = torch.empty(t.numel() + 64, dtype=t.dtype, device=DEV)
    view = room[elements:elements + t.numel()].view(t.shape)
    view.copy_(t)
    return view


EDGES = [  # dtype, dim, K, n, shift of the queries
    ("f32", 32, 1, 1, 0), ("f32", 33, 31, 32, 0), ("f32", 31, 129, 33, 1), ("f32", 300, 1000, 65, 0),
    ("f32", 384, 64, 64, 2), ("f32", 384, 65, 63, 0), ("f32", 2, 500, 5, 0), ("f32", 1024, 9000, 900, 0),
    ("f32", 100, 9001, 1025, 3), ("bf16", 300, 1000, 65, 0), ("bf16", 300, 9001, 1025, 4), ("bf16", 12, 77, 3, 0),
    ("bf16", 7, 129, 40, 0), ("bf16", 65, 300, 64, 1), ("bf16", 4095, 130, 33, 0), ("f32", 4096, 40, 2, 0),
]


def _workload(dtype, dim, K, n):
    wl = W.c2_mid(n_clusters=16, per_cluster=(K + 15) // 16, n_queries=n, dim=dim, dtype=dtype, sigma=0.3, seed=77 + dim)
    wl.centroids = wl.centroids[:K].copy()
    return wl


@pytest.mark.parametrize("dtype,dim,K,n,shift", EDGES)
def test_lookup_at_the_edges_of_the_tiles(siso, oracle, dtype, dim, K, n, shift):
    print(f"case: tile lookup {dtype} dim={dim} K={K} n={n} shift={shift}", flush=True)
    wl = _workload(dtype, dim, K, n)
    cache = siso.SisoCache(dim, K + 3, siso_dtype(dtype))
    cache.load(to_dev(wl.centroids, dtype))
    out = cache.lookup(shifted(to_dev(wl.queries, dtype), shift), 0.85)
    torch.cuda.synchronize()
    st = check_lookup(out, oracle.lookup_rows(wl.centroids, wl.queries, 0.85, dtype), 0.85, dtype, "tile")
    # products and sums in single precision: |error| <= about dim * 2^-24 in the worst case, some 1e-7 in practice
    assert st["max_err"] < max(2e-6, dim * 2.0 ** -24)


@pytest.mark.parametrize("dtype,dim", [("f32", 33), ("bf16", 65), ("f32", 300), ("bf16", 300)])
def test_a_row_that_is_not_finite_stays_by_itself(siso, oracle, dtype, dim):
    """Slabs end inside rows here: what lies behind a row's end is the next row, and must not leak in."""
    print(f"case: tile non-finite rows {dtype} dim={dim}", flush=True)
    wl = _workload(dtype, dim, 200, 70)
    cents, q = to_dev(wl.centroids, dtype), to_dev(wl.queries, dtype)
    cents[1::3] = float("nan")
    cents[2::3] = float("inf")
    q[1::2] = float("nan")
    cache = siso.SisoCache(dim, 200, siso_dtype(dtype))
    cache.load(cents)
    idx, sim, hit = cache.lookup(q, 0.85)
    good = np.arange(0, 200, 3)
    ora = oracle.lookup_rows(wl.centroids[good], wl.queries[::2], 0.85, dtype)
    ora = (good[ora[0]].astype(ora[0].dtype),) + tuple(ora[1:])
    check_lookup([x[::2].contiguous() for x in (idx, sim, hit)], ora, 0.85, dtype, "finite rows")
    assert torch.isnan(sim[1::2]).all() and (idx[1::2] == -1).all() and (hit[1::2] == 0).all()


@pytest.mark.parametrize("dtype,dim,K", [("f32", 31, 2), ("f32", 33, 64), ("f32", 300, 65), ("f32", 64, 129), ("bf16", 300, 127),
                                         ("bf16", 7, 128), ("f32", 128, 4100), ("bf16", 100, 4101)])
def test_pairs_at_the_edges_of_the_tiles(siso, dtype, dim, K):
    print(f"case: tile pairs {dtype} dim={dim} K={K}", flush=True)
    wl = _workload(dtype, dim, K, 1)
    rows = to_dev(wl.centroids, dtype)
    cache = siso.SisoCache(dim, K, siso_dtype(dtype))
    cache.load(rows)
    u = rows.double()
    u = u / u.norm(dim=1, keepdim=True)
    p = torch.triu(u @ u.T, 1)
    # a threshold in the middle of a gap, so that no pair is within rounding of it
    v = torch.sort(p[p > 0.3])[0] if (p > 0.3).sum() > 1 else torch.tensor([0.4, 0.6], dtype=torch.float64, device=DEV)
    lo = v.numel() // 4
    gaps = v[lo + 1:] - v[lo:-1]
    at = int(torch.argmax(gaps))
    theta = float(v[lo + at] + gaps[at] / 2) if gaps.numel() else 0.5
    pairs, total = cache.merge(theta, K * K // 2 + 1)
    want = (p > theta).nonzero()
    got = torch.sort(pairs[:, 0].long() * K + pairs[:, 1].long())[0]
    assert total == want.shape[0] and torch.equal(got, torch.sort(want[:, 0] * K + want[:, 1])[0])


@pytest.mark.parametrize("dtype,dim,K", [("f32", 8, 760000), ("bf16", 12, 1048577)])
def test_pairs_of_more_tiles_than_one_launch_holds(siso, dtype, dim, K):
    """17.6 million pairs of 128-row tiles, and 33.6 million: 5 and 9 launches.  Almost all rows have no length and are near
    nothing; the others are copies of one row, in the first and last tiles, on both sides of a tile's edge, and in tiles
    whose pairs lie in every launch."""
    print(f"case: tile pairs {dtype} dim={dim} K={K}", flush=True)
    rows = torch.zeros(K, dim, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    at = torch.tensor(sorted({0, 1, 127, 128, K // 3, K // 2, K // 2 + 129, 4 * K // 5, K // 128 * 128 - 1, K - 2, K - 1}), device=DEV)
    rows[at] = torch.arange(1, dim + 1, device=DEV).to(rows.dtype)
    cache = siso.SisoCache(dim, K, siso_dtype(dtype))
    cache.load(rows)
    pairs, total = cache.merge(0.9, 1000)
    want = torch.combinations(at, 2)
    assert total == want.shape[0]
    got = pairs.long()
    assert torch.equal(torch.sort(got[:, 0] * K + got[:, 1])[0], torch.sort(want[:, 0] * K + want[:, 1])[0])


@pytest.mark.parametrize("dtype,dim,K,n,k", [("f32", 300, 7000, 33, 10), ("bf16", 300, 3100, 130, 32), ("f32", 33, 31, 5, 32),
                                             ("f32", 384, 16400, 3, 1), ("bf16", 256, 33, 64, 2), ("bf16", 512, 70000, 40, 5)])
def test_topk_at_the_edges_of_the_groups(siso, oracle, dtype, dim, K, n, k):
    """Rows one past a group of 32, fewer groups than k, more groups than a list, rows that tie inside a group of 16."""
    print(f"case: tile topk {dtype} dim={dim} K={K} n={n} k={k}", flush=True)
    wl = _workload(dtype, dim, K, n)
    for a in range(0, K - 9, max(9, K // 50)):
        wl.centroids[a + 8] = wl.centroids[a]     # both in one group of 16
    cache = siso.SisoCache(dim, K, siso_dtype(dtype))
    cache.load(to_dev(wl.centroids, dtype))
    out = cache.lookup_topk(to_dev(wl.queries, dtype), k)
    oc = oracle.OracleCache(dim, K, dtype)
    oc.load(wl.centroids)
    st = check_topk(out, oc.lookup_topk(wl.queries, k + 1 if k < min(K, 32) else k), dtype, "topk")
    assert st["max_err"] < max(2e-6, dim * 2.0 ** -24)
