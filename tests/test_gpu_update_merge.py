"""GPU parity of the centroid update, the pair search and the group merge against the
CPU oracle, through the C ABI."""

import time

import numpy as np
import pytest
import torch

from paper_2508_18736_amd import workloads as W
from gpu_util import DEV, check_lookup, siso_dtype, to_dev, to_host

pytestmark = pytest.mark.gpu

MEAN_TOL = 2e-6       # fp32 running mean against the oracle's float64 mean, entries <= 1 in size
STORE_TOL_F32 = 2e-6  # fp32 stored centroid


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


def compare_state(cache, oc, dtype, label):
    gc, gm, gs = cache.export()
    torch.cuda.synchronize()
    oc_c, oc_m, oc_s = oc.export()
    assert cache.count == oc.count, label
    assert np.array_equal(gs.cpu().numpy(), oc_s), f"{label}: cluster sizes differ"
    err = np.abs(gm.cpu().numpy().astype(np.float64) - oc_m).max() if oc.count else 0.0
    assert err <= MEAN_TOL, f"{label}: mean error {err:.3e}"
    g = to_host(gc, dtype)
    if dtype == "f32":
        assert np.abs(g.astype(np.float64) - oc_c).max() <= STORE_TOL_F32, label
    else:
        # the stored bf16 value may differ by one step where the fp32 mean sits next to a rounding
        # boundary; everywhere else it is bit-identical
        diff = g != oc_c
        assert diff.mean() < 2e-3, f"{label}: {diff.mean():.2e} of stored bf16 values differ"
        a = W.bf16_bits_to_f32(g).astype(np.float64); b = W.bf16_bits_to_f32(oc_c).astype(np.float64)
        assert np.abs(a - b).max() <= 2.0 ** -8, label
    # the two numbers of Algorithm 1 per centroid: same single-precision sums in the same order, exact counts
    gl, ga = cache.export_meta()
    ol, oa = oc.export_meta()
    assert np.array_equal(gl.cpu().numpy().view(np.uint32), ol.view(np.uint32)), f"{label}: cluster_size (Algorithm 1) differs"
    assert np.array_equal(ga.cpu().numpy().astype(np.uint32), oa), f"{label}: access_count differs"
    return err


def test_c1_lookup_then_update_hits(siso, oracle):
    print("case: c1 lookup + update of hit centroids", flush=True)
    wl = W.c1_tiny()
    cache = siso.SisoCache(wl.dim, wl.K, siso.F32)
    cache.load(to_dev(wl.centroids, "f32"))
    q = to_dev(wl.queries, "f32")
    idx, sim, hit = cache.lookup(q, 0.80)
    cache.update(q, idx, hit)            # hits fold into their centroid, on the device
    oc = oracle.OracleCache(wl.dim, wl.K, "f32")
    oc.load(wl.centroids)
    ora = oc.lookup(wl.queries, 0.80)
    check_lookup((idx, sim, hit), ora, 0.80, "f32", "c1")
    assert np.array_equal(idx.cpu().numpy(), ora[0]) and np.array_equal(hit.cpu().numpy(), ora[2])
    oc.update(wl.queries, np.where(ora[2] == 1, ora[0], -1).astype(np.int32))
    compare_state(cache, oc, "f32", "c1 update")
    assert oc.export()[2].sum() == wl.K + int(ora[2].sum()) and ora[2].sum() > 200
    # a second lookup sees the updated centroids
    out2 = cache.lookup(q, 0.80)
    check_lookup(out2, oc.lookup(wl.queries, 0.80), 0.80, "f32", "c1 after update")
    assert cache.bad_indices() == 0


@pytest.mark.parametrize("dtype,dim,n", [("bf16", 768, 64), ("bf16", 1024, 700), ("f32", 100, 333), ("bf16", 4096, 40)])
def test_update_matches_oracle(siso, oracle, dtype, dim, n):
    print(f"case: update {dtype} dim={dim} n={n}", flush=True)
    wl = W.c4_stream(n_clusters=16, per_cluster=8, batches=1, batch=n, dim=dim, sigma=0.3, zipf_s=1.2,
                     dtype=dtype, seed=51)
    counts = W.random_counts(51, wl.K, 1, 20)
    r = np.random.default_rng(10)
    idx = wl.planted.astype(np.int32).copy()
    idx[r.random(n) < 0.2] = -1                 # skipped entries
    idx[: n // 4] = idx[0] if idx[0] >= 0 else 3  # a hot centroid with many members
    q = wl.queries_f32().copy()
    q[1] = 0.0                                  # zero-length member: skipped
    q[2, 0] = np.nan                            # non-finite member: skipped
    q[3] *= 37.0                                # members are normalised first
    wl.queries = W.to_storage(q, dtype)
    cache = siso.SisoCache(dim, wl.K + 3, siso_dtype(dtype))
    cache.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    oc = oracle.OracleCache(dim, wl.K + 3, dtype)
    oc.load(wl.centroids, counts)
    cache.update(to_dev(wl.queries, dtype), torch.from_numpy(idx).to(DEV))
    oc.update(wl.queries, idx)
    compare_state(cache, oc, dtype, "update")
    # a second batch on top, given in a permuted order: the result must not depend on the order
    perm = r.permutation(n)
    cache.update(to_dev(wl.queries[perm].copy(), dtype), torch.from_numpy(idx[perm].copy()).to(DEV))
    oc.update(wl.queries, idx)
    compare_state(cache, oc, dtype, "update, permuted second batch")
    # lookups after the update use the new centroids and their new lengths
    out = cache.lookup(to_dev(wl.queries, dtype), 0.85)
    gc = to_host(cache.export()[0], dtype)
    ora = oracle.lookup_rows(gc, wl.queries, 0.85, dtype)   # oracle on the GPU's own stored rows
    check_lookup(out, ora, 0.85, dtype, "lookup after update")
    # out-of-range indices are skipped and counted
    bad = np.array([wl.K, wl.K + 100, 0], np.int32)
    before = cache.export()[1].clone()
    cache.update(to_dev(wl.queries[:3], dtype), torch.from_numpy(bad[:2].repeat(2)[:3].copy()).to(DEV))
    assert cache.bad_indices() == 3
    assert torch.equal(before, cache.export()[1])


@pytest.mark.parametrize("dtype,dim,n,hot", [("bf16", 256, 5000, 3000), ("f32", 384, 3000, 2200), ("bf16", 1024, 9000, 9000),
                                             ("bf16", 768, 40000, 20000)])
def test_update_with_a_centroid_that_takes_thousands_of_members(siso, oracle, dtype, dim, n, hot):
    """A burst of near-identical queries in one large batch: one centroid takes `hot` members, a second one 300, the
    rest a few each (the block that leads a centroid folds its members one after the other: slow for such a
    centroid, and exact).  Means, sizes and stored rows against the oracle; a zero row and a row with a NaN among
    the burst are passed over."""
    print(f"case: update with a hot centroid {dtype} dim={dim} n={n} hot={hot}", flush=True)
    K = 2000
    wl = W.c2_mid(n_clusters=50, per_cluster=40, n_queries=n, dim=dim, dtype=dtype, seed=88)
    r = np.random.default_rng(5)
    idx = r.integers(0, K, size=n).astype(np.int32)
    where = r.permutation(n)
    idx[where[:hot]] = 777
    idx[where[hot:hot + 300]] = 1500 if hot + 300 <= n else 777
    c32 = W.storage_to_f32(wl.centroids, dtype)
    q32 = c32[idx] + r.standard_normal((n, dim)).astype(np.float32) * np.float32(0.1 / np.sqrt(dim))
    q32 *= r.uniform(0.5, 2.0, size=(n, 1)).astype(np.float32)
    q32[where[3]] = 0.0                        # members without length or with a NaN: passed over
    q32[where[7], 5] = np.nan
    queries = W.to_storage(q32, dtype)
    counts = W.random_counts(89, K, 1, 9)
    cache = siso.SisoCache(dim, K, siso_dtype(dtype))
    cache.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    oc = oracle.OracleCache(dim, K, dtype)
    oc.load(wl.centroids, counts)
    q = to_dev(queries, dtype)
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    cache.update(q, torch.from_numpy(idx).to(DEV))            # allocates the notes of a large batch
    cache.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    t0.record()
    cache.update(q, torch.from_numpy(idx).to(DEV))
    t1.record()
    torch.cuda.synchronize()
    print(f"  update of {n} queries, {hot} of them into one centroid: {t0.elapsed_time(t1) * 1e3:.0f} us", flush=True)
    oc.update(queries, idx)
    compare_state(cache, oc, dtype, "hot centroid")
    sizes = cache.export()[2].cpu().numpy()
    assert sizes[777] == counts[777] + int((idx == 777).sum()) - int(idx[where[3]] == 777) - int(idx[where[7]] == 777)
    assert cache.bad_indices() == 0
    # the same batch again in a different order: the same means within the tolerance, the same sizes
    perm = r.permutation(n)
    cache2 = siso.SisoCache(dim, K, siso_dtype(dtype))
    cache2.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    cache2.update(to_dev(queries[perm], dtype), torch.from_numpy(idx[perm]).to(DEV))
    a, b = cache.export(), cache2.export()
    assert torch.equal(a[2], b[2]) and (a[1] - b[1]).abs().max().item() <= MEAN_TOL


def test_update_fold_misses_policy(siso, oracle):
    """The library folds whatever it is told to: here the misses instead of the hits."""
    print("case: update folding misses", flush=True)
    wl = W.c2_mid(n_clusters=32, per_cluster=8, n_queries=300, dim=128, seed=52)
    cache = siso.SisoCache(wl.dim, wl.K, siso.BF16)
    cache.load(to_dev(wl.centroids, "bf16"))
    q = to_dev(wl.queries, "bf16")
    idx, sim, hit = cache.lookup(q, 0.85)
    cache.update(q, idx, (1 - hit).to(torch.uint8))
    oc = oracle.OracleCache(wl.dim, wl.K, "bf16")
    oc.load(wl.centroids)
    ora = oc.lookup(wl.queries, 0.85)
    assert np.array_equal(ora[2], hit.cpu().numpy()) and 50 < (1 - ora[2]).sum() < 150
    oc.update(wl.queries, np.where(ora[2] == 0, ora[0], -1).astype(np.int32))
    compare_state(cache, oc, "bf16", "fold misses")


def sorted_pairs(p):
    p = np.asarray(p).reshape(-1, 2)
    return p[np.lexsort((p[:, 1], p[:, 0]))]


@pytest.mark.parametrize("dtype,dim,groups,copies,sigma,theta", [
    ("bf16", 768, 300, 7, 0.03, 0.90), ("f32", 96, 100, 5, 0.05, 0.90), ("bf16", 128, 150, 9, 0.6, 0.7),
    ("bf16", 1024, 33, 31, 0.03, 0.90), ("bf16", 256, 429, 7, 0.03, 0.90)])
def test_merge_pairs_and_groups_match_oracle(siso, oracle, dtype, dim, groups, copies, sigma, theta):
    print(f"case: merge {dtype} dim={dim} K={groups * copies} sigma={sigma} theta={theta}", flush=True)
    wl = W.c5_merge(n_groups=groups, copies=copies, dim=dim, sigma=sigma, dtype=dtype, seed=53)
    counts = W.random_counts(53, wl.K, 1, 100)
    cache = siso.SisoCache(dim, wl.K, siso_dtype(dtype))
    cache.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    oc = oracle.OracleCache(dim, wl.K, dtype)
    oc.load(wl.centroids, counts)
    want, total = oc.merge(theta)
    # pairs whose cosine is within rounding of the threshold may legitimately differ
    c64 = wl.centroids_f32().astype(np.float64)
    u = c64 / np.linalg.norm(c64, axis=1, keepdims=True)
    S = u @ u.T
    edge = np.abs(S - np.float64(np.float32(theta))) < 2e-5
    np.fill_diagonal(edge, False)
    got, gtotal = cache.merge(theta, cap=total + 100)
    got = sorted_pairs(got.cpu().numpy())
    if not edge.any():
        assert gtotal == total and np.array_equal(got, want)
    else:
        gs, ws = set(map(tuple, got)), set(map(tuple, want))
        assert all(edge[i, j] for i, j in gs ^ ws)
    assert np.all(got[:, 0] < got[:, 1]) and len(np.unique(got, axis=0)) == len(got)
    # the general tiled kernel finds the same set (up to the pairs at the edge of the threshold; it is the default of
    # fewer than 2,900 bf16 rows as well)
    cache.set_option("merge_config", 1)
    got_s, total_s = cache.merge(theta, cap=total + 100)
    cache.set_option("merge_config", 0)
    got_s = sorted_pairs(got_s.cpu().numpy())
    assert all(edge[i, j] for i, j in set(map(tuple, got_s)) ^ set(map(tuple, got)))
    # and so do the four-wave MFMA kernel and the eight-wave one, the default of larger sets (where they apply at all)
    for config in (2, 3):
        cache.set_option("merge_config", config)
        got_8, total_8 = cache.merge(theta, cap=total + 100)
        cache.set_option("merge_config", 0)
        got_8 = sorted_pairs(got_8.cpu().numpy())
        assert total_8 == len(got_8) and all(edge[i, j] for i, j in set(map(tuple, got_8)) ^ set(map(tuple, got))), config
    # a second run gives the same set (the order of emission is free)
    again, total_a = cache.merge(theta, cap=total + 100)
    assert total_a == gtotal and np.array_equal(sorted_pairs(again.cpu().numpy()), got)
    if sigma < 0.1:
        assert total == groups * copies * (copies - 1) // 2
    # capped output: full count reported, only cap pairs written, all of them valid
    few, t2 = cache.merge(theta, cap=10)
    assert t2 == gtotal and few.shape[0] == 10
    assert set(map(tuple, few.cpu().numpy())) <= set(map(tuple, got))
    # group merge from the oracle's pair list on both sides
    pr = torch.from_numpy(want[np.random.default_rng(11).permutation(len(want))].copy()).to(DEV)
    surv = cache.merge_apply(pr)
    osurv = oc.merge_apply(want)
    assert np.array_equal(surv.cpu().numpy(), osurv)
    compare_state(cache, oc, dtype, "merge_apply")
    if sigma < 0.1:
        assert cache.count == groups
    # the merged cache still answers lookups consistently with its own stored rows
    qs = wl.centroids[:50].copy()
    out = cache.lookup(to_dev(qs, dtype), 0.9)
    ora = oracle.lookup_rows(to_host(cache.export()[0], dtype), qs, 0.9, dtype)
    check_lookup(out, ora, 0.9, dtype, "lookup after merge")


@pytest.mark.parametrize("K,dim", [(2800, 4096), (2899, 1024), (2900, 1024), (3299, 1088), (3300, 1088)])
def test_default_pair_search_of_few_thousand_rows(siso, K, dim):
    """On both sides of the lines between the tiled kernel and the pipelined one: the pairs of the tiled kernel, and no search of rows
    without pairs that takes longer than it."""
    print(f"case: default pair search K={K} dim={dim}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(K)
    rows = torch.randn(K, dim, device=DEV, generator=g)
    cache = siso.SisoCache(dim, K, siso.BF16)
    cache.load(rows.bfloat16())
    took = {0: [], 1: []}
    for _ in range(20):
        for config in took:
            cache.set_option("merge_config", config)
            begin = time.perf_counter()
            assert cache.merge(0.9, 10)[1] == 0
            took[config].append(time.perf_counter() - begin)
    assert min(took[0]) < 1.1 * min(took[1]), (min(took[0]), min(took[1]))
    cache.load((rows[torch.arange(K, device=DEV) // 5] + 0.1 * torch.randn(K, dim, device=DEV, generator=g)).bfloat16())
    got = []
    for config in took:
        cache.set_option("merge_config", config)
        pairs, total = cache.merge(0.9, 4 * K)
        got.append(sorted_pairs(pairs.cpu().numpy()))
        assert total == len(got[-1]) == K // 5 * 10 + (K % 5) * (K % 5 - 1) // 2
    assert np.array_equal(*got)


def test_merge_apply_chains_and_errors(siso, oracle):
    print("case: merge_apply chains / invalid pairs", flush=True)
    d = 64
    rows = np.eye(d, dtype=np.float32)[:6]
    counts = np.array([1, 2, 3, 4, 5, 6], np.int32)
    cache = siso.SisoCache(d, 6, siso.F32)
    cache.load(to_dev(rows, "f32"), torch.from_numpy(counts).to(DEV))
    oc = oracle.OracleCache(d, 6, "f32")
    oc.load(rows, counts)
    pairs = np.array([[3, 1], [3, 4]], np.int32)
    surv = cache.merge_apply(torch.from_numpy(pairs).to(DEV))
    assert np.array_equal(surv.cpu().numpy(), oc.merge_apply(pairs)) and cache.count == 4
    compare_state(cache, oc, "f32", "chain")
    for bad in ([[0, 0]], [[0, 9]], [[-1, 2]]):
        with pytest.raises(siso.SisoError):
            cache.merge_apply(torch.tensor(bad, dtype=torch.int32, device=DEV))
    assert cache.count == 4
    compare_state(cache, oc, "f32", "after rejected pairs")
    cache.merge_apply(torch.zeros((0, 2), dtype=torch.int32, device=DEV))
    assert cache.count == 4
    # fewer than two centroids: no pairs
    one = siso.SisoCache(d, 2, siso.F32)
    one.load(to_dev(rows[:1], "f32"))
    assert one.merge(0.5, cap=4)[1] == 0


def test_merge_dense_pairs_overflow_the_staging_buffer(siso, oracle):
    """Four groups of 300 exact copies: every tile pair holds tens of thousands of pairs, far more than a
    workgroup of the pipelined kernels stages at a time, so the staging buffer fills, spills and is flushed again and
    again (the tiled kernel, the default of so few rows, has none)."""
    dim, groups, copies = 128, 4, 300
    print(f"case: dense merge dim={dim} K={groups * copies}", flush=True)
    base = W.to_storage(W.uniform_directions(61, 3, groups, dim), "bf16")
    rows = np.repeat(base, copies, axis=0)[np.random.default_rng(62).permutation(groups * copies)]
    K = rows.shape[0]
    cache = siso.SisoCache(dim, K, siso.BF16)
    cache.load(to_dev(rows, "bf16"))
    oc = oracle.OracleCache(dim, K, "bf16")
    oc.load(rows)
    want, total = oc.merge(0.9)
    assert total == groups * copies * (copies - 1) // 2
    for config in (0, 1, 2, 3):  # the tiled kernel twice, the four-wave kernel, the eight-wave one
        cache.set_option("merge_config", config)
        got, gtotal = cache.merge(0.9, cap=total)
        assert gtotal == total, config
        assert np.array_equal(sorted_pairs(got.cpu().numpy()), want), config
    cache.set_option("merge_config", 0)
    # a cap in the middle of it all: full count, exactly cap valid pairs, no duplicates
    for config in (0, 2, 3):
        cache.set_option("merge_config", config)
        few, t2 = cache.merge(0.9, cap=5000)
        few = few.cpu().numpy()
        assert t2 == total and few.shape[0] == 5000 and len(np.unique(few, axis=0)) == 5000
        assert set(map(tuple, few)) <= set(map(tuple, want))


def test_merge_apply_groups_of_many_sizes(siso, oracle):
    """Groups given as chains of pairs in a shuffled order: of 2, 3, 257 and 700 rows (sorted by their
    block in LDS, several entries per thread) and of 1,500 rows (beyond the list a block sorts: the block
    searches the root array instead), with different weights, among rows that stay alone."""
    dim, dtype = 128, "bf16"
    sizes = [2, 3, 257, 700, 1500]
    K = sum(sizes) + 40
    print(f"case: merge_apply groups of {sizes} rows, K={K}", flush=True)
    rng = np.random.default_rng(77)
    rows = W.to_storage(W.uniform_directions(78, 2, K, dim), dtype)
    counts = rng.integers(1, 9, size=K).astype(np.int32)
    perm = rng.permutation(K)
    pairs, at = [], 0
    for m in sizes:
        mem = perm[at:at + m]
        at += m
        pairs += [(int(mem[i]), int(mem[i + 1])) for i in range(m - 1)]
    pairs = np.array(pairs, np.int32)[rng.permutation(len(pairs))]
    cache = siso.SisoCache(dim, K, siso.BF16)
    cache.load(to_dev(rows, dtype), torch.from_numpy(counts).to(DEV))
    oc = oracle.OracleCache(dim, K, dtype)
    oc.load(rows, counts)
    surv = cache.merge_apply(torch.from_numpy(pairs).to(DEV))
    assert np.array_equal(surv.cpu().numpy(), oc.merge_apply(pairs))
    assert cache.count == oc.count == K - sum(sizes) + len(sizes)
    compare_state(cache, oc, dtype, "groups of many sizes")


def test_merge_apply_meta_hand_worked_and_random(siso, oracle):
    """cluster_size and access_count of merged groups: the example worked by hand (a member at infinity, a sum that
    reaches infinity, a single-precision sum that depends on its order), then random groups with large access
    counts, state taken over from a snapshot on both sides."""
    from test_oracle_update_merge import merge_meta_state, read_merge_meta_example
    print("case: merge_apply cluster_size / access_count", flush=True)
    loc, acc, pairs, expect, surv = read_merge_meta_example()
    k = len(loc)
    cents, means, sizes = merge_meta_state(k, dim=64)
    cache = siso.SisoCache(64, k, siso.F32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    cache.import_state(dev(cents), dev(means.astype(np.float32)), dev(sizes), dev(loc), dev(acc.astype(np.int64)))
    gl, ga = cache.export_meta()
    assert np.array_equal(gl.cpu().numpy(), loc) and np.array_equal(ga.cpu().numpy().astype(np.uint32), acc)
    got = cache.merge_apply(dev(pairs)).cpu().numpy()
    assert np.array_equal(got, surv) and cache.count == len(expect)
    gl, ga = cache.export_meta()
    gl, ga = gl.cpu().numpy(), ga.cpu().numpy()
    for i, (want_l, want_a) in expect.items():
        assert gl[i].view(np.uint32) == np.float32(want_l).view(np.uint32) and int(ga[i]) == want_a, f"survivor {i}"
    # random: 600 rows, groups of 2..40 rows as shuffled chains, fractional cluster sizes, access counts up to 2^31
    rng = np.random.default_rng(91)
    K, dim = 600, 128
    rows = W.to_storage(W.uniform_directions(92, 2, K, dim), "bf16")
    u = W.bf16_bits_to_f32(rows).astype(np.float64)
    means = u / np.linalg.norm(u, axis=1, keepdims=True)
    sizes = rng.integers(1, 9, size=K).astype(np.int32)
    loc = (rng.integers(1, 4000, size=K) / np.float32(1.1)).astype(np.float32)
    acc = rng.integers(0, 2 ** 31, size=K).astype(np.uint32)
    acc[rng.random(K) < 0.05] = 0xFFFFFFFF
    acc[rng.random(K) < 0.5] //= 65536
    perm, at, pr = rng.permutation(K), 0, []
    for m in [2, 3, 5, 40, 17, 2, 2, 9, 33, 4, 4, 4, 8]:
        mem = perm[at:at + m]
        at += m
        pr += [(int(mem[i]), int(mem[i + 1])) for i in range(m - 1)]
    pr = np.array(pr, np.int32)[rng.permutation(len(pr))]
    cache = siso.SisoCache(dim, K, siso.BF16)
    cache.import_state(to_dev(rows, "bf16"), dev(means.astype(np.float32)), dev(sizes), dev(loc), dev(acc.astype(np.int64)))
    oc = oracle.OracleCache(dim, K, "bf16")
    oc.import_state(rows, means.astype(np.float32).astype(np.float64), sizes, loc, acc)
    compare_state(cache, oc, "bf16", "snapshot taken over")
    assert np.array_equal(cache.merge_apply(dev(pr)).cpu().numpy(), oc.merge_apply(pr))
    compare_state(cache, oc, "bf16", "merge_apply with cluster sizes and access counts")
    ol, oa = oc.export_meta()
    assert (oa == 0xFFFFFFFF).sum() >= 3 and len(np.unique(ol)) > 100


def same_state(a, b):
    """Two caches hold bit-identical centroids, means, sizes and metadata."""
    ea, eb = a.export(), b.export()
    ma, mb = a.export_meta(), b.export_meta()
    torch.cuda.synchronize()
    return all(torch.equal(x.view(torch.uint8) if x.dtype.is_floating_point else x,
                           y.view(torch.uint8) if y.dtype.is_floating_point else y) for x, y in zip(ea + ma, eb + mb))


@pytest.mark.parametrize("dtype,dim,K,n,clusters", [
    ("bf16", 768, 5000, 64, 256),      # batches of 64: the streaming shape (256 x 64 tiles)
    ("bf16", 256, 3000, 100, 8),       # 256 x 128 tiles; few clusters: many queries share a centroid
    ("bf16", 1024, 2000, 1, 16), ("bf16", 2048, 900, 37, 4),
    ("f32", 384, 1024, 256, 16),       # fp32 on the tiled kernel, a full board
    ("bf16", 768, 5000, 200, 64),      # a small bf16 problem on the tiled kernel
    ("bf16", 256, 30000, 200, 256),    # the 256 x 256 tiles name groups of rows: the two calls
    ("f32", 96, 700, 300, 16),         # more queries than the board has slots: the two calls, the notes of the
    ("bf16", 256, 4000, 700, 8),       # update taken by the end of the lookup (large batches, many members per
    ("bf16", 1024, 3000, 1500, 64)])   # centroid)
def test_lookup_update_is_lookup_then_update_hits(siso, oracle, dtype, dim, K, n, clusters):
    print(f"case: lookup_update {dtype} dim={dim} K={K} n={n}", flush=True)
    wl = W.c2_mid(n_clusters=clusters, per_cluster=(K + clusters - 1) // clusters, n_queries=n * 6, dim=dim, dtype=dtype, seed=77)
    wl.centroids = wl.centroids[:K].copy()
    counts = W.random_counts(78, K, 1, 5)
    one = siso.SisoCache(dim, K, siso_dtype(dtype))
    two = siso.SisoCache(dim, K, siso_dtype(dtype))
    oc = oracle.OracleCache(dim, K, dtype)
    for c in (one, two):
        c.load(to_dev(wl.centroids, dtype), torch.from_numpy(counts).to(DEV))
    oc.load(wl.centroids, counts)
    theta = 0.85
    for step in range(6):
        qs = wl.queries[step * n:(step + 1) * n].copy()
        if step == 2 and n >= 4:
            qs[1] = qs[0]                      # the same query twice: two members of one centroid for sure
            qs[3] = 0                          # a query without length: no hit, nothing folded
        q = to_dev(qs, dtype)
        out = one.lookup_update(q, theta)
        ref = two.lookup(q, theta)
        two.update(q, ref[0], ref[2])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out[:1] + out[2:], ref[:1] + ref[2:])), f"step {step}: idx / hit"
        assert torch.equal(out[1].view(torch.int32), ref[1].view(torch.int32)), f"step {step}: sim"
        assert same_state(one, two), f"step {step}: state differs from lookup + update_hits"
        # and against the oracle: lookup on its state, fold its hits
        ora = oc.lookup(qs, theta)
        st = check_lookup(out, ora, theta, dtype, f"lookup_update step {step}")
        gh = out[2].cpu().numpy()
        if np.array_equal(gh, ora[2]) and np.array_equal(out[0].cpu().numpy()[gh == 1], ora[0][gh == 1]):
            oc.update(qs, np.where(ora[2] == 1, ora[0], -1).astype(np.int32))
        else:   # a similarity within rounding of the threshold or of the runner-up: the oracle follows the GPU's choice
            oc.update(qs, np.where(gh == 1, out[0].cpu().numpy(), -1).astype(np.int32))
        compare_state(one, oc, dtype, f"lookup_update step {step}")
    assert int(one.export()[2].sum().item()) > int(counts.sum())        # something was folded
    assert one.bad_indices() == 0


def test_lookup_update_workgroups_that_give_up_leave_the_cache_alone(siso, oracle):
    """The wait of the one-kernel end is bounded.  With a limit of zero looks at the board every workgroup whose
    query hits gives up at once: the lookup's outputs are unchanged, no centroid is touched, and every hit is
    counted as not applied.  With the default limit again the same batch is folded."""
    print("case: lookup_update, bounded wait", flush=True)
    wl = W.c2_mid(n_clusters=64, per_cluster=16, n_queries=64, dim=256, seed=79)
    cache = siso.SisoCache(wl.dim, wl.K, siso.BF16)
    cache.load(to_dev(wl.centroids, "bf16"))
    q = to_dev(wl.queries, "bf16")
    ref = cache.lookup(q, 0.85)
    before = [x.clone() for x in cache.export()]
    cache.set_option("fold_spin_limit", 0)
    out = cache.lookup_update(q, 0.85)
    torch.cuda.synchronize()
    hits = int(ref[2].sum().item())
    assert hits > 20 and all(torch.equal(a, b) for a, b in zip(out, ref))
    assert all(torch.equal(a, b) for a, b in zip(cache.export(), before))
    assert cache.bad_indices() == hits
    cache.set_option("fold_spin_limit", -1)
    cache.lookup_update(q, 0.85)
    torch.cuda.synchronize()
    assert int(cache.export()[2].sum().item()) == wl.K + hits and cache.bad_indices() == hits
    oc = oracle.OracleCache(wl.dim, wl.K, "bf16")
    oc.load(wl.centroids)
    ora = oc.lookup(wl.queries, 0.85)
    oc.update(wl.queries, np.where(ora[2] == 1, ora[0], -1).astype(np.int32))
    # (the access counts saw three lookups on the GPU: compare what the update writes)
    assert np.array_equal(cache.export()[2].cpu().numpy(), oc.export()[2])
    assert np.abs(cache.export()[1].cpu().numpy().astype(np.float64) - oc.export()[1]).max() <= MEAN_TOL


def test_lookup_update_next_to_a_long_kernel_on_another_stream(siso, oracle):
    """The workgroups of the one-kernel end wait for each other; they must all get onto the chip even while another
    stream keeps it busy with large lookups of another cache."""
    print("case: lookup_update beside large lookups on another stream", flush=True)
    big = W.c2_mid(n_clusters=2048, per_cluster=16, n_queries=4096, dim=768, seed=80)
    big_cache = siso.SisoCache(big.dim, big.K, siso.BF16)
    big_cache.load(to_dev(big.centroids, "bf16"))
    bq = to_dev(big.queries, "bf16")
    big_out = big_cache.lookup(bq, 0.85)     # its outputs stay allocated: the other stream writes them while this one goes on
    wl = W.c4_stream(n_clusters=256, per_cluster=8, batches=40, batch=64, dim=256, seed=81)
    alone, beside = siso.SisoCache(wl.dim, wl.K, siso.BF16), siso.SisoCache(wl.dim, wl.K, siso.BF16)
    qs = to_dev(wl.queries, "bf16")
    for c in (alone, beside):
        c.load(to_dev(wl.centroids, "bf16"))
        c.reserve(64)
    outs_alone = [tuple(x.clone() for x in alone.lookup_update(qs[b * 64:(b + 1) * 64], 0.85)) for b in range(40)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    big_cache.set_stream(side)
    outs = []
    for b in range(40):
        big_cache.lookup(bq, 0.85, *big_out)       # 0.3 ms each, on the other stream
        outs.append(tuple(x.clone() for x in beside.lookup_update(qs[b * 64:(b + 1) * 64], 0.85)))
    torch.cuda.synchronize()
    big_cache.set_stream(torch.cuda.current_stream())
    for b in range(40):
        assert all(torch.equal(x, y) for x, y in zip(outs[b], outs_alone[b])), f"batch {b}"
    assert same_state(alone, beside) and beside.bad_indices() == 0
