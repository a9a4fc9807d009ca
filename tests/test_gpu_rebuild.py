"""The kernels behind the calls that fold and rebuild: updates with many members, group merges and clusterings at the
edges of their scans, lists and waves, against plain torch in 64 bits (and the host's walk over the pairs)."""

import time

import numpy as np
import pytest
import torch

from gpu_util import DEV, siso_dtype

pytestmark = pytest.mark.gpu
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


def rows_of(n, d, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(n, d, device=DEV, generator=g).to(TORCH[dtype])


def unit(x):
    return x / x.norm(dim=1, keepdim=True)


@pytest.mark.parametrize("dtype,d,n,targets", [("bf16", 256, 257, 3), ("f32", 100, 4097, 2), ("bf16", 768, 4354, 40),
                                               ("f32", 1028, 700, 5), ("bf16", 2048, 300, 7), ("f32", 64, 9000, 1),
                                               ("bf16", 128, 256, 1), ("f32", 96, 33000, 11)])
def test_an_update_with_many_members(siso, dtype, d, n, targets):
    """More entries than a block looks through at a time, members in every position, misses and queries without
    length among them."""
    print(f"case: update {dtype} d={d} n={n} targets={targets}", flush=True)
    K = 50
    cache = siso.SisoCache(d, K, siso_dtype(dtype))
    cents = rows_of(K, d, dtype, 1)
    cache.load(cents)
    q = rows_of(n, d, dtype, 2)
    q[5::97] = 0
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    idx = (torch.randint(0, targets, (n,), device=DEV, generator=g) * 7 % K).int()
    hit = (torch.rand(n, device=DEV, generator=g) < 0.9).to(torch.uint8)
    cache.update(q, idx, hit)
    mean, weight = unit(cents.double()), torch.ones(K, 1, dtype=torch.float64, device=DEV)
    use = (hit == 1) & (q.double().norm(dim=1) > 0)
    at = idx[use].long()
    total = (mean * weight).index_add_(0, at, unit(q[use].double()))
    weight = weight.index_add_(0, at, torch.ones(at.numel(), 1, dtype=torch.float64, device=DEV))
    want = total / weight
    got_c, got_m, got_s = cache.export()
    assert torch.equal(got_s.long(), weight[:, 0].long())
    # each of up to n additions and one division rounds to 2^-24 of a sum that stays below the weight
    assert (got_m.double() - want).abs().max() < 3e-7 * max(1.0, n ** 0.5)
    eps = 2.0 ** -8 if dtype == "bf16" else 2e-6
    touched = torch.zeros(K, dtype=torch.bool, device=DEV)
    touched[at] = True
    ref = unit(want[touched])
    assert ((got_c[touched].double() - ref).abs() <= eps * ref.abs() + 1e-4 * eps + 1e-6).all()


@pytest.mark.parametrize("dtype,d,n", [("bf16", 768, 250), ("f32", 1024, 251), ("bf16", 100, 5000), ("f32", 33, 4100), ("bf16", 1030, 300)])
def test_an_update_with_one_to_ten_members_each(siso, dtype, d, n):
    """Centroid k has 1 + k % 10 members: as many as are folded at a time, one more, one less, with the first and without."""
    print(f"case: update {dtype} d={d} n={n}, few members each", flush=True)
    idx = torch.repeat_interleave(torch.arange(n), torch.arange(n) % 10 + 1)[:n].int().to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    idx = idx[torch.randperm(n, device=DEV, generator=g)].contiguous()
    cents, q = rows_of(n, d, dtype, 5), rows_of(n, d, dtype, 6)
    cache = siso.SisoCache(d, n, siso_dtype(dtype))
    cache.load(cents)
    cache.update(q, idx)
    at = idx.long()
    weight = 1 + torch.bincount(at, minlength=n).double()[:, None]
    want = unit(cents.double()).index_add_(0, at, unit(q.double())) / weight
    _, mean, size = cache.export()
    assert torch.equal(size.long(), weight[:, 0].long())
    # at most 11 additions and a division of numbers below 11, each rounded to 2^-24, and an error of 2 * 2^-24 in every unit row
    assert (mean.double() - want).abs().max() < 20 * 2.0 ** -24


@pytest.mark.parametrize("dtype,d,K,sizes", [
    ("bf16", 64, 4096, [2, 3, 4, 5, 8, 9, 17]), ("f32", 100, 4097, [64, 1024, 1025]), ("bf16", 1032, 300, [2, 7]),
    ("f32", 33, 4095, [1300, 1700, 2]), ("bf16", 768, 17, [17]), ("bf16", 300, 8193, [2] * 1500 + [33] * 20)])
def test_group_merge_at_the_edges(siso, dtype, d, K, sizes):
    """Groups of every kind of list, groups in every position of a block of rows, one scan block more or less."""
    print(f"case: merge_apply {dtype} d={d} K={K} groups={len(sizes)}", flush=True)
    r = np.random.default_rng(K)
    order = r.permutation(K)
    pairs, group, lo = [], np.arange(K), 0
    for s in sizes:
        m = order[lo:lo + s]
        lo += s
        group[m] = m.min()
        pairs += [(int(m[i]), int(m[r.integers(0, i)])) for i in range(1, s)]  # a random tree holds it together
    pairs += pairs[:5]
    cents = rows_of(K, d, dtype, 4)
    counts = torch.from_numpy(r.integers(1, 40, K).astype(np.int32)).to(DEV)
    cache = siso.SisoCache(d, K, siso_dtype(dtype))
    cache.load(cents, counts)
    surv = cache.merge_apply(torch.tensor(pairs, dtype=torch.int32, device=DEV))
    roots, place = np.unique(group, return_inverse=True)
    assert np.array_equal(surv.cpu().numpy(), place) and cache.count == len(roots)
    at = torch.from_numpy(place).to(DEV)
    w = torch.zeros(len(roots), dtype=torch.float64, device=DEV).index_add_(0, at, counts.double())
    want = torch.zeros(len(roots), d, dtype=torch.float64, device=DEV).index_add_(0, at, unit(cents.double()) * counts[:, None]) / w[:, None]
    got_c, got_m, got_s = cache.export()
    loc, acc = cache.export_meta()
    assert torch.equal(got_s.double(), w) and torch.equal(loc.double(), w) and int(acc.sum()) == 0
    assert (got_m.double() - want).abs().max() < 1e-6
    alone = torch.from_numpy(np.bincount(place) == 1).to(DEV)
    assert torch.equal(got_c[alone], cents[torch.from_numpy(roots).to(DEV)][alone])
    # a pair that is none changes nothing
    before = [x.clone() for x in cache.export()]
    for bad in ([0, 0], [-1, 1], [0, cache.count]):
        with pytest.raises(siso.SisoError):
            cache.merge_apply(torch.tensor([[0, 1], bad], dtype=torch.int32, device=DEV))
    assert all(torch.equal(a, b) for a, b in zip(before, cache.export()))


def _graph_vectors(sizes, chains, d, seed):
    """Vectors whose neighbour graph at 0.9 has the given cliques, and chains of rows that turn by a little under the
    threshold's angle from one to the next (each a neighbour of a few others only)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = []
    for s in sizes:
        base = unit(torch.randn(1, d, device=DEV, generator=g))
        out.append(unit(base + 0.1 * unit(torch.randn(s, d, device=DEV, generator=g))))
    for s in chains:
        a, b = torch.linalg.qr(torch.randn(d, 2, device=DEV, generator=g))[0].T
        t = torch.arange(s, device=DEV) * 0.17 + 0.02 * torch.rand(s, device=DEV, generator=g)
        out.append(torch.cos(t)[:, None] * a + torch.sin(t)[:, None] * b)
    x = torch.cat(out)
    return x[torch.randperm(x.shape[0], device=DEV, generator=g)].contiguous()


@pytest.mark.parametrize("min_size", [1, 2, 4])
@pytest.mark.parametrize("sizes,chains", [([1] * 40 + [2, 3, 7, 12] * 30, []), ([64, 63, 2, 1], [30, 17, 9]), ([65, 5, 1], [12]),
                                          ([3], [18, 18, 18, 5]), ([1], []), ([2] * 600 + [9] * 100, [13] * 20)])
def test_communities_are_those_of_the_walk_over_the_pairs(siso, sizes, chains, min_size):
    """Components worked off by a wave, up to the largest that is; one more goes to the host."""
    print(f"case: cluster sizes={sizes[:4]}.. chains={chains[:4]} min_size={min_size}", flush=True)
    x = _graph_vectors(sizes, chains, 96, 5)
    n = x.shape[0]
    theta = 0.9
    u = unit(x.double())
    p = torch.triu(u @ u.T, 1)
    assert ((p - theta).abs() > 1e-6).all()
    pairs = (p > theta).nonzero().int().cpu().numpy()
    want, clusters = siso.choose_communities(pairs, n, min_size)
    cache = siso.SisoCache(96, n, siso.F32)
    labels, got, total = cache.cluster(x, theta, min_size)
    assert total == len(pairs) and got == clusters and np.array_equal(labels.cpu().numpy(), want)
    at = torch.from_numpy(want).to(DEV).long()
    size = torch.bincount(at[at >= 0], minlength=clusters).double()
    mean = torch.zeros(clusters, 96, dtype=torch.float64, device=DEV).index_add_(0, at[at >= 0], u[at >= 0]) / size[:, None]
    got_c, got_m, got_s = cache.export()
    assert torch.equal(got_s.double(), size) and (clusters == 0 or (got_m.double() - mean).abs().max() < 1e-6)
    if clusters > 1:  # too small a cache: an error, and nothing changed
        small = siso.SisoCache(96, clusters - 1, siso.F32)
        small.load(x[:1])
        with pytest.raises(siso.SisoError):
            small.cluster(x, theta, min_size)
        assert small.count == 1 and torch.equal(small.export()[0], x[:1])


def test_a_log_with_more_pairs_than_room_is_searched_again(siso):
    """1,600 equal vectors and a few others: 1,279,200 pairs, room for 1,048,576 at first; a component for the host."""
    print("case: cluster, second search", flush=True)
    x = rows_of(1700, 64, "f32", 6)
    x[:1600] = x[0]
    cache = siso.SisoCache(64, 1700, siso.F32)
    labels, clusters, total = cache.cluster(x, 0.95, 2)
    assert total == 1600 * 1599 // 2 and clusters == 1
    assert (labels[:1600] == 0).all() and (labels[1600:] == -1).all()


@pytest.mark.parametrize("order", ["forward", "backward", "shuffled"])
def test_long_chains_in_row_order(siso, order):
    """Rows that are only near their predecessors (a log that drifts in time): the groups are chains in row order, and finding
    them takes no longer than for the same chains over rows in any order."""
    K, d = 60000, 16
    print(f"case: merge_apply chains in row order, pairs {order}", flush=True)
    r = np.random.default_rng(1)
    pairs = np.stack([np.arange(K - 1), np.arange(1, K)], 1).astype(np.int32)
    pairs = pairs[(pairs[:, 1] % 20000 != 0)]  # three chains
    pairs = pairs[::-1] if order == "backward" else r.permutation(pairs) if order == "shuffled" else pairs
    cents = rows_of(K, d, "f32", 8)
    cache = siso.SisoCache(d, K, siso.F32)
    cache.load(cents)
    # a last pair that is none: the call is refused once the groups are known, so its time is theirs
    took = []
    for rows in (r.permutation(K).astype(np.int32), np.arange(K, dtype=np.int32)):
        p = torch.from_numpy(np.concatenate([rows[pairs], [[0, K]]]).astype(np.int32)).to(DEV)
        each = []
        for _ in range(4):
            torch.cuda.synchronize()
            begin = time.perf_counter()
            with pytest.raises(siso.SisoError):
                cache.merge_apply(p)
            each.append(time.perf_counter() - begin)
        took.append(min(each))
    assert took[1] < 3 * took[0], took
    surv = cache.merge_apply(torch.from_numpy(np.ascontiguousarray(pairs)).to(DEV)).cpu().numpy()
    assert np.array_equal(surv, np.arange(K) // 20000) and cache.count == 3
    assert cache.export()[2].tolist() == [20000] * 3
