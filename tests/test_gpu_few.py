"""A few queries in single precision (lookup_few.hip): remainders of its groups of 16 rows, blocks of 16 queries and rounds of
chunks, against double precision; and the sizes that are left to the tiled kernel."""

import numpy as np
import pytest
import torch

from gpu_util import DEV, SIM_TOL
from paper_2508_18736_amd import siso

pytestmark = pytest.mark.gpu


def few(K, d, n):
    """Whether k_lookup_few takes this batch (siso_few_slices); the tiled kernel does otherwise."""
    far = K * d * 4 > 384 << 20 and 7700 < 4 * d < 8600
    return d % 4 == 0 and d >= 64 and (n <= 16 or (n <= 32 and d < 1024)) and d <= 2496 and not far


def by_tiles(cache, queries):
    """The similarities of the tiled kernel, whose sums are added in another order."""
    cache.set_lookup_path(siso.PATH_SCALAR)
    sim = cache.lookup(queries, 0.5)[1].cpu().numpy()
    cache.set_lookup_path(siso.PATH_AUTO)
    return sim


# K: fewer rows than a group, a group and one row, an uneven number of groups per wave, for 16 queries more than all waves take
# at once; d: 300 and 65 * 4 end inside a round, 64 is the shortest row; 1,024 with 17 and 32 queries is the tiled kernel's
@pytest.mark.parametrize("K", [1, 17, 1000, 20011])
@pytest.mark.parametrize("d", [64, 260, 300, 384, 1024])
@pytest.mark.parametrize("n", [1, 15, 17, 32])
def test_few_queries_against_double_precision(K, d, n):
    g = torch.Generator().manual_seed(K * 31 + d * 7 + n)
    rows = torch.randn(K, d, generator=g)
    rows[K // 2] = rows[0]  # equal rows: the lower index wins
    q = rows[torch.randint(0, K, (n,), generator=g)] + 0.1 * torch.randn(n, d, generator=g)
    cache = siso.SisoCache(d, K + 3, siso.F32)
    cache.load(rows.to(DEV))
    padded = torch.empty(n * d + 1, device=DEV)
    for queries in (q.to(DEV), padded[1:].view(n, d).copy_(q)):  # 16-byte aligned and not
        idx, sim, hit = (x.cpu().numpy() for x in cache.lookup(queries.contiguous(), 0.5))
        r, x = rows.double().numpy(), q.double().numpy()
        cos = (x @ r.T) / np.linalg.norm(x, axis=1)[:, None] / np.linalg.norm(r, axis=1)[None, :]
        best = cos.max(1)
        # sums of d products of up to |x||r|, each sum and the two lengths within d * 2^-24 of exact at worst; and the bar of
        # single precision
        bound = min(3 * d * 2.0**-24, SIM_TOL["f32"])
        assert np.abs(sim - best).max() < bound
        assert (cos[np.arange(n), idx] > best - 2 * bound).all()
        assert not (idx == K // 2).any() or K // 2 == 0
        assert ((sim > 0.5) == (hit == 1)).all()
        if n >= 15 and d >= 260 and K >= 17:  # (some of so many sums differ in another order, none in the same)
            assert (sim != by_tiles(cache, queries.contiguous())).any() == few(K, d, n)


# Waves with several groups of rows each, for 17 to 32 queries too (256 workgroups of eight waves: 32,768 rows); d 1,020: 32
# queries take 128 KiB of LDS and end inside a round; 131,089 x 512 and 67,205 x 1,024 lie beyond 256 MiB, where 16 queries have twice the loads
# in flight; 52,000 x 2,000 and 17 x 2,500 are left to the tiles, 50,000 x 2,000 and 17 x 2,496 are not
@pytest.mark.parametrize("K,d,n", [(40003, 260, 17), (40003, 384, 32), (70001, 64, 32), (33000, 1020, 32), (131089, 512, 1), (131089, 512, 16),
                                   (131089, 512, 32), (67205, 1024, 15), (50000, 2000, 16), (52000, 2000, 16), (17, 2496, 16), (17, 2500, 16)])
def test_few_queries_and_several_groups_for_every_wave(K, d, n):
    print(f"case: few {K} x {d} n {n}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(K + n)
    rows = torch.randn(K, d, device=DEV, generator=g)
    # the closest rows: the last, others of the last group, some all over; and a second row equal to one of them, further on
    at = torch.cat([torch.tensor([K - 1, K - 2, 0, K // 2], device=DEV), torch.randint(0, K, (n,), device=DEV, generator=g)])[:n]
    q = rows[at] + 0.1 * torch.randn(n, d, device=DEV, generator=g)
    if n > 3 and K > 1000:
        rows[K // 2 + 700] = rows[K // 2]
    cache = siso.SisoCache(d, K, siso.F32)
    cache.load(rows)
    idx, sim, hit = cache.lookup(q, 0.5)
    cos = torch.empty(n, K, dtype=torch.float64, device=DEV)
    x = q.double() / q.double().norm(dim=1, keepdim=True)
    for lo in range(0, K, 16384):
        r = rows[lo:lo + 16384].double()
        cos[:, lo:lo + 16384] = x @ (r / r.norm(dim=1, keepdim=True)).T
    assert torch.equal(idx.long(), at) and bool((cos.gather(1, at[:, None])[:, 0] > cos.max(1).values - 1e-12).all())
    assert (sim.double() - cos.max(1).values).abs().max() < SIM_TOL["f32"] and bool((hit == 1).all())
    if n >= 15:
        assert (sim.cpu().numpy() != by_tiles(cache, q)).any() == few(K, d, n)


def test_few_queries_of_rows_without_a_length():
    d, K = 128, 100
    rows = torch.randn(K, d)
    rows[3] = 0
    rows[5, 7] = float("nan")
    rows[6, 0] = float("inf")
    cache = siso.SisoCache(d, K, siso.F32)
    cache.load(rows.to(DEV))
    q = torch.stack([rows[10], rows[20], torch.zeros(d), rows[5]]).to(DEV)
    idx, sim, hit = (x.cpu() for x in cache.lookup(q, 0.5))
    assert idx[:2].tolist() == [10, 20] and hit.tolist() == [1, 1, 0, 0]
    assert sim[2] == 0 and torch.isnan(sim[3])


def test_rows_about_8_kib_apart_are_left_to_the_tiles():
    """60,000 rows of 2,112 elements: not slower than the tiled kernel (where a load of 16 such rows would be)."""
    K, d, n = 60000, 2112, 16
    print(f"case: few {K} x {d}", flush=True)
    rows = torch.randn(K, d, device=DEV)
    q = rows[:n] + 0.1
    out = (torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV), torch.empty(n, dtype=torch.uint8, device=DEV))
    caches, took = [], [[], []]
    for path in (siso.PATH_AUTO, siso.PATH_SCALAR):
        caches.append(siso.SisoCache(d, K, siso.F32))
        caches[-1].set_lookup_path(path)
        caches[-1].load(rows)
    for i in range(12):
        for cache, t in zip(caches, took):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(8):
                cache.lookup(q, 0.5, *out)
            end.record()
            torch.cuda.synchronize()
            if i >= 2:
                t.append(begin.elapsed_time(end))
            assert out[0].tolist() == list(range(n))
    assert sorted(took[0])[5] < 1.08 * sorted(took[1])[5], took
