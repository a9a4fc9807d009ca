"""A few queries in single precision (lookup_few.hip): remainders of its groups of 16 rows, blocks of 16 queries and rounds of
chunks, against double precision."""

import numpy as np
import pytest
import torch

from gpu_util import DEV
from paper_2508_18736_amd import siso

pytestmark = pytest.mark.gpu


# K: fewer rows than a group, a group and one row, an uneven number of groups per wave, more than all waves take at once;
# d: 300 and 65 * 4 end inside a round, 64 is the shortest row, 1,024 x 32 queries fill LDS
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
        # sums of d products of up to |x||r|, each sum and the two lengths within d * 2^-24 of exact at worst
        bound = 3 * d * 2.0**-24
        assert np.abs(sim - best).max() < bound
        assert (cos[np.arange(n), idx] > best - 2 * bound).all()
        assert not (idx == K // 2).any() or K // 2 == 0
        assert ((sim > 0.5) == (hit == 1)).all()


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
