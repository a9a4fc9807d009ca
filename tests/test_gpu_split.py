"""Small single-precision lookups, whose dimension is split among the waves of a workgroup, against plain torch in 64 bits:
edges of the 32 x 32 tiles, dimensions that end inside a step, a chunk or a wave's share, rows at any alignment."""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("K,n", [(1, 33), (31, 255), (33, 100), (1000, 64), (1024, 256)])
@pytest.mark.parametrize("d", [1, 7, 30, 96, 97, 300, 384, 2048])
def test_lookup(K, n, d):
    from paper_2508_18736_amd import siso

    print(f"case: split lookup K={K} n={n} d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(K + n + d)
    c = torch.randn(K, d, device=DEV, generator=g)
    q = torch.randn(n, d, device=DEV, generator=g)
    if K > 40 and d > 1:
        c[3] = 0
        c[34, 1] = float("nan")
        c[36] = c[35]  # equal rows: the lower index
        q[5] = c[36]
        q[6, 0] = float("inf")
        q[7] = 0
    cache = siso.SisoCache(d, K, siso.F32)
    cache.load(c)
    idx, sim, hit = cache.lookup(q, 0.3)
    u, w = q.double(), c.double()
    s = (u / u.norm(dim=1, keepdim=True)) @ (w / w.norm(dim=1, keepdim=True)).T
    ok = torch.ones(n, dtype=torch.bool, device=DEV)
    if K > 40 and d > 1:
        s[:, 3] = 0  # (a row without length has similarity 0)
        s[:, 34] = -2
        assert torch.isnan(sim[6]) and idx[6] == -1 and sim[7] == 0 and idx[7] == 0 and (d < 7 or idx[5] == 35)
        ok[6:8] = False
    best = s[ok].max(1).values
    own = s[ok].gather(1, idx[ok].long()[:, None])[:, 0]
    # a sum of d products of unit vectors in single precision, four chains: at most (d / 4 + 8) roundings of 2^-24
    tol = (d / 4 + 8) * 2.0**-24
    assert (own - sim[ok].double()).abs().max() <= tol and (best - own).max() <= 2 * tol
    assert torch.equal(hit[ok], (sim[ok] > 0.3).to(torch.uint8))
