"""Lookups of up to 64 bf16 queries over the bytes of the rows, forced on by an option, against the kernel that reads the rows as
they are stored: the same bits, whatever the rows and queries, with and without the fold of the hits."""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SKINNY = 3
THETA = 0.85


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


def pair(siso, c, capacity=None):
    """Two caches of the same rows: over the bytes, and as they are stored."""
    out = []
    for screen in (4, 2):
        cache = siso.SisoCache(c.shape[1], capacity or c.shape[0], siso.BF16)
        cache.set_option("screen", screen)
        if screen == 2:
            cache.set_lookup_path(SKINNY)
        cache.load(c)
        out.append(cache)
    return out


def mixture(g, K, d, common=0.0, per=16):
    """Rows in groups around directions that share a common part (mean cosine `common`), of random lengths."""
    unit = torch.nn.functional.normalize
    base = unit(torch.randn(-(-K // per), d, device=DEV, generator=g), dim=1) * (1 - common) ** 0.5
    base = unit(base + common ** 0.5 * unit(torch.randn(1, d, device=DEV, generator=g), dim=1), dim=1)
    c = base[torch.randint(0, base.shape[0], (K,), device=DEV, generator=g)] + 0.08 / d ** 0.5 * torch.randn(K, d, device=DEV, generator=g)
    return (c * (0.5 + torch.rand(K, 1, device=DEV, generator=g))).bfloat16()


def queries(g, c, n, common=0.0):
    q = c[torch.randint(0, c.shape[0], (n,), device=DEV, generator=g)].float() + 0.05 / c.shape[1] ** 0.5 * torch.randn(n, c.shape[1], device=DEV, generator=g)
    miss = torch.rand(n, device=DEV, generator=g) < 0.4
    other = torch.randn(n, c.shape[1], device=DEV, generator=g)
    if common:
        other = mixture(g, max(n, 32), c.shape[1], 0.0)[:n].float() + c.float().mean(0)
    return torch.where(miss[:, None], other, q).bfloat16()


def same(a, b, what):
    for x, y in zip(a, b):
        assert torch.equal(x, y) or torch.equal(x.nan_to_num(nan=7.0), y.nan_to_num(nan=7.0)), what


@pytest.mark.parametrize("K,n,d", [(1, 1, 128), (31, 2, 256), (32, 33, 192), (33, 64, 320), (257, 7, 384), (2048, 64, 448), (8191, 32, 512),
                                   (20000, 64, 640), (65537, 31, 768), (65536 * 2 + 5, 64, 768), (70001, 1, 832), (70000, 40, 960), (90000, 64, 1024),
                                   (100003, 3, 1024)])
@pytest.mark.parametrize("common", [0.0, 0.7])
def test_the_same_bits(siso, K, n, d, common):
    print(f"case: few over bytes K={K} n={n} d={d} common={common}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(K + n)
    c = mixture(g, K, d, common)
    a, b = pair(siso, c)
    for seed in range(2):
        q = queries(g, c, n, common)
        same(a.lookup(q, THETA), b.lookup(q, THETA), "lookup")
    for seed in range(5):
        q = queries(g, c, n, common)
        same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), f"step {seed}")
    same(a.export() + a.export_meta(), b.export() + b.export_meta(), "state")
    assert a.bad_indices() == 0


def test_rows_and_queries_that_bytes_say_nothing_about(siso):
    print("case: few over bytes, odd rows", flush=True)
    g = torch.Generator(device=DEV).manual_seed(2)
    K, d, n = 9000, 768, 40
    c = mixture(g, K, d)
    c[5] = 0
    c[77, 3] = float("nan")
    c[200] *= 1e-20
    c[300, 9] = float("inf")
    c[400] *= 1e18
    c[8999] = 0
    c[1000:1100] = c[1000]  # equal rows: the lowest
    a, b = pair(siso, c)
    q = queries(g, c, n)
    same(a.lookup(q, THETA), b.lookup(q, THETA), "odd rows")
    q[0] = 0
    q[1, 5] = float("nan")
    q[2] = c[1050]
    q[3] = c[200] * 1e15
    same(a.lookup(q, THETA), b.lookup(q, THETA), "odd queries")
    same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), "odd queries, folded")
    q[4] = c[500] * 1e-19  # a length near the end of the range: nothing of the batch goes by the bytes
    q[5] = 1e-30
    same(a.lookup(q, THETA), b.lookup(q, THETA), "odd lengths")
    q = queries(g, c, n)
    same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), "behind them")
    c[0], c[1] = float("nan"), 0  # the first row with a weight
    a, b = pair(siso, c)
    q[0] = 0
    same(a.lookup(q, THETA), b.lookup(q, THETA), "a query of zeros")


@pytest.mark.parametrize("d", [128, 768])
def test_rows_close_together(siso, d):
    """More rows near the best than the lists hold: every workgroup that finds no room multiplies its rows as they are stored."""
    print(f"case: few over bytes, crowded d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(3)
    for K, common, n in ((40000, 0.98, 64), (40000, 0.9, 1), (9000, 1.0, 33)):
        c = mixture(g, K, d, common, per=1)
        a, b = pair(siso, c)
        q = queries(g, c, n, common)
        same(a.lookup(q, THETA), b.lookup(q, THETA), "lookup")
        same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), "step")
        q = queries(g, c, n, common)
        same(a.lookup(q, THETA), b.lookup(q, THETA), "lookup behind it")


def test_rows_that_change(siso):
    """Updates of every size, loads, rows whose largest element outgrows the scale of its block, and replays of a recorded step:
    blocks whose bytes are behind are multiplied as they are stored, or written anew."""
    print("case: few over bytes, changing rows", flush=True)
    g = torch.Generator(device=DEV).manual_seed(4)
    K, d = 12000, 384
    c = mixture(g, K, d)
    a, b = pair(siso, c)
    for seed, n in enumerate((64, 300, 1, 5, 64)):
        q = queries(g, c, n)
        if seed == 3:  # spikes
            q = torch.zeros(n, d, device=DEV, dtype=torch.bfloat16)
            q[:, 7] = 1
        idx = torch.randint(0, K, (n,), device=DEV, generator=g, dtype=torch.int32)
        for cache in (a, b):
            cache.update(q, idx)
        p = queries(g, c, 64)
        p[:5, 7] += 20
        same(a.lookup(p, THETA), b.lookup(p, THETA), f"update {seed}")
        same(a.lookup_update(p, 0.3), b.lookup_update(p, 0.3), f"step {seed}")
        same(a.lookup(p, THETA), b.lookup(p, THETA), f"behind step {seed}")
    q, out = queries(g, c, 64), [[torch.empty(64, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.uint8)] for _ in range(2)]
    graphs = []
    torch.cuda.synchronize()
    for cache, o in zip((a, b), out):
        side = torch.cuda.Stream()
        cache.set_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            cache.lookup_update(q, THETA, *o)
        graphs.append(graph)
    for seed in range(5):
        q.copy_(queries(g, c, 64))
        more = mixture(g, K, d)
        torch.cuda.synchronize()
        if seed == 2:
            a.load(more)
            b.load(more)
        if seed == 3:
            a.update(q, out[1][0])
            b.update(q, out[1][0])
        torch.cuda.synchronize()
        for graph in graphs:
            graph.replay()
        torch.cuda.synchronize()
        same(*out, f"replay {seed}")
    same(a.export(), b.export(), "state behind the replays")
    torch.cuda.synchronize()
    got = a.lookup(q, THETA), b.lookup(q, THETA)  # (on two streams)
    torch.cuda.synchronize()
    same(*got, "behind the replays")


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()  # (all but torch's own)


@pytest.mark.parametrize("capacity,K,d,n,batches", [(100000, 90000, 768, 64, (1, 8)), (139999, 135000, 768, 64, (9, 32)), (280000, 275000, 256, 8, (1, 8)),
                                                    (2097153, 270000, 256, 1000, (1, 64))])
@pytest.mark.parametrize("refused", [False, True])
def test_a_reservation_serves_every_smaller_batch(siso, capacity, K, d, n, batches, refused):
    """Also the batches that go over the bytes from fewer rows on than the reserved one, a cache that holds fewer rows than it can, and a reservation
    that found no room: none of them allocates."""
    print(f"case: few over bytes, reserved capacity={capacity} n={n} refused={refused}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    cache = siso.SisoCache(d, capacity, siso.BF16)
    c = torch.randn(K, d, device=DEV, generator=g).bfloat16()
    cache.load(c)
    assert all(cache.screened(b) for b in batches[:1])
    if refused:
        cache.set_option("screen_room", 1)
    before = free()
    cache.reserve(n)
    assert (before - free() >= K * d) == (not refused)
    cache.set_option("screen_room", 0)
    before = free()
    for b in batches:
        q = queries(g, c, b)
        for _ in range(6):
            cache.lookup_update(q, THETA)
    assert abs(before - free()) < 2 << 20  # (a reservation of the driver's)


@pytest.mark.parametrize("K,d,over,stored", [(65536, 1024, (), (1, 8, 64)), (65537, 1024, (1, 8), (9, 64)), (131072, 768, (8,), (9, 64)), (131073, 768, (9, 64), ()),
                                             (131072, 1024, (8, 16), (17, 64)), (131073, 1024, (17, 32), (33, 64)), (196608, 896, (33, 64), ()),
                                             (196608, 960, (32,), (33,)), (196609, 960, (33, 64), ())])
def test_where_small_lookups_go_over_bytes(siso, K, d, over, stored):
    """On both sides of every line: where steps over the bytes take longer, with few or many misses, they stay with the stored rows."""
    print(f"case: lines of small lookups K={K} d={d}", flush=True)
    cache = siso.SisoCache(d, K, siso.BF16)
    cache.load(torch.ones(K, d, dtype=torch.bfloat16, device=DEV))
    assert [n for n in over + stored if cache.screened(n)] == list(over)


def test_lists_without_room_are_not_asked_for_again(siso):
    """Room for the bytes (1 MiB) and none for the lists (1.7 MiB): the rows as they are stored, also when there would be room, until siso_reserve."""
    print("case: few over bytes, no room for lists", flush=True)
    g = torch.Generator(device=DEV).manual_seed(9)
    c = mixture(g, 4096, 256)
    a, b = pair(siso, c)
    q = queries(g, c, 64)
    want = b.lookup(q, THETA)
    a.set_option("screen", 2)
    a.reserve(64)  # (keys)
    a.set_option("screen", 4)
    a.set_option("screen_room", 1200)
    before = free()
    same(a.lookup(q, THETA), want, "no room")
    with_bytes = free()
    a.set_option("screen_room", 0)
    for _ in range(3):
        same(a.lookup(q, THETA), want, "not asked for again")
    assert free() == with_bytes
    a.reserve(64)
    assert free() < with_bytes <= before
    same(a.lookup(q, THETA), want, "room")


@pytest.mark.parametrize("d,n,units,folds", [(1024, 64, 63, False), (1024, 64, 64, True), (768, 3, 2, False), (256, 64, 21, False), (256, 64, 22, True), (768, 64, 0, True)])
def test_workgroups_that_do_not_fit_together_do_not_wait_for_each_other(siso, d, n, units, folds):
    """With a limit of zero looks at the board a fold gives up on every hit; the two calls wait for nothing."""
    print(f"case: few over bytes on {units} units, d={d} n={n}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(d)
    c = mixture(g, 5000, d)
    a, b = pair(siso, c)
    a.set_option("fold_units", units)
    a.set_option("fold_spin_limit", 0)
    q = queries(g, c, n)
    before = a.export()
    got, want = a.lookup_update(q, THETA), b.lookup_update(q, THETA)
    same(got, want, "step")
    hits = int(want[2].sum().item())
    assert hits > 0 and a.bad_indices() == (hits if folds else 0)
    same(a.export(), before if folds else b.export(), "state")
    if not folds:
        same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), "step behind it")
        same(a.export(), b.export(), "state behind it")


def test_the_units_of_a_stream_are_asked_for_under_capture(siso):
    print("case: few over bytes, stream set under capture", flush=True)
    g = torch.Generator(device=DEV).manual_seed(12)
    c = mixture(g, 5000, 512)
    a, b = pair(siso, c)
    q = queries(g, c, 64)
    for cache in (a, b):
        cache.lookup(q, THETA)
    out = [torch.empty(64, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.uint8)]
    main, graph = torch.cuda.current_stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        a.set_stream(torch.cuda.current_stream())
        a.lookup_update(q, THETA, *out)
    a.set_stream(main)
    for seed in range(3):
        graph.replay()
        torch.cuda.synchronize()
        same(out, b.lookup_update(q, THETA), f"replay {seed}")
    same(a.export(), b.export(), "state")


@pytest.mark.parametrize("K,d,common,n", [(131072, 768, 0.8, 32), (140001, 768, 0.6, 64), (64000, 1024, 0.8, 8), (64000, 1024, 0.6, 8), (100000, 256, 0.9, 33), (262144, 384, 0.8, 1)])
def test_rows_that_fill_the_lists_in_part(siso, K, d, common, n):
    """Some workgroups find places in a query's list, others do not and multiply their rows as they are stored, in turn over several calls."""
    print(f"case: few over bytes, lists that fill K={K} d={d} n={n}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(K + d)
    c = mixture(g, K, d, common)
    a, b = pair(siso, c)
    for seed in range(4):
        q = queries(g, c, n, common)
        same(a.lookup_update(q, THETA), b.lookup_update(q, THETA), f"step {seed}")
    same(a.export(), b.export(), "state")


def took(f, reps):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(3):
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_a_recorded_step_goes_over_the_stored_rows(siso):
    """A graph cannot turn back once its lists flood: recorded on rows without a common direction and replayed on rows with one, it takes the time of the rows as
    they are stored (over the bytes five times that; the line is far above what machines and runs differ by), with the same results."""
    print("case: few over bytes, recorded by default", flush=True)
    g = torch.Generator(device=DEV).manual_seed(21)
    K, d, n = 140001, 768, 64
    c, crowded = mixture(g, K, d), mixture(g, K, d, 0.8)
    q, main = queries(g, c, n), torch.cuda.current_stream()
    times, out = [], []
    for screen in (0, 2):
        cache = siso.SisoCache(d, K, siso.BF16)
        cache.set_option("screen", screen)
        cache.load(c)
        assert cache.screened(n) == (screen == 0)
        for _ in range(6):
            cache.lookup_update(q, THETA)
        out.append([torch.empty(n, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.uint8)])
        torch.cuda.synchronize()
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        cache.set_stream(side)
        with torch.cuda.graph(graph, stream=side):
            cache.lookup_update(q, THETA, *out[-1])
        cache.set_stream(main)
        cache.load(crowded)
        p = queries(torch.Generator(device=DEV).manual_seed(22), crowded, n, 0.8)
        q.copy_(p)
        torch.cuda.synchronize()
        times.append(took(graph.replay, 20))
        q.copy_(queries(torch.Generator(device=DEV).manual_seed(23), crowded, n, 0.8))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
    same(out[0], out[1], "replays")
    assert times[0] < 2 * times[1], times


def kernel_us(cache, f, reps):
    """Time of the kernel that reads the rows, over the bytes about half of what it takes over the stored ones."""
    cache.profile_enable(1)
    for _ in range(reps):
        f()
    ms, times = cache.profile_read()
    cache.profile_enable(0)
    return ms / times * 1e3


@pytest.mark.parametrize("K,d,n,common", [(66000, 1024, 8, 0.6), (262144, 768, 64, 0.6), (140001, 768, 32, 0.8)])
def test_lookups_that_leave_many_rows_turn_to_the_stored_rows(siso, K, d, n, common):
    """Rows with a common direction, whether the lists run over or are only long: most of a stream of lookups goes over the rows as they are stored."""
    print(f"case: few over bytes, long lists by default K={K} d={d} n={n} common={common}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(26)
    c = mixture(g, K, d, common)
    q = [queries(g, c, n, common) for _ in range(8)]
    caches = []
    for screen in (0, 2):
        caches.append(siso.SisoCache(d, K, siso.BF16))
        caches[-1].set_option("screen", screen)
        caches[-1].load(c)
        assert caches[-1].screened(n) == (screen == 0)
    for seed in range(100):
        same(caches[0].lookup(q[seed % 8], THETA), caches[1].lookup(q[seed % 8], THETA), f"lookup {seed}")
    for _ in range(200):
        for x in q:
            caches[0].lookup(x, THETA)
        torch.cuda.synchronize()
    times = [kernel_us(cache, lambda: [cache.lookup(x, THETA) for x in q], 40) for cache in caches]
    assert 0.85 * times[1] < times[0] < 1.25 * times[1], times


def test_which_way_lookups_go_by_default(siso):
    """Steps that fold their hits go over the bytes from the second one behind a load on, steps of two calls over the stored rows (the bytes would be
    written each time), lookups alone over the bytes again."""
    print("case: few over bytes, ways by default", flush=True)
    g = torch.Generator(device=DEV).manual_seed(24)
    K, d, n = 262144, 768, 64
    c = mixture(g, K, d)
    q = queries(g, c, n)
    cache, plain = siso.SisoCache(d, K, siso.BF16), siso.SisoCache(d, K, siso.BF16)
    plain.set_option("screen", 2)
    for x in (cache, plain):
        x.load(c)
        x.reserve(n)

    def two(x=cache):
        idx, sim, hit = x.lookup(q, THETA)
        x.update(q, idx, hit)
        return idx, sim, hit

    stored = kernel_us(plain, lambda: plain.lookup(q, THETA), 20)
    for load in range(2):
        for x in (cache, plain):
            x.load(c)
        cache.lookup_update(q, THETA)
        plain.lookup_update(q, THETA)
        for step in range(70):  # (through the writing behind 64 lookups)
            same(cache.lookup_update(q, THETA), plain.lookup_update(q, THETA), f"step {step}")
        assert kernel_us(cache, lambda: cache.lookup_update(q, THETA), 20) < 0.8 * stored
        for _ in range(20):
            plain.lookup_update(q, THETA)
        for step in range(40):
            same(two(), two(plain), f"two calls {step}")
        assert kernel_us(cache, two, 20) > 0.85 * stored
        for _ in range(130):  # (twice as many as the 60 steps have come to)
            cache.lookup(q, THETA)
        assert kernel_us(cache, lambda: cache.lookup(q, THETA), 20) < 0.8 * stored
