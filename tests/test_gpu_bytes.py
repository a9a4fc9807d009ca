"""The rows of a cache as bytes are kept from one screened lookup to the next: behind everything that changes rows, and behind
graphs replayed in between, a lookup names what it names on a fresh cache that holds the same rows."""

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
THETA = 0.85
SKINNY = 3


@pytest.fixture(scope="module")
def siso():
    from paper_2508_18736_amd import siso as m
    return m


def rows(g, n, d, dtype, base=None):
    x = torch.randn(n, d, device=DEV, generator=g)
    if base is not None:
        x = 0.1 * x / d ** 0.5 + torch.nn.functional.normalize(base[torch.randint(0, base.shape[0], (n,), device=DEV, generator=g)].float(), dim=1)
    return (x * (0.5 + torch.rand(n, 1, device=DEV, generator=g))).to(TYPES[dtype])


def make(siso, capacity, d, dtype):
    cache = siso.SisoCache(d, capacity, siso.F32 if dtype == "f32" else siso.BF16)
    cache.set_option("screen", 1)
    return cache


def as_fresh(siso, cache, d, dtype, q, what):
    """The lookup on this cache, bit for bit what a cache gives that has just been loaded with its rows."""
    c = cache.export()[0]
    other = make(siso, c.shape[0], d, dtype)
    other.load(c)
    got, want = cache.lookup(q, THETA), other.lookup(q, THETA)
    for a, b in zip(got, want):
        assert torch.equal(a, b), what


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [128, 300, 768])
def test_behind_every_change_of_rows(siso, dtype, d):
    print(f"case: kept bytes {dtype} d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(d)
    K = 3000
    cache = make(siso, 4000, d, dtype)
    c = rows(g, K, d, dtype, rows(g, 300, d, dtype))
    cache.load(c)
    q = torch.cat([rows(g, 400, d, dtype, c), rows(g, 100, d, dtype)])
    as_fresh(siso, cache, d, dtype, q, "load")
    as_fresh(siso, cache, d, dtype, q, "nothing")
    for n in (1, 64, 300, 500):
        cache.lookup_update(q[:n], THETA)
        as_fresh(siso, cache, d, dtype, q, f"update of {n}")
    idx = torch.randint(0, K, (200,), device=DEV, generator=g, dtype=torch.int32)
    cache.update(rows(g, 200, d, dtype), idx)
    as_fresh(siso, cache, d, dtype, q, "update")
    for k in (2011, 33, 3999, 31, 2048, 2047, 1):  # rows that are left behind the last one, and come back
        cache.load(rows(g, k, d, dtype, c))
        as_fresh(siso, cache, d, dtype, q, f"load of {k}")
    cache.load(c)
    snapshot = cache.export() + cache.export_meta()
    cache.lookup_update(q, THETA)
    cache.lookup(q, THETA)
    cache.import_state(*snapshot)
    as_fresh(siso, cache, d, dtype, q, "import")
    pairs, _ = cache.merge(0.9, 1 << 20)
    cache.merge_apply(pairs)
    assert cache.count < K
    as_fresh(siso, cache, d, dtype, q, "merge")
    for seed in range(3):  # the two sets of arrays in turn
        cache.refresh(rows(g, 200, d, dtype), torch.ones(200, device=DEV), 0.9, 2000)
        as_fresh(siso, cache, d, dtype, q, f"refresh {seed}")
        cache.lookup_update(q, 0.3)
        as_fresh(siso, cache, d, dtype, q, f"update behind refresh {seed}")
    cache.cluster(rows(g, 2500, d, dtype, c[:300]), 0.86, 2)
    as_fresh(siso, cache, d, dtype, q, "cluster")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_behind_replayed_graphs(siso, dtype):
    """A recorded step and a recorded lookup, replayed with other steps and a load in between, before and behind a growth of the room."""
    print(f"case: kept bytes graph {dtype}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(5)
    d, K, n = 256, 2000, 300
    cache = make(siso, 6000, d, dtype)
    c = rows(g, K, d, dtype, rows(g, 200, d, dtype))
    cache.load(c)
    q, p = rows(g, n, d, dtype, c), rows(g, n, d, dtype, c)
    out = [(torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV), torch.empty(n, dtype=torch.uint8, device=DEV)) for _ in range(2)]
    cache.reserve(n)
    cache.lookup_update(q, THETA)
    side = torch.cuda.Stream()
    cache.set_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        cache.lookup_update(q, THETA, *out[0])
        cache.lookup(p, THETA, *out[1])
    for seed in range(4):
        q.copy_(rows(g, n, d, dtype, c))
        p.copy_(rows(g, n, d, dtype, c))
        torch.cuda.synchronize()
        other = make(siso, 6000, d, dtype)
        snapshot = cache.export() + cache.export_meta()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        other.import_state(*snapshot)
        want = [other.lookup_update(q, THETA), other.lookup(p, THETA)]
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            for x, y in zip(a, b):
                assert torch.equal(x, y), seed
        if seed == 1:
            more = rows(g, 5000, d, dtype, c)
            torch.cuda.synchronize()
            cache.load(more)  # (bytes for more rows than the recorded launches know of)
            cache.lookup(q, THETA)
            torch.cuda.synchronize()
            cache.load(more[:K])
            torch.cuda.synchronize()
        if seed == 2:
            cache.update(rows(g, 100, d, dtype), torch.randint(0, K, (100,), device=DEV, generator=g, dtype=torch.int32))
            torch.cuda.synchronize()
            as_fresh(siso, cache, d, dtype, q, "update between replays")


@pytest.mark.parametrize("copy", [False, True])
def test_bytes_that_a_recorded_fold_writes_to_stay(siso, copy):
    """A step whose lookup goes over the stored rows (here: more than 64 queries, or an 8-bit copy) writes the bytes of the rows it folds.  A graph that
    holds it refers to them: they stay when the cache outgrows them, which is looked at before the graph is replayed, and replays then leave the rows and the
    later lookups that they leave on a cache without bytes."""
    print(f"case: kept bytes of a recorded fold, copy={copy}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(17)
    d, K, capacity, n = 256, 40000, 200000, 64 if copy else 100

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()  # (all but torch's own)

    c, more = rows(g, K, d, "bf16", rows(g, 4000, d, "bf16")), rows(g, capacity, d, "bf16")
    q, few = rows(g, n, d, "bf16", c), rows(g, 64, d, "bf16", c)
    out = [(torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV), torch.empty(n, dtype=torch.uint8, device=DEV)) for _ in range(2)]
    caches, others, graphs = [], [], []
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    for screen, o in zip((4, 2), out):
        cache = siso.SisoCache(d, capacity, siso.BF16)
        cache.set_option("screen", screen)
        cache.load(c)
        cache.lookup(few, THETA)  # (of the first: makes its bytes)
        other = siso.SisoCache(d, capacity, siso.FP8) if copy else None
        if copy:
            other.load(c)
        for stream in (main, side):
            torch.cuda.synchronize()
            for x in filter(None, (cache, other)):
                x.set_stream(stream)
            step = (lambda: other.lookup_update_with(cache, q, THETA, *o)) if copy else (lambda: cache.lookup_update(q, THETA, *o))
            if stream is main:
                step()
            else:
                graphs.append(torch.cuda.CUDAGraph())
                with torch.cuda.graph(graphs[-1], stream=side):
                    step()
        for x in filter(None, (cache, other)):
            x.set_stream(main)
        caches.append(cache)
        others.append(other)
    torch.cuda.synchronize()
    caches[0].load(more)
    before = free()
    caches[0].lookup(few, THETA)  # (bytes for all of the capacity: 51 MB, and the 10 MB of before stay)
    assert before - free() > capacity * d
    caches[1].load(more)
    for cache in caches:
        cache.load(c)
    for seed in range(4):
        q.copy_(rows(g, n, d, "bf16", c))
        torch.cuda.synchronize()
        for graph in graphs:
            graph.replay()
            torch.cuda.synchronize()
        for x, y in zip(*out):
            assert torch.equal(x, y), seed
        assert out[0][2].sum() > 0
        for x, y in zip(caches[0].export(), caches[1].export()):
            assert torch.equal(x, y), seed
        caches[1].set_lookup_path(SKINNY)  # (the kernel with the same sums)
        for x, y in zip(caches[0].lookup(few, THETA), caches[1].lookup(few, THETA)):
            assert torch.equal(x, y), seed


@pytest.mark.parametrize("room,grows", [(0, True), (55, True), (40, False)])
def test_bytes_that_grow(siso, room, grows):
    """Beside the bytes of before (10 MB), in their place where both do not fit, or not at all: then those of before serve as many rows as before."""
    print(f"case: growing bytes, room={room}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(19)
    d, K, capacity = 256, 40000, 200000
    c = rows(g, capacity, d, "bf16", rows(g, 4000, d, "bf16"))
    q = rows(g, 64, d, "bf16", c[:K])
    caches = []
    for screen in (4, 2):
        caches.append(siso.SisoCache(d, capacity, siso.BF16))
        caches[-1].set_option("screen", screen)
        caches[-1].set_lookup_path(SKINNY)

    def step(k, what):
        for cache in caches:
            cache.load(c[:k])
        for _ in range(2):
            for x, y in zip(caches[0].lookup_update(q, THETA), caches[1].lookup_update(q, THETA)):
                assert torch.equal(x, y), what

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()  # (all but torch's own)

    step(K, "few rows")
    caches[1].reserve(64)
    caches[0].set_option("screen", 2)
    caches[0].reserve(64)  # (keys)
    caches[0].set_option("screen", 4)
    caches[0].set_option("screen_room", room << 10)
    before = free()
    step(capacity, "all rows")
    more = before - free()
    assert 36 << 20 < more < 45 << 20 if grows else abs(more) < 4 << 20
    step(K, "few rows again")
    assert abs(before - more - free()) < 4 << 20


@pytest.mark.parametrize("room,moves", [(0, False), (52, True)])
def test_bytes_of_a_cache_that_is_nearly_full(siso, room, moves):
    """They have room for all it can hold (54 MB), so the last rows do not move them; where that is not to be had, for the rows that there are (48 MB)."""
    print(f"case: bytes of a nearly full cache, room={room}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(23)
    d, K, capacity = 1024, 48000, 54000
    c = rows(g, capacity, d, "bf16", rows(g, 4000, d, "bf16"))
    q = rows(g, 300, d, "bf16", c[:K])
    cache = make(siso, capacity, d, "bf16")
    cache.load(c[:K])

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()  # (all but torch's own)

    cache.set_option("screen_room", room << 10)
    before = free()
    cache.lookup(q, THETA)
    first = free()
    assert before - first > K * d
    cache.set_option("screen_room", 0)
    cache.load(c)
    cache.lookup(q, THETA)
    assert (free() < first - (2 << 20)) == moves
    as_fresh(siso, cache, d, "bf16", q, "all rows")


@pytest.mark.parametrize("kind", ["f32", "bf16", "copy"])
@pytest.mark.parametrize("d", [256, 384, 1024])
def test_small_folds_over_rows_with_bytes(siso, kind, d):
    """Steps whose lookup goes over the stored rows, on a cache that has bytes: current ones (which follow, if they are bf16), ones that an update has left
    behind, and none yet.  Later lookups over the bytes name what they name on a fresh cache."""
    print(f"case: small folds, {kind} d={d}", flush=True)
    dtype = "f32" if kind == "f32" else "bf16"
    g = torch.Generator(device=DEV).manual_seed(d + 1)
    K = 6000
    c = rows(g, K, d, dtype, rows(g, 600, d, dtype))
    cache, twin = make(siso, K, d, dtype), make(siso, K, d, dtype)
    copies = [siso.SisoCache(d, K, siso.FP8) if kind == "copy" else None for _ in range(2)]
    for x, y in zip((cache, twin), copies):
        x.load(c)
        if y is not None:
            y.load(c)
    big = torch.cat([rows(g, 400, d, dtype, c), rows(g, 100, d, dtype)])

    def step(x, y, q):
        return x.lookup_update(q, 0.5) if y is None else y.lookup_update_with(x, q, 0.5)

    def small(what):
        for n in (1, 64, 128, 200 if kind == "f32" else 100, 7):
            q = rows(g, n, d, dtype, c)
            q[::5, 7] += 3 * q[::5].float().norm(dim=1).to(q.dtype)  # (rows whose largest element outgrows the scale of their bytes)
            cache.set_option("screen", 2)
            twin.set_option("screen", 2)
            for a, b in zip(step(cache, copies[0], q), step(twin, copies[1], q)):
                assert torch.equal(a, b), (what, n)
            cache.set_option("screen", 1)
            as_fresh(siso, cache, d, dtype, big, f"{what}, {n}")
            if dtype == "bf16":
                cache.set_option("screen", 4)
                cache.lookup(big[:64], THETA)
                cache.set_option("screen", 1)
        for a, b in zip(cache.export(), twin.export()):
            assert torch.equal(a, b), what

    for n in (1, 100):  # (no bytes yet)
        for x, y in zip((cache, twin), copies):
            x.set_option("screen", 2)
            step(x, y, big[:n])
    cache.set_option("screen", 1)
    cache.lookup(big, THETA)
    small("current")
    idx, q = torch.randint(0, K, (50,), device=DEV, generator=g, dtype=torch.int32), rows(g, 50, d, dtype)
    for x in (cache, twin):
        x.update(q, idx)
    for _ in range(2):
        small("behind an update")
