"""The work that a user of the centroid cache has it do, as cases whose time can be measured.

Every case goes through ``SisoCache``.  A pass is one of

``step``     the online loop: ``batches`` batches one after the other, each looked up and its hits folded into
             their centroids before the next (``lookup_update``).  Popularity is skewed, so later batches meet
             centroids that earlier ones have moved: their similarities show the updated state.
``copy``     the same loop with an 8-bit serving copy (``lookup_update_with`` on the copy and its bf16 master).
``lookup``   batches that are only looked up, on a cache of any storage type.
``topk``     the k closest centroids of a batch.
``merge``    a centroid set is loaded, its near-duplicates are found and merged, the result is exported.
``cluster``  a query log becomes a repository: community detection, one row per cluster, exported.
``refresh``  a snapshot is taken over, a repository is merged into it and the smallest rows leave (Algorithm 1),
             the threshold-to-hit-ratio table is taken anew, the new set is exported.

The vectors are Gaussian mixtures on the unit sphere like those of ``workloads.py`` (16 centroids per cluster in a
random order, noise of a given total length), drawn on the GPU.
"""

import math

import numpy as np
import torch

from paper_2508_18736_amd import siso

DEV = "cuda:0"
DTYPES = {"f32": (siso.F32, torch.float32, 4), "bf16": (siso.BF16, torch.bfloat16, 2), "fp8": (siso.FP8, torch.bfloat16, 1)}
THETA = 0.85        # retrieval threshold of the online cases
THETA_MERGE = 0.90  # clustering threshold of merge and refresh
THETA_LOG = 0.86    # and of the community detection
SWEEP = np.round(np.arange(0.98, 0.599, -0.02), 2).astype(np.float32)


def listed():
    return [
        # a small application's cache in single precision (the tiny configuration): latency of a handful of launches
        {"name": "f32_tiny_step", "op": "step", "dtype": "f32", "K": 1024, "d": 384, "n": 256, "batches": 4, "fresh": 0.0},
        # a cache of 60,000 centroids kept in single precision, requests in batches of a thousand
        {"name": "f32_mid_step", "op": "step", "dtype": "f32", "K": 60000, "d": 384, "n": 1000, "batches": 2, "fresh": 0.3},
        # interactive use: one request at a time against 60,000 centroids
        {"name": "bf16_one_step", "op": "step", "dtype": "bf16", "K": 60000, "d": 768, "n": 1, "batches": 16, "fresh": 0.3},
        # the streaming configuration: micro-batches of 64 with the update between them
        {"name": "bf16_stream_step", "op": "step", "dtype": "bf16", "K": 262144, "d": 768, "n": 64, "batches": 16, "fresh": 0.0},
        # the mid configuration: 30 % of the queries are new directions and miss
        {"name": "bf16_mid_step", "op": "step", "dtype": "bf16", "K": 65536, "d": 768, "n": 4096, "batches": 2, "fresh": 0.3},
        # the large configuration, the benchmark's default
        {"name": "bf16_large_step", "op": "step", "dtype": "bf16", "K": 1048576, "d": 1024, "n": 16384, "batches": 2, "fresh": 0.0},
        # the streaming configuration on an 8-bit serving copy that follows its bf16 master
        {"name": "fp8_stream_copy", "op": "copy", "dtype": "fp8", "K": 262144, "d": 768, "n": 64, "batches": 16, "fresh": 0.0},
        # bulk lookups on an 8-bit cache, sizes that fill no tile
        {"name": "fp8_bulk_lookup", "op": "lookup", "dtype": "fp8", "K": 300001, "d": 768, "n": 5000, "batches": 1, "fresh": 0.3},
        # candidates for re-ranking: the 8 closest of a ragged batch
        {"name": "bf16_topk", "op": "topk", "dtype": "bf16", "K": 60000, "d": 768, "n": 1000, "k": 8, "fresh": 0.3},
        # the merge configuration: eight near-duplicates of everything
        {"name": "bf16_merge", "op": "merge", "dtype": "bf16", "K": 131072, "d": 768, "copies": 8},
        # a day's query log, topics of 2 to 12 questions
        {"name": "bf16_cluster_log", "op": "cluster", "dtype": "bf16", "n": 50001, "d": 768},
        # the periodic replacement: a repository of a tenth of the cache
        {"name": "bf16_refresh", "op": "refresh", "dtype": "bf16", "K": 65536, "d": 768, "r": 6553},
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; half of them odd sizes, the others rounded to 64."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= 256 and rng.random() < 0.4:
        v = v // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "copy", "lookup", "lookup", "topk", "topk", "merge", "cluster", "refresh"])
    if op in ("step", "lookup", "topk"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"] if op == "step" else ["bf16", "fp8", "fp8", "f32"] if op == "lookup" else ["bf16", "bf16", "fp8", "f32"])
        d = rng.choice([256, 384, 512, 768, 1024] if dtype == "fp8" else [128, 256, 300, 384, 512, 768, 768, 1024])
        # (300: averaged word vectors; a dimension the tiled kernels have to pad)
        K = _log_int(rng, 1000, 400000)
        n = _log_int(rng, 1, 8192)
        # single precision and odd dimensions are for small and middling caches
        most = (2e10 if op == "topk" else 1e11) if dtype == "f32" or d % 64 else 5e12
        while n > 1 and 2.0 * n * K * d > most:
            n = max(1, n // 2)
        case = {"op": op, "dtype": dtype, "K": K, "d": d, "n": n, "fresh": rng.choice([0.0, 0.3, 0.6])}
        if op == "topk":
            case["k"] = rng.choice([2, 4, 5, 8, 10, 16, 32])
            case["K"] = max(case["K"], 100 * case["k"])
        else:
            case["batches"] = 1 if op == "lookup" else 16 if n <= 8 else 8 if n <= 256 else 2
        return case
    if op == "copy":
        return {"op": op, "dtype": "fp8", "K": _log_int(rng, 8000, 400000), "d": rng.choice([384, 512, 768, 1024]),
                "n": _log_int(rng, 1, 1024), "batches": 8, "fresh": rng.choice([0.0, 0.3])}
    d = rng.choice([256, 384, 768, 1024])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    if op == "merge":
        return {"op": op, "dtype": dtype, "K": _log_int(rng, 2000, 8000 if dtype == "f32" else 131072), "d": d, "copies": rng.choice([2, 4, 8])}
    if op == "cluster":
        return {"op": op, "dtype": dtype, "n": _log_int(rng, 2000, 8000 if dtype == "f32" else 80000), "d": d}
    K = _log_int(rng, 4000, 16000 if dtype == "f32" else 200000)
    return {"op": op, "dtype": dtype, "K": K, "d": d, "r": max(64, K // rng.choice([8, 10, 20, 40]))}


# ------------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------------
def _unit(x):
    return x / x.square().sum(1, keepdim=True).sqrt()


def _directions(g, n, d):
    return _unit(torch.randn(n, d, device=DEV, generator=g))


def _near(g, base, rows, sigma, dtype):
    """normalize(base[rows[i]] + noise of total length sigma), in pieces."""
    d = base.shape[1]
    out = torch.empty(rows.shape[0], d, dtype=dtype, device=DEV)
    for lo in range(0, rows.shape[0], 131072):
        x = torch.randn(min(131072, rows.shape[0] - lo), d, device=DEV, generator=g)
        s = sigma[lo:lo + 131072, None] if isinstance(sigma, torch.Tensor) else sigma
        x = x * (s / math.sqrt(d)) + base[rows[lo:lo + 131072]].float()
        out[lo:lo + 131072] = _unit(x).to(dtype)
    return out


def _mixture(g, K, d, per, sigma, dtype):
    """K rows, `per` jittered copies of each mean in a random order; and the cluster of every row."""
    clusters = -(-K // per)
    of = (torch.arange(K, device=DEV) // per)[torch.randperm(K, device=DEV, generator=g)]
    return _near(g, _directions(g, clusters, d), of, sigma, dtype), of


def _requests(g, cents, of, n, fresh):
    """n queries: clusters by Zipf(1.1) over a random ranking, a random row of the cluster, jittered; a share of
    `fresh` of them are new directions."""
    K, d = cents.shape
    clusters = int(of.max().item()) + 1
    order = torch.argsort(of, stable=True)
    size = torch.bincount(of, minlength=clusters)
    start = torch.cumsum(size, 0) - size
    p = torch.arange(1, clusters + 1, device=DEV, dtype=torch.float64).pow(-1.1)
    cdf = torch.cumsum(p / p.sum(), 0)
    rank = torch.searchsorted(cdf, torch.rand(n, device=DEV, generator=g, dtype=torch.float64)).clamp_(max=clusters - 1)
    cl = torch.randperm(clusters, device=DEV, generator=g)[rank]
    pick = (torch.rand(n, device=DEV, generator=g) * size[cl]).long()
    rows = order[start[cl] + torch.minimum(pick, size[cl] - 1)]
    q = _near(g, cents, rows, 0.08, cents.dtype)
    new = torch.rand(n, device=DEV, generator=g) < fresh
    return torch.where(new[:, None], _directions(g, n, d).to(q.dtype), q).contiguous()


def _query_log(g, n, d, dtype):
    """n log entries in a random order: topics of 2 to 12 entries (cosine about 0.99 inside a topic), and one entry in
    twenty unrelated to all others.  The sizes of the topics do not depend on the draw."""
    grouped = n - n // 20
    topics = grouped // 7 + 2
    members = torch.arange(topics, device=DEV) % 11 + 2
    topic_of = torch.repeat_interleave(torch.arange(topics, device=DEV), members)[:grouped]
    rows = torch.cat([_near(g, _directions(g, topics, d), topic_of, 0.1, dtype), _directions(g, n - topic_of.shape[0], d).to(dtype)])
    return rows[torch.randperm(n, device=DEV, generator=g)].contiguous()


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    op, d = case["op"], case["d"]
    dtype = DTYPES[case["dtype"]][1]
    s = {}
    if op in ("step", "copy", "lookup", "topk"):
        n = case["n"]
        s["cents"], of = _mixture(g, case["K"], d, 16, 0.08, dtype)
        s["batches"] = list(_requests(g, s["cents"], of, n * case.get("batches", 1), case["fresh"]).split(n))
    elif op == "merge":
        s["rows"], _ = _mixture(g, case["K"], d, case["copies"], 0.03, dtype)
        s["counts"] = torch.randint(1, 40, (case["K"],), device=DEV, generator=g, dtype=torch.int32)
    elif op == "cluster":
        s["log"] = _query_log(g, case["n"], d, dtype)
    elif op == "refresh":
        K, r = case["K"], case["r"]
        s["cents"], of = _mixture(g, K, d, 16, 0.08, dtype)
        cents = s["cents"]
        s["counts"] = torch.randint(1, 40, (K,), device=DEV, generator=g, dtype=torch.int32)
        s["references"] = list(_requests(g, cents, of, min(K, 16384), 0.3).split(4096))
        near = torch.randint(0, K, (r // 2,), device=DEV, generator=g)
        repo = torch.cat([_near(g, cents, near, 0.06, dtype), _directions(g, r - r // 2, d).to(dtype)])
        s["repo"] = repo[torch.randperm(r, device=DEV, generator=g)].contiguous()
        s["sizes"] = torch.randint(1, 40, (r,), device=DEV, generator=g).float()
        # the sample of the table: a twentieth of the cache's size, similarities spread over the sweep
        m = max(64, K // 20)
        length = torch.rand(m, device=DEV, generator=g) * 1.2 + 0.1
        s["sample"] = _near(g, cents, torch.randint(0, K, (m,), device=DEV, generator=g), length, dtype)
    return s


def prepare(case, seed):
    op, d, kind = case["op"], case["d"], DTYPES[case["dtype"]][0]
    s = {"op": op, "case": case, **_inputs(case, seed)}
    if op in ("step", "copy", "lookup", "topk"):
        K, n = case["K"], case["n"]
        cents = s.pop("cents")
        s["cache"] = siso.SisoCache(d, K, kind)
        s["cache"].load(cents)
        if op == "copy":
            s["master"] = siso.SisoCache(d, K, siso.BF16)
            s["master"].load(cents)
        for c in (s["cache"], s.get("master")):
            if c is not None:
                c.reserve(n)  # a serving loop sizes its workspaces once
    elif op == "merge":
        s["cache"] = siso.SisoCache(d, case["K"], kind)
        s["cap"] = case["K"] * (case["copies"] - 1) // 2 + 1024
        s["cache"].set_option("second_set", 1)  # (a cache that is rebuilt now and then keeps its second set)
    elif op == "cluster":
        s["cache"] = siso.SisoCache(d, case["n"], kind)
    elif op == "refresh":
        s["cache"] = siso.SisoCache(d, case["K"] + case["r"], kind)
        s["cache"].set_option("second_set", 1)
        s["cache"].load(s.pop("cents"), s.pop("counts"))
        for q in s.pop("references"):  # they decide who leaves
            s["cache"].lookup(q, THETA)
        s["snapshot"] = s["cache"].export() + s["cache"].export_meta()
    torch.cuda.synchronize()
    return s


def run(s):
    op, cache, case = s["op"], s["cache"], s["case"]
    if op == "step":
        return [cache.lookup_update(q, THETA) for q in s["batches"]]
    if op == "copy":
        return [cache.lookup_update_with(s["master"], q, THETA) for q in s["batches"]]
    if op == "lookup":
        return [cache.lookup(q, THETA) for q in s["batches"]]
    if op == "topk":
        return cache.lookup_topk(s["batches"][0], case["k"])
    if op == "merge":
        cache.load(s["rows"], s["counts"])
        pairs, total = cache.merge(THETA_MERGE, s["cap"])
        survivors = cache.merge_apply(pairs)
        return total, survivors, cache.export(), cache.export_meta()
    if op == "cluster":
        labels, clusters, total = cache.cluster(s["log"], THETA_LOG, 2)
        return labels, clusters, total, cache.export(), cache.export_meta()
    cents, means, counts, size, access = s["snapshot"]
    cache.import_state(cents, means, counts, size, access)
    stats = cache.refresh(s["repo"], s["sizes"], THETA_MERGE, case["K"] + case["K"] // 50)
    hits = cache.t2h(s["sample"], SWEEP)
    return stats, hits, cache.export(), cache.export_meta()


def work(case):
    op, d = case["op"], case["d"]
    e = DTYPES[case["dtype"]][2]
    if op in ("step", "copy", "lookup", "topk"):
        K, n, b = case["K"], case["n"], case.get("batches", 1)
        inp = n * d * (4 if case["dtype"] == "f32" else 2)
        # every batch waits for the fold of the one before it, so each reads the centroids and their inverse lengths anew
        each = K * (d * e + 4) + inp + n * 8 * case.get("k", 1) + n
        if op in ("step", "copy"):  # mean read and written, stored row written (and its codes)
            each += int(n * (1 - case["fresh"])) * d * (8 + max(e, 2) + (1 if op == "copy" else 0))
        return {"bytes": b * each, "flops": 2.0 * b * n * K * d}
    if op == "merge":
        K = case["K"]
        live = K // case["copies"]
        # load: rows in, rows and means out; search: rows; groups: means in; gather and export: survivors twice
        return {"bytes": K * d * (e + e + 4 + e + 4) + live * d * (e + 4) * 4, "flops": float(K) * K * d}
    if op == "cluster":
        n = case["n"]
        return {"bytes": n * d * e * 3 + n // 7 * d * (e + 4) * 3, "flops": float(n) * n * d}
    K, r = case["K"], case["r"]
    m = max(64, K // 20)
    # import and the gather and the export of the new set: rows and means in and out; the searches: rows
    return {"bytes": K * d * (e + 4) * 6 + (2 * K + 3 * r) * d * e + m * d * e, "flops": 2.0 * r * K * d + float(r) * r * d + 2.0 * m * K * d}


def tolerance(case):
    # Similarities are single-precision sums of 128 to 1,024 exact products.  The same passes with the sums in another
    # order (another kernel of the library) differ by up to 6.6e-7 in the 2-norm and 1.5e-6 at one value, and name the
    # same rows; 8-bit lookups by 2.8e-8, but a centroid that rounds to another code moves a similarity by about 1e-5.
    # Exported rows are means rounded to bf16: where a mean lies on a rounding boundary (under 0.2 % of the elements)
    # the last bit may go either way: sqrt(0.002) * 2^-8 in the 2-norm, one step of 2^-7 at one value.
    if case["op"] in ("merge", "cluster", "refresh"):
        return {"rel": 2e-4, "max": 0.01, "differ": 1e-4}
    return {"rel": 1e-5 if case["op"] == "copy" else 3e-6, "max": 1e-4, "differ": 5e-4}


# ------------------------------------------------------------------------------------------------------------------
# the same passes in 64 bits, by plain torch
# ------------------------------------------------------------------------------------------------------------------
def _dir64(x):
    """Rows at unit length, in 64 bits."""
    return _unit(x.double())


def _codes64(x):
    """The E4M3 codes of 8-bit rows (scale = largest element / 448, in single precision), as 64-bit numbers."""
    x = x.float()
    most = x.abs().amax(1, keepdim=True)
    return (x / (most / torch.full_like(most, 448.0))).to(torch.float8_e4m3fn).double()


def _best64(q, c, k=1):
    """(index, cosine) of the k closest rows of c for every row of q; both hold unit rows."""
    best_i, best_s = [], []
    block = max(1, (1 << 30) // c.shape[0])
    for lo in range(0, q.shape[0], block):
        p = q[lo:lo + block] @ c.T
        v, i = p.topk(k, dim=1) if k > 1 else p.max(1, keepdim=True)
        best_i.append(i)
        best_s.append(v)
    return torch.cat(best_i), torch.cat(best_s)


def _first_neighbour64(u, theta):
    """Per row the lowest index among itself and the rows closer than theta, and their number (u: unit rows)."""
    n = u.shape[0]
    first, degree = [], []
    block = max(1, (1 << 29) // n)
    for lo in range(0, n, block):
        near = u[lo:lo + block] @ u.T > theta
        i = torch.arange(near.shape[0], device=DEV)
        near[i, i + lo] = True
        first.append(near.to(torch.uint8).argmax(1))
        degree.append(near.sum(1))
    return torch.cat(first), torch.cat(degree)


def _exact_steps(case, s):
    dtype, theta = DTYPES[case["dtype"]][1], torch.tensor(THETA, dtype=torch.float32).double().to(DEV)
    stored = (lambda x: _unit(_codes64(x))) if case["dtype"] == "fp8" else _dir64
    mean = _dir64(s["cents"])
    weight = torch.ones(case["K"], 1, dtype=torch.float64, device=DEV)
    c = stored(s["cents"])
    out = []
    for q in s["batches"]:
        idx, sim = _best64(stored(q), c)
        idx, sim = idx[:, 0], sim[:, 0]
        hit = sim > theta
        out.append((idx.int(), sim, hit.to(torch.uint8)))
        rows, at = idx[hit].unique(return_inverse=True)
        if rows.numel():
            total = (mean[rows] * weight[rows]).index_add_(0, at, _dir64(q[hit]))
            weight[rows] += torch.bincount(at, minlength=rows.numel()).double()[:, None]
            mean[rows] = total / weight[rows]
            c[rows] = stored(_unit(mean[rows]).to(dtype))
    return out


def _exact_refresh(case, s):
    K, r = case["K"], case["r"]
    mean = _dir64(s["cents"])
    access = torch.zeros(K, dtype=torch.int64, device=DEV)
    for q in s["references"]:
        idx, sim = _best64(_dir64(q), mean)
        access += torch.bincount(idx[:, 0][sim[:, 0] > float(np.float32(THETA))], minlength=K)
    repo = _dir64(s["repo"])
    theta = float(np.float32(THETA_MERGE))
    idx, sim = (x[:, 0].tolist() for x in _best64(repo, mean))
    candidates = [[] for _ in range(r)]  # earlier rows of the repository above the threshold
    block = max(1, (1 << 29) // r)
    for lo in range(0, r, block):
        p = repo[lo:lo + block] @ repo.T
        for i, j in (p > theta).nonzero().tolist():
            if j < i + lo:
                candidates[i + lo].append((p[i, j].item(), j))
    size = s["counts"].double().tolist()
    refs = access.tolist()
    source, place, merged = list(range(K)), {}, 0
    for i, w in enumerate(s["sizes"].tolist()):
        best, at = sim[i], idx[i]
        for v, j in candidates[i]:
            if j in place and v > best:
                best, at = v, place[j]
        if best > theta:
            size[at] += w
            merged += 1
        else:
            place[i] = len(source)
            source.append(K + i)
            size.append(w)
            refs.append(0xFFFFFFFF)
    order = sorted(range(len(source)), key=lambda j: (size[j], refs[j], j))
    evicted = max(0, len(source) - (K + K // 50))
    kept = sorted(order[evicted:])
    src = torch.tensor([source[j] for j in kept], device=DEV)
    weight = torch.cat([s["counts"], s["sizes"].round().int()])[src]
    loc = torch.tensor([size[j] for j in kept], dtype=torch.float64, device=DEV) / 1.1
    cents = torch.cat([s["cents"], s["repo"]])[src]
    new = torch.cat([mean, repo])[src]
    _, best = _best64(_dir64(s["sample"]), _dir64(cents))
    hits = np.array([int((best > float(t)).sum()) for t in SWEEP], dtype=np.int64)
    return (merged, len(place), evicted), hits, (cents.double(), new, weight), (loc, torch.zeros_like(loc, dtype=torch.int64))


def exact(case, seed):
    op, s = case["op"], _inputs(case, seed)
    if op in ("step", "copy", "lookup"):
        return _exact_steps(case, s)  # (a lookup is one batch: what would follow it is not looked at)
    if op == "topk":
        rows = (lambda x: _unit(_codes64(x))) if case["dtype"] == "fp8" else _dir64
        idx, sim = _best64(rows(s["batches"][0]), rows(s["cents"]), case["k"])
        return idx.int(), sim
    if op == "refresh":
        return _exact_refresh(case, s)
    # merge and cluster: groups whose rows are all neighbours of each other
    rows = s["rows"] if op == "merge" else s["log"]
    u = _dir64(rows)
    n = rows.shape[0]
    first, degree = _first_neighbour64(u, THETA_MERGE if op == "merge" else THETA_LOG)
    total = (int(degree.sum()) - n) // 2
    if op == "merge":
        leaders, group = first.unique(return_inverse=True)
        count = s["counts"].double()
    else:
        leaders, group = first.unique(return_inverse=True)
        members = torch.bincount(group)
        order = torch.argsort(members, descending=True, stable=True)
        order = order[members[order] > 1]
        number = torch.full_like(members, -1)
        number[order] = torch.arange(order.numel(), device=DEV)
        labels, group, leaders = number[group], number[group], leaders[order]
        count = torch.ones(n, dtype=torch.float64, device=DEV)
    keep = group >= 0
    weight = torch.zeros(leaders.numel(), dtype=torch.float64, device=DEV).index_add_(0, group[keep], count[keep])
    mean = torch.zeros(leaders.numel(), case["d"], dtype=torch.float64, device=DEV)
    mean = mean.index_add_(0, group[keep], u[keep] * count[keep, None]) / weight[:, None]
    cents = _unit(mean)
    if op == "merge":
        alone = torch.bincount(group) == 1
        cents[alone] = rows[leaders[alone]].double()
    state = (cents, mean, weight.int()), (weight, torch.zeros(leaders.numel(), dtype=torch.int64, device=DEV))
    return (total, group.int(), *state) if op == "merge" else (labels.int(), leaders.numel(), total, *state)
