// Cache replacement: Algorithm 1 (SISO-CacheManager) of section 4.2 — MergeCentroids,
// FilteringCentroids, UpdateCentroids.
//
// The merge step takes the repository centroids one after the other and compares each with
// C_new as it stands then, so its decisions form a chain.  What is heavy in it is data
// parallel and runs in the library's kernels:
//   * every repository row against every cached centroid: one batched lookup;
//   * every repository row against every other one: the pair search, which lists the pairs above
//     the clustering threshold (only those can change a decision: a row joins C_new when nothing
//     in it is closer than the threshold, whatever is closest then);
//   * the cosines of the listed pairs (to tell which candidate is the closest).
// The chain itself (who joined, who took whose cluster size) and the choice of the survivors
// (the smallest (cluster_size, access_count) go first) are bookkeeping over a few numbers per
// row and are done on the host, in the order the algorithm states; then the new centroid set is
// gathered on the GPU and becomes the cache between two lookups of the stream (a lookup sees
// the old set or the new one, never a mixture; nothing is locked, so nothing needs to be
// replaced piecemeal).
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <utility>
#include <vector>

#include "siso_internal.h"

struct RefreshCandidate {  // an earlier repository row above the threshold
    int row;
    float cosine;
};

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// both counters of the call: rows that cannot be taken, pairs found
__global__ void k_clear(u64 *bad, u64 *pairs) {
    *bad = 0;
    *pairs = 0;
}

// What the host decides on, to pinned host memory (a copy engine takes longer to get going than these few hundred
// kilobytes take): five arrays of r or K0 numbers, one behind the other.
__global__ void k_report(const int *__restrict__ idx, const float *__restrict__ sim, const float *__restrict__ rsize, long r,
                         const float *__restrict__ loc, const unsigned *__restrict__ acc, long K0, int *h_idx, float *h_sim,
                         float *h_rsize, float *h_loc, unsigned *h_acc) {
    const long n = r > K0 ? r : K0;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        if (i < r) {
            h_idx[i] = idx[i];
            h_sim[i] = sim[i];
            h_rsize[i] = rsize[i];
        }
        if (i < K0) {
            h_loc[i] = loc[i];
            h_acc[i] = acc[i];
        }
    }
}

__global__ void k_nan_tail(float *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = __uint_as_float(0x7FC00000u);
}

// Copy the repository rows into a buffer with readable rows behind them, with 1 / |row|; count the
// rows that hold a NaN or an infinity and the cluster sizes that are not positive finite numbers.
template <typename T>
__global__ __launch_bounds__(256) void k_stage_repo(const T *__restrict__ src, const float *__restrict__ sizes, T *dst,
                                                     float *invn, int d, u64 *bad) {
    __shared__ float sh[4];
    const long k = blockIdx.x;
    float ss = 0.f;
    for (int e = threadIdx.x; e < d; e += 256) {
        const T x = src[(size_t)k * d + e];
        dst[(size_t)k * d + e] = x;
        const float f = widen(x);
        ss += f * f;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float inv = inv_length((sh[0] + sh[1]) + (sh[2] + sh[3]));
        invn[k] = inv;
        const float s = sizes[k];
        if (!(inv == inv) || !(s > 0.f) || s > 3.0e38f) atomicAdd(bad, 1ull);
    }
}

// cosine of the two rows of every listed pair, one wave per pair (the arithmetic of the lookup's
// last step: fp32 products summed per lane, then over the lanes, then scaled by both inverse lengths); the pairs and
// their cosines go to the host.  The number of pairs is read from the device, so that the host need not know it yet; at
// most `most` are looked at from `from` on.
template <typename T>
__global__ __launch_bounds__(256) void k_pair_cosines(const T *__restrict__ rows, const float *__restrict__ invn,
                                                       const int *__restrict__ pairs, const u64 *__restrict__ n_pairs, long from,
                                                       long most, int d, int *h_pairs, float *h_cos) {
    const long n = *n_pairs < (u64)(from + most) ? (long)*n_pairs : from + most;
    const int lane = threadIdx.x & 63;
    for (long p = from + (long)blockIdx.x * 4 + (threadIdx.x >> 6); p < n; p += (long)gridDim.x * 4) {
        const long a = pairs[2 * p], b = pairs[2 * p + 1];
        float acc = 0.f;
        for (int e = lane; e < d; e += 64) acc += widen(rows[(size_t)a * d + e]) * widen(rows[(size_t)b * d + e]);
        acc = wave_sum(acc);
        if (lane == 0) {
            h_pairs[2 * p] = (int)a;
            h_pairs[2 * p + 1] = (int)b;
            h_cos[p] = acc * invn[a] * invn[b];
        }
    }
}

// New row j <- source src[j]: a cached row (src < K0) with all it carries, or repository row
// src - K0, which starts a cluster of its own: stored as it is, mean = its direction, weight of
// the mean = its cluster size rounded to a whole number of members (at least 1).
template <typename T>
__global__ __launch_bounds__(256) void k_refresh_gather(const int *__restrict__ src, long K0, const T *__restrict__ cent,
                                                         const float *__restrict__ mean, const int *__restrict__ size,
                                                         const float *__restrict__ invn, const T *__restrict__ repo,
                                                         const float *__restrict__ repo_invn,
                                                         const float *__restrict__ repo_size,
                                                         const float *__restrict__ loc, T *cent2, float *mean2,
                                                         int *size2, float *invn2, float *loc2, unsigned *acc2,
                                                         unsigned *version2, int d) {
    const long j = blockIdx.x;
    const long s = src[j];
    if (threadIdx.x == 0) {
        loc2[j] = loc[j];
        acc2[j] = 0u;
        raise_version_once(version2, j);
    }
    if (s < K0) {
        for (int e = threadIdx.x; e < d; e += 256) {
            cent2[(size_t)j * d + e] = cent[(size_t)s * d + e];
            mean2[(size_t)j * d + e] = mean[(size_t)s * d + e];
        }
        if (threadIdx.x == 0) {
            size2[j] = size[s];
            invn2[j] = invn[s];
        }
    } else {
        const long r = s - K0;
        const float inv = repo_invn[r];
        for (int e = threadIdx.x; e < d; e += 256) {
            const T x = repo[(size_t)r * d + e];
            cent2[(size_t)j * d + e] = x;
            mean2[(size_t)j * d + e] = widen(x) * inv;  // inv = 0 for a zero row
        }
        if (threadIdx.x == 0) {
            const float w = rintf(repo_size[r]);
            size2[j] = w < 1.f ? 1 : (w > 2147483647.f ? 2147483647 : (int)w);
            invn2[j] = inv;
        }
    }
}

struct DeviceBuf {  // frees on every way out
    void *p = nullptr;
    ~DeviceBuf() {
        if (p) (void)hipFree(p);
    }
    bool alloc(size_t bytes) { return hipMalloc(&p, bytes ? bytes : 1) == hipSuccess; }
    template <class U>
    U *as() const {
        return (U *)p;
    }
};

}  // namespace

// The lists of plan_refresh, kept by a cache from one refresh to the next: taken anew they are megabytes of fresh pages each
// time, and touching those for the first time took longer than the bookkeeping (65,536 rows: 340 us between the last
// kernel of the searches and the gather, 260 with kept lists).
struct RefreshLists {
    std::vector<long> first, fill, place;
    std::vector<RefreshCandidate> cand;
    std::vector<int> src;
    std::vector<float> loc, decayed;  // cluster sizes, and what they are behind the decay
    std::vector<unsigned> acc, with;
    std::vector<u64> key, same;
    bool keyed = false;  // key and with are those of loc and acc
    hipEvent_t reported = nullptr;
    ~RefreshLists() {
        if (reported) (void)hipEventDestroy(reported);
    }
    size_t bytes() const {
        return (first.capacity() + fill.capacity() + place.capacity()) * sizeof(long) + cand.capacity() * sizeof(RefreshCandidate) +
               (src.capacity() + loc.capacity() + decayed.capacity() + acc.capacity() + with.capacity()) * 4 +
               (key.capacity() + same.capacity()) * sizeof(u64);
    }
};

void siso_refresh_release(siso_cache *c) {
    delete c->refresh_lists;
    c->refresh_lists = nullptr;
}

namespace {

// (cluster_size, access_count) as one number that orders alike; -0 and 0 are the same size
inline u64 refresh_key(float size, unsigned references) {
    const float f = size + 0.0f;
    unsigned u;
    memcpy(&u, &f, 4);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((u64)u << 32) | references;
}

// What can be done before the searches have ended: the lists as they stand before the first repository row, and, if rows may have
// to go, their numbers and how many share the upper 16 bits of one.
void plan_prepare(long K0, long r, const float *h_loc, const unsigned *h_acc, long max_centroids, RefreshLists &l) {
    l.loc.reserve((size_t)(K0 + r));
    l.acc.reserve((size_t)(K0 + r));
    l.src.reserve((size_t)(K0 + r));
    l.key.reserve((size_t)(K0 + r));
    l.decayed.reserve((size_t)(K0 + r));
    l.loc.assign(h_loc, h_loc + K0);
    l.acc.assign(h_acc, h_acc + K0);
    l.decayed.resize((size_t)K0);
    for (long j = 0; j < K0; ++j) l.decayed[(size_t)j] = l.loc[(size_t)j] / 1.1f;
    l.src.resize((size_t)K0);  // C_new: source of every row (cached row, or K0 + repository row)
    for (long j = 0; j < K0; ++j) l.src[(size_t)j] = (int)j;
    l.keyed = K0 + r > max_centroids;
    if (!l.keyed) return;
    l.key.resize((size_t)K0);
    l.with.assign((size_t)1 << 16, 0);
    for (long j = 0; j < K0; ++j) l.key[(size_t)j] = refresh_key(l.loc[(size_t)j], l.acc[(size_t)j]);
    for (long j = 0; j < K0; ++j) l.with[(size_t)(l.key[(size_t)j] >> 48)] += 1;
}

// The decisions of Algorithm 1 from what the kernels found, behind plan_prepare.  Per repository row i: h_idx / h_sim = its closest
// cached centroid and the cosine; h_pairs / h_cos = the pairs (a, b), a < b, of repository rows above the
// threshold with their cosines.  l.loc / l.acc = cluster_size and access_count of the cached centroids (they grow
// by the rows that join).  The outcome: out_src = the source of every surviving row in order (cached row, or K0 + repository
// row), out_loc = its cluster size behind the decay; their number is returned.
long plan_refresh(long K0, long r, const int *h_idx, const float *h_sim, const float *h_rsize, const int *h_pairs,
                  const float *h_cos, long n_pairs, float theta_c, long max_centroids, RefreshLists &l, int *out_src, float *out_loc,
                  long &merged, long &added, long &evicted) {
    std::vector<float> &loc = l.loc, &decayed = l.decayed;
    std::vector<unsigned> &acc = l.acc, &with = l.with;
    std::vector<int> &src = l.src;
    std::vector<u64> &key = l.key;
    std::vector<long> &first = l.first, &place = l.place;
    std::vector<RefreshCandidate> &cand = l.cand;
    // ---- the chain of the merge step, in the order of the repository ---------------------
    // candidates of row b: the earlier rows a < b with cosine above the threshold (pairs come as a < b)
    first.assign((size_t)r + 1, 0);
    for (long p = 0; p < n_pairs; ++p) first[(size_t)h_pairs[2 * p + 1] + 1] += 1;
    for (long i = 0; i < r; ++i) first[(size_t)i + 1] += first[(size_t)i];
    cand.resize((size_t)n_pairs);
    {
        std::vector<long> &fill = l.fill;
        fill.assign(first.begin(), first.end() - 1);
        for (long p = 0; p < n_pairs; ++p) {
            const int b = h_pairs[2 * p + 1];
            cand[(size_t)fill[(size_t)b]++] = RefreshCandidate{h_pairs[2 * p], h_cos[(size_t)p]};
        }
    }
    place.assign((size_t)r, -1);  // position in C_new of a repository row that joined
    merged = added = 0;
    for (long i = 0; i < r; ++i) {
        long best = h_idx[(size_t)i];
        float bsim = h_sim[(size_t)i];
        if (best < 0 || !(bsim == bsim)) {
            best = -1;
            bsim = -INFINITY;
        }
        for (long q = first[(size_t)i]; q < first[(size_t)i + 1]; ++q) {
            const long pos = place[(size_t)cand[(size_t)q].row];
            if (pos < 0) continue;  // that row did not join: it is not in C_new
            const float s = cand[(size_t)q].cosine;
            if (s > bsim || (s == bsim && pos < best)) {
                bsim = s;
                best = pos;
            }
        }
        if (best >= 0 && bsim > theta_c) {
            loc[(size_t)best] = loc[(size_t)best] + h_rsize[(size_t)i];
            decayed[(size_t)best] = loc[(size_t)best] / 1.1f;
            if (l.keyed) {
                with[(size_t)(key[(size_t)best] >> 48)] -= 1;
                key[(size_t)best] = refresh_key(loc[(size_t)best], acc[(size_t)best]);
                with[(size_t)(key[(size_t)best] >> 48)] += 1;
            }
            ++merged;
        } else {
            place[(size_t)i] = (long)src.size();
            src.push_back((int)(K0 + i));
            loc.push_back(h_rsize[(size_t)i]);
            decayed.push_back(loc.back() / 1.1f);
            acc.push_back(SISO_ACCESS_INF);
            if (l.keyed) {
                key.push_back(refresh_key(loc.back(), SISO_ACCESS_INF));
                with[(size_t)(key.back() >> 48)] += 1;
            }
            ++added;
        }
    }

    // ---- filtering step: the smallest (cluster_size, access_count) go, the first such first ----
    const long n_new = (long)src.size();
    evicted = n_new > max_centroids ? n_new - max_centroids : 0;
    long out = 0;
    auto stay = [&](long from, long to) {  // these rows, one behind the other
        if (from >= to) return;
        memcpy(out_src + out, src.data() + from, (size_t)(to - from) * sizeof(int));
        memcpy(out_loc + out, decayed.data() + from, (size_t)(to - from) * sizeof(float));
        out += to - from;
    };
    if (evicted == 0) {
        stay(0, n_new);
        return out;
    }
    // the evicted-th smallest number: its upper 16 bits from the count of them, the rest among the rows that share those
    std::vector<u64> &same = l.same;
    long below = 0;
    size_t top = 0;
    while (below + with[top] < evicted) below += with[top++];
    same.clear();
    same.reserve((size_t)with[top]);
    for (long j = 0; j < n_new; ++j)
        if ((key[(size_t)j] >> 48) == top) same.push_back(key[(size_t)j]);
    std::nth_element(same.begin(), same.begin() + (evicted - below - 1), same.end());
    const u64 last = same[(size_t)(evicted - below - 1)];  // rows with a smaller number go,
    long at_last = evicted - below;                        // and of those with this one so many, the first ones
    for (u64 v : same) at_last -= v < last ? 1 : 0;
    long from = 0;
    for (long j = 0; j < n_new; ++j) {
        const u64 v = key[(size_t)j];
        if (v > last || (v == last && at_last-- <= 0)) continue;
        stay(from, j);
        from = j + 1;
    }
    stay(from, n_new);
    return out;
}

}  // namespace

static int refresh_impl(siso_cache *c, const void *repo, const float *repo_size, long r, float theta_c,
                        long max_centroids, long *out_stats) {
    if (!c) return SISO_EINVAL;
    if (c->dtype == SISO_FP8) return siso_fail(c, SISO_EINVAL, "siso_refresh: not available with the 8-bit storage");
    if (out_stats) out_stats[0] = out_stats[1] = out_stats[2] = 0;
    if (r < 0 || max_centroids < 1 || max_centroids > c->capacity || (r > 0 && (!repo || !repo_size)))
        return siso_fail(c, SISO_EINVAL, "siso_refresh: bad arguments (1 <= max_centroids <= capacity %ld)", c->capacity);
    if (r > 2147483647L / 4 || c->count + r > 2147483647L)
        return siso_fail(c, SISO_EINVAL, "siso_refresh: %ld repository rows are too many", r);
    if (((uintptr_t)repo & 15) != 0) return siso_fail(c, SISO_EINVAL, "siso_refresh: repository rows must be 16-byte aligned");
    const long K0 = c->count;
    const int d = c->dim;
    const size_t eb = c->dtype == SISO_F32 ? 4 : 2;
    hipStream_t st = c->stream;
#define REFRESH_TRY(expr, what)                                   \
    do {                                                          \
        const int rc_ = siso_check_hip(c, (expr), what);          \
        if (rc_ != SISO_OK) return rc_;                           \
    } while (0)

    // ---- device side of the merge step -------------------------------------------------
    // Everything the host decides on is on its way before it waits for the first time: the lookups, the pair search and
    // the cosines of the first pairs do no harm if the check of the repository rows, read at the same time, then fails.
    long cap = r * 4 > (1L << 20) ? r * 4 : (1L << 20);  // room for pairs
    const long early = 16384;                            // of which the cosines are formed before their number is known
    char *d_rows;
    float *d_rinv, *d_sim, *d_loc2, *h_sim, *h_rsize, *h_loc, *h_cos, *h_loc2;
    int *d_idx, *d_pairs, *d_src, *h_idx, *h_pairs, *h_src;
    unsigned *h_acc;
    auto layout = [&](Carver a, Carver h) {
        d_rows = a.take<char>((size_t)(r + SISO_PAD_ROWS) * d * eb);
        d_rinv = a.take<float>(r + SISO_PAD_ROWS);
        d_idx = a.take<int>(r);
        d_sim = a.take<float>(r);
        d_pairs = a.take<int>(2 * cap);
        d_src = a.take<int>(2 * (K0 + r));
        h_idx = h.take<int>(r);
        h_sim = h.take<float>(r);
        h_rsize = h.take<float>(r);
        h_loc = h.take<float>(K0);
        h_acc = h.take<unsigned>(K0);
        h_pairs = h.take<int>(2 * early);
        h_cos = h.take<float>(early);
        h_src = h.take<int>(2 * (K0 + r));
        return std::pair<size_t, size_t>(a.used, h.used);
    };
    {
        const std::pair<size_t, size_t> need = layout(Carver{nullptr}, Carver{nullptr});
        const int rc = siso_arena(c, need.first, need.second);
        if (rc != SISO_OK) return rc;
        layout(Carver{c->arena}, Carver{c->pinned});
    }
    DeviceBuf more_pairs;  // a list that turned out too short
    std::vector<int> all_pairs;
    std::vector<float> all_cos;
    long n_pairs = 0;
    u64 *bad_at = c->counters + 2, *found_at = c->counters + 1;
    auto search = [&](int *pairs, long room) { return siso_pairs_launch(c, d_rows, d_rinv, r, theta_c, pairs, room, found_at); };
    auto cosines = [&](const int *pairs, long from, long most, int *to_pairs, float *to_cos) {
        const dim3 grid((unsigned)(most < 4096 ? (most + 3) / 4 : 1024)), block(256);
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_pair_cosines<float>, grid, block, 0, st, (const float *)d_rows, d_rinv, pairs, found_at, from, most,
                               d, to_pairs, to_cos);
        else
            hipLaunchKernelGGL(k_pair_cosines<bf16_t>, grid, block, 0, st, (const bf16_t *)d_rows, d_rinv, pairs, found_at, from, most,
                               d, to_pairs, to_cos);
        return siso_check_hip(c, hipGetLastError(), "k_pair_cosines");
    };
    if (c->refresh_lists == nullptr) c->refresh_lists = new RefreshLists;
    RefreshLists &lists = *c->refresh_lists;
    if (lists.reported == nullptr) REFRESH_TRY(hipEventCreateWithFlags(&lists.reported, hipEventDisableTiming), "siso_refresh: event");
    auto report = [&](long rows, long kept) {
        const long widest = rows > kept ? rows : kept;
        hipLaunchKernelGGL(k_report, dim3((unsigned)(widest < 262144 ? (widest + 255) / 256 : 1024)), dim3(256), 0, st, d_idx, d_sim,
                           repo_size, rows, c->locality, c->access, kept, h_idx, h_sim, h_rsize, h_loc, h_acc);
        return siso_check_hip(c, hipGetLastError(), "k_report");
    };
    // What the plan needs of a large cache's rows goes to the host first, which works on it while the searches run, and what is left
    // behind them is a look at the numbers and copies; small ones do not make up for a launch and an event more (us, all at the end / ahead, x 256
    // bf16 by a tenth and by 20 rows: 1,000 94 / 99, 99 / 107; 4,000 111 / 113, 109 / 113; 8,000 129 / 131, 122 / 128; 12,000 147 / 148,
    // 137 / 140; 16,384 177 / 164, 151 / 155; 20,000 210 / 190, 168 / 167; 30,000 280 / 245, 206 / 200; fp32 x 768: 8,000 201 / 197, 16,384
    // 283 / 271, 65,536 951 / 893).
    const bool ahead = K0 >= 16384;
    if (ahead) {
        const int rc = report(0, K0);
        if (rc != SISO_OK) return rc;
        REFRESH_TRY(hipEventRecord(lists.reported, st), "siso_refresh: event");
    }
    if (r > 0) {
        REFRESH_TRY(hipMemsetAsync(d_rows + (size_t)r * d * eb, 0, (size_t)SISO_PAD_ROWS * d * eb, st), "clear pad rows");
        hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, st, bad_at, found_at);
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_stage_repo<float>, dim3((unsigned)r), dim3(256), 0, st, (const float *)repo, repo_size,
                               (float *)d_rows, d_rinv, d, bad_at);
        else
            hipLaunchKernelGGL(k_stage_repo<bf16_t>, dim3((unsigned)r), dim3(256), 0, st, (const bf16_t *)repo, repo_size,
                               (bf16_t *)d_rows, d_rinv, d, bad_at);
        hipLaunchKernelGGL(k_nan_tail, dim3(1), dim3(SISO_PAD_ROWS), 0, st, d_rinv + r, SISO_PAD_ROWS);
        REFRESH_TRY(hipGetLastError(), "stage repository rows");
        // every repository row against the cache (test lookups: no references are counted); what does not exceed theta_c joins
        int rc = siso_lookup_impl(c, d_rows, r, &theta_c, 1, -1, d_idx, d_sim, nullptr, nullptr, 0, nullptr, theta_c);
        // repository rows among themselves: the pairs above the threshold, then their cosines
        if (rc == SISO_OK && r >= 2) rc = search(d_pairs, cap);
        if (rc == SISO_OK && r >= 2) rc = cosines(d_pairs, 0, early, h_pairs, h_cos);
        if (rc != SISO_OK) return rc;
    }
    if (r > 0 || (K0 > 0 && !ahead)) {
        const int rc = report(r, ahead ? 0 : K0);
        if (rc != SISO_OK) return rc;
    }
    if (ahead) {
        REFRESH_TRY(hipEventSynchronize(lists.reported), "siso_refresh: synchronize");
        plan_prepare(K0, r, h_loc, h_acc, max_centroids, lists);
    }
    if (r > 0 || (K0 > 0 && !ahead)) {
        u64 bad = 0;
        int rc = siso_read_counter(c, 2, &bad);  // (all counters come at once)
        if (rc != SISO_OK) return rc;
        if (r > 0 && bad != 0)
            return siso_fail(c, SISO_EINVAL, "siso_refresh: %llu repository rows are not finite or have no positive cluster size", bad);
        n_pairs = r >= 2 ? (long)c->host_pin[1] : 0;
    }
    if (n_pairs > cap) {  // once more with room for all of them
        const long need = n_pairs;
        if (!more_pairs.alloc((size_t)need * 2 * sizeof(int))) {
            (void)hipGetLastError();
            return siso_fail(c, SISO_ENOMEM, "siso_refresh: room for %ld pairs", need);
        }
        hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, st, bad_at, found_at);
        int rc = search(more_pairs.as<int>(), need);
        u64 total = 0;
        if (rc == SISO_OK) rc = siso_read_counter(c, 1, &total);
        if (rc != SISO_OK) return rc;
        if ((long)total > need) return siso_fail(c, SISO_ENOMEM, "siso_refresh: %llu pairs above the threshold", total);
        n_pairs = (long)total;
        cap = need;
    }
    if (n_pairs > early || more_pairs.p) {
        DeviceBuf d_found;  // pairs and cosines, to be copied
        if (!d_found.alloc((size_t)n_pairs * (2 * sizeof(int) + sizeof(float)))) {
            (void)hipGetLastError();
            return siso_fail(c, SISO_ENOMEM, "siso_refresh: cosines of %ld pairs", n_pairs);
        }
        int *found_pairs = d_found.as<int>();
        float *found_cos = (float *)(found_pairs + 2 * n_pairs);
        const int rc = cosines(more_pairs.p ? more_pairs.as<int>() : d_pairs, 0, n_pairs, found_pairs, found_cos);
        if (rc != SISO_OK) return rc;
        all_pairs.resize((size_t)n_pairs * 2);
        all_cos.resize((size_t)n_pairs);
        REFRESH_TRY(hipMemcpyAsync(all_pairs.data(), found_pairs, (size_t)n_pairs * 2 * sizeof(int), hipMemcpyDeviceToHost, st), "pairs to host");
        REFRESH_TRY(hipMemcpyAsync(all_cos.data(), found_cos, (size_t)n_pairs * sizeof(float), hipMemcpyDeviceToHost, st), "cosines to host");
        REFRESH_TRY(hipStreamSynchronize(st), "siso_refresh: synchronize");
        h_pairs = all_pairs.data();
        h_cos = all_cos.data();
    }

    // ---- merge step and filtering step: bookkeeping on the host ----------------------------------
    long merged = 0, added = 0, evicted = 0;
    if (!ahead) plan_prepare(K0, r, h_loc, h_acc, max_centroids, lists);
    h_loc2 = (float *)(h_src + K0 + r);
    const long live = plan_refresh(K0, r, h_idx, h_sim, h_rsize, h_pairs, h_cos, n_pairs, theta_c, max_centroids, lists, h_src, h_loc2, merged,
                                   added, evicted);

    // ---- update step: gather the new set, then it becomes the cache ---------------------------
    if (live > 0) {
        const int rc2 = siso_second_set(c);
        if (rc2 != SISO_OK) return rc2;
        REFRESH_TRY(hipMemcpyAsync(d_src, h_src, (size_t)(K0 + r + live) * sizeof(int), hipMemcpyHostToDevice, st), "sources to device");
        d_loc2 = (float *)(d_src + K0 + r);
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_refresh_gather<float>, dim3((unsigned)live), dim3(256), 0, st, d_src, K0, (const float *)c->cent,
                               c->mean, c->size, c->invn, (const float *)d_rows, d_rinv, repo_size, d_loc2, (float *)c->cent_b,
                               c->mean_b, c->size_b, c->invn_b, c->locality_b, c->access_b, c->version_b, d);
        else
            hipLaunchKernelGGL(k_refresh_gather<bf16_t>, dim3((unsigned)live), dim3(256), 0, st, d_src, K0, (const bf16_t *)c->cent,
                               c->mean, c->size, c->invn, (const bf16_t *)d_rows, d_rinv, repo_size, d_loc2, (bf16_t *)c->cent_b,
                               c->mean_b, c->size_b, c->invn_b, c->locality_b, c->access_b, c->version_b, d);
        REFRESH_TRY(hipGetLastError(), "k_refresh_gather");
        siso_swap_sets(c);  // lookups enqueued from here on see the new set
    }
    hipLaunchKernelGGL(k_nan_tail, dim3(1), dim3(SISO_PAD_ROWS), 0, st, c->invn + live, SISO_PAD_ROWS);
    REFRESH_TRY(hipGetLastError(), "k_nan_tail");
    REFRESH_TRY(hipStreamSynchronize(st), "siso_refresh: synchronize");
    c->count = live;
    if (out_stats) {
        out_stats[0] = merged;
        out_stats[1] = added;
        out_stats[2] = evicted;
    }
#undef REFRESH_TRY
    return SISO_OK;
}

extern "C" int siso_refresh(siso_cache *c, const void *repo, const float *repo_size, long r, float theta_c,
                            long max_centroids, long *out_stats) {
    if (!c) return SISO_EINVAL;
    int rc;
    try {
        rc = refresh_impl(c, repo, repo_size, r, theta_c, max_centroids, out_stats);
    } catch (const std::bad_alloc &) {  // the host lists; they are all built before the update step
        (void)hipStreamSynchronize(c->stream);  // (the searches may be running)
        rc = siso_fail(c, SISO_ENOMEM, "siso_refresh: host memory for the bookkeeping");
    }
    if (c->refresh_lists && c->refresh_lists->bytes() > (size_t)SISO_PINNED_KEEP) siso_refresh_release(c);
    siso_arena_done(c);
    return rc;
}

// The host part of siso_refresh alone (all pointers are HOST pointers).
extern "C" long siso_refresh_plan(long k0, const float *cluster_size, const unsigned *access_count, long r,
                                  const float *repo_size, const int *best_idx, const float *best_sim, const int *pairs,
                                  const float *pair_cosine, long n_pairs, float theta_c, long max_centroids,
                                  int *out_source, float *out_cluster_size, long *out_stats) {
    if (k0 < 0 || r < 0 || n_pairs < 0 || max_centroids < 1 || !out_source || !out_cluster_size) return SISO_EINVAL;
    if ((k0 > 0 && (!cluster_size || !access_count)) || (r > 0 && (!repo_size || !best_idx || !best_sim)) ||
        (n_pairs > 0 && (!pairs || !pair_cosine)))
        return SISO_EINVAL;
    for (long p = 0; p < n_pairs; ++p)
        if (pairs[2 * p] < 0 || pairs[2 * p] >= pairs[2 * p + 1] || pairs[2 * p + 1] >= r) return SISO_EINVAL;
    for (long i = 0; i < r; ++i)
        if (best_idx[i] >= k0 || !(repo_size[i] > 0.f)) return SISO_EINVAL;
    try {
        RefreshLists lists;
        long merged = 0, added = 0, evicted = 0;
        plan_prepare(k0, r, cluster_size, access_count, max_centroids, lists);
        const long live = plan_refresh(k0, r, best_idx, best_sim, repo_size, pairs, pair_cosine, n_pairs, theta_c, max_centroids, lists, out_source,
                                       out_cluster_size, merged, added, evicted);
        if (out_stats) {
            out_stats[0] = merged;
            out_stats[1] = added;
            out_stats[2] = evicted;
        }
        return live;
    } catch (const std::bad_alloc &) {
        return SISO_ENOMEM;
    }
}
