// The k closest centroids of every query (FindClosestCentroid of Algorithm 1 taken k times).
//
// One pass of the tiled products, whose epilogue keeps of every group of 16 rows (what one lane of an MFMA accumulator
// holds) the largest scaled product <q, c> / |c|, with the row it came from in its lowest four bits, and the second
// largest: 1/8 of the similarity matrix.  Then one kernel picks the rows that can be among the k best: the k-th largest
// group maximum is reached by at least k rows, so the k best are in groups that reach it (with a margin for the order of
// the sums and for those four bits), and of a group whose second largest product does not reach it only the one row.
// Their cosines are formed anew, as the finalize step of a lookup does, and ranked: larger cosine first, lower index
// among equal cosines.  Against two passes of products (the second listing the rows at a bound that the first supplied)
// this halves the matrix work: 1,000 queries x 60,000 bf16 rows of 768, k = 8: 201 -> 115 us.  With the group maxima
// alone all 16 rows of a group had to be formed anew: 220 MB of them, 55 us of 144; now 20 us.
// For an 8-bit cache the batch is quantised first, as in a lookup, and everything here sees codes and the inverse
// lengths of code rows; large 8-bit caches take two passes (siso_lookup_topk tells why).
// Queries whose candidates do not fit the lists (hundreds of rows equal to the k-th best, a query without length) are
// taken row by row by their workgroups.
#include "siso_internal.h"

namespace {

// (value, index): larger value first, then the lower index; index -1 = no entry (worse than any entry)
__device__ __forceinline__ bool ranks_before(float va, int ia, float vb, int ib) {
    if (ia < 0) return false;
    if (ib < 0) return true;
    return va > vb || (va == vb && ia < ib);
}

// Row by row, by a 256-thread block: wave w takes rows w, w + 4, ...; lane j of a wave holds the wave's j-th best so far,
// a better row is inserted by shifting the lanes behind its place.  The four lists are merged by counting.
// sh_q = the query (chunks if vec, else elements), qi = 1 / |q|, finite; val, idx = 4 * SISO_TOPK_MAX entries each.
template <typename T>
__device__ __forceinline__ void scan_query(const u32x4_t *sh_q, float qi, const T *__restrict__ cent, const float *__restrict__ invn,
                                           long K, int d, int k, int vec, long q, float *val, int *idx, int *out_idx,
                                           float *out_sim) {
    constexpr int EPC = 16 / (int)sizeof(T);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const T *qrow = (const T *)sh_q;
    float mv = -INFINITY;  // this lane's entry of the wave's list
    int mi = -1;
    for (long r = wave; r < K; r += 4) {
        const T *crow = cent + (size_t)r * d;
        float acc = 0.f;
        if (vec) {
            for (int e0 = lane * EPC; e0 < d; e0 += 64 * EPC)
                acc += chunk_dot(sh_q[e0 / EPC], *(const u32x4_t *)(crow + e0), T());
        } else {
            for (int e = lane; e < d; e += 64) acc += widen(qrow[e]) * widen(crow[e]);
        }
        acc = wave_sum(acc);
        const float sv = acc * qi * invn[r];
        if (!(sv == sv)) continue;  // uniform over the wave
        // place = number of entries that stay before the new one (rows ascend, so an equal value stays before)
        const u64 stay = __ballot(lane < k && ranks_before(mv, mi, sv, (int)r));
        const int place = __popcll(stay);
        if (place >= k) continue;
        const float uv = __shfl_up(mv, 1);
        const int ui = __shfl_up(mi, 1);
        if (lane > place) {
            mv = uv;
            mi = ui;
        } else if (lane == place) {
            mv = sv;
            mi = (int)r;
        }
    }
    if (lane < k) {
        val[wave * SISO_TOPK_MAX + lane] = mv;
        idx[wave * SISO_TOPK_MAX + lane] = mi;
    }
    __syncthreads();
    int usable = 0;
    for (int w = 0; w < 4; ++w)
        for (int j = 0; j < k; ++j) usable += idx[w * SISO_TOPK_MAX + j] >= 0 ? 1 : 0;
    if (t < 4 * SISO_TOPK_MAX && (t % SISO_TOPK_MAX) < k && idx[t] >= 0) {
        int before = 0;
        for (int w = 0; w < 4; ++w)
            for (int j = 0; j < k; ++j) {
                const int o = w * SISO_TOPK_MAX + j;
                before += ranks_before(val[o], idx[o], val[t], idx[t]) ? 1 : 0;
            }
        if (before < k) {
            out_idx[(size_t)q * k + before] = idx[t];
            out_sim[(size_t)q * k + before] = val[t];
        }
    }
    for (int r = usable + t; r < k; r += 256) {
        out_idx[(size_t)q * k + r] = -1;
        out_sim[(size_t)q * k + r] = -INFINITY;
    }
}

// the query to LDS (chunks if vec, else elements); returns this thread's share of its squared length
template <typename T>
__device__ __forceinline__ float stage_query(const T *qrow, int d, int vec, bool lengths, u32x4_t *sh_q) {
    constexpr int EPC = 16 / (int)sizeof(T);
    float ss = 0.f;
    if (vec) {
        for (int e = threadIdx.x * EPC; e < d; e += 256 * EPC) {
            const u32x4_t v = *(const u32x4_t *)(qrow + e);
            sh_q[e / EPC] = v;
            if (lengths) ss += chunk_dot(v, v, T());
        }
    } else {
        for (int e = threadIdx.x; e < d; e += 256) {
            const T x = qrow[e];
            ((T *)sh_q)[e] = x;
            ss += widen(x) * widen(x);
        }
    }
    return ss;
}

// a query holding a NaN or an infinity: no entry
__device__ __forceinline__ void write_nan(long q, int k, int *out_idx, float *out_sim) {
    for (int r = threadIdx.x; r < k; r += 256) {
        out_idx[(size_t)q * k + r] = -1;
        out_sim[(size_t)q * k + r] = __uint_as_float(0x7FC00000u);
    }
}

#define TOPK_GROUPS 512  // groups a query may list
#define TOPK_CAND 2048   // rows of them that may have to be formed anew
#define TOPK_ROWS 512    // and of those that may come near the k-th best

// Group maxima -> result.  One 256-thread block per query:
//   1. every thread takes the maximum of its share of the groups, and every wave the ceil(k / 4)-th largest of its 64: the
//      least of the four is reached by at least k groups (a first bound, cheap);
//   2. the groups that reach it (some more than k) are listed, and the k-th largest of them is the bound that counts;
//   3. the rows that reach that, less the margin, are multiplied with the query, four rows a wave at a time;
//   4. those that still reach it are ranked by counting.
// The sums of the first phase and those of step 3 take the same products in another order.  `slack` bounds how far a group
// maximum can be from the cosine formed in step 3, as a share of |q| (topk_slack): at least k rows come within it of the
// k-th largest maximum, so a row that belongs to the k best has a product within twice that.
// `vec` = rows are 16-byte aligned and a whole number of 16-byte chunks.
template <typename T>
__global__ __launch_bounds__(256) void k_topk_pick(const T *__restrict__ Q, const T *__restrict__ cent,
                                                    const float *__restrict__ invn, long K, int d, int k, int vec,
                                                    const float2 *__restrict__ groups, int ng, float slack,
                                                    const float *__restrict__ q_inv, int *out_idx, float *out_sim) {
    constexpr int EPC = 16 / (int)sizeof(T);
    __shared__ u32x4_t sh_q[SISO_MAX_DIM / EPC];
    __shared__ float sh_f[4];
    __shared__ unsigned part[4];
    __shared__ float gval[TOPK_GROUPS], gnext[TOPK_GROUPS];
    __shared__ int gid[TOPK_GROUPS];
    __shared__ int cand[TOPK_CAND];
    __shared__ float val[TOPK_ROWS];
    __shared__ int idx[TOPK_ROWS];
    __shared__ int listed_s, cand_s, rows_s;
    __shared__ float bound_s;
    const long q = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const float2 *grow = groups + (size_t)q * ng;
    float ss = stage_query(Q + (size_t)q * d, d, vec, q_inv == nullptr, sh_q);
    float mine = -INFINITY;
#pragma unroll 8
    for (int g = t; g < ng; g += 256) mine = fmaxf(mine, grow[g].x);
    // The first bound: the ceil(k / 4)-th largest of the 64 maxima of each wave, or a little less (its upper 20 bits, found
    // bit by bit with a ballot each), the least of the four waves': at least k groups reach it.
    {
        const unsigned key = ordered_bits(mine);
        const int want = (k + 3) / 4;
        unsigned at = 0;
        for (int bit = 31; bit >= 12; --bit) {
            const unsigned up = at | (1u << bit);
            if (__popcll(__ballot(key >= up)) >= want) at = up;
        }
        if (lane == 0) part[wave] = at;
    }
    ss = wave_sum(ss);
    if (lane == 0) sh_f[wave] = ss;
    if (t == 0) {
        listed_s = 0;
        cand_s = 0;
        rows_s = 0;
        bound_s = -INFINITY;
    }
    __syncthreads();
    // (q_inv: the inverse lengths that came with the quantised batch)
    const float qi = q_inv ? q_inv[q] : inv_length((sh_f[0] + sh_f[1]) + (sh_f[2] + sh_f[3]));
    if (!(qi == qi)) {
        write_nan(q, k, out_idx, out_sim);
        return;
    }
    // false = more candidates than a list holds (uniform over the block, behind a barrier)
    auto from_lists = [&]() __attribute__((always_inline)) -> bool {
        unsigned least = part[0];
#pragma unroll
        for (int w = 1; w < 4; ++w) least = part[w] < least ? part[w] : least;
        // (below the image of -inf lie NaNs only: then everything is listed)
        const float first_bound = least <= ordered_bits(-INFINITY) ? -INFINITY : unordered_bits(least);
#pragma unroll 4
        for (int g = t; g < ng; g += 256) {
            const float2 v = grow[g];
            if (v.x >= first_bound) {
                const int at = atomicAdd(&listed_s, 1);
                if (at < TOPK_GROUPS) {
                    gval[at] = v.x;
                    gnext[at] = v.y;
                    gid[at] = g;
                }
            }
        }
        __syncthreads();
        const int listed = listed_s;
        if (listed > TOPK_GROUPS) return false;
        for (int i = t; i < listed; i += 256) {  // (fewer than k groups in all: the bound stays -inf)
            int before = 0;
            for (int j = 0; j < listed; ++j) before += (gval[j] > gval[i] || (gval[j] == gval[i] && j < i)) ? 1 : 0;
            if (before == k - 1) bound_s = gval[i];
        }
        __syncthreads();
        const float bound = listed < k ? -INFINITY : bound_s - 2.f * slack / qi;
        const float row_bound = bound * qi;  // (in cosines: slack below what the k-th of them can be)
        // groups within the margin below the first bound do not stand in the list: they are looked for now (rarely: the
        // first bound is usually further below the k-th largest maximum than that)
        if (first_bound > bound) {
            for (int g = t; g < ng; g += 256) {
                const float2 v = grow[g];
                if (v.x >= bound && v.x < first_bound) {
                    const int at = atomicAdd(&listed_s, 1);
                    if (at < TOPK_GROUPS) {
                        gval[at] = v.x;
                        gnext[at] = v.y;
                        gid[at] = g;
                    }
                }
            }
        }
        __syncthreads();
        const int all = listed_s;
        if (all > TOPK_GROUPS) return false;
        for (int i = t; i < all; i += 256) {
            if (gval[i] < bound) continue;
            const int g = gid[i], r0 = 32 * (g >> 1) + 4 * (g & 1);
            const int own = (int)(__float_as_uint(gval[i]) & 15u);
            const bool one = gnext[i] < bound;  // (a NaN counts as reaching it)
            const int at = atomicAdd(&cand_s, one ? 1 : 16);
            for (int j = one ? own : 0, to = at; j < 16; ++j, ++to) {
                if (to < TOPK_CAND) cand[to] = r0 + 8 * (j >> 2) + (j & 3);
                if (one) break;
            }
        }
        __syncthreads();
        const int cands = cand_s;
        if (cands > TOPK_CAND) return false;
        // four rows a wave, their loads in flight together; each is summed as the scan does it (a chunk per lane, then over
        // the lanes), so that a query's cosines do not depend on which of the two takes it
        for (int i = 4 * wave; i < cands; i += 16) {
            const T *crow[4];
            float acc[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int r = cand[i + p < cands ? i + p : i];
                crow[p] = cent + (size_t)(r < K ? r : K - 1) * d;
                acc[p] = 0.f;
            }
            if (vec) {
#pragma unroll 2
                for (int e = lane * EPC; e < d; e += 64 * EPC) {
                    u32x4_t x[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) x[p] = *(const u32x4_t *)(crow[p] + e);
                    const u32x4_t y = sh_q[e / EPC];
#pragma unroll
                    for (int p = 0; p < 4; ++p) acc[p] += chunk_dot(y, x[p], T());
                }
            } else {
#pragma unroll 2
                for (int e = lane; e < d; e += 64) {
                    const float y = widen(((const T *)sh_q)[e]);
#pragma unroll
                    for (int p = 0; p < 4; ++p) acc[p] += y * widen(crow[p][e]);
                }
            }
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                acc[p] = wave_sum(acc[p]);
                if (lane == 0 && i + p < cands && cand[i + p] < K) {
                    const int r = cand[i + p];
                    const float sv = acc[p] * qi * invn[r];
                    if (sv == sv && !(sv < row_bound)) {  // a NaN is never chosen
                        const int at = atomicAdd(&rows_s, 1);
                        if (at < TOPK_ROWS) {
                            val[at] = sv;
                            idx[at] = r;
                        }
                    }
                }
            }
        }
        __syncthreads();
        const int rows = rows_s;
        if (rows > TOPK_ROWS || (rows < k && listed >= k)) return false;  // (the bound left k rows, or it is no bound)
        // rank by counting the entries that come before (all differ in their index)
        for (int i = t; i < rows; i += 256) {
            int before = 0;
            for (int j = 0; j < rows; ++j) before += ranks_before(val[j], idx[j], val[i], idx[i]) ? 1 : 0;
            if (before < k) {
                out_idx[(size_t)q * k + before] = idx[i];
                out_sim[(size_t)q * k + before] = val[i];
            }
        }
        // fewer usable rows than k: the rest is empty
        for (int r = rows + t; r < k; r += 256) {
            out_idx[(size_t)q * k + r] = -1;
            out_sim[(size_t)q * k + r] = -INFINITY;
        }
        return true;
    };
    // Queries without length (1 / |q| = 0: every cosine is 0, but the maxima still differ in their lowest bits, and those
    // of a query whose squares underflow in more) and queries whose products come near the smallest numbers, where
    // errors are no longer a share of |q|, are taken row by row.
    const bool measurable = qi > 0.f && qi < 1e15f;
    if (!measurable || !from_lists()) scan_query(sh_q, qi, cent, invn, K, d, k, vec, q, val, idx, out_idx, out_sim);
}

// Codes of a large cache, pass 1 -> bound: tau[q] = value of the k-th largest key of query q (-inf with fewer than k keys: every
// row is wanted then).  One 256-thread block per query; the keys sit in LDS, k rounds of "largest left".
__global__ __launch_bounds__(256) void k_topk_bound(const u64 *__restrict__ keys, int slices, int k, float *tau, int *cnt,
                                                     int *scan) {
    extern __shared__ u64 sk[];  // [slices]
    __shared__ u64 wmax[4];
    __shared__ int wpos[4];
    const long q = blockIdx.x;
    const int t = threadIdx.x;
    for (int s = t; s < slices; s += 256) sk[s] = keys[(size_t)q * slices + s];
    __syncthreads();
    u64 kth = 0;
    for (int r = 0; r < k; ++r) {
        u64 best = 0;
        int pos = -1;
        for (int s = t; s < slices; s += 256)
            if (sk[s] > best) {
                best = sk[s];
                pos = s;
            }
        // keys of different slices differ (they name different rows)
        const u64 top = wave_max(best);
        pos = __builtin_amdgcn_readlane(pos, __ffsll((long long)__ballot(best == top)) - 1);
        best = top;
        if ((t & 63) == 0) {
            wmax[t >> 6] = best;
            wpos[t >> 6] = pos;
        }
        __syncthreads();
        best = wmax[0];
        pos = wpos[0];
        for (int w = 1; w < 4; ++w)
            if (wmax[w] > best) {
                best = wmax[w];
                pos = wpos[w];
            }
        kth = best;
        __syncthreads();
        if (best == 0) break;  // fewer than k keys
        if (t == 0) sk[pos] = 0;
        __syncthreads();
    }
    if (t == 0) {
        tau[q] = kth == 0 ? -INFINITY : unordered_bits((unsigned)(kth >> 32));
        cnt[q] = 0;
        scan[q] = 0;
    }
}

// Listed rows of codes -> result: exact cosines of the listed rows of query q (one wave per row), ranked; queries
// whose list overflowed are marked for the scan instead.  One 256-thread block per query.
__global__ __launch_bounds__(256) void k_topk_select(const fp8_t *__restrict__ Q, const fp8_t *__restrict__ cent,
                                                      const float *__restrict__ invn, long K, int d, int k,
                                                      const int *__restrict__ cand, const int *__restrict__ cnt, int cap,
                                                      const float *__restrict__ q_inv, int *scan, int *out_idx,
                                                      float *out_sim) {
    constexpr int EPC = 16;
    __shared__ u32x4_t sh_q[SISO_MAX_DIM / EPC];
    __shared__ float val[SISO_TOPK_CAND];
    __shared__ int idx[SISO_TOPK_CAND];
    const long q = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const fp8_t *qrow = Q + (size_t)q * d;
    for (int e = t * EPC; e < d; e += 256 * EPC) sh_q[e / EPC] = *(const u32x4_t *)(qrow + e);
    __syncthreads();
    const float qi = q_inv[q];  // (the inverse lengths that came with the quantised batch)
    const int listed = cnt[q];
    if (!(qi == qi)) {  // a query holding a NaN or an infinity
        for (int r = t; r < k; r += 256) {
            out_idx[(size_t)q * k + r] = -1;
            out_sim[(size_t)q * k + r] = __uint_as_float(0x7FC00000u);
        }
        return;
    }
    if (listed > cap) {  // more rows at the bound than the list holds: the scan takes this query
        if (t == 0) scan[q] = 1;
        return;
    }
    for (int i = wave; i < listed; i += 4) {
        const int r = cand[(size_t)q * cap + i];
        const fp8_t *crow = cent + (size_t)r * d;
        float acc = 0.f;
        for (int e0 = lane * EPC; e0 < d; e0 += 64 * EPC) acc += chunk_dot(sh_q[e0 / EPC], *(const u32x4_t *)(crow + e0), fp8_t());
        acc = wave_sum(acc);
        const float sv = acc * qi * invn[r];
        if (lane == 0) {
            val[i] = sv;
            idx[i] = sv == sv ? r : -1;  // a NaN is never chosen
        }
    }
    __syncthreads();
    // rank by counting the entries that come before (all differ in their index)
    if (t < listed && idx[t] >= 0) {
        int before = 0;
        for (int j = 0; j < listed; ++j) before += ranks_before(val[j], idx[j], val[t], idx[t]) ? 1 : 0;
        if (before < k) {
            out_idx[(size_t)q * k + before] = idx[t];
            out_sim[(size_t)q * k + before] = val[t];
        }
    }
    // fewer usable rows than k: the rest is empty
    int usable = 0;
    for (int j = 0; j < listed; ++j) usable += idx[j] >= 0 ? 1 : 0;
    for (int r = usable + t; r < k; r += 256) {
        out_idx[(size_t)q * k + r] = -1;
        out_sim[(size_t)q * k + r] = -INFINITY;
    }
}

// Every query row by row, where no first phase serves the cache (with `scan`: those with scan[q] != 0).
template <typename T>
__global__ __launch_bounds__(256) void k_topk_scan(const T *__restrict__ Q, const T *__restrict__ cent,
                                                    const float *__restrict__ invn, long K, int d, int k, int vec,
                                                    const float *__restrict__ q_inv, const int *__restrict__ scan, int *out_idx,
                                                    float *out_sim) {
    __shared__ float sh_f[4];
    __shared__ u32x4_t sh_q[SISO_MAX_DIM * sizeof(T) / 16];
    __shared__ float val[4 * SISO_TOPK_MAX];
    __shared__ int idx[4 * SISO_TOPK_MAX];
    const long q = blockIdx.x;
    if (scan && !scan[q]) return;
    const float ss = wave_sum(stage_query(Q + (size_t)q * d, d, vec, true, sh_q));
    if ((threadIdx.x & 63) == 0) sh_f[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float qi = q_inv ? q_inv[q] : inv_length((sh_f[0] + sh_f[1]) + (sh_f[2] + sh_f[3]));
    if (!(qi == qi)) write_nan(q, k, out_idx, out_sim);
    else scan_query(sh_q, qi, cent, invn, K, d, k, vec, q, val, idx, out_idx, out_sim);
}

// room for `cells` pairs of the first phase
int ensure_topk_workspace(siso_cache *c, long cells) {
    if (cells <= c->topk_groups_cap) return SISO_OK;
    const int rc = siso_check_hip(c, hipStreamSynchronize(c->stream), "siso_lookup_topk: synchronize");
    if (rc != SISO_OK) return rc;
    if (c->topk_groups) (void)hipFree(c->topk_groups);
    c->topk_groups = nullptr;
    c->topk_groups_cap = 0;
    if (hipMalloc((void **)&c->topk_groups, (size_t)cells * sizeof(float2)) != hipSuccess) {
        (void)hipGetLastError();
        return siso_fail(c, SISO_ENOMEM, "siso_lookup_topk: workspace of %ld pairs", cells);
    }
    c->topk_groups_cap = cells;
    return SISO_OK;
}

int ensure_two_pass_workspace(siso_cache *c, long n) {
    if (n <= c->topk_cap) return SISO_OK;
    if (c->topk_tau) {
        const int rc = siso_check_hip(c, hipStreamSynchronize(c->stream), "siso_lookup_topk: synchronize");
        if (rc != SISO_OK) return rc;
        (void)hipFree(c->topk_tau);
        (void)hipFree(c->topk_cnt);
        (void)hipFree(c->topk_cand);
        c->topk_tau = nullptr;
        c->topk_cnt = nullptr;
        c->topk_cand = nullptr;
        c->topk_cap = 0;
    }
    bool ok = hipMalloc((void **)&c->topk_tau, (size_t)n * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->topk_cnt, (size_t)n * 2 * sizeof(int)) == hipSuccess;  // counts, then scan flags
    ok = ok && hipMalloc((void **)&c->topk_cand, (size_t)n * SISO_TOPK_CAND * sizeof(int)) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (c->topk_tau) (void)hipFree(c->topk_tau);
        if (c->topk_cnt) (void)hipFree(c->topk_cnt);
        c->topk_tau = nullptr;
        c->topk_cnt = nullptr;
        c->topk_cand = nullptr;
        return siso_fail(c, SISO_ENOMEM, "siso_lookup_topk: workspace for %ld queries", n);
    }
    c->topk_cap = n;
    return SISO_OK;
}

// Codes of a large cache: see siso_lookup_topk.
int two_pass_launch(siso_cache *c, long n, int k, int slices, int *out_idx, float *out_sim) {
    int rc = ensure_two_pass_workspace(c, n);
    if (rc == SISO_OK) rc = siso_ensure_keys(c, n * (long)slices);
    if (rc == SISO_OK) rc = siso_topk_fp8_pass1(c, n, slices, c->keys);
    if (rc != SISO_OK) return rc;
    const fp8_t *Q = (const fp8_t *)c->fp8_q, *cent = (const fp8_t *)c->cent;
    int *cnt = c->topk_cnt, *flags = c->topk_cnt + c->topk_cap;
    hipLaunchKernelGGL(k_topk_bound, dim3((unsigned)n), dim3(256), (size_t)slices * sizeof(u64), c->stream, c->keys, slices, k,
                       c->topk_tau, cnt, flags);
    rc = siso_check_hip(c, hipGetLastError(), "k_topk_bound");
    if (rc == SISO_OK) rc = siso_topk_fp8_collect(c, n, slices, c->topk_tau, c->topk_cand, cnt, SISO_TOPK_CAND);
    if (rc != SISO_OK) return rc;
    hipLaunchKernelGGL(k_topk_select, dim3((unsigned)n), dim3(256), 0, c->stream, Q, cent, c->invn, c->count, c->dim, k,
                       c->topk_cand, cnt, SISO_TOPK_CAND, c->fp8_qinv, flags, out_idx, out_sim);
    hipLaunchKernelGGL(k_topk_scan<fp8_t>, dim3((unsigned)n), dim3(256), 0, c->stream, Q, cent, c->invn, c->count, c->dim, k, 1,
                       c->fp8_qinv, flags, out_idx, out_sim);
    return siso_check_hip(c, hipGetLastError(), "k_topk_select, k_topk_scan");
}

// How far the largest product of a group, as the first phase keeps it, can be from the cosine that k_topk_pick forms, as a
// share of |q|.  Measured on single instructions: one of two fp32 products is off by at most 2^-23 of the magnitudes it adds,
// the accumulator's among them, one of sixteen bf16 products by 2^-21.7.  Over d / 2 or d / 16 of them that stays below
// d * 2^-24 (bf16: half of that) of the sum of all magnitudes, which |q| |c| bounds (whole sums, the worst found: d / 4 * 2^-24
// for fp32 rows with elements +-c, where all roundings go the same way, d / 32 * 2^-24 in bf16).  The sum formed anew adds
// d / 64 + 8 roundings, the row number in the lowest four bits up to 15 * 2^-23.  Codes: the 8-bit instructions cut the
// products of eight elements at 2^-13 of the largest of them before they add them (seven are cut, by less than that each; the
// worst found: 1.9e-4 of |q|, on rows of one large and many small elements), and the sums at 2^-23 of the accumulator.
// 768 elements: 5.0e-5, bf16 2.7e-5, codes 8.8e-4.  1,000 queries x 60,000 bf16 rows, k = 8: 121.0 us with a margin of 8e-6
// that did not hold, 121.9 us with this one (fp32 and bf16 alike at d * 2^-24: 118.2 against 119.5).
template <typename T>
float topk_slack(int d) {
    const float unit = 5.9604645e-8f, f = (float)d;  // 2^-24
    const float again = (f / 64.f + 64.f) * unit;    // the sum formed anew, the row number, the scaling
    if (sizeof(T) == 4) return f * unit + again;
    if (sizeof(T) == 2) return 0.5f * f * unit + again;
    return 0.25f * f * unit + 7.f / 8192.f + again;
}

// what the first phase runs on: the pipelined kernels, the tiled kernel, or neither (then every query is scanned)
enum { PHASE_NONE, PHASE_MFMA, PHASE_TILE };

// Room for the group maxima (ng pairs a query) of `piece` queries, or of as many as it gets: fewer where the memory is short
// or the option says so; under capture, where nothing can be allocated, as many as fit what is there.  *piece = 0: none.
int topk_room(siso_cache *c, int ng, long *piece) {
    const long limit = c->opt_topk_room ? c->opt_topk_room * 1024L / (long)sizeof(float2) / ng : *piece;
    if (*piece > limit) *piece = limit;
    if (*piece * ng <= c->topk_groups_cap) return SISO_OK;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &status) != hipSuccess) (void)hipGetLastError();
    if (status != hipStreamCaptureStatusNone) {
        *piece = c->topk_groups_cap / ng;
        return SISO_OK;
    }
    int rc = SISO_ENOMEM;
    for (; *piece > 0; *piece /= 2) {
        rc = ensure_topk_workspace(c, *piece * ng);
        if (rc != SISO_ENOMEM) return rc;
    }
    return SISO_OK;
}

template <typename T>
int topk_launch(siso_cache *c, const T *Q, long n, int k, int phase, const float *q_inv, int *out_idx, float *out_sim) {
    const T *cent = (const T *)c->cent;
    const int vec = ((c->dim * sizeof(T)) % 16 == 0 && ((uintptr_t)Q & 15) == 0) ? 1 : 0;
    // pieces of the batch whose maxima take about SISO_TOPK_GROUP_BYTES: they stay in the memory-side cache
    const int ng = (int)(2 * ((c->count + 31) / 32));
    long piece = 0;
    if (phase != PHASE_NONE) {
        const long most = SISO_TOPK_GROUP_BYTES / ((long)ng * 8) / 256 * 256;
        piece = n <= most ? n : n <= 256 ? n : most > 256 ? most : 256;
        const int rc = topk_room(c, ng, &piece);
        if (rc != SISO_OK) return rc;
    }
    if (piece == 0) {
        hipLaunchKernelGGL(k_topk_scan<T>, dim3((unsigned)n), dim3(256), 0, c->stream, Q, cent, c->invn, c->count, c->dim, k, vec,
                           q_inv, (const int *)nullptr, out_idx, out_sim);
        return siso_check_hip(c, hipGetLastError(), "k_topk_scan");
    }
    int rc = SISO_OK;
    for (long lo = 0; lo < n && rc == SISO_OK; lo += piece) {
        const long m = n - lo < piece ? n - lo : piece;
        const T *rows = Q + (size_t)lo * c->dim;
        rc = phase == PHASE_MFMA ? siso_mfma_groups_launch(c, rows, m, c->topk_groups, ng)
                                 : siso_tile_groups_launch(c, rows, m, c->topk_groups, ng);
        if (rc != SISO_OK) return rc;
        hipLaunchKernelGGL(k_topk_pick<T>, dim3((unsigned)m), dim3(256), 0, c->stream, rows, cent, c->invn, c->count, c->dim, k, vec,
                           c->topk_groups, ng, topk_slack<T>(c->dim), q_inv ? q_inv + lo : nullptr, out_idx + lo * k,
                           out_sim + lo * k);
        rc = siso_check_hip(c, hipGetLastError(), "k_topk_pick");
    }
    return rc;
}

}  // namespace

// (siso_reserve has no part for top-k lookups: the call says that it may allocate.)
extern "C" int siso_lookup_topk(siso_cache *c, const void *queries, long n, int k, int *out_idx, float *out_sim) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || k < 1 || k > SISO_TOPK_MAX || (n > 0 && (!queries || !out_idx || !out_sim)))
        return siso_fail(c, SISO_EINVAL, "siso_lookup_topk: bad arguments (1 <= k <= %d)", SISO_TOPK_MAX);
    if (n == 0) return SISO_OK;
    if (n > 2147483647L / 4) return siso_fail(c, SISO_EINVAL, "siso_lookup_topk: batch of %ld is too large", n);
    const bool fp8 = c->dtype == SISO_FP8;
    const void *rows = queries;  // what the kernels read: the batch, or its codes
    if (fp8) {
        int rc = siso_fp8_ensure_batch(c, n);
        if (rc == SISO_OK) rc = siso_fp8_quantize_batch(c, queries, n);
        if (rc != SISO_OK) return rc;
        rows = c->fp8_q;
    }
    // Codes of a cache of at least 512 * k rows: two passes, the second of which lists the rows at a bound from the first.  The
    // products of the 8-bit matrix instructions are some 1e-5 off, which decides between neighbours at that bound; one
    // pass with a margin for that would rank about one entry in a thousand otherwise than it has been.
    if (fp8 && c->count >= 512L * k) {
        c->plan_min_slices = 8 * k;
        const int slices = siso_topk_fp8_slices(c, n);
        if (slices >= 2 * k && slices <= 4096) {  // (the bound kernel keeps a query's keys in LDS)
            const int rc = two_pass_launch(c, n, k, slices, out_idx, out_sim);
            c->plan_min_slices = 0;
            return rc;
        }
        c->plan_min_slices = 0;
    }
    // (pieces of a batch start whole rows further on, so where the batch is aligned they are)
    int phase = PHASE_NONE;
    if (c->count > 0) {
        if (((uintptr_t)rows & 15) == 0 && !siso_tile_preferred(c, n) && siso_mfma_groups_supported(c, n)) phase = PHASE_MFMA;
        else if (!fp8 || siso_tile_preferred(c, n)) phase = PHASE_TILE;
    }
    return c->dtype == SISO_F32 ? topk_launch<float>(c, (const float *)rows, n, k, phase, nullptr, out_idx, out_sim)
           : fp8              ? topk_launch<fp8_t>(c, (const fp8_t *)rows, n, k, phase, c->fp8_qinv, out_idx, out_sim)
                              : topk_launch<bf16_t>(c, (const bf16_t *)rows, n, k, phase, nullptr, out_idx, out_sim);
}
