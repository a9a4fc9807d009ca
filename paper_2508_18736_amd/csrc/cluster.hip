// Clustering of a query log into the centroid repository (section 4.1): community detection at the
// clustering threshold ("Selecting a clustering algorithm"), then one repository row per cluster
// ("Keeping centroids in a repository": id, centroid = the average of the members (section 3.1),
// cluster_size = their number).
//
// The heavy part is the all-pairs similarity of the n vectors, n * n * dim / 2 products: that is the
// pair search of the merge (the pairs above the threshold are the edges of the neighbour graph), and
// the member averages; both run in kernels.  Between them sits the greedy choice of the communities
// (largest candidate first; a candidate keeps the vectors no earlier community took).  It is a chain, but only inside a
// connected component of the graph: components of at most 64 vectors are worked off by a wave each, the neighbours of a
// vector being one 64-bit mask, and the clusters are numbered afterwards by the candidates they came from (50,001
// vectors in topics of 2 to 12: 150 us of kernels, where copying the pairs out and walking them on the host took
// 1,500).  A graph with a larger component is walked on the host, linear in vectors + edges.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "siso_internal.h"

namespace {

// the counters of the call: pairs found, vectors that cannot be taken, room of the component lists handed out
__global__ void k_clear_counters(u64 *p) { p[0] = p[1] = p[2] = 0; }

__global__ void k_nan_fill(float *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = __uint_as_float(0x7FC00000u);
}

// Copy the vectors into a buffer with readable rows behind them, with 1 / |row|; count the rows that
// hold a NaN or an infinity or have no length.  A wave for each row: its lanes sum as the threads of a block of 256 would, one sum
// for each of the block's waves, and copy whole 16-byte chunks (`vec`), which they find in the caches.  (A block for each row,
// element by element: 50,001 x 768 bf16 53.0 us, so 45.6.)
template <typename T>
__global__ __launch_bounds__(256) void k_stage_vectors(const T *__restrict__ src, T *__restrict__ dst, float *__restrict__ invn, long n,
                                                        int d, int vec, u64 *bad) {
    const long k = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (k >= n) return;
    const T *row = src + (size_t)k * d;
    T *to = dst + (size_t)k * d;
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int e = lane; e < d; e += 256) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float f = e + 64 * v < d ? widen(row[e + 64 * v]) : 0.f;
            ss[v] += f * f;
        }
    }
    if (vec) {
        constexpr int EPC = 16 / (int)sizeof(T);
#pragma unroll 2
        for (int e = lane * EPC; e < d; e += 64 * EPC) *(u32x4_t *)(to + e) = *(const u32x4_t *)(row + e);
    } else {
        for (int e = lane; e < d; e += 64) to[e] = row[e];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) ss[v] = wave_sum(ss[v]);
    if (lane == 0) {
        const float inv = inv_length((ss[0] + ss[1]) + (ss[2] + ss[3]));
        invn[k] = inv;
        if (!(inv == inv) || inv == 0.f) atomicAdd(bad, 1ull);
    }
}

__device__ __forceinline__ float block_total(float v, float *sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// One block per cluster k: members member[first[k] .. first[k+1]) in ascending order.
// mean = average of the unit-length members; stored centroid = mean / |mean| rounded to the element
// type (a zero row when the mean has no length); size = cluster_size = number of members; no references yet.
// rep (nullable): the member with the largest cosine to the mean, the lowest index among equals.
template <typename T>
__global__ __launch_bounds__(256) void k_cluster_rows(const T *__restrict__ vec, const float *__restrict__ vinv,
                                                       const int *__restrict__ first, const int *__restrict__ member,
                                                       T *cent, float *mean, int *size, float *invn, float *locality,
                                                       unsigned *access, unsigned *version, int *rep, int d) {
    __shared__ float sh[4];
    __shared__ float sh_mean[SISO_MAX_DIM];
    __shared__ float sh_best[4];
    __shared__ int sh_who[4];
    const long k = blockIdx.x;
    const int t = threadIdx.x;
    const long lo = first[k], hi = first[k + 1];
    const float count = (float)(hi - lo);
    float ss = 0.f;
    for (int col = t; col < d; col += 256) {
        float acc = 0.f;
#pragma unroll 4
        for (long p = lo; p < hi; ++p) {
            const long j = member[p];
            acc += widen(vec[(size_t)j * d + col]) * vinv[j];
        }
        const float m = acc / count;
        mean[(size_t)k * d + col] = m;
        sh_mean[col] = m;
        ss += m * m;
    }
    const float n2 = block_total(ss, sh);
    const bool has_length = n2 > 0.f && n2 <= 3.0e38f;
    const float nrm = has_length ? sqrtf(n2) : 1.f;
    float cs = 0.f;
    for (int col = t; col < d; col += 256) {
        T v;
        narrow(has_length ? mean[(size_t)k * d + col] / nrm : 0.f, &v);  // this thread wrote that element itself
        cent[(size_t)k * d + col] = v;
        const float back = widen(v);
        cs += back * back;
    }
    const float c2 = block_total(cs, sh);  // (its barriers also make the whole mean in LDS visible)
    if (t == 0) {
        size[k] = hi - lo > 2147483647L ? 2147483647 : (int)(hi - lo);
        invn[k] = inv_length(c2);
        locality[k] = count;
        access[k] = 0u;
        raise_version_once(version, k);
    }
    if (!rep) return;
    // the member closest to the centroid: cosine(x_j, m) = <x_j, m> / (|x_j| |m|), and |m| is the same for
    // all of them.  One wave per member, members in ascending order within a wave.
    const int lane = t & 63, wave = t >> 6;
    float best = -INFINITY;
    int who = 0x7FFFFFFF;
    for (long p = lo + wave; p < hi; p += 4) {
        const long j = member[p];
        float dot = 0.f;
        for (int col = lane; col < d; col += 64) dot += widen(vec[(size_t)j * d + col]) * sh_mean[col];
        dot = wave_sum(dot) * vinv[j];
        if (dot > best) {
            best = dot;
            who = (int)j;
        }
    }
    if (lane == 0) {
        sh_best[wave] = best;
        sh_who[wave] = who;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < 4; ++w)
            if (sh_best[w] > best || (sh_best[w] == best && sh_who[w] < who)) {
                best = sh_best[w];
                who = sh_who[w];
            }
        rep[k] = who;
    }
}

// ============================================================================
// the choice of the communities on the device
// ============================================================================
#define COMPONENT_MAX 64                 // vectors of a component that a wave works off
#define COMPONENT_TOO_LARGE (1ull << 63)  // in the counter of bad vectors: some component is larger

__global__ void k_graph_init(int *parent, int *size_of, int *cursor, u64 *mask, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    parent[i] = (int)i;
    size_of[i] = 0;
    cursor[i] = 0;
    mask[i] = 0;
}
// (the number of pairs is read from the device: the host need not have seen it yet; more than `cap` were not written)
__global__ void k_graph_first(const int *__restrict__ pairs, const u64 *__restrict__ found, long cap, int *parent) {
    const long n_pairs = *found < (u64)cap ? (long)*found : cap;
    for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < n_pairs; p += (long)gridDim.x * blockDim.x)
        uf_first(parent, pairs[2 * p], pairs[2 * p + 1]);
}
__global__ void k_graph_join(const int *__restrict__ pairs, const u64 *__restrict__ found, long cap, int *parent) {
    const long n_pairs = *found < (u64)cap ? (long)*found : cap;
    for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < n_pairs; p += (long)gridDim.x * blockDim.x)
        uf_join(parent, pairs[2 * p], pairs[2 * p + 1]);
}
__global__ void k_graph_roots(int *parent, int *root, int *size_of, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = uf_find(parent, (int)i);
    root[i] = r;
    atomicAdd(&size_of[r], 1);
}
// room for the vectors of every component, in the order the blocks arrive
__global__ __launch_bounds__(256) void k_graph_starts(const int *__restrict__ root, const int *__restrict__ size_of, long n,
                                                       int *start, u64 *room, u64 *bad) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int mine = i < n && root[i] == (int)i ? size_of[i] : 0;
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    __shared__ int wave_all[4];
    __shared__ u64 base;
    const int wave = threadIdx.x >> 6;
    if (lane == 63) wave_all[wave] = incl;
    __syncthreads();
    // (10 ns each, one after the other: with one for every wave 11.6 us for 50,001 vectors, so 4.7)
    if (threadIdx.x == 0) base = atomicAdd(room, (u64)(wave_all[0] + wave_all[1] + wave_all[2] + wave_all[3]));
    __syncthreads();
    u64 at = base;
    for (int w = 0; w < wave; ++w) at += (u64)wave_all[w];
    if (mine > 0) start[i] = (int)at + incl - mine;
    if (__ballot(mine > COMPONENT_MAX) != 0 && lane == 0) atomicOr(bad, COMPONENT_TOO_LARGE);
}
__global__ void k_graph_fill(const int *__restrict__ root, const int *__restrict__ start, long n, int *cursor, int *list,
                             int *place) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = root[i];
    const int at = atomicAdd(&cursor[r], 1);
    place[i] = at;
    list[start[r] + at] = (int)i;
}
// mask[v]: the places of v's neighbours in the list of their component
__global__ void k_graph_masks(const int *__restrict__ pairs, const u64 *__restrict__ found, long cap,
                              const int *__restrict__ root, const int *__restrict__ size_of, const int *__restrict__ place,
                              u64 *mask) {
    const long n_pairs = *found < (u64)cap ? (long)*found : cap;
    for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < n_pairs; p += (long)gridDim.x * blockDim.x) {
        const int a = pairs[2 * p], b = pairs[2 * p + 1];
        if (size_of[root[a]] > COMPONENT_MAX) continue;
        atomicOr(&mask[a], 1ull << place[b]);
        atomicOr(&mask[b], 1ull << place[a]);
    }
}

// One component after the other, a wave each (a wave looks after 8 vectors: those that are the root of one).  Lane l holds
// the l-th vector of the component in ascending order and the mask of its candidate community (itself and its
// neighbours).  Candidates are taken by size, largest first, equal sizes by index; of a candidate the vectors that no
// earlier cluster holds remain, and if at least min_size do they are the next cluster.  Per vector: seed_of = the
// candidate whose cluster it is in or -1, pos = its place among that cluster's members in ascending order; and
// per candidate that became a cluster: its number of neighbours (255: it did not) and the members that were left.
#define NO_SEED 255
__global__ __launch_bounds__(256) void k_communities(const int *__restrict__ root, const int *__restrict__ size_of,
                                                      const int *__restrict__ start, const int *__restrict__ list,
                                                      const u64 *__restrict__ mask, long n, int min_size, int *seed_of,
                                                      int *pos, int *seed_size, unsigned char *seed_degree) {
    const int lane = threadIdx.x & 63;
    const long base = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 8;
    const long mine = base + (lane & 7);
    u64 roots = __ballot(lane < 8 && mine < n && root[mine < n ? mine : 0] == (int)mine);
    for (; roots != 0; roots &= roots - 1) {
        const long r = base + __ffsll((long long)roots) - 1;
        const int c = size_of[r];
        if (c > COMPONENT_MAX) continue;
        int v = lane < c ? list[start[r] + lane] : 0x7FFFFFFF;
        u64 m = lane < c ? mask[v] : 0ull;
        // into ascending order (the lists are in the order the vectors arrived): lane -> up
        int up = 0;
        for (int j = 0; j < c; ++j) up += __shfl(v, j) < v ? 1 : 0;
        u64 turned = 0;
        for (int j = 0; j < c; ++j)
            if (m >> j & 1) turned |= 1ull << __builtin_amdgcn_readlane(up, j);
        // (the lanes past the component all go to the first place behind it)
        const int lo = __builtin_amdgcn_ds_permute(up * 4, (int)(unsigned)turned);
        const int hi = __builtin_amdgcn_ds_permute(up * 4, (int)(unsigned)(turned >> 32));
        v = __builtin_amdgcn_ds_permute(up * 4, v);
        const bool in = lane < c;
        m = in ? ((u64)(unsigned)hi << 32 | (unsigned)lo) | 1ull << lane : 0ull;
        const int degree = __popcll(m) - 1;
        int rank = 0;
        for (int j = 0; j < c; ++j) {
            const int o = __shfl(degree, j);
            rank += o > degree || (o == degree && j < lane) ? 1 : 0;
        }
        u64 left = c == 64 ? ~0ull : (1ull << c) - 1;
        int seed = -1, at = 0, size = 0;
        unsigned char deg = NO_SEED;
        for (int s = 0; s < c && __popcll(left) >= min_size; ++s) {
            const int src = __ffsll((long long)__ballot(in && rank == s)) - 1;
            const u64 candidate = __shfl(m, src);
            if (__popcll(candidate) < min_size) break;  // every later candidate is smaller still
            const u64 take = candidate & left;
            if (__popcll(take) < min_size) continue;
            left &= ~take;
            const int who = __shfl(v, src);
            if (take >> lane & 1) {
                seed = who;
                at = __popcll(take & ((1ull << lane) - 1));
            }
            if (lane == src) {
                size = __popcll(take);
                deg = (unsigned char)(__popcll(candidate) - 1);
            }
        }
        if (in) {
            seed_of[v] = seed;
            pos[v] = at;
            seed_size[v] = size;
            seed_degree[v] = deg;
        }
    }
}

// The clusters in the order of their candidates: by number of neighbours, largest first, then by index.  SEED_ROWS vectors
// per block: clusters and members per block and number of neighbours (k_seed_sums), summed up in that order
// (k_seed_base), then every block numbers its own (k_seed_place).
#define SEED_ROWS 256
__global__ __launch_bounds__(SEED_ROWS) void k_seed_sums(const unsigned char *__restrict__ seed_degree,
                                                          const int *__restrict__ seed_size, long n, int2 *sums) {
    __shared__ int cnt[COMPONENT_MAX], members[COMPONENT_MAX];
    const int t = threadIdx.x;
    if (t < COMPONENT_MAX) cnt[t] = members[t] = 0;
    __syncthreads();
    const long i = (long)blockIdx.x * SEED_ROWS + t;
    const int deg = i < n ? seed_degree[i] : NO_SEED;
    if (deg != NO_SEED) {
        atomicAdd(&cnt[deg], 1);
        atomicAdd(&members[deg], seed_size[i]);
    }
    __syncthreads();
    if (t < COMPONENT_MAX) sums[(size_t)(COMPONENT_MAX - 1 - t) * gridDim.x + blockIdx.x] = make_int2(cnt[t], members[t]);
}
// exclusive sums in place, by one block; total: clusters, and the members in the upper half
__global__ __launch_bounds__(1024) void k_seed_base(int2 *sums, long count, u64 *total) {
    __shared__ int2 wsum[16];
    __shared__ int2 carry;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t == 0) carry = make_int2(0, 0);
    __syncthreads();
    for (long base = 0; base < count; base += 4096) {
        const long i0 = base + 4 * t;
        int2 v[4];
        int a = 0, b = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < count ? sums[i0 + k] : make_int2(0, 0);
            a += v[k].x;
            b += v[k].y;
        }
        int ia = a, ib = b;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int oa = __shfl_up(ia, off), ob = __shfl_up(ib, off);
            if (lane >= off) {
                ia += oa;
                ib += ob;
            }
        }
        if (lane == 63) wsum[w] = make_int2(ia, ib);
        __syncthreads();
        int ra = carry.x + ia - a, rb = carry.y + ib - b;
        for (int k = 0; k < w; ++k) {
            ra += wsum[k].x;
            rb += wsum[k].y;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < count) sums[i0 + k] = make_int2(ra, rb);
            ra += v[k].x;
            rb += v[k].y;
        }
        __syncthreads();
        if (t == 1023) carry = make_int2(ra, rb);
        __syncthreads();
    }
    if (t == 0) *total = (u64)(unsigned)carry.x | (u64)(unsigned)carry.y << 32;
}
__global__ __launch_bounds__(SEED_ROWS) void k_seed_place(const unsigned char *__restrict__ seed_degree,
                                                           const int *__restrict__ seed_size, long n,
                                                           const int2 *__restrict__ sums, int *id_of, int *first) {
    __shared__ int2 at[COMPONENT_MAX];
    const int t = threadIdx.x, lane = t & 63;
    if (t < COMPONENT_MAX) at[t] = sums[(size_t)(COMPONENT_MAX - 1 - t) * gridDim.x + blockIdx.x];
    const long i = (long)blockIdx.x * SEED_ROWS + t;
    const int deg = i < n ? seed_degree[i] : NO_SEED;
    const int size = deg != NO_SEED ? seed_size[i] : 0;
    for (int w = 0; w < SEED_ROWS / 64; ++w) {  // the waves one after the other
        __syncthreads();
        if (w != t >> 6) continue;
        u64 rest = __ballot(deg != NO_SEED);
        while (rest) {
            const int bin = __shfl(deg, __ffsll((long long)rest) - 1);
            const u64 same = __ballot(deg == bin);
            rest &= ~same;
            int incl = deg == bin ? size : 0;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(incl, off);
                if (lane >= off) incl += o;
            }
            const int2 from = at[bin];
            if (deg == bin) {
                const int id = from.x + __popcll(same & ((1ull << lane) - 1));
                id_of[i] = id;
                first[id] = from.y + incl - size;
            }
            const int members = __shfl(incl, 63);
            if (lane == 0) at[bin] = make_int2(from.x + __popcll(same), from.y + members);
        }
    }
}
__global__ void k_members(const int *__restrict__ seed_of, const int *__restrict__ pos, const int *__restrict__ id_of, long n,
                          int clusters, int members, int *first, int *member, int *out_label) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) first[clusters] = members;
    if (i >= n) return;
    const int seed = seed_of[i];
    const int id = seed < 0 ? -1 : id_of[seed];
    if (id >= 0) member[first[id] + pos[i]] = (int)i;
    if (out_label) out_label[i] = id;
}

struct DeviceMem {  // frees on every way out
    void *p = nullptr;
    ~DeviceMem() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
    }
    bool alloc(size_t bytes) {
        release();
        return hipMalloc(&p, bytes ? bytes : 1) == hipSuccess;
    }
    template <class U>
    U *as() const {
        return (U *)p;
    }
};

// The greedy choice of the communities from the list of neighbour pairs (host memory, each pair once, in any
// order): candidates = every vector with its neighbours, largest first, equal sizes by index; a candidate
// keeps the vectors no earlier cluster took and becomes a cluster if at least min_size remain.
// label[i] = cluster of vector i or -1; the members of cluster k, in ascending order, are
// member[first[k] .. first[k+1]).  Linear in vectors + pairs (counting sort, one pass over the lists).
void choose_communities(const int *h_pairs, long n_pairs, long n, int min_size, std::vector<int> &label,
                        std::vector<int> &first, std::vector<int> &member) {
    // ---- neighbour lists -----------------------------------------------------------------------
    std::vector<long> start((size_t)n + 1, 0);
    for (long p = 0; p < 2 * n_pairs; ++p) start[(size_t)h_pairs[(size_t)p] + 1] += 1;
    long largest = 0;
    for (long i = 0; i < n; ++i) {
        if (start[(size_t)i + 1] > largest) largest = start[(size_t)i + 1];
        start[(size_t)i + 1] += start[(size_t)i];
    }
    std::vector<int> nbr((size_t)(2 * n_pairs));
    {
        std::vector<long> fill(start.begin(), start.end() - 1);
        for (long p = 0; p < n_pairs; ++p) {
            const int a = h_pairs[(size_t)(2 * p)], b = h_pairs[(size_t)(2 * p + 1)];
            nbr[(size_t)fill[(size_t)a]++] = b;
            nbr[(size_t)fill[(size_t)b]++] = a;
        }
    }
    // ---- candidates by size (itself + neighbours), largest first, equal sizes by index ------------
    // a counting sort over the sizes 1 .. largest + 1
    std::vector<long> bucket((size_t)largest + 3, 0);
    for (long i = 0; i < n; ++i) bucket[(size_t)(largest + 1 - (start[(size_t)i + 1] - start[(size_t)i])) + 1] += 1;
    for (long s = 0; s <= largest + 1; ++s) bucket[(size_t)s + 1] += bucket[(size_t)s];
    std::vector<int> order((size_t)n);
    for (long i = 0; i < n; ++i) order[(size_t)bucket[(size_t)(largest + 1 - (start[(size_t)i + 1] - start[(size_t)i]))]++] = (int)i;

    // ---- greedy choice ----------------------------------------------------------------------------
    label.assign((size_t)n, -1);
    first.assign(1, 0);
    member.clear();
    member.reserve((size_t)n);
    for (long q = 0; q < n; ++q) {
        const long i = order[(size_t)q];
        const long lo = start[(size_t)i], hi = start[(size_t)i + 1];
        if (hi - lo + 1 < (long)min_size) break;   // every later candidate is smaller still
        long left = label[(size_t)i] < 0 ? 1 : 0;
        for (long p = lo; p < hi; ++p) left += label[(size_t)nbr[(size_t)p]] < 0 ? 1 : 0;
        if (left < (long)min_size) continue;
        const int id = (int)(first.size() - 1);
        if (label[(size_t)i] < 0) {
            label[(size_t)i] = id;
            member.push_back((int)i);
        }
        for (long p = lo; p < hi; ++p) {
            const int j = nbr[(size_t)p];
            if (label[(size_t)j] < 0) {
                label[(size_t)j] = id;
                member.push_back(j);
            }
        }
        std::sort(member.begin() + first.back(), member.end());   // averages take the members in ascending order
        first.push_back((int)member.size());
    }
}

}  // namespace

static long cluster_impl(siso_cache *c, const void *vectors, long n, float theta_c, int min_size, int *out_label,
                         int *out_representative, long *out_stats) {
    if (!c) return SISO_EINVAL;
    if (out_stats) out_stats[0] = out_stats[1] = 0;
    if (n < 0 || min_size < 1 || (n > 0 && !vectors))
        return siso_fail(c, SISO_EINVAL, "siso_cluster: bad arguments (n >= 0, min_size >= 1)");
    if (n > 2147483647L / 4) return siso_fail(c, SISO_EINVAL, "siso_cluster: %ld vectors are too many", n);
    if (((uintptr_t)vectors & 15) != 0) return siso_fail(c, SISO_EINVAL, "siso_cluster: vectors must be 16-byte aligned");
    const int d = c->dim;
    const size_t eb = c->dtype == SISO_F32 ? 4 : 2;
    hipStream_t st = c->stream;
#define CLUSTER_TRY(expr, what)                                   \
    do {                                                          \
        const int rc_ = siso_check_hip(c, (expr), what);          \
        if (rc_ != SISO_OK) return rc_;                           \
    } while (0)

    if (n == 0) {
        hipLaunchKernelGGL(k_nan_fill, dim3(1), dim3(SISO_PAD_ROWS), 0, st, c->invn, SISO_PAD_ROWS);
        CLUSTER_TRY(hipGetLastError(), "k_nan_fill");
        CLUSTER_TRY(hipStreamSynchronize(st), "siso_cluster: synchronize");
        c->count = 0;
        return 0;
    }

    // ---- the neighbour graph: every pair of vectors above the threshold; its communities ----------
    // room for 32 pairs per vector at first (256 bytes each); a log with more gets a second pass with the exact room
    long cap = n * 32 > (1L << 20) ? n * 32 : (1L << 20);
    const unsigned sblocks = (unsigned)((n + SEED_ROWS - 1) / SEED_ROWS), vblocks = (unsigned)((n + 255) / 256);
    char *rows;
    float *inv;
    int *pairs, *parent, *root, *size_of, *cursor, *start, *list, *place, *seed_of, *pos, *seed_size, *id_of, *first, *member;
    unsigned char *seed_degree;
    u64 *mask;
    int2 *sums;
    auto layout = [&](Carver a) {
        rows = a.take<char>((size_t)(n + SISO_PAD_ROWS) * d * eb);
        inv = a.take<float>(n + SISO_PAD_ROWS);
        mask = a.take<u64>(n);
        parent = a.take<int>(n);
        root = a.take<int>(n);
        size_of = a.take<int>(n);
        cursor = a.take<int>(n);
        start = a.take<int>(n);
        list = a.take<int>(n);
        place = a.take<int>(n);
        seed_of = a.take<int>(n);
        pos = a.take<int>(n);
        seed_size = a.take<int>(n);
        id_of = a.take<int>(n);
        first = a.take<int>(n + 1);
        member = a.take<int>(n);
        seed_degree = a.take<unsigned char>(n);
        sums = a.take<int2>((size_t)sblocks * COMPONENT_MAX);
        pairs = a.take<int>(2 * cap);
        return a.used;
    };
    DeviceMem more_pairs;  // a list that turned out too short
    {
        const int rc = siso_arena(c, layout(Carver{nullptr}), 0);
        if (rc != SISO_OK) return rc;
        layout(Carver{c->arena});
    }
    long n_pairs = 0;
    u64 *found = c->counters + 1, *bad_at = c->counters + 2, *room = c->counters + 3;
    u64 state[4];
    for (int attempt = 0; attempt < 2; ++attempt) {
        hipLaunchKernelGGL(k_clear_counters, dim3(1), dim3(1), 0, st, found);
        if (attempt == 0) {
            CLUSTER_TRY(hipMemsetAsync(rows + (size_t)n * d * eb, 0, (size_t)SISO_PAD_ROWS * d * eb, st), "clear pad rows");
            const dim3 four_rows((unsigned)((n + 3) / 4));
            const int vec = (size_t)d * eb % 16 == 0 && (((uintptr_t)vectors | (uintptr_t)rows) & 15) == 0 ? 1 : 0;
            if (c->dtype == SISO_F32)
                hipLaunchKernelGGL(k_stage_vectors<float>, four_rows, dim3(256), 0, st, (const float *)vectors,
                                   (float *)rows, inv, n, d, vec, bad_at);
            else
                hipLaunchKernelGGL(k_stage_vectors<bf16_t>, four_rows, dim3(256), 0, st, (const bf16_t *)vectors,
                                   (bf16_t *)rows, inv, n, d, vec, bad_at);
            hipLaunchKernelGGL(k_nan_fill, dim3(1), dim3(SISO_PAD_ROWS), 0, st, inv + n, SISO_PAD_ROWS);
        }
        CLUSTER_TRY(hipGetLastError(), "stage vectors");
        int rc = SISO_OK;
        if (n >= 2) {
            rc = siso_pairs_launch(c, rows, inv, n, theta_c, pairs, cap, found);
        }
        if (rc != SISO_OK) return rc;
        // (all of this stays within its arrays whatever the list holds: nothing is looked at if it turns out too short, if
        // a vector cannot be taken, or if a component is too large for a wave)
        const dim3 per_vector(vblocks), per_pair((unsigned)(cap < 262144 ? (cap + 255) / 256 : 1024)), block(256);
        hipLaunchKernelGGL(k_graph_init, per_vector, block, 0, st, parent, size_of, cursor, mask, n);
        hipLaunchKernelGGL(k_graph_first, per_pair, block, 0, st, pairs, found, cap, parent);
        hipLaunchKernelGGL(k_graph_join, per_pair, block, 0, st, pairs, found, cap, parent);
        hipLaunchKernelGGL(k_graph_roots, per_vector, block, 0, st, parent, root, size_of, n);
        hipLaunchKernelGGL(k_graph_starts, per_vector, block, 0, st, root, size_of, n, start, room, bad_at);
        hipLaunchKernelGGL(k_graph_fill, per_vector, block, 0, st, root, start, n, cursor, list, place);
        hipLaunchKernelGGL(k_graph_masks, per_pair, block, 0, st, pairs, found, cap, root, size_of, place, mask);
        // (vectors of a component that is too large keep what is set here)
        CLUSTER_TRY(hipMemsetAsync(seed_degree, NO_SEED, (size_t)n, st), "no cluster yet");
        hipLaunchKernelGGL(k_communities, dim3((unsigned)((n + 31) / 32)), block, 0, st, root, size_of, start, list, mask, n, min_size,
                           seed_of, pos, seed_size, seed_degree);
        hipLaunchKernelGGL(k_seed_sums, dim3(sblocks), dim3(SEED_ROWS), 0, st, seed_degree, seed_size, n, sums);
        hipLaunchKernelGGL(k_seed_base, dim3(1), dim3(1024), 0, st, sums, (long)sblocks * COMPONENT_MAX, room);
        hipLaunchKernelGGL(k_seed_place, dim3(sblocks), dim3(SEED_ROWS), 0, st, seed_degree, seed_size, n, sums, id_of, first);
        CLUSTER_TRY(hipGetLastError(), "communities");
        rc = siso_read_counter(c, 1, &state[1]);  // (all four counters come at once)
        if (rc != SISO_OK) return rc;
        state[2] = c->host_pin[2];
        state[3] = c->host_pin[3];
        const u64 bad = state[2] & ~COMPONENT_TOO_LARGE;
        if (bad != 0) return siso_fail(c, SISO_EINVAL, "siso_cluster: %llu vectors are not finite or have no length", bad);
        n_pairs = (long)state[1];
        if (n_pairs <= cap) break;
        if (attempt == 1) return siso_fail(c, SISO_ENOMEM, "siso_cluster: %ld pairs above the threshold", n_pairs);
        cap = n_pairs;  // once more with room for all of them
        if (!more_pairs.alloc((size_t)cap * 2 * sizeof(int))) {
            (void)hipGetLastError();
            return siso_fail(c, SISO_ENOMEM, "siso_cluster: room for %ld pairs", cap);
        }
        pairs = more_pairs.as<int>();
    }
    long clusters = (long)(unsigned)state[3], members = (long)(state[3] >> 32);
    std::vector<int> label;
    const bool on_host = (state[2] & COMPONENT_TOO_LARGE) != 0;
    if (on_host) {
        // ---- the communities: a walk over the pairs on the host --------------------------------------
        std::vector<int> h_first;   // members of cluster k: h_member[h_first[k] .. h_first[k+1])
        std::vector<int> h_member;
        std::vector<int> h_pairs((size_t)n_pairs * 2);
        CLUSTER_TRY(hipMemcpyAsync(h_pairs.data(), pairs, (size_t)n_pairs * 2 * sizeof(int), hipMemcpyDeviceToHost, st), "pairs to host");
        CLUSTER_TRY(hipStreamSynchronize(st), "siso_cluster: synchronize");
        more_pairs.release();
        choose_communities(h_pairs.data(), n_pairs, n, min_size, label, h_first, h_member);
        std::vector<int>().swap(h_pairs);
        clusters = (long)h_first.size() - 1;
        members = (long)h_member.size();
        if (clusters > 0 && clusters <= c->capacity) {
            CLUSTER_TRY(hipMemcpyAsync(first, h_first.data(), h_first.size() * sizeof(int), hipMemcpyHostToDevice, st), "member offsets");
            CLUSTER_TRY(hipMemcpyAsync(member, h_member.data(), h_member.size() * sizeof(int), hipMemcpyHostToDevice, st), "members");
            CLUSTER_TRY(hipStreamSynchronize(st), "siso_cluster: synchronize");  // (before the lists go out of scope)
        }
    }
    if (clusters > c->capacity)
        return siso_fail(c, SISO_ECAPACITY, "siso_cluster: %ld clusters, capacity %ld", clusters, c->capacity);

    // ---- the repository: one row per cluster -----------------------------------------------------
    if (!on_host) {
        hipLaunchKernelGGL(k_members, dim3(vblocks), dim3(256), 0, st, seed_of, pos, id_of, n, (int)clusters, (int)members, first,
                           member, out_label);
        CLUSTER_TRY(hipGetLastError(), "k_members");
    }
    if (clusters > 0) {
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_cluster_rows<float>, dim3((unsigned)clusters), dim3(256), 0, st, (const float *)rows, inv, first,
                               member, (float *)c->cent, c->mean, c->size, c->invn, c->locality, c->access, c->version, out_representative, d);
        else
            hipLaunchKernelGGL(k_cluster_rows<bf16_t>, dim3((unsigned)clusters), dim3(256), 0, st, (const bf16_t *)rows, inv, first,
                               member, (bf16_t *)c->cent, c->mean, c->size, c->invn, c->locality, c->access, c->version, out_representative, d);
        CLUSTER_TRY(hipGetLastError(), "k_cluster_rows");
    }
    hipLaunchKernelGGL(k_nan_fill, dim3(1), dim3(SISO_PAD_ROWS), 0, st, c->invn + clusters, SISO_PAD_ROWS);
    CLUSTER_TRY(hipGetLastError(), "k_nan_fill");
    if (out_label && on_host)
        CLUSTER_TRY(hipMemcpyAsync(out_label, label.data(), (size_t)n * sizeof(int), hipMemcpyHostToDevice, st), "labels");
    CLUSTER_TRY(hipStreamSynchronize(st), "siso_cluster: synchronize");
    c->count = clusters;
    siso_bytes_all_behind(c);
    if (out_stats) {
        out_stats[0] = n_pairs;
        out_stats[1] = members;
    }
#undef CLUSTER_TRY
    return clusters;
}

extern "C" long siso_cluster(siso_cache *c, const void *vectors, long n, float theta_c, int min_size, int *out_label,
                             int *out_representative, long *out_stats) {
    if (!c) return SISO_EINVAL;
    if (c->dtype == SISO_FP8) return siso_fail(c, SISO_EINVAL, "siso_cluster: not available with the 8-bit storage");
    long rc;
    try {
        rc = cluster_impl(c, vectors, n, theta_c, min_size, out_label, out_representative, out_stats);
    } catch (const std::bad_alloc &) {  // the host lists; nothing has been changed yet when they are built
        rc = siso_fail(c, SISO_ENOMEM, "siso_cluster: host memory for the neighbour lists");
    }
    siso_arena_done(c);
    return rc;
}

// The host part of siso_cluster alone: pairs and labels are HOST arrays.
extern "C" long siso_choose_communities(const int *pairs, long n_pairs, long n, int min_size, int *out_label) {
    if (n < 0 || n_pairs < 0 || min_size < 1 || (n_pairs > 0 && !pairs) || (n > 0 && !out_label)) return SISO_EINVAL;
    for (long p = 0; p < 2 * n_pairs; ++p)
        if (pairs[p] < 0 || pairs[p] >= n) return SISO_EINVAL;
    for (long p = 0; p < n_pairs; ++p)
        if (pairs[2 * p] == pairs[2 * p + 1]) return SISO_EINVAL;
    try {
        std::vector<int> label, member;
        std::vector<int> first;
        choose_communities(pairs, n_pairs, n, min_size, label, first, member);
        for (long i = 0; i < n; ++i) out_label[i] = label[(size_t)i];
        return (long)first.size() - 1;
    } catch (const std::bad_alloc &) {
        return SISO_ENOMEM;
    }
}
