// Internal declarations shared by the translation units of libsiso.so.
// Nothing here is visible through the C ABI (include/siso.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#include "siso.h"
#include "siso_bench.h"

typedef unsigned long long u64;
typedef unsigned short bf16_t;  // bfloat16 bit pattern

// A phase-1 lookup kernel reduces, for every query q and every slice s of the
// centroid range, the scaled dot products <q, c_k> / |c_k| to one 64-bit key
//     key = ordered(value) << 32 | (0xFFFFFFFF - id)
// so that an unsigned max over keys picks the largest value and, among equal
// values, the lowest id.  Key 0 means "no candidate".  The id is either the row
// itself (kernels that can afford the exact arg-max in their epilogue: the value
// then is the similarity but for the factor 1 / |q|), or the number k / 4 of a
// group of four consecutive rows that holds the best one (what a lane of a
// 32 x 32 MFMA accumulator holds in four consecutive registers: rows 8*g + 4*h
// + j of an aligned run of 32, j = 0..3); the finalize kernel then recomputes
// the four cosines exactly and picks the lowest index among their maxima.  Ids
// ascend with the rows, so "the lowest id among equal values" always holds the
// lowest index among equal maxima.
// SISO_KEY_ROWS_ANEW: the id is the row, and its cosine is formed anew all the same, with the sums of the finalize kernel
// (where a screened lookup of the same batch would do so: the similarities are then the same bits on either way).
enum { SISO_KEY_ROWS = 1, SISO_KEY_ROWS_ANEW = 2, SISO_KEY_GROUPS4 = 3 };
#define SISO_ACCESS_INF 0xFFFFFFFFu
#define SISO_MAX_DIM 4096
#define SISO_FOLD_BOARD 256  // queries of a siso_lookup_update that ends in one kernel: one slot each
#define SISO_MULTI_MAX 32  // thresholds one lookup can be judged against
#define SISO_PAD_ROWS 256  // readable rows past the capacity of the stored-centroid array

struct ScreenSpace {
    char *at;
    size_t cap;
    size_t refused;  // the smallest size that could not be had (0 = none): not asked for again until siso_reserve or a release
};

// The cache's rows as bytes (screen.hip), kept from one screened lookup to the next.  Every set of arrays has a count for every 32
// rows (`version`), which each kernel that writes a stored row raises (raise_version), and the bytes carry the counts that they
// were made from, so that a lookup writes anew only what has changed since.  All of that lives on the device, where the
// order of the stream, a captured graph's launches among them, is the order in which rows are written and read.  The
// counts of the two sets begin far apart: what was made from one is never taken for the other.
struct ByteView {  // where they lie
    signed char *codes;  // NULL: nowhere
    float4 *meta;        // for 32 rows: scale, error, error for lower ends, 1 / scale
    u64 *made;           // for 32 rows: the count they were made from << 8 | how many of them there were
    int dp;              // bytes of a row
};
struct ByteRows {
    char *at;  // room for the bytes of `rows` rows, or NULL; see byte_store in screen.hip
    long rows;
    long refused;  // the smallest number of rows that found no room (0 = none): not asked for again until siso_reserve or a release
    int recorded;  // a graph refers to them: outgrown, they stay until the cache goes (screen_kept)
    // How many rows may have changed since all bytes were current (an estimate of the host's, that only the choice of a route goes
    // by), how many elements small lookups have read as they are stored since then that would have gone over the bytes, and how many of
    // them there were, and have to be before the bytes are written for the next.
    long behind;
    double forgone;
    int waited, wait;
    int written;  // some bytes have been made, or are by a recorded launch
    int served;  // small lookups over them since they were written for one
};

// A lookup of few queries over the bytes (lookup_bytes.hip, k_finalize_update), per query; best and cnt are left as they were found, all zeros.
#define SISO_FEW 64
#define SISO_FEW_WORKGROUPS 256
#define SISO_FEW_SLOTS 8  // words of a workgroup for each of 64 queries; of 32 twice, of eight as many times: its largest lower end, how many rows it names, and those that need no place in the list
#define SISO_FEW_LIST 2048   // places
#define SISO_FEW_MOST_ROWS (32L * 256 * SISO_FEW_WORKGROUPS)
struct FewLists {
    u64 *best;        // largest key of the blocks that were multiplied as they are stored
    u64 *table;       // [SISO_FEW_WORKGROUPS][SISO_FEW]: number of the call << 32 | the largest lower end (ordered bits) that a workgroup knows
    unsigned *call;   // the number of the call
    int *cnt;         // rows in the list
    uint2 *rows;      // [SISO_FEW_LIST]: row, entry
    unsigned *slots;  // for as many workgroups as there are: [query][workgroup][words]
};

struct siso_cache {
    int dim;
    long capacity;
    int dtype;
    long count;
    int device;
    int path;
    hipStream_t stream;

    void *cent;   // [capacity][dim] stored centroids (bf16 bits or float)
    float *mean;  // [capacity][dim] mean of the unit-length members
    int *size;    // [capacity] cluster_size
    float *invn;  // [capacity] 1 / |stored centroid| (0 for a zero row, NaN for a non-finite row)
    float *locality;   // [capacity] cluster_size of Algorithm 1: grows by merges, decays by 1.1 per refresh
    unsigned *access;  // [capacity] access_count of Algorithm 1: hits since the last refresh; SISO_ACCESS_INF = infinity
    unsigned *version; // see ByteRows: [capacity / 32, of whole tiles of 256 rows]; NULL for an 8-bit cache
    // A second set of the seven arrays, allocated the first time a call rebuilds the cache (group merge, refresh):
    // the new set is gathered there and the two sets change places, so nothing is copied back and such calls
    // allocate nothing afterwards.
    void *cent_b;
    float *mean_b;
    int *size_b;
    float *invn_b;
    float *locality_b;
    unsigned *access_b;
    unsigned *version_b;

    // large update batches: first member and number of members per centroid, [capacity] each, allocated at
    // the first such batch; between calls every entry is back at (INT_MAX, 0)
    int *upd_owner;
    int *upd_members;

    // workspace, grown on demand
    u64 *keys;     // [keys_cap] phase-1 keys, n * slices
    long keys_cap;

    // temporaries of the calls that rebuild the cache (group merge, refresh, clustering): device memory, and pinned host
    // memory that kernels write their findings to; kept from one such call to the next (siso_arena)
    char *arena;
    size_t arena_cap;
    char *pinned;
    size_t pinned_cap;

    struct RefreshLists *refresh_lists;  // host lists of siso_refresh, kept (refresh.hip)

    u64 *static_keys;  // this device's copy of the library's static key array (siso_lookup_static)

    u64 *counters;  // device: [0] bad update indices, [1] merge pair count, [2] scratch, [3] scratch; behind them the
                    // board of siso_lookup_update (SISO_FOLD_BOARD slots)
    u64 *host_pin;  // pinned host mirror for counter read-back (4 entries)

    // 8-bit storage (SISO_FP8): cent holds one E4M3 code per element, scale [capacity] the scale of every row
    // (NaN for a non-finite row), invn the inverse lengths of the code rows; there is no running mean.
    // fp8_q / fp8_qinv: codes and inverse code lengths of the batch being looked up, [fp8_q_cap] rows, grown on demand
    float *scale;
    void *fp8_q;
    float *fp8_qinv;
    long fp8_q_cap;

    // top-k lookups: the two largest products of every group of 16 rows, per query ([topk_groups_cap] pairs; larger batches
    // go in pieces of at least 256 queries that take at most SISO_TOPK_GROUP_BYTES if they can), grown on demand
    float2 *topk_groups;
    long topk_groups_cap;
    // over the codes of a large 8-bit cache: per query the bound, the number of listed rows, a flag "scan this query row by
    // row" and the listed rows ([topk_cap] floats / ints / ints, [topk_cap][SISO_TOPK_CAND] ints), grown on demand
    float *topk_tau;
    int *topk_cnt;
    int *topk_cand;
    long topk_cap;
    int plan_min_slices;  // > 0 while such a lookup plans its passes: at least this many slices (if the tiles allow)
    const siso_cache *fold_master;  // not NULL while siso_fp8_lookup_update runs its lookup on this 8-bit copy
    int mark_in_finalize;  // siso_lookup_update on a large batch: 1 = the finalize step shall take the update's notes
                           // (first member and number of members per centroid), 2 = it has; 0 otherwise
    u64 *board_to_clear;  // not NULL while siso_lookup_update launches its first phase: a kernel that empties these
                          // slots sets it back to NULL

    // screened lookups and pair searches (screen.hip): bytes of rows and queries, bounds, lists; grown on demand.  Two
    // workspaces, so that a pair search does not move what a captured lookup refers to.
    ScreenSpace screen, screen_pairs;
    ByteRows bytes;
    FewLists few;  // room for them from few.best on, or NULL
    int few_refused;  // there was none: not asked for again until siso_reserve or a release
    int *few_flooded;  // pinned: a workgroup found no room for its lists, or a query was left with very many rows; such lookups are better off on the rows as they are stored:
    long few_rest, few_rests;  // as many more of them, and how many that were the last time
    long few_went;  // lookups over the bytes since then
    long few_reserved;  // batches that siso_reserve has made room for such lookups for, or tried to: they do not ask for any
    long screen_reserved;  // batches that siso_reserve has sized `screen` for, or tried to: their lookups leave it as it is
    int screen_recorded;  // a graph holds a screened lookup on `screen`: outgrown, it stays until the cache goes (screen_kept)
    std::vector<char *> *screen_kept;

    // tuning knobs (siso_set_option); 0 = library default
    int opt_screen;  // 1 = screen wherever the kernels can and give no batch up, 2 = never, 3 = screen wherever the kernels can
    int opt_screen_room;  // > 0: KiB that a workspace of screen.hip may take
    int opt_mfma_config;
    int opt_tiles_per_slice;
    int opt_merge_config;
    int opt_mfma_qblock;
    int opt_fold_spin_limit;  // -1 = default
    int opt_fold_units;
    int units;  // compute units that `stream` may use, 0 = not asked yet
    int opt_topk_room;        // KiB that topk_groups may take
    int opt_stream_hint;      // 0 = default; 1 = mark the centroid loads of the eight-wave lookups as streaming, 2 = never

    // kernel timing (siso_profile_enable / siso_profile_read)
    int profile_on;       // 0 = off, N = bracket every N-th call
    long prof_calls;      // calls seen since profiling was enabled
    int prof_open;        // a bracket was opened by the current call
    hipEvent_t *prof_ev;  // pairs: [2*i] start, [2*i+1] stop
    int prof_count;       // recorded pairs
    double prof_empty_ms; // what a pair of events with nothing between them measures on this stream

    char err[256];
};

// ----------------------------------------------------------------------------
// device helpers
// ----------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((unsigned)v) << 16); }

// round-to-nearest-even float -> bf16 bit pattern (NaN stays NaN)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    unsigned u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (bf16_t)0x7FC0;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(bf16_t v) { return bf16_to_f32(v); }

// One OCP E4M3 code of the 8-bit storage (1 sign, 4 exponent bits with bias 7, 3 mantissa bits, subnormals
// m/8 * 2^-6); a type of its own so that templates can tell a code from a byte.
struct fp8_t {
    unsigned char v;
};
__device__ __forceinline__ float e4m3_to_f32(unsigned code) {
    const unsigned e = (code >> 3) & 15u, m = code & 7u;
    const float v = e == 0 ? (float)m * 0.001953125f : __uint_as_float(((e + 120u) << 23) | (m << 20));
    return (code & 0x80u) ? -v : v;
}
__device__ __forceinline__ float widen(fp8_t c) { return e4m3_to_f32(c.v); }

__device__ __forceinline__ void narrow(float v, float *out) { *out = v; }
__device__ __forceinline__ void narrow(float v, bf16_t *out) { *out = f32_to_bf16(v); }

// monotone map float -> unsigned (larger float <=> larger unsigned; NaN excluded by callers)
__device__ __forceinline__ unsigned ordered_bits(float f) {
    unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unordered_bits(unsigned o) {
    unsigned u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(u);
}
__device__ __forceinline__ u64 pack_key(float value, unsigned block) {
    return ((u64)ordered_bits(value) << 32) | (u64)(0xFFFFFFFFu - block);
}

// The two largest of the products a lane meets, each tagged with a number in its lowest four bits (top-k lookups).  A NaN
// is passed over by the maximum, and by the median of three, which then is the smallest of the other two.
struct TwoLargest {
    float first = -INFINITY, second = -INFINITY;
    __device__ __forceinline__ void take(float v, unsigned tag) {
        v = __uint_as_float((__float_as_uint(v) & ~15u) | tag);
        second = __builtin_amdgcn_fmed3f(first, second, v);
        first = fmaxf(first, v);
    }
};

// 1/|x| from the sum of squares: 0 for a zero vector, NaN if the sum is not finite
__device__ __forceinline__ float inv_length(float sumsq) {
    if (!(sumsq == sumsq) || sumsq > 3.0e38f) return __uint_as_float(0x7FC00000u);
    if (sumsq == 0.0f) return 0.0f;
    return 1.0f / sqrtf(sumsq);
}

// Reductions over the 64 lanes of a wave (all of them must call); every lane gets the result.  A butterfly over 32, 16, 8, 4, 2, 1
// whose partners come by v_permlane32_swap, v_permlane16_swap and, within 16 lanes, DPP moves: ten vector instructions.
// __shfl_xor sends each step through the LDS crossbar, a round trip of some hundred cycles that a compute unit's waves queue
// for: six in a row are what the small kernels around a lookup waited for.  Pairs and order are the same, and so are the bits of
// a sum.  Batches with their updates, us: 4 of 256 against 1,024 x 384 fp32 74.5 -> 69.8, 2 of 1,000 against 60,000 x 384 257 -> 243,
// 16 of one against 60,000 x 768 bf16 381 -> 364 (371 of which the barrier between slabs had left), 16 of 64 against
// 262,144 x 768 codes 771 -> 743.
// Of a swap, the first number returned holds the lower half (the even rows of 16 lanes) in both, the second the upper.
template <class V>
struct LanePair {
    V a, b;
};
template <int OFF, class V>
__device__ __forceinline__ LanePair<V> lane_pair(V v) {
    static_assert(sizeof(V) % 4 == 0, "whole registers");
    constexpr int N = (int)sizeof(V) / 4;
    struct Words {
        unsigned w[N];
    };
    const Words in = __builtin_bit_cast(Words, v);
    Words a, b;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        a.w[i] = in.w[i];
        if constexpr (OFF == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(in.w[i], in.w[i], false, false);
            a.w[i] = r[0];
            b.w[i] = r[1];
        } else if constexpr (OFF == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(in.w[i], in.w[i], false, false);
            a.w[i] = r[0];
            b.w[i] = r[1];
        } else if constexpr (OFF == 8) {
            b.w[i] = (unsigned)__builtin_amdgcn_mov_dpp((int)in.w[i], 0x128, 0xF, 0xF, true);  // row_ror:8
        } else if constexpr (OFF == 4) {  // l ^ 7, then l ^ 3
            const int t = __builtin_amdgcn_mov_dpp((int)in.w[i], 0x141, 0xF, 0xF, true);  // row_half_mirror
            b.w[i] = (unsigned)__builtin_amdgcn_mov_dpp(t, 0x1B, 0xF, 0xF, true);         // quad_perm:[3,2,1,0]
        } else if constexpr (OFF == 2) {
            b.w[i] = (unsigned)__builtin_amdgcn_mov_dpp((int)in.w[i], 0x4E, 0xF, 0xF, true);  // quad_perm:[2,3,0,1]
        } else {
            static_assert(OFF == 1, "a power of two below 64");
            b.w[i] = (unsigned)__builtin_amdgcn_mov_dpp((int)in.w[i], 0xB1, 0xF, 0xF, true);  // quad_perm:[1,0,3,2]
        }
    }
    return LanePair<V>{__builtin_bit_cast(V, a), __builtin_bit_cast(V, b)};
}
template <int OFF = 32, class V, class Op>
__device__ __forceinline__ V wave_fold(V v, Op op) {
    const LanePair<V> p = lane_pair<OFF>(v);
    const V both = op(p.a, p.b);
    if constexpr (OFF == 1) return both;
    else return wave_fold<OFF / 2>(both, op);
}
__device__ __forceinline__ float wave_sum(float v) {
    return wave_fold(v, [](float a, float b) __attribute__((always_inline)) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
    return wave_fold(v, [](float a, float b) __attribute__((always_inline)) { return fmaxf(a, b); });
}
__device__ __forceinline__ u64 wave_max(u64 v) {
    return wave_fold(v, [](u64 a, u64 b) __attribute__((always_inline)) { return b > a ? b : a; });
}

// 16-byte chunk dot products (finalize, top-k re-ranking)
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float chunk_dot(const float *a, const float *b) {
    const float4 x = *(const float4 *)a, y = *(const float4 *)b;
    return x.x * y.x + x.y * y.y + x.z * y.z + x.w * y.w;
}
__device__ __forceinline__ float chunk_dot(const bf16_t *a, const bf16_t *b) {
    const u32x4_t x = *(const u32x4_t *)a, y = *(const u32x4_t *)b;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s += __uint_as_float(x[i] << 16) * __uint_as_float(y[i] << 16);
        s += __uint_as_float(x[i] & 0xFFFF0000u) * __uint_as_float(y[i] & 0xFFFF0000u);
    }
    return s;
}

// the same sums from chunks that are already in registers
__device__ __forceinline__ float chunk_dot(u32x4_t x, u32x4_t y, float) {
    return __uint_as_float(x[0]) * __uint_as_float(y[0]) + __uint_as_float(x[1]) * __uint_as_float(y[1]) +
           __uint_as_float(x[2]) * __uint_as_float(y[2]) + __uint_as_float(x[3]) * __uint_as_float(y[3]);
}
__device__ __forceinline__ float chunk_dot(u32x4_t x, u32x4_t y, bf16_t) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s += __uint_as_float(x[i] << 16) * __uint_as_float(y[i] << 16);
        s += __uint_as_float(x[i] & 0xFFFF0000u) * __uint_as_float(y[i] & 0xFFFF0000u);
    }
    return s;
}

__device__ __forceinline__ float chunk_dot(u32x4_t x, u32x4_t y, fp8_t) {  // sixteen codes, two decoded per instruction
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto xl = __builtin_amdgcn_cvt_pk_f32_fp8((int)x[i], false), xh = __builtin_amdgcn_cvt_pk_f32_fp8((int)x[i], true);
        const auto yl = __builtin_amdgcn_cvt_pk_f32_fp8((int)y[i], false), yh = __builtin_amdgcn_cvt_pk_f32_fp8((int)y[i], true);
        s += xl[0] * yl[0];
        s += xl[1] * yl[1];
        s += xh[0] * yh[0];
        s += xh[1] * yh[1];
    }
    return s;
}

// Products of queries with R rows, this lane's share of the sums (the whole wave must call): row r with the query whose chunks
// are at sh_q[r] in LDS (vec: rows are 16-byte aligned and a whole number of 16-byte chunks), or with the one at
// qrows[r].  Two chunks of every row in flight.
template <typename T, int R>
__device__ __forceinline__ void row_products(const T *const (&qrows)[R], const u32x4_t *const (&sh_q)[R], int vec,
                                             const T *const (&rows)[R], int d, int lane, float (&sum)[R]) {
    constexpr int EPC = 16 / (int)sizeof(T);
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] = 0.f;
    if (vec) {
#pragma unroll 1
        for (int e0 = lane * EPC; e0 < d; e0 += 2 * 64 * EPC) {
            const int e1 = e0 + 64 * EPC;
            u32x4_t c0[R], c1[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                c0[r] = *(const u32x4_t *)(rows[r] + e0);
                c1[r] = *(const u32x4_t *)(rows[r] + (e1 < d ? e1 : 0));
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                sum[r] += chunk_dot(sh_q[r][e0 / EPC], c0[r], T());
                const float part = chunk_dot(sh_q[r][(e1 < d ? e1 : 0) / EPC], c1[r], T());
                sum[r] += e1 < d ? part : 0.f;
            }
        }
    } else {
        for (int e = lane; e < d; e += 64)
#pragma unroll
            for (int r = 0; r < R; ++r) sum[r] += widen(qrows[r][e]) * widen(rows[r][e]);
    }
}
template <typename T>
__device__ __forceinline__ float row_product(const T *qrow, const u32x4_t *sh_q, int vec, const T *row, int d, int lane) {
    const T *const rows[1] = {row}, *const qrows[1] = {qrow};
    const u32x4_t *const chunks[1] = {sh_q};
    float sum[1];
    row_products<T, 1>(qrows, chunks, vec, rows, d, lane, sum);
    return wave_sum(sum[0]);
}

// A row that a workgroup of k_bytes_few names, in 32 bits: the query, the row's number in the workgroup, and the upper end of its cosine in thirteen
// bits, rounded up (the largest stands for anything above).
__device__ __forceinline__ unsigned few_upper_bits(float v) {
    const float x = (v + 1.25f) * (8191.f / 2.5f);
    return x >= 8190.f ? 8191u : x <= 0.f ? 1u : (unsigned)x + 1u;
}
__device__ __forceinline__ float few_upper(unsigned e) {
    return (e & 8191u) == 8191u ? INFINITY : (float)(e & 8191u) * (2.5f / 8191.f) - 1.25f + 1e-6f;
}
__device__ __forceinline__ unsigned few_row(unsigned e, unsigned workgroup, unsigned workgroups) {  // (32 rows to a block, eight blocks to a round)
    return (((e >> 18) & 255u) * workgroups + workgroup) * 32u + ((e >> 13) & 31u);
}

// By one thread for a stored row that its block writes (see ByteRows); _once: in a launch that writes all rows from the first on.
__device__ __forceinline__ void raise_version(unsigned *version, long row) { atomicAdd(version + (row >> 5), 1u); }
__device__ __forceinline__ void raise_version_once(unsigned *version, long row) {
    if ((row & 31) == 0) raise_version(version, row);
}

// The thresholds of a call travel as kernel arguments (nothing to allocate or copy): out_hit[q * m + j] = 1 where
// the similarity of query q exceeds v[j]; the hits at v[count_at] are the references that access counts.
struct ThetaList {
    float v[SISO_MULTI_MAX];
    int m, count_at;
};
// What a lookup leaves of query q, by one thread (q_base + q = its number in the whole batch).
__device__ __forceinline__ void write_lookup(long q, long q_base, long best_i, float best_s, const ThetaList &thetas, int *out_idx,
                                             float *out_sim, unsigned char *out_hit, unsigned *access, int *upd_owner,
                                             int *upd_members) {
    out_idx[q] = (int)best_i;
    out_sim[q] = best_s;
    for (int j = 0; j < thetas.m; ++j) {
        const bool hit = best_i >= 0 && best_s > thetas.v[j];
        if (out_hit) out_hit[(size_t)q * thetas.m + j] = hit ? 1 : 0;
        // a hit is a reference to its centroid (access_count of Algorithm 1); infinity stays infinity
        if (hit && j == thetas.count_at && access && access[best_i] != SISO_ACCESS_INF) atomicAdd(&access[best_i], 1u);
        // siso_lookup_update on a large batch: the notes that k_update_mark would take (first member and
        // number of members of each centroid), taken here, a launch earlier
        if (hit && j == 0 && upd_owner) {
            atomicMin(&upd_owner[best_i], (int)(q_base + q));
            atomicAdd(&upd_members[best_i], 1);
        }
    }
}

// ---- the quantiser of the 8-bit storage (k_fp8_quantize, and the end of siso_fp8_lookup_update)
__device__ __forceinline__ unsigned f32_to_e4m3(float y) {
    const unsigned sign = (__float_as_uint(y) >> 24) & 0x80u;
    const float a = fabsf(y);
    if (a >= 448.f) return sign | 0x7Eu;
    if (a < 0.015625f) return sign | (unsigned)(int)rintf(a * 512.f);  // multiples of 2^-9; 8 of them is 2^-6 = code 0x08
    unsigned v = __float_as_uint(a);
    v += 0x7FFFFu + ((v >> 20) & 1u);  // to three mantissa bits, ties to even (may carry into the exponent)
    return sign | ((((v >> 23) - 120u) << 3) | ((v >> 20) & 7u));
}
__device__ __forceinline__ float block_max256(float v, float *sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}
__device__ __forceinline__ float block_sum256f(float v, float *sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}
// One row by a 256-thread block: x = this thread's elements (columns t + 256 e; 0 beyond d).  Writes the codes,
// the scale (if asked for) and 1 / |code row| (0 for a row without length, NaN for a non-finite one).
template <int E>
__device__ __forceinline__ void fp8_store_row(const float (&x)[E], int d, unsigned char *codes_row, float *scale_out,
                                              float *inv_out, float *sh) {
    const int t = threadIdx.x;
    float amax = 0.f;
    bool finite = true;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        finite = finite && fabsf(x[e]) <= 3.4e38f;  // false for NaN and infinity
        amax = fmaxf(amax, fabsf(x[e]));
    }
    const float bad = block_max256(finite ? 0.f : 1.f, sh);
    amax = block_max256(amax, sh);
    const float sc = amax / 448.0f;
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int col = t + e * 256;
        if (col < d) {
            const unsigned code = (bad > 0.f || amax == 0.f) ? 0u : f32_to_e4m3(__fdiv_rn(x[e], sc));
            codes_row[col] = (unsigned char)code;
            const float back = e4m3_to_f32(code);
            ss = __fmaf_rn(back, back, ss);
        }
    }
    ss = block_sum256f(ss, sh);
    if (t == 0) {
        const float nanv = __uint_as_float(0x7FC00000u);
        if (scale_out) *scale_out = bad > 0.f ? nanv : sc;
        *inv_out = bad > 0.f ? nanv : inv_length(ss);
    }
}

// Pairs (i, j) into out[cap][2], up to 32 candidates per lane at once: bit I of `mask` says that this lane has the
// pair (i, j0 + row_of(I)); the wave takes one slot range with a single atomic and every lane writes its pairs behind
// those of the lanes before it.  counter accumulates the total number of pairs, also beyond cap.  Every lane of the wave
// must call it.
template <class RowOf>
__device__ __forceinline__ void emit_pairs(unsigned mask, int i, RowOf row_of, int *out, long cap, u64 *counter) {
    const int lane = threadIdx.x & 63;
    const int cnt = __popc(mask);
    int incl = cnt;  // inclusive prefix sum over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
    }
    const int total = __shfl(incl, 63);
    if (total == 0) return;
    u64 base = 0;
    if (lane == 63) base = atomicAdd(counter, (u64)total);
    base = __shfl(base, 63);
    u64 pos = base + (u64)(incl - cnt);
    while (mask != 0) {
        const int I = __ffs((int)mask) - 1;
        mask &= mask - 1;
        if (pos < (u64)cap) {
            out[2 * pos] = i;
            out[2 * pos + 1] = row_of(I);
        }
        ++pos;
    }
}

// The same with a staging buffer of the workgroup in LDS (stage[room][2], *staged = entries taken):
// the lanes take their slots with LDS atomics, which cost a fraction of the round trip of a global
// one; what does not fit any more goes straight to the global list.  Every lane must call it.
template <class RowOf>
__device__ __forceinline__ void emit_pairs_staged(unsigned mask, int i, RowOf row_of, int *stage, int *staged, int room,
                                                  int *out, long cap, u64 *counter) {
    // few lanes hold pairs (a block of 32 x 32 products with one group of near-duplicates in it): each of them
    // takes its slots with an LDS atomic of its own, which is cheaper than a prefix sum over the wave
    const int cnt = __popc(mask);
    if (__ballot(cnt != 0) == 0) return;
    int pos = cnt != 0 ? atomicAdd(staged, cnt) : 0;
    unsigned rest = 0;  // pairs of this lane that found no room
    while (mask != 0) {
        const int I = __ffs((int)mask) - 1;
        mask &= mask - 1;
        if (pos < room) {
            stage[2 * pos] = i;
            stage[2 * pos + 1] = row_of(I);
        } else {
            rest |= 1u << I;
        }
        ++pos;
    }
    if (__ballot(rest != 0) != 0) emit_pairs(rest, i, row_of, out, cap, counter);  // uniform over the wave
}

// Move the staged pairs of the workgroup to the global list and empty the buffer.  Every thread of
// the workgroup must call it (it synchronises); `slot` = one u64 of LDS for the broadcast.
__device__ __forceinline__ void flush_staged_pairs(const int *stage, int *staged, int room, u64 *slot, int *out, long cap,
                                                   u64 *counter) {
    __syncthreads();
    const int n = *staged < room ? *staged : room;
    if (threadIdx.x == 0 && n > 0) *slot = atomicAdd(counter, (u64)n);
    __syncthreads();
    if (n > 0) {
        const u64 base = *slot;
        for (int p = threadIdx.x; p < n; p += blockDim.x) {
            if (base + (u64)p < (u64)cap) {
                out[2 * (base + p)] = stage[2 * p];
                out[2 * (base + p) + 1] = stage[2 * p + 1];
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) *staged = 0;
    __syncthreads();
}

// Lock-free union-find: parent[i] <= i, the lowest index of a group is its root.  Parents only ever decrease, so every
// retry makes progress and the loops end.  A search leaves every other row that it passes below its grandparent, so that the
// searches of a long chain shorten it for each other: after the first pass (uf_first) rows that are only near their
// predecessors are one chain as long as the group (one of 20,000 rows in row order, all of siso_merge_apply: 13.4 ms without, 6.8 so,
// 6.8 for the same chain over rows in any order; 50 chains of 1,000 1,120 and 720 us).
__device__ __forceinline__ int uf_find(int *parent, int x) {
    int p = __atomic_load_n(parent + x, __ATOMIC_RELAXED);
    while (p != x) {
        const int g = __atomic_load_n(parent + p, __ATOMIC_RELAXED);
        if (g == p) return p;
        atomicMin(parent + x, g);  // (x is no root any more: only searches write there)
        x = g;
        p = __atomic_load_n(parent + x, __ATOMIC_RELAXED);
    }
    return x;
}
// A first pass over all pairs, in a launch of its own, leaves every row below the lowest row it is paired with (parents of
// freshly made trees only): that is all there is to do in a group whose rows are all paired with each other, and no pair of it
// searches for its roots, whose every step waits for memory behind the caches; nor does a pair of which one row hangs below the other.
__device__ __forceinline__ void uf_first(int *parent, int a, int b) { atomicMin(parent + (a > b ? a : b), a > b ? b : a); }
__device__ __forceinline__ void uf_join(int *parent, int a, int b) {
    if (a == b) return;
    // (old values will do: what is joined stays joined)
    const int pa = *(volatile int *)(parent + a), pb = *(volatile int *)(parent + b);
    if (pa == pb || pa == b || pb == a) return;
    for (;;) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) break;
        const int hi = a > b ? a : b, lo = a > b ? b : a;
        const int old = atomicCAS(parent + hi, hi, lo);
        if (old == hi) break;
        a = old;  // someone re-parented hi meanwhile: continue from there
        b = lo;
    }
}

// ----------------------------------------------------------------------------
// host-side plumbing shared by the translation units
// ----------------------------------------------------------------------------
int siso_fail(siso_cache *c, int code, const char *fmt, ...);
void siso_prof_begin(siso_cache *c);  // bracket the dominant kernel of a call (no-ops unless enabled)
void siso_prof_end(siso_cache *c);
int siso_check_hip(siso_cache *c, hipError_t e, const char *what);

// Phase-1 launchers.  Each fills keys[q * slices + s] for all q < n, s < slices (every entry is written,
// nothing has to be cleared beforehand).
// *_slices returns the number of slices the launcher will use (0 = path cannot
// handle this cache / batch).
//
// `many` (NULL = n): on the device, how many of the n queries there are: a workgroup beyond them leaves at once.
int siso_tile_preferred(const siso_cache *c, long n);  // 1 = small: rather these kernels, also where siso_mfma_* could
int siso_tile_slices(const siso_cache *c, long n, bool left = false);
long siso_tile_keys_bound(const siso_cache *c, long n);
int siso_tile_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys, const int *many = nullptr);
#define SISO_MFMA_UNALIGNED "bf16 lookup: queries must be 16-byte aligned"
inline bool siso_mfma_aligned(const void *queries) { return ((uintptr_t)queries & 15) == 0; }
int siso_mfma_slices(const siso_cache *c, long n);
int siso_mfma_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys, int *row_keys, const int *many = nullptr);
// Up to 32 queries in single precision: the rows straight from memory into the matrix cores (lookup_few.hip).  Keys name rows.
#define SISO_PATH_FEW 4  // (chosen, never set)
int siso_few_slices(const siso_cache *c, long n);
int siso_few_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys);
int siso_skinny_slices(const siso_cache *c, long n);
int siso_skinny_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys, int *row_keys);

// Up to SISO_FEW queries over the bytes of bf16 rows (lookup_bytes.hip): fills c->few, which k_finalize_update goes on with.
int siso_bytes_few_workgroups(const siso_cache *c);
int siso_bytes_few_launch(siso_cache *c, const void *queries, long n, const ByteView &v);
// Is a lookup of n queries to go that way?  If so: room and bytes for it (may synchronise and allocate, not under capture); 0 = without.
int siso_bytes_few_wanted(const siso_cache *c, long n);
int siso_bytes_few_room(siso_cache *c, long n);
void siso_bytes_few_reserve(siso_cache *c, long n);
// The host's note that rows of the cache are about to be written by something that leaves the bytes behind (see ByteRows).
inline void siso_bytes_behind(siso_cache *c, long rows) {
    c->bytes.behind = c->bytes.behind + rows < c->capacity ? c->bytes.behind + rows : c->capacity;
}
inline void siso_bytes_current(siso_cache *c) {
    c->bytes.behind = 0;
    c->bytes.forgone = 0;
    c->bytes.waited = 0;
}
inline void siso_bytes_all_behind(siso_cache *c) {
    siso_bytes_current(c);
    c->bytes.behind = c->capacity;
    c->bytes.wait = 0;
    c->bytes.served = 16;  // (what was written has served its time)
    c->few_rest = c->few_rests = c->few_went = 0;  // (other rows: perhaps no flood)
}
ByteView siso_byte_view(const siso_cache *c);
// Before every launch that is given the address of the bytes: a graph that records it goes on using them, so they stay when they are outgrown.  False: that
// could not be noted, and the launch has to do without them.
bool siso_bytes_may_record(siso_cache *c);
// The counts of the rows for a launch that raises them, or NULL where nobody can ask: no bytes have been made yet (those that come are made from all rows),
// and no graph records the launch, to be replayed when there are.
unsigned *siso_counted(const siso_cache *c);

// Top-k lookups, first phase: groups[q * ng + g].x = the largest scaled product <q, c> / |c| among the 16 rows of group g
// (-inf if none is finite), its lowest four bits replaced by the row's number in the group; .y = the second largest (its
// lowest bits are anything).  Row r of group g = 2 * (row / 32) + h is the row 32 * (g / 2) + 4 * (g % 2) + 8 * (r / 4) +
// r % 4.  ng = 2 * ceil(count / 32); every entry is written.
#define SISO_TOPK_MAX 32
#define SISO_TOPK_GROUP_BYTES (128l << 20)
int siso_mfma_groups_supported(const siso_cache *c, long n);
int siso_mfma_groups_launch(siso_cache *c, const void *queries, long n, float2 *groups, int ng);
// Over the codes of a large 8-bit cache, two passes: the phase-1 keys of a lookup planned with c->plan_min_slices (0 slices =
// these kernels cannot serve the cache), then the rows whose scaled product reaches tau[q] are listed (cand[q * cap + i],
// i < min(cnt[q], cap); cnt counts all of them; cnt must be zero before).  Both passes sum every product in the same order.
#define SISO_TOPK_CAND 128
int siso_topk_fp8_slices(const siso_cache *c, long n);
int siso_topk_fp8_pass1(siso_cache *c, long n, int slices, u64 *keys);
int siso_topk_fp8_collect(siso_cache *c, long n, int slices, const float *tau, int *cand, int *cnt, int cap);
int siso_tile_groups_launch(siso_cache *c, const void *queries, long n, float2 *groups, int ng);

// Screened lookups and pair searches (screen.hip).
// siso_screen_wanted: is a lookup of n queries to be screened?  If so, and if siso_screen_room finds room (0 = there is
// none: the lookup goes without), siso_screen_lookup takes up to SISO_SCREEN_PIECE queries at a time (with_rows: the rows have to
// be written as bytes, for the first piece of a call; whole: it is the only one) and leaves some to the other kernels: *plain names them (all on the
// device, written by the launch): how many, which, and their rows one behind the other; vec: how their products are summed
// (see k_lookup_finalize).
#define SISO_SCREEN_DIM 1024  // largest dimension
#define SISO_SCREEN_PIECE 16384L
struct ScreenPlain {
    const int *many, *query;
    const void *rows;
    int vec;
};
int siso_screen_wanted(const siso_cache *c, long n);
// The same for a lookup that only asks for cosines above `floor`: a query that nothing exceeds it by may get any row that does not,
// or none.  Rows below it are not even listed, so queries that miss cost nothing behind the products of the bytes.
int siso_screen_above_wanted(const siso_cache *c, long n, float floor);
int siso_screen_room(siso_cache *c, long n);  // may synchronise and allocate, but not under capture
void siso_screen_reserve(siso_cache *c, long n);  // siso_reserve: room for a full cache
int siso_screen_pairs_room(siso_cache *c, long rows);
void siso_screen_done(siso_cache *c);
void siso_screen_release(siso_cache *c);
int siso_screen_lookup(siso_cache *c, const void *queries, long n, bool with_rows, bool whole, const ThetaList &tl, long q_base, int *out_idx,
                       float *out_sim, unsigned char *out_hit, unsigned *access, int *owner, int *members, ScreenPlain *plain, float floor);
// The same for pairs above a threshold (room: siso_screen_pairs_room; siso_screen_done, at the end of a call, gives
// back what is larger than the library keeps between calls).  Behind it the search of all pairs has to be
// launched with `redo`: its workgroups leave at once unless more than redo.above pairs were in doubt.
struct PairsRedo {
    const u64 *count;  // NULL = search all pairs
    u64 above;
};
int siso_screen_pairs_wanted(const siso_cache *c, long count, float threshold);
int siso_screen_pairs_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                             u64 *counter, PairsRedo *redo);
struct BytePlan {
    int tiles_per_slice, slices, nqt, qb;
    long grid;
};
int siso_byte_plan(const siso_cache *c, long rows, long n, int dp, int most_tiles, BytePlan *p);  // 256 x 256 tiles of dp bytes a row

// All pairs above a threshold, on the kernels that serve the cache best.
int siso_pairs_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                      u64 *counter);

// Self-similarity pair search over `count` rows of the cache's element type and dimension with
// their inverse lengths (counter already zeroed).  The MFMA kernel reads whole tiles: rows and invn
// must be readable for SISO_PAD_ROWS entries past count, the invn entries there holding NaN.
int siso_pairs_tile_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold,
                           int *out_pairs, long cap, u64 *counter, PairsRedo redo);
int siso_pairs_mfma_supported(const siso_cache *c, long count);
int siso_pairs_mfma_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold,
                           int *out_pairs, long cap, u64 *counter, PairsRedo redo);

// siso_lookup without the argument checks of the ABI, against m thresholds (host pointer, 1 <= m <=
// SISO_MULTI_MAX; out_hit is [n][m] or NULL); the hits at thetas[count_index] are references to their
// centroids (access_count goes up), as in serving; count_index = -1 for test lookups.  static_keys: NULL = the phase-1
// keys go to the cache's own workspace (grown on demand); otherwise they go there (room for static_cap keys:
// a larger need is an error), and the call allocates nothing and records no timing events.
// folded: NULL = a lookup and nothing else; otherwise the caller is about to fold the hits into their centroids
// and *folded tells whether the lookup has already done it (small batches: one kernel ends the lookup and
// applies the update).
// floor: only cosines above it matter to the caller (see siso_screen_above_wanted).
int siso_lookup_impl(siso_cache *c, const void *queries, long n, const float *thetas, int m, int count_index,
                     int *out_idx, float *out_sim, unsigned char *out_hit, u64 *static_keys = nullptr,
                     long static_cap = 0, int *folded = nullptr, float floor = -INFINITY);
int siso_fp8_load(siso_cache *c, const void *centroids, const int *counts, long k);  // siso_load of an 8-bit cache
int siso_fp8_ensure_batch(siso_cache *c, long n);
int siso_fp8_quantize_batch(siso_cache *c, const void *queries, long n);  // bf16 queries -> c->fp8_q, c->fp8_qinv
int siso_read_counter(siso_cache *c, int which, u64 *value);
int siso_ensure_keys(siso_cache *c, long need);  // room for `need` phase-1 keys in c->keys (may synchronise and allocate)
// Temporaries of a call that rebuilds the cache.  siso_arena makes room for `device_bytes` and `host_bytes` (c->arena,
// c->pinned; earlier contents are lost: it synchronises before it lets go of them); siso_arena_done, at the
// call's end, gives back what is larger than the library keeps between calls.
#define SISO_ARENA_KEEP (512l << 20)
#define SISO_PINNED_KEEP (64l << 20)
int siso_arena(siso_cache *c, size_t device_bytes, size_t host_bytes);
void siso_arena_done(siso_cache *c);
void siso_refresh_release(siso_cache *c);
struct Carver {  // hands out aligned pieces; with a null base it only adds up
    char *base;
    size_t used = 0;
    template <class U>
    U *take(size_t count) {
        U *at = (U *)(base + used);
        used += (count * sizeof(U) + 255) & ~(size_t)255;
        return at;
    }
};
int siso_second_set(siso_cache *c);    // make sure the second set of arrays exists (allocates once; synchronises then)
void siso_swap_sets(siso_cache *c);    // the second set becomes the cache, the old arrays the second set  // synchronises
