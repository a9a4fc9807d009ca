// C ABI of the centroid cache (include/siso.h): state management, the kernels
// that are not matrix-shaped (row norms, finalize, update, group merge).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>
#include <utility>

#include "siso_internal.h"

// ============================================================================
// error plumbing
// ============================================================================
int siso_fail(siso_cache *c, int code, const char *fmt, ...) {
    if (c) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(c->err, sizeof(c->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

int siso_check_hip(siso_cache *c, hipError_t e, const char *what) {
    if (e == hipSuccess) return SISO_OK;
    return siso_fail(c, SISO_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(c, call)                                          \
    do {                                                          \
        int rc_ = siso_check_hip((c), (call), #call);             \
        if (rc_ != SISO_OK) return rc_;                           \
    } while (0)

#define SISO_PROF_MAX 8192

void siso_prof_begin(siso_cache *c) {
    c->prof_open = 0;
    if (!c->profile_on || c->prof_count >= SISO_PROF_MAX) return;
    if (c->prof_calls++ % c->profile_on != 0) return;
    if (!c->prof_ev) {
        c->prof_ev = (hipEvent_t *)calloc(2 * SISO_PROF_MAX, sizeof(hipEvent_t));
        if (!c->prof_ev) return;
    }
    hipEvent_t *e = c->prof_ev + 2 * c->prof_count;
    if (hipEventCreate(&e[0]) != hipSuccess || hipEventCreate(&e[1]) != hipSuccess) return;
    (void)hipEventRecord(e[0], c->stream);
    c->prof_open = 1;
}

void siso_prof_end(siso_cache *c) {
    if (!c->prof_open) return;
    hipEvent_t *e = c->prof_ev + 2 * c->prof_count;
    if (!e[0] || !e[1]) return;
    (void)hipEventRecord(e[1], c->stream);
    c->prof_count++;
}

static inline size_t elem_bytes(int dtype) { return dtype == SISO_F32 ? 4 : dtype == SISO_FP8 ? 1 : 2; }

// the calls an 8-bit cache does not offer (it is a read-only serving copy: lookups, and siso_load to rebuild it)
#define SISO_NOT_FP8(c, what)                                                                                        \
    do {                                                                                                             \
        if ((c)->dtype == SISO_FP8) return siso_fail((c), SISO_EINVAL, what ": not available with the 8-bit storage"); \
    } while (0)

// ============================================================================
// small kernels
// ============================================================================
// Block-wide sum for 256-thread blocks; every thread gets the result.
__device__ __forceinline__ float block_sum256(float v, float *sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// siso_load: store rows verbatim, mean = row / |row|, size = counts or 1, invn = 1/|row|.  One wave per row; the rows are
// copied in whole 16-byte chunks per lane if they allow it (`vec`), on a second pass that finds them in the caches.  A lane
// sums the squares of the elements lane + 64 v + 256 e, one sum for every v, and the four are added as a block of 256
// threads adds its waves (block_sum256): import and update find lengths in that order too.  Bound by memory: 131,072
// rows of 768 bf16 elements move 805 MB; element by element, a block per row, they took 341 us, this way 183 us.
template <typename T>
__global__ __launch_bounds__(256) void k_load_rows(const T *__restrict__ src, const int *__restrict__ counts, T *cent,
                                                    float *mean, int *size, float *invn, float *locality,
                                                    unsigned *access, unsigned *version, long K, int d, int vec) {
    constexpr int EPC = 16 / (int)sizeof(T);
    const long k = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (k >= K) return;
    const T *row = src + (size_t)k * d;
    T *cent_row = cent + (size_t)k * d;
    float *mean_row = mean + (size_t)k * d;
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
    const int whole = d / 256 * 256;
#pragma unroll 4
    for (int e = lane; e < whole; e += 256) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float x = widen(row[e + 64 * v]);
            ss[v] += x * x;
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int e = whole + lane + 64 * v;
        if (e < d) {
            const float x = widen(row[e]);
            ss[v] += x * x;
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) ss[v] = wave_sum(ss[v]);
    const float n2 = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    const float inv = inv_length(n2);
    const bool ok = (inv == inv) && inv > 0.f;
    const float nrm = sqrtf(n2);
    if (vec) {
#pragma unroll 2
        for (int e = lane * EPC; e < d; e += 64 * EPC) {
            const u32x4_t v = *(const u32x4_t *)(row + e);
            *(u32x4_t *)(cent_row + e) = v;
            float x[EPC];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (sizeof(T) == 4) {
                    x[i] = __uint_as_float(v[i]);
                } else {
                    x[2 * i] = __uint_as_float(v[i] << 16);
                    x[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
                }
            }
#pragma unroll
            for (int i = 0; i < EPC; i += 4)
                *(float4 *)(mean_row + e + i) = ok ? make_float4(x[i] / nrm, x[i + 1] / nrm, x[i + 2] / nrm, x[i + 3] / nrm)
                                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else {
        for (int e = lane; e < d; e += 64) {
            const T x = row[e];
            cent_row[e] = x;
            mean_row[e] = ok ? widen(x) / nrm : 0.f;
        }
    }
    if (lane == 0) {
        int s = counts ? counts[k] : 1;
        size[k] = s < 1 ? 1 : s;
        invn[k] = inv;
        locality[k] = (float)(s < 1 ? 1 : s);
        access[k] = 0;
        raise_version_once(version, k);
    }
}

// siso_import: take over a snapshot as it is; only the inverse length of the stored row is computed.
template <typename T>
__global__ __launch_bounds__(256) void k_import_rows(const T *__restrict__ src, const float *__restrict__ src_mean,
                                                      const int *__restrict__ src_size, const float *__restrict__ src_loc,
                                                      const unsigned *__restrict__ src_acc, T *cent, float *mean, int *size,
                                                      float *invn, float *locality, unsigned *access, unsigned *version, int d) {
    __shared__ float sh[4];
    const long k = blockIdx.x;
    float ss = 0.f;
    for (int e = threadIdx.x; e < d; e += 256) {
        const T x = src[(size_t)k * d + e];
        cent[(size_t)k * d + e] = x;
        mean[(size_t)k * d + e] = src_mean[(size_t)k * d + e];
        ss += widen(x) * widen(x);
    }
    const float n2 = block_sum256(ss, sh);
    if (threadIdx.x == 0) {
        const int s = src_size[k] < 1 ? 1 : src_size[k];
        size[k] = s;
        invn[k] = inv_length(n2);
        locality[k] = src_loc ? src_loc[k] : (float)s;
        access[k] = src_acc ? src_acc[k] : 0u;
        raise_version_once(version, k);
    }
}

// Finalize: per query, max over the slice keys; then either the key names the row (nothing to read), or it
// names a group of four consecutive rows: their exact cosines (one wave per row; strict ">" in ascending
// row order, so the lowest index keeps a tie); then the strict threshold test.  One 256-thread block
// per query.  `vec` = rows are 16-byte aligned and a whole number of 16-byte chunks.
// LEFT: what a screened lookup has left over: the first *many of the queries, whose results go to of[q].
template <typename T, bool LEFT>
__global__ __launch_bounds__(256) void k_lookup_finalize(const T *__restrict__ Q, const T *__restrict__ cent,
                                                          const float *__restrict__ invn, const u64 *__restrict__ keys,
                                                          long n, long K, int d, int slices, ThetaList thetas, int vec,
                                                          int key_kind, int *out_idx, float *out_sim,
                                                          unsigned char *out_hit, unsigned *access,
                                                          const float *__restrict__ q_inv, int *upd_owner,
                                                          int *upd_members, const int *__restrict__ many,
                                                          const int *__restrict__ of, long q_base) {
    constexpr int EPC = 16 / (int)sizeof(T);  // elements per 16-byte chunk
    __shared__ float sh_f[4];
    __shared__ u64 sh_k[4];
    __shared__ float sh_s[16];
    __shared__ long sh_i[16];
    __shared__ u32x4_t sh_q[SISO_MAX_DIM / EPC];  // the query row
    const long q = blockIdx.x;
    long to = q;  // where its results go
    if constexpr (LEFT) {
        if (q >= *many) return;
        to = of[q];
    }
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, grp = t >> 4, gl = t & 15;
    const T *qrow = Q + (size_t)q * d;
    // 1/|q|: 0 for a zero-length query, NaN for a non-finite one
    float ss = 0.f;
    if (q_inv) {
        // 1 / |q| is given (the batch was quantised: Q is not read at all; such keys always name rows)
    } else if (vec) {  // the row also goes to LDS: sixteen groups of lanes will read it again
        for (int e = t * EPC; e < d; e += 256 * EPC) {
            const u32x4_t v = *(const u32x4_t *)(qrow + e);
            sh_q[e / EPC] = v;
            ss += chunk_dot(v, v, T());
        }
    } else {
        for (int e = t; e < d; e += 256) ss += widen(qrow[e]) * widen(qrow[e]);
    }
    u64 key = 0;
    for (int s = t; s < slices; s += 256) {
        const u64 k2 = keys[(size_t)q * slices + s];
        key = k2 > key ? k2 : key;
    }
    ss = wave_sum(ss);
    key = wave_max(key);
    if (lane == 0) {
        sh_f[wave] = ss;
        sh_k[wave] = key;
    }
    __syncthreads();
    const float qi = q_inv ? q_inv[q] : inv_length((sh_f[0] + sh_f[1]) + (sh_f[2] + sh_f[3]));
#pragma unroll
    for (int w = 0; w < 4; ++w) key = sh_k[w] > key ? sh_k[w] : key;

    long best_i = -1;
    float best_s = -INFINITY;
    const bool finite_q = qi == qi;
    if (key_kind == SISO_KEY_ROWS) {
        // the key names the row and carries <q, c> / |c| as the kernel summed it: nothing left to read
        if (finite_q && K > 0 && key != 0) {
            best_i = (long)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
            best_s = unordered_bits((unsigned)(key >> 32)) * qi;
        }
    } else if (finite_q && K > 0 && key != 0) {
        // the key names a group of four consecutive rows: one wave per row, its lanes share the row's chunks (a row past the
        // end reads the last row and is discarded); or one row, whose cosine is formed anew: every wave forms the same sum
        const long id = (long)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
        const long r = key_kind == SISO_KEY_GROUPS4 ? 4L * id + wave : id;
        const long at = r < K ? r : K - 1;
        const float acc = row_product<T>(qrow, sh_q, vec, cent + (size_t)at * d, d, lane);
        const float sv = r < K ? acc * qi * invn[at] : __uint_as_float(0x7FC00000u);
        if (sv == sv) {  // a NaN never wins
            best_s = sv;
            best_i = r;
        }
    }
    if (gl == 0) {
        sh_s[grp] = best_s;
        sh_i[grp] = best_i;
    }
    __syncthreads();
    if (t == 0) {
        // rows ascend with the group number inside a pass, and pass 1 lies above pass 0
        // (with groups of four every wave holds one row, ascending with the wave: the 16 entries repeat them)
        for (int g = 1; g < (key_kind == SISO_KEY_GROUPS4 ? 16 : 1); ++g) {
            const float os = sh_s[g];
            const long oi = sh_i[g];
            if (oi >= 0 && (best_i < 0 || os > best_s || (os == best_s && oi < best_i))) {
                best_s = os;
                best_i = oi;
            }
        }
        if (!finite_q) best_s = __uint_as_float(0x7FC00000u);
        write_lookup(to, LEFT ? q_base : 0L, best_i, best_s, thetas, out_idx, out_sim, out_hit, access, upd_owner, upd_members);
    }
}

// ============================================================================
// centroid update: one block per query; the block of the first member of a
// centroid sums all members in ascending order and rewrites the centroid.
// ============================================================================
#define UPD_MAXE (SISO_MAX_DIM / 256)

// Large batches: every block searching the whole index array for the members of its centroid costs
// n^2 / 256 steps.  A first pass notes, per centroid, its first member and the number of its members;
// then only the first member's block does anything, and it looks through the index array only if
// there is more than one member (queries of one batch rarely share a centroid).
#define UPD_NO_OWNER 0x7FFFFFFF
__global__ void k_update_mark(const int *__restrict__ idx, const unsigned char *__restrict__ hit, long n, long count,
                              int *owner, int *members) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || (hit && !hit[i])) return;
    const int k = idx[i];
    if (k < 0 || k >= count) return;
    atomicMin(&owner[k], (int)i);
    atomicAdd(&members[k], 1);
}
__global__ void k_update_mark_init(int *owner, int *members, long capacity) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < capacity) {
        owner[i] = UPD_NO_OWNER;
        members[i] = 0;
    }
}

// a vector with this sum of squares can be scaled to unit length (inv_length is a number above 0)
__device__ __forceinline__ bool has_length(float n2) { return n2 > 0.f && n2 <= 3.0e38f; }

// One member of a centroid: x = this thread's elements (t + 256 e) of the query; the query at unit length is
// added to acc (queries without length or with a non-finite element are passed over).  Uniform over the
// block.  Every operation is spelled out with its rounding, here and in update_write, so that k_update and
// k_finalize_update do the same arithmetic whatever the compiler would fuse in either of them.
template <int UPD_MAXE_T>
__device__ __forceinline__ bool fold_member(const float (&x)[UPD_MAXE_T], float (&acc)[UPD_MAXE_T], float *sh) {
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) ss = __fmaf_rn(x[e], x[e], ss);
    const float n2 = block_sum256(ss, sh);
    if (!has_length(n2)) return false;
    const float nrm = sqrtf(n2);
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] = __fadd_rn(acc[e], __fdiv_rn(x[e], nrm));
    return true;
}

#define FOLD_SUMS (2 * 4 * 8)
// The members list[from .. to) of a centroid (the caller folds the first): M at a time, so that their rows are on their way
// together (AHEAD: while the M before them are folded) and their lengths share a barrier; the sums take them in the order of the
// list, with the arithmetic of fold_member.  A block alone works through its members one round after the other: four at a time, their rows
// asked for when their turn had come, took 0.37 us a member, eight with the next eight on their way 0.28 (a centroid with 200 of 300
// members, 768 elements: the update 91.6 -> 65.6 us; k_finalize_update has few members and is quicker with four, none ahead; 8,192 queries on 1,000 x 128 rows, lookup and update, 118.8 -> 93.5).
// OFFSETS: 32-bit offsets in bytes leave the rows' addresses in scalar registers, without which k_update<bf16, 4> needs scratch (4,096 queries
// of 65,536 x 768, all apart, 18.5 -> 16.6 us); for long rows, and four at a time, they are not worth their own registers (4,096 Zipf queries
// of 20,000 x 2,048 fp32 154 -> 163).
// sums: FOLD_SUMS of them.
template <typename T, int UPD_MAXE_T, int M, bool AHEAD, bool OFFSETS>
__device__ __forceinline__ int fold_list(const int *list, int from, int to, const T *__restrict__ Q, int d,
                                         float (&acc)[UPD_MAXE_T], float *sums) {
    static_assert(2 * 4 * M <= FOLD_SUMS, "two buffers of a sum for every wave and member");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int members = 0;
    bool odd = false;
    if (from >= to) return 0;
    to = __builtin_amdgcn_readfirstlane(to);  // (the same for the whole block)
    T raw[M][UPD_MAXE_T];
    unsigned col[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) col[e] = (unsigned)(t + e * 256 < d ? t + e * 256 : 0) * (unsigned)sizeof(T);
    // (without a condition, also behind the last member: the registers of a load that may not happen are copied at the
    // end of the round, which waits for it)
    auto ask = [&](int p) __attribute__((always_inline)) {
        int row[M];
#pragma unroll
        for (int m = 0; m < M; ++m) row[m] = list[p + m < to ? p + m : to - 1];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const T *at = Q + (size_t)__builtin_amdgcn_readfirstlane(row[m]) * d;
#pragma unroll
            for (int e = 0; e < UPD_MAXE_T; ++e) {
                if constexpr (OFFSETS) raw[m][e] = *(const T *)((const char *)at + col[e]);
                else raw[m][e] = at[(unsigned)(t + e * 256 < d ? t + e * 256 : 0)];
            }
        }
    };
    if (AHEAD) ask(from);
    for (int p = from; p < to; p += M) {
        if (!AHEAD) ask(p);
        float x[M][UPD_MAXE_T], n2[M];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int e = 0; e < UPD_MAXE_T; ++e) x[m][e] = t + e * 256 < d ? widen(raw[m][e]) : 0.f;
        if (AHEAD) {
            ask(p + M);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < UPD_MAXE_T; ++e) ss = __fmaf_rn(x[m][e], x[m][e], ss);
            n2[m] = wave_sum(ss);
        }
        float *const at = sums + (odd ? 4 * M : 0);  // (two buffers in turn: one barrier a round)
        odd = !odd;
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (lane == 0) at[wave * M + m] = n2[m];
        __syncthreads();
        // lane l finds the length of member l % M
        const float n2_l = (at[lane % M] + at[M + lane % M]) + (at[2 * M + lane % M] + at[3 * M + lane % M]);
        const float nrm_l = sqrtf(n2_l);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (p + m >= to) break;
            if (!has_length(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(n2_l), m)))) continue;
            const float nrm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nrm_l), m));
#pragma unroll
            for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] = __fadd_rn(acc[e], __fdiv_rn(x[m][e], nrm));
            ++members;
        }
    }
    return members;
}

// Up to four members: no others to be asked for meanwhile, and half of the loads (eight at a time / four, us: 64 queries, two for
// each centroid, x 768 bf16 5.8 / 5.0, 4,096 by three 25.4 / 23.0; by one, where nothing is folded, the same).
template <typename T, int UPD_MAXE_T>
__device__ __forceinline__ int fold_some(const int *list, int from, int to, const T *__restrict__ Q, int d, float (&acc)[UPD_MAXE_T],
                                         float *sums) {
    if (UPD_MAXE_T <= 4 && to - from <= 4) return fold_list<T, UPD_MAXE_T, 4, false, true>(list, from, to, Q, d, acc, sums);
    return fold_list<T, UPD_MAXE_T, UPD_MAXE_T <= 4 ? 8 : 2, true, UPD_MAXE_T <= 4>(list, from, to, Q, d, acc, sums);
}

// The end of an update, by the block that leads centroid k: acc = the sum of its `members` unit-length members
// (this thread's elements t + 256 e), m_old / size_old = the mean and its weight as they were.  Writes the
// new mean and weight, the stored row (the mean at unit length, rounded to the storage type; left alone when
// the mean has no length: false then) and its inverse length; `stored` receives this thread's elements of the
// stored row.
template <typename T, int UPD_MAXE_T>
__device__ __forceinline__ bool update_write(int k, int d, int size_old, int members, const float (&m_old)[UPD_MAXE_T],
                                             const float (&acc)[UPD_MAXE_T], T *cent, float *mean, int *size, float *invn,
                                             float *sh, float (&stored)[UPD_MAXE_T], float &inv) {
    const int t = threadIdx.x;
    const float n_old = (float)size_old;
    const float n_new = n_old + (float)members;
    float m[UPD_MAXE_T];
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        const int col = t + e * 256;
        m[e] = 0.f;
        if (col < d) {
            m[e] = __fdiv_rn(__fmaf_rn(n_old, m_old[e], acc[e]), n_new);
            mean[(size_t)k * d + col] = m[e];
            ss = __fmaf_rn(m[e], m[e], ss);
        }
    }
    const float n2 = block_sum256(ss, sh);
    if (t == 0) size[k] = size_old + members;
    if (!(n2 > 0.f) || n2 > 3.0e38f) return false;
    const float nrm = sqrtf(n2);
    float cs = 0.f;
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        const int col = t + e * 256;
        stored[e] = 0.f;
        if (col < d) {
            T r;
            narrow(__fdiv_rn(m[e], nrm), &r);
            cent[(size_t)k * d + col] = r;
            const float back = widen(r);
            stored[e] = back;
            cs = __fmaf_rn(back, back, cs);
        }
    }
    inv = inv_length(block_sum256(cs, sh));
    if (t == 0) invn[k] = inv;
    return true;
}

#define UPD_SCAN 4096  // entries of the index array that a block looks through at a time
// UPD_MAXE_T = elements of a row per thread (4 for dim <= 1024, else 16).  owner / marked = the notes
// of k_update_mark, or NULL: then every block finds out by itself whether it is the first member.
template <typename T, int UPD_MAXE_T>
__global__ __launch_bounds__(256, UPD_MAXE_T <= 4 ? 4 : 2) void k_update(const T *__restrict__ Q, const int *__restrict__ idx,
                                                 const unsigned char *__restrict__ hit, int n, T *cent, float *mean,
                                                 int *size, float *invn, unsigned *version, int count, int d, u64 *bad, int *owner,
                                                 int *marked) {
    __shared__ float sh[4];
    __shared__ float sums[FOLD_SUMS];
    __shared__ u64 masks[4];
    __shared__ int cells[UPD_SCAN / 64];
    __shared__ int list[UPD_SCAN];
    const long me = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // what does not depend on anything else is asked for first: the first 256 entries of the index
    // array (all of it in a small batch), this block's own entry
    const bool first_ok = !owner && t < n;
    const int first_idx = first_ok ? idx[t] : -1;
    const unsigned char first_hit = first_ok && hit ? hit[t] : 1;
    if (hit && !hit[me]) return;
    const int k = idx[me];
    if (k < 0) return;
    if (k >= count) {
        if (t == 0) atomicAdd(bad, 1ull);
        return;
    }
    // ... then this block's own query and the centroid's mean, before it is known whether this block
    // leads the centroid: most do, and the rows are on their way while the notes are read
    // (without notes the two loads read this block's own index entry instead: no branch, no wait here)
    const int lead_raw = *(owner ? owner + k : idx + me);
    const int noted_raw = *(owner ? marked + k : idx + me);
    // loads without conditions (a column past the end reads column 0 and is zeroed afterwards), so
    // that all of them are in flight together
    float x_me[UPD_MAXE_T], m_old[UPD_MAXE_T];
    T xr[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        const int col = t + e * 256;
        xr[e] = Q[(size_t)me * d + (col < d ? col : 0)];
        m_old[e] = mean[(size_t)k * d + (col < d ? col : 0)];
    }
    const int size_old = size[k];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        x_me[e] = t + e * 256 < d ? widen(xr[e]) : 0.f;
        // the values exist from here on: otherwise the compiler moves the loads behind the test below,
        // where they would only start once the notes have arrived
        asm volatile("" ::"v"(x_me[e]), "v"(m_old[e]));
    }
    if (owner && lead_raw != (int)me) return;  // an earlier member leads this centroid
    if (owner) {
        __syncthreads();  // everyone has read the notes
        if (t == 0) {     // leave them as they were found
            owner[k] = UPD_NO_OWNER;
            marked[k] = 0;
            raise_version(version, k);  // (here: its address would take registers that the folding needs)
        }
    }
    float acc[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] = 0.f;
    int members = 0;
    if (!owner) {
        // at most 256 queries: one look tells who leads and who follows
        const u64 mask = __ballot(first_ok && first_idx == k && first_hit);
        if (lane == 0) masks[wave] = mask;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) before += __popcll(masks[w]);
            all += __popcll(masks[w]);
        }
        if (mask >> lane & 1) list[before + __popcll(mask & ((1ull << lane) - 1))] = t;
        __syncthreads();
        if (list[0] != (int)me) return;  // an earlier member leads this centroid
        if (t == 0) raise_version(version, k);
        if (fold_member<UPD_MAXE_T>(x_me, acc, sh)) ++members;
        members += fold_some<T, UPD_MAXE_T>(list, 1, all, Q, d, acc, sums);
    } else {
        if (fold_member<UPD_MAXE_T>(x_me, acc, sh)) ++members;
        // the others lie behind: UPD_SCAN entries of the index array at a time, all of them on their way together, the
        // members in ascending order into the list
        int found = 1;
        for (long base = me + 1; found < noted_raw && base < n; base += UPD_SCAN) {
            unsigned mine = 0;  // bit i: entry base + 256 i + t is a member
            int entry[UPD_SCAN / 256];
            unsigned char is_hit[UPD_SCAN / 256];
            // (nothing conditional, or each load would wait for the one before it: 16 x 2 of them in a row took 5 us)
#pragma unroll
            for (int i = 0; i < UPD_SCAN / 256; ++i) {
                const unsigned j = (unsigned)(base + 256 * i) + (unsigned)t;  // (32 bits: a chunk of an update at most)
                entry[i] = *(const int *)((const char *)idx + 4u * (j < (unsigned)n ? j : (unsigned)me));
            }
            if (hit) {
#pragma unroll
                for (int i = 0; i < UPD_SCAN / 256; ++i) {
                    const unsigned j = (unsigned)(base + 256 * i) + (unsigned)t;
                    is_hit[i] = hit[j < (unsigned)n ? j : (unsigned)me];
                }
            } else {
#pragma unroll
                for (int i = 0; i < UPD_SCAN / 256; ++i) is_hit[i] = 1;
            }
#pragma unroll
            for (int i = 0; i < UPD_SCAN / 256; ++i)
                mine |= (entry[i] == k && (unsigned)(base + 256 * i) + (unsigned)t < (unsigned)n && is_hit[i] != 0 ? 1u : 0u) << i;
            __syncthreads();  // (the list of the last round has been read)
#pragma unroll
            for (int i = 0; i < UPD_SCAN / 256; ++i) {
                const u64 mask = __ballot(mine >> i & 1);
                if (lane == 0) cells[4 * i + wave] = __popcll(mask);
            }
            __syncthreads();
            int at = lane < UPD_SCAN / 64 ? cells[lane] : 0;  // exclusive sums over the cells, in every wave
            const int own = at;
#pragma unroll
            for (int off = 1; off < UPD_SCAN / 64; off <<= 1) {
                const int o = __shfl_up(at, off);
                if (lane >= off) at += o;
            }
            const int all = __shfl(at, UPD_SCAN / 64 - 1);
            at -= own;
#pragma unroll
            for (int i = 0; i < UPD_SCAN / 256; ++i) {
                const u64 mask = __ballot(mine >> i & 1);
                const int to = __builtin_amdgcn_readlane(at, 4 * i + __builtin_amdgcn_readfirstlane(wave)) + __popcll(mask & ((1ull << lane) - 1));
                if (mine >> i & 1) list[to] = (int)(base + 256 * i + t);
            }
            __syncthreads();
            members += fold_some<T, UPD_MAXE_T>(list, 0, all, Q, d, acc, sums);
            found += all;
        }
    }
    if (members == 0) return;
    float stored[UPD_MAXE_T], inv;
    update_write<T, UPD_MAXE_T>(k, d, size_old, members, m_old, acc, cent, mean, size, invn, sh, stored, inv);
}

// The bytes of a rewritten row follow in place (see ByteRows): x = this thread's elements (t + 256 e) of the stored row, inv = 1 / its length, block = the scale and
// the errors of its 32 rows.  Where the scale does not fit the row any more, or there are no bytes, only the count of the rows goes up (k_finalize_update), and
// whoever writes bytes next writes all 32 rows anew.  Otherwise the counts of the rows and of the bytes go up alike: bytes that were current stay
// so, and bytes that were not do not become so.
template <int E>
__device__ __forceinline__ void follow_bytes(const float (&x)[E], float inv, int k, int d, const ByteView &bytes, const float4 &block, float *sh) {
    const int t = threadIdx.x;
    // An element beyond the scale counts as its largest, and what that leaves out as error, up to half as much again as rounding leaves of
    // a row on average (steps of block.x, each off by 12^-1/2 of one).
    const float by = inv * block.w;
    float off2 = 0.f;
    int code[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float y = fminf(fmaxf(rintf(x[e] * by), -127.f), 127.f), off = fmaf(x[e], by, -y);
        off2 = fmaf(off, off, off2);
        code[e] = (int)y;
    }
    off2 = block_sum256f(off2, sh);
    const bool fits = inv > 1e-15f && inv < 1e15f && block.y < INFINITY && off2 <= 2.25f / 12.f * (float)d;
    if (fits) {
        signed char *row = bytes.codes + (size_t)(k >> 5) * 32 * bytes.dp + (k & 31) * 16;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int col = t + e * 256;
            if (col < d) row[(col >> 5) * 1024 + ((col >> 4) & 1) * 512 + (col & 15)] = (signed char)code[e];
        }
        if (t == 0) {
            const float err = block.x * sqrtf(off2) * 1.0005f + 1e-6f;
            unsigned *errs = (unsigned *)(bytes.meta + (k >> 5));  // (not negative: they compare as integers)
            atomicMax(errs + 1, __float_as_uint(err));
            atomicMax(errs + 2, __float_as_uint(err));
            atomicAdd(bytes.made + (k >> 5), (u64)1 << 8);
        }
    }
}

// ============================================================================
// The end of a small lookup and the update of its hits as one kernel (siso_lookup_update, at most 256
// queries, keys that name rows): block q does what k_lookup_finalize does for query q, then what k_update
// does for it, with the same arithmetic in the same order, so the outputs and the state are those of the
// two kernels bit for bit.  What a block needs from the others is their (index, hit) - to know whether it
// leads its centroid and which other queries fold into it - and that crosses the grid through a board of
// one 64-bit slot per query: (written, hit, index), written and read with device-scope atomic operations.
// The slots are emptied by the kernel before this one - the first phase of the same lookup, whose first
// block does it when siso_lookup_update asks for it - so the end of that kernel stands between the emptying
// and the first entry, also when the launches are replayed from a captured graph, and no fence is needed
// (the rows and means the blocks read were written by earlier kernels too).  All blocks of the grid
// are resident together (at most 256 small blocks), so the wait for the slots ends; it is bounded all the
// same: a block that gives up leaves its centroid as it was and counts its query as not applied.
// Saves a launch and the gap before it, and the loads of the update (own row, mean of the centroid) are on
// their way while the block waits for the board.
// With an 8-bit serving copy (siso_fp8_lookup_update) the keys and 1/|q| are the copy's, the centroid arrays the
// bf16 master's, and the block that rewrites a centroid quantises the new stored row into the copy as well
// (fp8_store_row: what k_fp8_quantize would store).
// ============================================================================
__device__ __forceinline__ u64 board_entry(bool hit, int idx) {
    return (1ull << 63) | ((u64)(hit ? 1 : 0) << 32) | (u64)(unsigned)idx;
}
// LISTED: behind k_bytes_few.  What that has left of query q - the rows whose cosine may be the largest, by workgroup and in the query's list -
// is judged once more by the largest lower end of all, and multiplied: 32 rows at a time, a wave for each, with the instruction and in the order
// of k_lookup_pipe, so that the key is the one which that kernel's workgroups would have left.  (Rows of other blocks are not written
// meanwhile: a block folds when all have been heard of, and they are by then done with their rows.)
// (All columns of the instruction are the one query.  A lane supplies row `row`, one of the wave's 32 by lane % 32, and gets the products of sixteen.)
#define LISTED_ROWS 1024  // rows that are gathered before they are multiplied
typedef __bf16 listed_frag __attribute__((ext_vector_type(8)));
typedef float listed_acc __attribute__((ext_vector_type(16)));
__device__ __forceinline__ u64 listed_key(const listed_acc &acc, float w, int row) {
    const int h = (threadIdx.x & 63) >> 5;
    u64 key = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int from = 8 * (i >> 2) + 4 * h + (i & 3);
        const float v = acc[i] * __shfl(w, from);
        const u64 k = pack_key(v, (unsigned)__shfl(row, from));
        if (v > -INFINITY && k > key) key = k;
    }
    const LanePair<u64> both = lane_pair<32>(key);
    return both.a > both.b ? both.a : both.b;
}
// Many rows: each wave loads its own from memory, 32 bytes of each at a time.
__device__ __forceinline__ u64 listed_product(const bf16_t *__restrict__ cent, const float *__restrict__ invn, int row, const u32x4_t *sh_q, int d) {
    constexpr int AHEAD = 6;  // groups of four steps on their way together
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const bf16_t *at = cent + (size_t)row * d + h * 8;
    const float w = invn[row];
    listed_acc acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int e0 = 0; e0 < d; e0 += 64 * AHEAD) {
        u32x4_t x[AHEAD][4];
#pragma unroll
        for (int g = 0; g < AHEAD; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = e0 + g * 64 + i * 16;
                x[g][i] = *(const u32x4_t *)(at + (e < d ? e : 0));
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) {
            if (e0 + g * 64 >= d) break;  // (d is a multiple of 64)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(listed_frag, x[g][i]),
                                                              __builtin_bit_cast(listed_frag, sh_q[(e0 + g * 64 + i * 16) / 8 + h]), acc, 0, 0, 0);
        }
    }
    return listed_key(acc, w, row);
}
// Up to LISTED_FEW rows, what mostly is left: all waves bring them to LDS, whole rows at a time (in the wave's own loads they took 5 us of 13),
// a pad of 16 bytes behind each, and a wave for 32 of them multiplies.
#define LISTED_FEW 64
// Rows of one query that take longer than the bytes save, 0.1 us each (a step of eight against 66,000 x 1,024, mean cosine 0.6, up to 591 of them: 66 us,
// 41 over the stored rows): the host hears of them as of lists that found no room.  Rows without a common direction leave up to 330, a
// mean cosine of 0.4 mostly fewer than 260.
#define LISTED_MANY 512
#define LISTED_LDS(d) (LISTED_FEW * (2 * (d) + 16))
#define LISTED_STATIC (14 * 1024)  // and what else the kernel keeps there, 13,952 bytes
__device__ __forceinline__ u64 listed_products_few(const bf16_t *__restrict__ cent, const float *__restrict__ invn, const int *sh_rows, int many,
                                               const u32x4_t *sh_q, int d, unsigned char *room) {
    constexpr int AHEAD = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, pitch = 2 * d + 16;
    const int mine = wave * 32 + (lane & 31) < many ? wave * 32 + (lane & 31) : 0;  // this lane's row
    const int row = sh_rows[mine];
    const float w = invn[row];
    for (int r0 = wave; r0 < many; r0 += 4 * AHEAD) {
        u32x4_t x[AHEAD][2];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const bf16_t *at = cent + (size_t)sh_rows[r0 + 4 * k < many ? r0 + 4 * k : r0] * d;
#pragma unroll
            for (int c = 0; c < 2; ++c) x[k][c] = *(const u32x4_t *)(at + ((lane + 64 * c) * 8 < d ? (lane + 64 * c) * 8 : 0));
        }
#pragma unroll
        for (int k = 0; k < AHEAD; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (r0 + 4 * k < many && (lane + 64 * c) * 8 < d) *(u32x4_t *)(room + (size_t)(r0 + 4 * k) * pitch + (lane + 64 * c) * 16) = x[k][c];
    }
    __syncthreads();
    if (wave * 32 >= many) return 0;
    listed_acc acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const unsigned char *at = room + (size_t)mine * pitch + h * 16;
    u32x4_t x[4], q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = *(const u32x4_t *)(at + i * 32);
        q[i] = sh_q[i * 2 + h];
    }
    for (int e = 64; e <= d; e += 64) {  // (the next four steps are read while four are multiplied)
        u32x4_t y[4], p[4];
        const int n = e < d ? e : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            y[i] = *(const u32x4_t *)(at + n * 2 + i * 32);
            p[i] = sh_q[(n + i * 16) / 8 + h];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(listed_frag, x[i]), __builtin_bit_cast(listed_frag, q[i]), acc, 0, 0, 0);
            x[i] = y[i];
            q[i] = p[i];
        }
    }
    return listed_key(acc, w, row);
}

// What the kernel does beside that, as types and not as conditions: arguments, loads and code that are not needed cost 1 to 2 % of a small step.
struct FoldPlain {  // nobody asks about changed rows (no bytes have been made, and no graph records the launch)
    static constexpr bool LISTED = false, BYTES = false, COUNTED = false;
};
struct FoldCounted {  // the counts of the rows that are rewritten change (see ByteRows)
    static constexpr bool LISTED = false, BYTES = false, COUNTED = true;
    unsigned *version;
};
struct FoldBytes {  // and their bytes follow
    static constexpr bool LISTED = false, BYTES = true, COUNTED = true;
    unsigned *version;
    ByteView bytes;
};
struct FoldListed {
    static constexpr bool LISTED = true, BYTES = true, COUNTED = true;
    unsigned *version;
    ByteView bytes;
    FewLists few;
    int fold;  // 0 = a lookup and nothing else
    int *flooded;
};
template <typename T, int UPD_MAXE_T, class More>
__global__ __launch_bounds__(256) void k_finalize_update(const T *__restrict__ Q, const u64 *__restrict__ keys, long n, long K,
                                                          int d, int slices, float theta, int vec, int *out_idx,
                                                          float *out_sim, unsigned char *out_hit, unsigned *access, T *cent,
                                                          float *mean, int *size, float *invn, u64 *board,
                                                          int spin_limit, u64 *gave_up, const float *__restrict__ q_inv,
                                                          unsigned char *copy_codes, float *copy_scale, float *copy_inv,
                                                          int *copy_size, More more) {
    constexpr bool LISTED = More::LISTED, BYTES = More::BYTES, COUNTED = More::COUNTED;
    constexpr int EPC = 16 / (int)sizeof(T);
    __shared__ float sh[4];
    __shared__ float sh_f[4];
    __shared__ u64 sh_k[4];
    __shared__ u64 masks[4];
    __shared__ u64 sh_board[SISO_FOLD_BOARD];
    __shared__ float sums[FOLD_SUMS];
    __shared__ int list[SISO_FOLD_BOARD];
    __shared__ int sh_all;
    __shared__ u32x4_t sh_q[LISTED ? SISO_SCREEN_DIM / EPC : 1];
    __shared__ int sh_rows[LISTED ? LISTED_ROWS : 1];
    __shared__ unsigned sh_upper[LISTED ? LISTED_ROWS : 1];
    __shared__ int sh_rows_n;
    __shared__ unsigned sh_low[4];
    extern __shared__ __attribute__((aligned(16))) unsigned char listed_room[];  // LISTED: LISTED_LDS(d)
    const long me = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const T *qrow = Q + (size_t)me * d;
    // this block's own query in the layout of the update, asked for first
    T xr[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        const int col = t + e * 256;
        xr[e] = qrow[col < d ? col : 0];
    }
    // --- k_lookup_finalize for keys that name rows: 1/|q| (given, if the batch was quantised) and the largest key
    float ss = 0.f;
    if (q_inv) {
    } else if (vec) {
        for (int e = t * EPC; e < d; e += 256 * EPC) {
            const u32x4_t v = *(const u32x4_t *)(qrow + e);
            ss += chunk_dot(v, v, T());
            if constexpr (LISTED) sh_q[e / EPC] = v;
        }
    } else {
        for (int e = t; e < d; e += 256) ss += widen(qrow[e]) * widen(qrow[e]);
    }
    u64 key = 0;
    unsigned entry[6], low = 0;
    int listed = 0, named = 0, words = 0;
    uint2 place = make_uint2(0, 0);
    if constexpr (LISTED) {  // all of it in one round trip
        static_assert(SISO_FEW_WORKGROUPS <= 256 && SISO_FEW_SLOTS == 8, "a workgroup's words to a thread");
        words = SISO_FEW_SLOTS * 64 / (n <= 8 ? 8 : n <= 32 ? 32 : 64);
        const u32x4_t *from = (const u32x4_t *)(more.few.slots + ((size_t)me * slices + (t < slices ? t : 0)) * words);
        const u32x4_t e0 = from[0], e1 = from[1];
        place = more.few.rows[(size_t)me * SISO_FEW_LIST + t];
        listed = more.few.cnt[me];
        key = more.few.best[me];
        low = t >= slices || e0[0] == ordered_bits(INFINITY) ? 0 : e0[0];  // (of a query that lists nothing: +inf)
        named = t >= slices ? 0 : (int)e0[1] < words - 2 ? (int)e0[1] : words - 2;
#pragma unroll
        for (int i = 0; i < 6; ++i) entry[i] = i < 2 ? e0[2 + i] : e1[i - 2];
        if (t == 0) sh_rows_n = 0;
    } else {
        for (int s = t; s < slices; s += 256) {
            const u64 k2 = keys[(size_t)me * slices + s];
            key = k2 > key ? k2 : key;
        }
    }
    if constexpr (LISTED) {
        asm volatile("" ::"v"(listed));  // (has arrived: it is emptied behind the barrier)
        low = wave_fold(low, [](unsigned a, unsigned b) __attribute__((always_inline)) { return a > b ? a : b; });
        if (lane == 0) sh_low[wave] = low;
    }
    ss = wave_sum(ss);
    key = wave_max(key);
    if (lane == 0) {
        sh_f[wave] = ss;
        sh_k[wave] = key;
    }
    __syncthreads();
    const float qi = q_inv ? q_inv[me] : inv_length((sh_f[0] + sh_f[1]) + (sh_f[2] + sh_f[3]));
#pragma unroll
    for (int w = 0; w < 4; ++w) key = sh_k[w] > key ? sh_k[w] : key;
    if constexpr (LISTED) {
        if (t == 0) {  // (everyone has read them)
            more.few.cnt[me] = 0;
            more.few.best[me] = 0;
            if (me == 0) *more.few.call += 1;
        }
        low = max(max(sh_low[0], sh_low[1]), max(sh_low[2], sh_low[3]));
        float bound = unordered_bits(low);
        auto multiply = [&](int many) {
            for (int g = wave * 32; g < many; g += 128) {
                const u64 k2 = listed_product((const bf16_t *)cent, invn, sh_rows[g + (lane & 31) < many ? g + (lane & 31) : g], sh_q, d);
                key = k2 > key ? k2 : key;
            }
        };
        // the rows that this thread has been given and that reach the bound: of workgroup t, and every 256th of the list
        const int places = listed < SISO_FEW_LIST ? listed : SISO_FEW_LIST;
        auto each = [&](auto &&take) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 6; ++i)
                if (i < named && few_upper(entry[i]) >= bound) take((int)few_row(entry[i], (unsigned)t, (unsigned)slices), entry[i]);
            for (int i = 6; i < named; i += 4) {
                const u32x4_t e = *(const u32x4_t *)(more.few.slots + ((size_t)me * slices + t) * words + 2 + i);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (i + k < named && few_upper(e[k]) >= bound) take((int)few_row(e[k], (unsigned)t, (unsigned)slices), e[k]);
            }
            for (int i = t; i < places; i += 256) {
                const uint2 e = i < 256 ? place : more.few.rows[(size_t)me * SISO_FEW_LIST + i];
                if (few_upper(e.y) >= bound) take((int)e.x, e.y);
            }
        };
        int own = 0;
        each([&](int row, unsigned e) __attribute__((always_inline)) {
            const int to = atomicAdd(&sh_rows_n, 1);
            if (to < LISTED_ROWS) {
                sh_rows[to] = row;
                sh_upper[to] = e & 8191u;
            }
            ++own;
        });
        __syncthreads();
        int all_rows = sh_rows_n;
        if (all_rows > LISTED_FEW) {
            // Rather many: the bound is short of the best by as much as the bytes may be off.  The cosine of the row of the highest upper end, as
            // k_screen_pick forms it, is not, and rows that cannot reach that are left out.
            u64 high = 0;
            const int kept = all_rows < LISTED_ROWS ? all_rows : LISTED_ROWS;
            for (int i = t; i < kept; i += 256) {
                const u64 k2 = (u64)sh_upper[i] << 32 | (unsigned)i;
                high = k2 > high ? k2 : high;
            }
            high = wave_max(high);
            if (lane == 0) sh_k[wave] = high;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < 4; ++w) high = sh_k[w] > high ? sh_k[w] : high;
            const int best_row = sh_rows[(unsigned)high];
            const float cosine = row_product<bf16_t>((const bf16_t *)qrow, sh_q, 1, (const bf16_t *)cent + (size_t)best_row * d, d, lane) * qi * invn[best_row];
            if (cosine == cosine) bound = fmaxf(bound, cosine - 2e-5f);
            __syncthreads();
            if (t == 0) sh_rows_n = 0;
            __syncthreads();
            own = 0;
            each([&](int row, unsigned) __attribute__((always_inline)) {
                const int to = atomicAdd(&sh_rows_n, 1);
                if (to < LISTED_ROWS) sh_rows[to] = row;
                ++own;
            });
            __syncthreads();
            all_rows = sh_rows_n;
        }
        if (all_rows > LISTED_MANY && t == 0) __hip_atomic_store(more.flooded, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (all_rows <= LISTED_FEW) {
            const u64 k2 = all_rows > 0 ? listed_products_few((const bf16_t *)cent, invn, sh_rows, all_rows, sh_q, d, listed_room) : 0;
            key = k2 > key ? k2 : key;
        } else if (all_rows <= LISTED_ROWS) {
            multiply(all_rows);
        } else {  // more than LDS holds: one part of them after the other, by their numbers
            int before = own;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(before, off);
                if (lane >= off) before += o;
            }
            if (lane == 63) list[wave] = before;
            __syncthreads();
            before -= own;
            for (int w = 0; w < wave; ++w) before += list[w];
            for (int from = 0; from < all_rows; from += LISTED_ROWS) {
                int number = before - from;
                each([&](int row, unsigned) __attribute__((always_inline)) {
                    if (number >= 0 && number < LISTED_ROWS) sh_rows[number] = row;
                    ++number;
                });
                __syncthreads();
                multiply(all_rows - from < LISTED_ROWS ? all_rows - from : LISTED_ROWS);
                __syncthreads();
            }
        }
        if (lane == 0) sh_k[wave] = key;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) key = sh_k[w] > key ? sh_k[w] : key;
        if (qi == 0.f) {  // without a single element: all products are 0, and the first row that has a length, or none, is named
            bool none = true;
            for (int e = t; e < d; e += 256) none = none && (__float_as_uint(widen(qrow[e])) << 1) == 0;
            if (!__syncthreads_or(!none)) {
                key = 0;
                for (long r0 = 0; r0 < K && key == 0; r0 += 256) {
                    const bool ok = r0 + t < K && invn[r0 + t] == invn[r0 + t];
                    __syncthreads();
                    if (lane == 0) masks[wave] = 0;
                    const u64 mask = __ballot(ok);
                    if (lane == 0) masks[wave] = mask;
                    __syncthreads();
                    for (int w = 3; w >= 0; --w)
                        if (masks[w] != 0) key = pack_key(0.f, (unsigned)(r0 + 64 * w + __ffsll((long long)masks[w]) - 1));
                }
            }
        }
    }
    long best_i = -1;
    float best_s = -INFINITY;
    const bool finite_q = qi == qi;
    if (finite_q && K > 0 && key != 0) {
        best_i = (long)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
        best_s = unordered_bits((unsigned)(key >> 32)) * qi;
    }
    if (!finite_q) best_s = __uint_as_float(0x7FC00000u);
    const bool hit = best_i >= 0 && best_s > theta;
    if (t == 0) {
        out_idx[me] = (int)best_i;
        out_sim[me] = best_s;
        if (!LISTED || out_hit) out_hit[me] = hit ? 1 : 0;  // (a lookup alone may do without)
        if (hit && access && access[best_i] != SISO_ACCESS_INF) atomicAdd(&access[best_i], 1u);
        __hip_atomic_store(board + me, board_entry(hit, (int)best_i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!hit) return;
    if constexpr (LISTED)
        if (!more.fold) return;
    // --- k_update for query `me`: its centroid's mean and weight, on their way during the wait
    const int k = (int)best_i;
    float x_me[UPD_MAXE_T], m_old[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        const int col = t + e * 256;
        m_old[e] = mean[(size_t)k * d + (col < d ? col : 0)];
    }
    const int size_old = size[k];
    float4 block = make_float4(0.f, 0.f, 0.f, 0.f);  // what the bytes of the centroid's 32 rows are made with
    if constexpr (BYTES) block = more.bytes.meta[k >> 5];
    // (without bytes to keep step with, that the count changes is all that is asked of it: a store, where 256 additions to the one line of a small
    // cache's counts are 2 us)
    unsigned counted = 0;
    if constexpr (COUNTED && !BYTES) counted = more.version[k >> 5];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) {
        x_me[e] = t + e * 256 < d ? widen(xr[e]) : 0.f;
        asm volatile("" ::"v"(x_me[e]), "v"(m_old[e]));  // (the loads are issued here, not behind the wait)
    }
    // the board: wave 0 reads the slots until all of them are written (one query has nobody to wait for)
    if (wave == 0) {
        bool all = n == 1;
        if (all && lane == 0) sh_board[0] = board_entry(hit, k);
        for (int tries = 0; tries < spin_limit && !all; ++tries) {
            bool mine = true;
            for (int j = lane; j < (int)n; j += 64) {
                const u64 v = __hip_atomic_load(board + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh_board[j] = v;
                mine = mine && (v >> 63) != 0;
            }
            all = __ballot(!mine) == 0;
            if (!all) __builtin_amdgcn_s_sleep(4);
        }
        if (lane == 0) sh_all = all ? 1 : 0;
    }
    __syncthreads();
    if (!sh_all) {
        if (t == 0) atomicAdd(gave_up, 1ull);
        return;
    }
    float acc[UPD_MAXE_T];
#pragma unroll
    for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] = 0.f;
    // the members of centroid k in ascending order (a hit whose index is k)
    const bool m = t < (int)n && sh_board[t] == board_entry(true, k);
    const u64 mask = __ballot(m);
    if (lane == 0) masks[wave] = mask;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) before += __popcll(masks[w]);
        all += __popcll(masks[w]);
    }
    if (m) list[before + __popcll(mask & ((1ull << lane) - 1))] = t;
    __syncthreads();
    if (list[0] != (int)me) return;  // an earlier member leads this centroid (uniform over the block)
    if (t == 0) {
        if constexpr (BYTES) raise_version(more.version, k);
        else if constexpr (COUNTED) more.version[k >> 5] = counted + 1;
    }
    int members = fold_member<UPD_MAXE_T>(x_me, acc, sh) ? 1 : 0;
    members += fold_list<T, UPD_MAXE_T, UPD_MAXE_T <= 4 ? 4 : 2, false, false>(list, 1, all, Q, d, acc, sums);
    if (members == 0) return;
    float stored[UPD_MAXE_T], inv;
    const bool rewritten = update_write<T, UPD_MAXE_T>(k, d, size_old, members, m_old, acc, cent, mean, size, invn, sh, stored, inv);
    if constexpr (BYTES)
        if (rewritten) follow_bytes<UPD_MAXE_T>(stored, inv, k, d, more.bytes, block, sh);
    if (copy_codes) {  // the 8-bit copy follows
        if (t == 0) copy_size[k] = size_old + members;
        if (rewritten) fp8_store_row<UPD_MAXE_T>(stored, d, copy_codes + (size_t)k * d, copy_scale + k, copy_inv + k, sh);
    }
}


// ============================================================================
// group merge: lock-free union-find (the lower index becomes the root), group
// means by the group's root, stable compaction.
// ============================================================================
__global__ void k_uf_init(int *parent, unsigned char *touched, int *members_of, int *cursor, long K) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < K) {
        parent[i] = (int)i;
        touched[i] = 0;
        members_of[i] = 0;
        cursor[i] = 0;
    }
}

// Member lists of the groups: how many rows each root leads (k_uf_roots counts them, itself included), then, once the
// counts have been scanned into list starts, the rows themselves (in the order they arrive; the root's block sorts
// its list).  Only rows that occur in a pair take part.
__global__ void k_group_fill(const int *__restrict__ root, const unsigned char *__restrict__ touched, long K,
                             const int *__restrict__ first, int *cursor, int *list) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= K || !touched[i]) return;
    const int r = root[i];
    list[first[r] + atomicAdd(&cursor[r], 1)] = (int)i;
}

__global__ void k_uf_first(const int *__restrict__ pairs, long n_pairs, long K, int *parent) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_pairs) return;
    const int a = pairs[2 * p], b = pairs[2 * p + 1];
    if (a >= 0 && b >= 0 && a < K && b < K) uf_first(parent, a, b);
}

// Pairs that name a row twice or one that is not there are passed over and counted: the host looks at the count before
// anything of the cache is touched.
__global__ void k_uf_hook(const int *__restrict__ pairs, long n_pairs, long K, int *parent, unsigned char *touched, u64 *bad) {
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_pairs) return;
    const int a = pairs[2 * p], b = pairs[2 * p + 1];
    if (a < 0 || b < 0 || a >= K || b >= K || a == b) {
        atomicAdd(bad, 1ull);
        return;
    }
    touched[a] = 1;
    touched[b] = 1;
    uf_join(parent, a, b);
}

__global__ void k_uf_roots(int *parent, const unsigned char *__restrict__ touched, int *root, int *members_of,
                           long K) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= K) return;
    const int r = uf_find(parent, (int)i);
    root[i] = r;
    if (touched[i]) atomicAdd(&members_of[r], 1);
}

// A block looks after rows_per_block (at most 64) consecutive rows: those that are the root of a group of at least two rows are
// given their group's mean, one after the other, four members' loads in flight.  (A block per row has nothing to do in
// most of them: 131,072 rows in groups of eight took 252 us, 16 rows per block 152 us; 403 MB of means are read.  A few
// thousand rows are better off with a block each: all groups at the same time.)
// UPD_MAXE_T = elements of a row per thread (4 for dim <= 1024, else 16).
#define GROUP_LIST_MAX 1024  // members of a group that its block sorts in LDS; larger groups are searched for
template <typename T, int UPD_MAXE_T>
__global__ __launch_bounds__(256) void k_group_mean(const int *__restrict__ root, const unsigned char *__restrict__ touched,
                                                     long K, const int *__restrict__ members_of,
                                                     const int *__restrict__ first, const int *__restrict__ list,
                                                     T *cent, float *mean, int *size, float *invn,
                                                     float *locality, unsigned *access, unsigned *version, int d, int rows_per_block) {
    __shared__ float sh[4];
    __shared__ u64 masks[4];
    __shared__ int raw[GROUP_LIST_MAX], sorted[GROUP_LIST_MAX];
    const int t = threadIdx.x, lane = t & 63;
    const long r_lane = (long)blockIdx.x * rows_per_block + lane;
    u64 roots = __ballot(lane < rows_per_block && r_lane < K && touched[r_lane] && root[r_lane] == (int)r_lane);  // the same in every wave
    for (; roots != 0; roots &= roots - 1) {
        const long r = (long)blockIdx.x * rows_per_block + __ffsll((long long)roots) - 1;
        float acc[UPD_MAXE_T];
#pragma unroll
        for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] = 0.f;
        double wsum = 0.0;
        int members = 0;
        float loc = 0.f;  // cluster sizes of Algorithm 1 add up, in ascending order of the members
        u64 refs = 0;     // so do the access counts, saturating at infinity
        // up to four members at a time: their loads are in flight together, the sums take them in order
        auto take = [&](const long(&jj)[4], int many) __attribute__((always_inline)) {
            float x[4][UPD_MAXE_T], lo[4];
            int sz[4];
            unsigned ac[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int e = 0; e < UPD_MAXE_T; ++e) {
                    const int col = t + e * 256;
                    x[m][e] = mean[(size_t)jj[m] * d + (col < d ? col : 0)];
                }
                sz[m] = size[jj[m]];
                lo[m] = locality[jj[m]];
                ac[m] = access[jj[m]];
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                if (m >= many) break;
                const float wgt = (float)sz[m];
#pragma unroll
                for (int e = 0; e < UPD_MAXE_T; ++e) acc[e] += wgt * x[m][e];
                wsum += (double)sz[m];
                loc = loc + lo[m];
                refs += ac[m];
            }
            members += many;
        };
        const int listed = members_of[r];
        if (listed <= GROUP_LIST_MAX) {
            // the list arrives in no particular order; the sums take the members in ascending order, so the
            // result does not depend on scheduling: every thread places its entries by counting the smaller ones
            const int lo = first[r];
            for (int i = t; i < listed; i += 256) raw[i] = list[lo + i];
            __syncthreads();
            for (int i = t; i < listed; i += 256) {
                const int mine = raw[i];
                int below = 0;
                for (int k = 0; k < listed; ++k) below += raw[k] < mine ? 1 : 0;
                sorted[below] = mine;
            }
            __syncthreads();
            for (int p = 0; p < listed; p += 4) {
                const int many = listed - p < 4 ? listed - p : 4;
                const long jj[4] = {sorted[p], sorted[p + (many > 1 ? 1 : 0)], sorted[p + (many > 2 ? 2 : 0)],
                                    sorted[p + (many > 3 ? 3 : 0)]};
                take(jj, many);
            }
        } else {
            for (long base = r - (r & 255); base < K; base += 256) {
                const long j = base + t;
                const bool m = j < K && j >= r && root[j] == (int)r;
                const u64 mask = __ballot(m);
                __syncthreads();
                if (lane == 0) masks[t >> 6] = mask;
                __syncthreads();
                for (int w = 0; w < 4; ++w) {
                    u64 mm = masks[w];
                    while (mm) {
                        long jj[4];
                        int many = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (mm) {
                                jj[i] = base + w * 64 + __ffsll((long long)mm) - 1;
                                mm &= mm - 1;
                                ++many;
                            } else {
                                jj[i] = r;
                            }
                        }
                        take(jj, many);
                    }
                }
            }
        }
        if (members >= 2) {
            const float wtot = (float)wsum;
            float m[UPD_MAXE_T];
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < UPD_MAXE_T; ++e) {
                const int col = t + e * 256;
                m[e] = 0.f;
                if (col < d) {
                    m[e] = acc[e] / wtot;
                    mean[(size_t)r * d + col] = m[e];
                    ss += m[e] * m[e];
                }
            }
            const float n2 = block_sum256(ss, sh);
            if (t == 0) {
                size[r] = wsum > 2147483647.0 ? 2147483647 : (int)wsum;
                locality[r] = loc;
                access[r] = refs >= (u64)SISO_ACCESS_INF ? SISO_ACCESS_INF : (unsigned)refs;
            }
            if ((n2 > 0.f) && n2 <= 3.0e38f) {
                const float nrm = sqrtf(n2);
                float cs = 0.f;
#pragma unroll
                for (int e = 0; e < UPD_MAXE_T; ++e) {
                    const int col = t + e * 256;
                    if (col < d) {
                        T v;
                        narrow(m[e] / nrm, &v);
                        cent[(size_t)r * d + col] = v;
                        const float back = widen(v);
                        cs += back * back;
                    }
                }
                const float c2 = block_sum256(cs, sh);
                if (t == 0) {
                    invn[r] = inv_length(c2);
                    raise_version(version, r);
                }
            }
        }
        __syncthreads();  // the lists of this group have been read
    }
}

// Exclusive scans of the group sizes (into the starts of the member lists) and of the survivors (root[i] == i, into their
// new places) together, SCAN_ROWS rows per 1024-thread block: the sums of the blocks first, then every block adds up
// those before its own.  (One block for everything took 73 us a scan for 131,072 rows; two launches take 11 us for both.)
#define SCAN_ROWS 4096
__device__ __forceinline__ void scan_load(const int *__restrict__ members_of, const int *__restrict__ root, long K, long i0,
                                          int (&m)[4], int (&f)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const long i = i0 + k;
        m[k] = i < K ? members_of[i] : 0;
        f[k] = i < K && root[i] == (int)i ? 1 : 0;
    }
}
// sum over a 1024-thread block of two numbers; every thread gets both
__device__ __forceinline__ int2 block_sum1024(int a, int b, int2 *sh) {
    const auto sum = [](int x, int y) __attribute__((always_inline)) { return x + y; };
    a = wave_fold(a, sum);
    b = wave_fold(b, sum);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_int2(a, b);
    __syncthreads();
    int2 s = make_int2(0, 0);
    for (int w = 0; w < 16; ++w) {
        s.x += sh[w].x;
        s.y += sh[w].y;
    }
    return s;
}
__global__ __launch_bounds__(1024) void k_scan_sums(const int *__restrict__ members_of, const int *__restrict__ root, long K,
                                                     int2 *sums) {
    __shared__ int2 sh[16];
    int m[4], f[4];
    scan_load(members_of, root, K, (long)blockIdx.x * SCAN_ROWS + 4 * threadIdx.x, m, f);
    const int2 s = block_sum1024((m[0] + m[1]) + (m[2] + m[3]), (f[0] + f[1]) + (f[2] + f[3]), sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}
__global__ __launch_bounds__(1024) void k_scan_exclusive(const int *__restrict__ members_of, const int *__restrict__ root,
                                                          long K, const int2 *__restrict__ sums, int *first, int *newpos,
                                                          u64 *total) {
    __shared__ int2 sh[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int a = 0, b = 0;
    for (int k = t; k < (int)blockIdx.x; k += 1024) {
        a += sums[k].x;
        b += sums[k].y;
    }
    const int2 before = block_sum1024(a, b, sh);
    const long i0 = (long)blockIdx.x * SCAN_ROWS + 4 * t;
    int m[4], f[4];
    scan_load(members_of, root, K, i0, m, f);
    const int mine_m = (m[0] + m[1]) + (m[2] + m[3]), mine_f = (f[0] + f[1]) + (f[2] + f[3]);
    int incl_m = mine_m, incl_f = mine_f;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int om = __shfl_up(incl_m, off), of = __shfl_up(incl_f, off);
        if (lane >= off) {
            incl_m += om;
            incl_f += of;
        }
    }
    __syncthreads();
    if (lane == 63) sh[w] = make_int2(incl_m, incl_f);
    __syncthreads();
    int run_m = before.x + incl_m - mine_m, run_f = before.y + incl_f - mine_f;
    for (int k = 0; k < w; ++k) {
        run_m += sh[k].x;
        run_f += sh[k].y;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (i0 + k < K) {
            first[i0 + k] = run_m;
            newpos[i0 + k] = run_f;
        }
        run_m += m[k];
        run_f += f[k];
    }
    if (blockIdx.x == gridDim.x - 1 && t == 1023) *total = (u64)run_f;
}
template <typename T>
__global__ __launch_bounds__(256) void k_gather_rows(const int *__restrict__ root, const int *__restrict__ newpos,
                                                      const T *__restrict__ cent, const float *__restrict__ mean,
                                                      const int *__restrict__ size, const float *__restrict__ invn,
                                                      const float *__restrict__ locality,
                                                      const unsigned *__restrict__ access, T *cent2, float *mean2,
                                                      int *size2, float *invn2, float *locality2, unsigned *access2,
                                                      unsigned *version2, int d) {
    const long i = blockIdx.x;
    if (root[i] != (int)i) return;
    const long p = newpos[i];
    for (int e = threadIdx.x; e < d; e += 256) {
        cent2[(size_t)p * d + e] = cent[(size_t)i * d + e];
        mean2[(size_t)p * d + e] = mean[(size_t)i * d + e];
    }
    if (threadIdx.x == 0) {
        size2[p] = size[i];
        invn2[p] = invn[i];
        locality2[p] = locality[i];
        access2[p] = access[i];
        raise_version_once(version2, p);
    }
}

__global__ void k_survivor_map(const int *__restrict__ root, const int *__restrict__ newpos, long K, int *out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < K) out[i] = newpos[root[i]];
}

// ============================================================================
// C ABI
// ============================================================================
// Key workspace of siso_lookup_static: part of the library's image, so a caller that must not allocate
// (graph capture, a serving loop, a harness that forbids it) still has room for the phase-1 keys.  Every
// GPU the library runs on holds its own copy at its own address until the process ends; in host code the
// array's name is only a handle for hipGetSymbolAddress, never an address to pass on.
#define SISO_STATIC_KEYS (1L << 20)  // 8 MiB
static __device__ __align__(256) u64 scratch[SISO_STATIC_KEYS];
#define SISO_MAX_DEVICES 64
static u64 *scratch_ptr[SISO_MAX_DEVICES];  // device address of `scratch` per device, resolved by siso_create_ex

// the current device's copy of the array (the device must be current)
static int resolve_scratch(int device, u64 **out) {
    *out = nullptr;
    if (device < 0 || device >= SISO_MAX_DEVICES) return SISO_EINVAL;
    if (!scratch_ptr[device]) {
        u64 *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return SISO_EHIP;
        }
        scratch_ptr[device] = ptr;
    }
    *out = scratch_ptr[device];
    return SISO_OK;
}

static int ensure_workspace(siso_cache *c, long n, int slices) {
    const long need_keys = n * (long)slices;
    if (need_keys > c->keys_cap) {
        if (c->keys) {
            HIP_TRY(c, hipStreamSynchronize(c->stream));
            HIP_TRY(c, hipFree(c->keys));
            c->keys = nullptr;
            c->keys_cap = 0;
        }
        if (hipMalloc((void **)&c->keys, (size_t)need_keys * sizeof(u64)) != hipSuccess) {
            (void)hipGetLastError();
            return siso_fail(c, SISO_ENOMEM, "workspace of %ld keys", need_keys);
        }
        c->keys_cap = need_keys;
    }
    return SISO_OK;
}

int siso_ensure_keys(siso_cache *c, long need) { return ensure_workspace(c, need, 1); }

// hipMalloc and hipFree of something large cost tens to hundreds of microseconds each (a refresh of 65,536 rows, with the rest
// of its host side: 2,490 -> 1,868 us; a merge of 6,208 rows, whose temporaries are small: 258 -> 250).
int siso_arena(siso_cache *c, size_t device_bytes, size_t host_bytes) {
    if (device_bytes > c->arena_cap || host_bytes > c->pinned_cap) HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (device_bytes > c->arena_cap) {
        if (c->arena) (void)hipFree(c->arena);
        c->arena = nullptr;
        c->arena_cap = 0;
        if (hipMalloc((void **)&c->arena, device_bytes) != hipSuccess) {
            (void)hipGetLastError();
            c->arena = nullptr;
            return siso_fail(c, SISO_ENOMEM, "temporaries of %zu bytes", device_bytes);
        }
        c->arena_cap = device_bytes;
    }
    if (host_bytes > c->pinned_cap) {
        if (c->pinned) (void)hipHostFree(c->pinned);
        c->pinned = nullptr;
        c->pinned_cap = 0;
        if (hipHostMalloc((void **)&c->pinned, host_bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            c->pinned = nullptr;
            return siso_fail(c, SISO_ENOMEM, "pinned temporaries of %zu bytes", host_bytes);
        }
        c->pinned_cap = host_bytes;
    }
    return SISO_OK;
}

void siso_arena_done(siso_cache *c) {
    siso_screen_done(c);
    if (c->arena_cap <= (size_t)SISO_ARENA_KEEP && c->pinned_cap <= (size_t)SISO_PINNED_KEEP) return;
    (void)hipStreamSynchronize(c->stream);
    if (c->arena_cap > (size_t)SISO_ARENA_KEEP) {
        (void)hipFree(c->arena);
        c->arena = nullptr;
        c->arena_cap = 0;
    }
    if (c->pinned_cap > (size_t)SISO_PINNED_KEEP) {
        (void)hipHostFree(c->pinned);
        c->pinned = nullptr;
        c->pinned_cap = 0;
    }
}

// How often the rows of 32 have changed (ByteRows) stands behind other numbers of its set, `words` of them, in their allocation: one
// of its own would move what is allocated after it.  (With the board of a cache of 1,024 rows 4 KiB further on, 256 queries' steps take 1 % longer.)
// first_byte: 0 is nobody's, bytes that are not made yet.
static bool take_with_versions(siso_cache *c, void **at, size_t words, unsigned **version, int first_byte) {
    const size_t before = (words + 63) / 64 * 64, counts = c->dtype == SISO_FP8 ? 0 : ((size_t)c->capacity + 255) / 256 * 8;  // (8-bit rows are never screened)
    if (hipMalloc(at, (before + counts) * sizeof(unsigned)) != hipSuccess) return false;
    if (counts == 0) return true;
    *version = (unsigned *)*at + before;
    return hipMemset(*version, first_byte, counts * sizeof(unsigned)) == hipSuccess;
}

int siso_second_set(siso_cache *c) {
    if (c->cent_b) return SISO_OK;
    const size_t cells = (size_t)c->capacity * c->dim;
    const size_t cent_bytes = (cells + (size_t)SISO_PAD_ROWS * c->dim) * elem_bytes(c->dtype);
    bool ok = hipMalloc(&c->cent_b, cent_bytes) == hipSuccess;
    ok = ok && hipMemset(c->cent_b, 0, cent_bytes) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->mean_b, cells * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->size_b, (size_t)c->capacity * sizeof(int)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->invn_b, ((size_t)c->capacity + SISO_PAD_ROWS) * sizeof(float)) == hipSuccess;
    ok = ok && hipMemset(c->invn_b, 0, ((size_t)c->capacity + SISO_PAD_ROWS) * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->locality_b, (size_t)c->capacity * sizeof(float)) == hipSuccess;
    ok = ok && take_with_versions(c, (void **)&c->access_b, (size_t)c->capacity, &c->version_b, 0x81);
    ok = ok && hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (c->cent_b) (void)hipFree(c->cent_b);
        if (c->mean_b) (void)hipFree(c->mean_b);
        if (c->size_b) (void)hipFree(c->size_b);
        if (c->invn_b) (void)hipFree(c->invn_b);
        if (c->locality_b) (void)hipFree(c->locality_b);
        if (c->access_b) (void)hipFree(c->access_b);
        c->version_b = nullptr;
        c->cent_b = nullptr;
        c->mean_b = nullptr;
        c->size_b = nullptr;
        c->invn_b = nullptr;
        c->locality_b = nullptr;
        c->access_b = nullptr;
        return siso_fail(c, SISO_ENOMEM, "second set of arrays for %ld centroids", c->capacity);
    }
    return SISO_OK;
}

// Work already enqueued keeps the pointers it was launched with; work enqueued from now on sees the new set.
void siso_swap_sets(siso_cache *c) {
    std::swap(c->cent, c->cent_b);
    std::swap(c->mean, c->mean_b);
    std::swap(c->size, c->size_b);
    std::swap(c->invn, c->invn_b);
    std::swap(c->locality, c->locality_b);
    std::swap(c->access, c->access_b);
    std::swap(c->version, c->version_b);
    siso_bytes_all_behind(c);
}

extern "C" int siso_create_ex(int dim, long capacity, int dtype, siso_cache **out) {
    if (!out) return SISO_EINVAL;
    *out = nullptr;
    if (dim < 1 || dim > SISO_MAX_DIM || capacity < 1 || capacity > 2147483647L ||
        (dtype != SISO_F32 && dtype != SISO_BF16 && dtype != SISO_FP8))
        return SISO_EINVAL;
    if (dtype == SISO_FP8 && (dim % 128 != 0 || dim < 256)) return SISO_EINVAL;  // slabs of 128 codes, two per tile
    siso_cache *c = new (std::nothrow) siso_cache();
    if (!c) return SISO_ENOMEM;
    memset(c, 0, sizeof(*c));
    c->opt_fold_spin_limit = -1;
    c->dim = dim;
    c->capacity = capacity;
    c->dtype = dtype;
    c->path = SISO_PATH_AUTO;
    const size_t cells = (size_t)capacity * dim;
    bool ok = hipGetDevice(&c->device) == hipSuccess;
    ok = ok && resolve_scratch(c->device, &c->static_keys) == SISO_OK;
    // The stored centroids carry SISO_PAD_ROWS readable rows past the capacity, so that the
    // tiled kernels may load a whole last tile; their results are discarded.
    const size_t cent_bytes = (cells + (size_t)SISO_PAD_ROWS * dim) * elem_bytes(dtype);
    ok = ok && hipMalloc(&c->cent, cent_bytes) == hipSuccess;
    ok = ok && hipMemset(c->cent, 0, cent_bytes) == hipSuccess;
    if (dtype == SISO_FP8) ok = ok && hipMalloc((void **)&c->scale, (size_t)capacity * sizeof(float)) == hipSuccess;
    else ok = ok && hipMalloc((void **)&c->mean, cells * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->size, (size_t)capacity * sizeof(int)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->invn, ((size_t)capacity + SISO_PAD_ROWS) * sizeof(float)) == hipSuccess;
    ok = ok && hipMemset(c->invn, 0, ((size_t)capacity + SISO_PAD_ROWS) * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->locality, (size_t)capacity * sizeof(float)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->access, (size_t)capacity * sizeof(unsigned)) == hipSuccess;
    // (behind the four counters: the board of siso_lookup_update, one slot per query of a small batch)
    ok = ok && take_with_versions(c, (void **)&c->counters, (4 + SISO_FOLD_BOARD) * 2, &c->version, 0x01);
    ok = ok && hipHostMalloc((void **)&c->host_pin, 4 * sizeof(u64), hipHostMallocDefault) == hipSuccess;
    ok = ok && hipMemset(c->counters, 0, (4 + SISO_FOLD_BOARD) * sizeof(u64)) == hipSuccess;
    ok = ok && hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        siso_destroy(c);
        return SISO_ENOMEM;
    }
    *out = c;
    return SISO_OK;
}

extern "C" int siso_create(int dim, long capacity, siso_cache **out) {
    return siso_create_ex(dim, capacity, SISO_BF16, out);
}

extern "C" void siso_destroy(siso_cache *c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    if (c->cent) (void)hipFree(c->cent);
    if (c->mean) (void)hipFree(c->mean);
    if (c->size) (void)hipFree(c->size);
    if (c->invn) (void)hipFree(c->invn);
    if (c->locality) (void)hipFree(c->locality);
    if (c->upd_owner) (void)hipFree(c->upd_owner);
    if (c->upd_members) (void)hipFree(c->upd_members);
    if (c->access) (void)hipFree(c->access);
    if (c->cent_b) (void)hipFree(c->cent_b);
    if (c->mean_b) (void)hipFree(c->mean_b);
    if (c->size_b) (void)hipFree(c->size_b);
    if (c->invn_b) (void)hipFree(c->invn_b);
    if (c->locality_b) (void)hipFree(c->locality_b);
    if (c->access_b) (void)hipFree(c->access_b);
    if (c->keys) (void)hipFree(c->keys);
    if (c->scale) (void)hipFree(c->scale);
    if (c->fp8_q) (void)hipFree(c->fp8_q);
    if (c->fp8_qinv) (void)hipFree(c->fp8_qinv);
    if (c->topk_groups) (void)hipFree(c->topk_groups);
    if (c->topk_tau) (void)hipFree(c->topk_tau);
    if (c->topk_cnt) (void)hipFree(c->topk_cnt);
    if (c->topk_cand) (void)hipFree(c->topk_cand);
    if (c->arena) (void)hipFree(c->arena);
    siso_screen_release(c);
    if (c->pinned) (void)hipHostFree(c->pinned);
    siso_refresh_release(c);
    if (c->counters) (void)hipFree(c->counters);
    if (c->host_pin) (void)hipHostFree(c->host_pin);
    if (c->prof_ev) {
        for (int i = 0; i < 2 * SISO_PROF_MAX; ++i)
            if (c->prof_ev[i]) (void)hipEventDestroy(c->prof_ev[i]);
        free(c->prof_ev);
    }
    delete c;
}

extern "C" int siso_set_stream(siso_cache *c, void *hip_stream) {
    if (!c) return SISO_EINVAL;
    c->stream = (hipStream_t)hip_stream;
    c->units = 0;
    return SISO_OK;
}

extern "C" int siso_set_lookup_path(siso_cache *c, int path) {
    if (!c) return SISO_EINVAL;
    if (c->dtype == SISO_FP8 && path == SISO_PATH_SCALAR) return siso_fail(c, SISO_EINVAL, "the 8-bit storage has no scalar kernel");
    if (path < SISO_PATH_AUTO || path > SISO_PATH_SKINNY) return siso_fail(c, SISO_EINVAL, "unknown lookup path %d", path);
    c->path = path;
    return SISO_OK;
}

extern "C" int siso_set_option(siso_cache *c, const char *name, long value) {
    if (!c || !name) return SISO_EINVAL;
    if (!strcmp(name, "fold_spin_limit") && value == -1) {
        c->opt_fold_spin_limit = -1;
        return SISO_OK;
    }
    if (value < 0 || value > 1000000) return siso_fail(c, SISO_EINVAL, "option %s: value %ld out of range", name, value);
    if (!strcmp(name, "mfma_config")) c->opt_mfma_config = (int)value;
    else if (!strcmp(name, "tiles_per_slice")) c->opt_tiles_per_slice = (int)value;
    else if (!strcmp(name, "merge_config")) c->opt_merge_config = (int)value;
    else if (!strcmp(name, "screen") && value <= 4) c->opt_screen = (int)value;
    else if (!strcmp(name, "screen_room")) c->opt_screen_room = (int)value;
    else if (!strcmp(name, "mfma_qblock")) c->opt_mfma_qblock = (int)value;
    else if (!strcmp(name, "fold_spin_limit")) c->opt_fold_spin_limit = (int)value;
    else if (!strcmp(name, "fold_units")) c->opt_fold_units = (int)value;
    else if (!strcmp(name, "topk_room")) c->opt_topk_room = (int)value;
    else if (!strcmp(name, "stream_hint") && value <= 2) c->opt_stream_hint = (int)value;
    else if (!strcmp(name, "second_set")) return value ? siso_second_set(c) : SISO_OK;
    else return siso_fail(c, SISO_EINVAL, "unknown option %s", name);
    return SISO_OK;
}

extern "C" long siso_count(const siso_cache *c) { return c ? c->count : (long)SISO_EINVAL; }

extern "C" const char *siso_last_error(const siso_cache *c) { return c ? c->err : "null cache"; }

__global__ void k_fill_nan(float *p, int count);

extern "C" int siso_load(siso_cache *c, const void *centroids, const int *counts, long k) {
    if (!c) return SISO_EINVAL;
    if (k < 0 || (k > 0 && !centroids)) return siso_fail(c, SISO_EINVAL, "siso_load: bad arguments");
    if (k > c->capacity) return siso_fail(c, SISO_ECAPACITY, "siso_load: %ld rows exceed capacity %ld", k, c->capacity);
    if (c->dtype == SISO_FP8) {
        const int rc = siso_fp8_load(c, centroids, counts, k);
        if (rc != SISO_OK) return rc;
    } else if (k > 0) {
        const dim3 grid((unsigned)((k + 3) / 4));
        const int vec = (c->dim * elem_bytes(c->dtype)) % 16 == 0 && ((uintptr_t)centroids & 15) == 0 ? 1 : 0;
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_load_rows<float>, grid, dim3(256), 0, c->stream, (const float *)centroids, counts,
                               (float *)c->cent, c->mean, c->size, c->invn, c->locality, c->access, c->version, k, c->dim, vec);
        else
            hipLaunchKernelGGL(k_load_rows<bf16_t>, grid, dim3(256), 0, c->stream, (const bf16_t *)centroids, counts,
                               (bf16_t *)c->cent, c->mean, c->size, c->invn, c->locality, c->access, c->version, k, c->dim, vec);
        HIP_TRY(c, hipGetLastError());
    }
    hipLaunchKernelGGL(k_fill_nan, dim3(1), dim3(SISO_PAD_ROWS), 0, c->stream, c->invn + k, SISO_PAD_ROWS);
    HIP_TRY(c, hipGetLastError());
    c->count = k;
    siso_bytes_all_behind(c);
    return SISO_OK;
}

extern "C" int siso_import(siso_cache *c, const void *centroids, const float *means, const int *counts,
                           const float *cluster_size, const unsigned *access_count, long k) {
    if (!c) return SISO_EINVAL;
    if (k < 0 || (k > 0 && (!centroids || !means || !counts))) return siso_fail(c, SISO_EINVAL, "siso_import: bad arguments");
    SISO_NOT_FP8(c, "siso_import");
    if (k > c->capacity) return siso_fail(c, SISO_ECAPACITY, "siso_import: %ld rows exceed capacity %ld", k, c->capacity);
    if (k > 0) {
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_import_rows<float>, dim3((unsigned)k), dim3(256), 0, c->stream, (const float *)centroids,
                               means, counts, cluster_size, access_count, (float *)c->cent, c->mean, c->size, c->invn,
                               c->locality, c->access, c->version, c->dim);
        else
            hipLaunchKernelGGL(k_import_rows<bf16_t>, dim3((unsigned)k), dim3(256), 0, c->stream, (const bf16_t *)centroids,
                               means, counts, cluster_size, access_count, (bf16_t *)c->cent, c->mean, c->size, c->invn,
                               c->locality, c->access, c->version, c->dim);
        HIP_TRY(c, hipGetLastError());
    }
    hipLaunchKernelGGL(k_fill_nan, dim3(1), dim3(SISO_PAD_ROWS), 0, c->stream, c->invn + k, SISO_PAD_ROWS);
    HIP_TRY(c, hipGetLastError());
    c->count = k;
    siso_bytes_all_behind(c);
    return SISO_OK;
}

// left: for what a screened lookup leaves over (k_lookup_few does not know how many queries that are)
static int choose_path(const siso_cache *c, long n, bool left = false) {
    if (c->path != SISO_PATH_AUTO) return c->path;
    if (!left && siso_few_slices(c, n) > 0) return SISO_PATH_FEW;
    if (siso_tile_preferred(c, n)) return SISO_PATH_SCALAR;
    if (n <= 64 && siso_skinny_slices(c, n) > 0) return SISO_PATH_SKINNY;
    if (siso_mfma_slices(c, n) > 0) return SISO_PATH_MFMA;
    return SISO_PATH_SCALAR;
}

extern "C" int siso_lookup_static(siso_cache *c, const void *queries, long n, float threshold, int *out_idx,
                                  float *out_sim, unsigned char *out_hit) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || (n > 0 && (!queries || !out_idx || !out_sim)))
        return siso_fail(c, SISO_EINVAL, "siso_lookup_static: bad arguments");
    // (an 8-bit cache quantises the batch into a workspace that siso_reserve sizes: this call does not grow it)
    if (c->dtype == SISO_FP8 && n > c->fp8_q_cap)
        return siso_fail(c, SISO_ECAPACITY, "siso_lookup_static: room for the codes of %ld queries, %ld asked for (siso_reserve sizes it)",
                         c->fp8_q_cap, n);
    if (!c->static_keys) return siso_fail(c, SISO_EHIP, "siso_lookup_static: the static workspace was not found on device %d", c->device);
    return siso_lookup_impl(c, queries, n, &threshold, 1, 0, out_idx, out_sim, out_hit, c->static_keys, SISO_STATIC_KEYS);
}

// keys a lookup of n queries writes in its first phase, for the kernel the library would choose
static long keys_needed(const siso_cache *c, long n) {
    if (n < 1 || c->count < 1) return n > 0 ? n : 0;
    int slices = 0;
    switch (choose_path(c, n)) {
        case SISO_PATH_SCALAR: slices = siso_tile_slices(c, n); break;
        case SISO_PATH_MFMA: slices = siso_mfma_slices(c, n); break;
        case SISO_PATH_SKINNY: slices = siso_skinny_slices(c, n); break;
        case SISO_PATH_FEW: slices = siso_few_slices(c, n); break;
    }
    return slices > 0 ? n * (long)slices : 0;
}

static int ensure_update_notes(siso_cache *c) {
    if (c->upd_owner) return SISO_OK;
    bool ok = hipMalloc((void **)&c->upd_owner, (size_t)c->capacity * sizeof(int)) == hipSuccess;
    ok = ok && hipMalloc((void **)&c->upd_members, (size_t)c->capacity * sizeof(int)) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (c->upd_owner) (void)hipFree(c->upd_owner);
        c->upd_owner = nullptr;
        return siso_fail(c, SISO_ENOMEM, "siso_update: notes for %ld centroids", c->capacity);
    }
    hipLaunchKernelGGL(k_update_mark_init, dim3((unsigned)((c->capacity + 255) / 256)), dim3(256), 0, c->stream,
                       c->upd_owner, c->upd_members, c->capacity);
    return siso_check_hip(c, hipGetLastError(), "k_update_mark_init");
}

extern "C" int siso_reserve(siso_cache *c, long n) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || n > 2147483647L / 4) return siso_fail(c, SISO_EINVAL, "siso_reserve: bad batch size %ld", n);
    if (n == 0) return SISO_OK;
    // The number of keys per query depends on the batch size only through the number of query tiles (64 rows
    // is the smallest tile of any kernel) and on the number of centroids: take the largest need over all batch
    // sizes up to n, for the cache as full as it is now and for a full cache.
    long need = 0;
    siso_cache full = *c;
    full.count = c->capacity;
    for (long m = 64;; m += 64) {
        const long b = m < n ? m : n;
        const long a = keys_needed(c, b), f = keys_needed(&full, b);
        need = a > need ? a : need;
        need = f > need ? f : need;
        const long t = siso_tile_keys_bound(c, b);
        need = t > need ? t : need;
        if (b == n) break;
    }
    if (need > c->keys_cap) {
        const int rc = ensure_workspace(c, need, 1);
        if (rc != SISO_OK) return rc;
    }
    if (c->dtype == SISO_FP8) return siso_fp8_ensure_batch(c, n);
    // (no room for the bytes of a screened lookup is no error: such lookups then go without)
    if (siso_screen_wanted(&full, n)) siso_screen_reserve(c, n);
    siso_bytes_few_reserve(c, n);
    if (n > 256) return ensure_update_notes(c);
    return SISO_OK;
}

extern "C" int siso_lookup(siso_cache *c, const void *queries, long n, float threshold, int *out_idx, float *out_sim,
                           unsigned char *out_hit) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || (n > 0 && (!queries || !out_idx || !out_sim)))
        return siso_fail(c, SISO_EINVAL, "siso_lookup: bad arguments");
    return siso_lookup_impl(c, queries, n, &threshold, 1, 0, out_idx, out_sim, out_hit);
}

extern "C" int siso_lookup_multi(siso_cache *c, const void *queries, long n, const float *thetas, int m, int count_index,
                                 int *out_idx, float *out_sim, unsigned char *out_hit) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || m < 1 || m > SISO_MULTI_MAX || !thetas || count_index < -1 || count_index >= m ||
        (n > 0 && (!queries || !out_idx || !out_sim || !out_hit)))
        return siso_fail(c, SISO_EINVAL, "siso_lookup_multi: bad arguments (1 to %d thresholds)", SISO_MULTI_MAX);
    return siso_lookup_impl(c, queries, n, thetas, m, count_index, out_idx, out_sim, out_hit);
}

// A lookup on the kernels that form every product in the cache's own type.  Its plan: which of them, with how many slices, and
// where the keys go.
struct PlainLookup {
    int path, slices;
    u64 *keys;
};
// left: for what a screened lookup leaves over
static int plan_plain(siso_cache *c, long n, u64 *static_keys, long static_cap, bool left, PlainLookup *p) {
    int slices = 1;
    const int path = c->count > 0 ? choose_path(c, n, left) : SISO_PATH_SCALAR;
    if (c->dtype == SISO_FP8 && c->count > 0 && path == SISO_PATH_SCALAR && !siso_tile_preferred(c, n))
        return siso_fail(c, SISO_EINVAL, "siso_lookup: the 8-bit storage has no scalar kernel");
    if (c->count > 0) {
        switch (path) {
            case SISO_PATH_SCALAR: slices = siso_tile_slices(c, n, left); break;
            case SISO_PATH_MFMA: slices = siso_mfma_slices(c, n); break;
            case SISO_PATH_SKINNY: slices = siso_skinny_slices(c, n); break;
            case SISO_PATH_FEW: slices = siso_few_slices(c, n); break;
        }
        if (slices <= 0)
            return siso_fail(c, SISO_EINVAL, "siso_lookup: path %d cannot serve dim %d, type %d, batch %ld", path,
                             c->dim, c->dtype, n);
    }
    if (static_keys) {
        if (n * (long)slices > static_cap)
            return siso_fail(c, SISO_ECAPACITY,
                             "siso_lookup_static: %ld queries x %d slices of the centroids need %ld keys, the static "
                             "workspace holds %ld", n, slices, n * (long)slices, static_cap);
    } else {
        const int rc = ensure_workspace(c, n, slices);
        if (rc != SISO_OK) return rc;
    }
    *p = PlainLookup{path, slices, static_keys ? static_keys : c->keys};
    return SISO_OK;
}

// `timed`: a kernel of siso_profile_enable.  folded: see siso_lookup_impl.  owner, members: the notes of an update to be taken,
// or NULL.  left: the queries that a screened lookup has left over (NULL: all are looked up).
static int plain_lookup(siso_cache *c, const PlainLookup &plan, const void *queries, long n, const ThetaList &tl, long q_base,
                        int *out_idx, float *out_sim, unsigned char *out_hit, bool timed, int *folded, int *owner, int *members,
                        const ScreenPlain *left, bool screen) {
    const int path = plan.path, slices = plan.slices, m = tl.m, count_index = tl.count_at;
    const bool fp8 = c->dtype == SISO_FP8;
    const int *many = left ? left->many : nullptr, *of = left ? left->query : nullptr;
    int rc = SISO_OK;
    u64 *keys = plan.keys;
    const void *kernel_queries = queries;
    if (fp8) {  // the batch as codes, quantised like the stored rows
        rc = siso_fp8_ensure_batch(c, n);
        if (rc == SISO_OK) rc = siso_fp8_quantize_batch(c, queries, n);
        if (rc != SISO_OK) return rc;
        kernel_queries = c->fp8_q;
    }
    const unsigned qblocks = (unsigned)n;
    // (left-over rows are gathered, and aligned whatever the batch is: they are summed as the rest of their batch is)
    const int vec = left ? left->vec : ((c->dim * elem_bytes(c->dtype)) % 16 == 0 && ((uintptr_t)queries & 15) == 0) ? 1 : 0;
    int row_keys = SISO_KEY_ROWS;  // what the keys of the chosen kernel carry: the winning row, or its group of four rows
    // (the similarities of a batch are the same bits whether it is screened, as it would be with enough memory, or not: then
    // they are formed anew, which the kernel that ends a lookup together with its update does not do)
    const bool anew = left || screen;
    const bool may_fold = folded && !anew && n <= SISO_FOLD_BOARD && c->count > 0 && (!fp8 || c->fold_master) && m == 1 && out_hit;
    c->board_to_clear = may_fold ? c->counters + 4 : nullptr;
    if (c->count > 0) {
        if (timed) siso_prof_begin(c);
        switch (path) {
            case SISO_PATH_SCALAR: rc = siso_tile_launch(c, kernel_queries, n, slices, keys, many); break;
            case SISO_PATH_MFMA: rc = siso_mfma_launch(c, kernel_queries, n, slices, keys, &row_keys, many); break;
            case SISO_PATH_SKINNY: rc = siso_skinny_launch(c, kernel_queries, n, slices, keys, &row_keys); break;
            case SISO_PATH_FEW: rc = siso_few_launch(c, kernel_queries, n, slices, keys); break;
        }
        if (timed) siso_prof_end(c);
        if (rc != SISO_OK) {
            c->board_to_clear = nullptr;
            return rc;
        }
    }
    // (a kernel that empties the board takes the pointer; one that does not know of it leaves it)
    const bool board_emptied = may_fold && c->board_to_clear == nullptr;
    c->board_to_clear = nullptr;
    if (board_emptied && row_keys == SISO_KEY_ROWS) {
        const siso_cache *ms = c->fold_master;  // the bf16 cache behind an 8-bit copy, or NULL
        siso_cache *tgt = ms ? const_cast<siso_cache *>(ms) : c;
        // Bytes (rows of up to 1,024 elements) follow where small lookups go over them, if they are current, or nearly so.  Otherwise they are left behind, as
        // those of fp32 rows are: the screened lookups that these serve write changed rows anew in any case, and to follow takes 2 to 3 % of a step (of 64
        // queries against 60,000 x 384 41.3 us without bytes, 41.6 so, 42.2 following).
        ByteView bytes = tgt->dtype == SISO_BF16 && tgt->bytes.behind == 0 ? siso_byte_view(tgt) : ByteView{nullptr, nullptr, nullptr, 0};
        if (bytes.codes && !siso_bytes_may_record(tgt)) bytes.codes = nullptr;
        unsigned *const version = c->dim <= SISO_SCREEN_DIM ? siso_counted(tgt) : nullptr;
        // the end of the lookup and the update of its hits as one kernel (see k_finalize_update)
        // polls of the board (a microsecond or two each) before a block gives up
        const int spin_limit = c->opt_fold_spin_limit >= 0 ? c->opt_fold_spin_limit : 1 << 18;
#define SISO_LAUNCH_FOLD(T, E, MORE, ...)                                                                                 \
    hipLaunchKernelGGL((k_finalize_update<T, E, MORE>), dim3(qblocks), dim3(256), 0, c->stream, (const T *)queries, keys, n, c->count, \
                       c->dim, slices, tl.v[0], vec, out_idx, out_sim, out_hit, count_index >= 0 ? c->access : nullptr, \
                       (T *)tgt->cent, tgt->mean, tgt->size, tgt->invn, c->counters + 4, spin_limit, c->counters,         \
                       ms ? (const float *)c->fp8_qinv : (const float *)nullptr, ms ? (unsigned char *)c->cent : nullptr, \
                       ms ? c->scale : nullptr, ms ? c->invn : nullptr, ms ? c->size : nullptr, MORE{__VA_ARGS__})
        if (tgt->dtype == SISO_F32) {
            if (c->dim > 1024) SISO_LAUNCH_FOLD(float, 16, FoldPlain);
            else if (version) SISO_LAUNCH_FOLD(float, 4, FoldCounted, version);
            else SISO_LAUNCH_FOLD(float, 4, FoldPlain);
        } else {
            if (c->dim > 1024) SISO_LAUNCH_FOLD(bf16_t, 16, FoldPlain);
            else if (bytes.codes) SISO_LAUNCH_FOLD(bf16_t, 4, FoldBytes, tgt->version, bytes);
            else if (version) SISO_LAUNCH_FOLD(bf16_t, 4, FoldCounted, version);
            else SISO_LAUNCH_FOLD(bf16_t, 4, FoldPlain);
        }
#undef SISO_LAUNCH_FOLD
        HIP_TRY(c, hipGetLastError());
        *folded = 1;
        return SISO_OK;
    }
    if (row_keys == SISO_KEY_ROWS && anew) row_keys = SISO_KEY_ROWS_ANEW;
#define SISO_LAUNCH_FINALIZE(T, LEFT)                                                                                        \
    hipLaunchKernelGGL((k_lookup_finalize<T, LEFT>), dim3(qblocks), dim3(256), 0, c->stream, (const T *)queries, (const T *)c->cent, c->invn, \
                       keys, n, c->count, c->dim, slices, tl, vec, row_keys, out_idx, out_sim, out_hit,                        \
                       count_index >= 0 ? c->access : nullptr, fp8 ? (const float *)c->fp8_qinv : (const float *)nullptr, owner, \
                       members, many, of, q_base)
    if (c->dtype == SISO_F32) {
        if (left) SISO_LAUNCH_FINALIZE(float, true);
        else SISO_LAUNCH_FINALIZE(float, false);
    } else {
        if (left) SISO_LAUNCH_FINALIZE(bf16_t, true);
        else SISO_LAUNCH_FINALIZE(bf16_t, false);
    }
#undef SISO_LAUNCH_FINALIZE
    return siso_check_hip(c, hipGetLastError(), "k_lookup_finalize");
}

// Compute units that the cache's stream may use: of a partitioned chip, or of a stream with a mask, fewer than 256.
static int stream_units(siso_cache *c) {
    if (c->units > 0) return c->units;
    int units = 0;
    if (hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) units = 0;
    unsigned mask[16] = {0};
    int masked = 0;
    if (hipExtStreamGetCUMask(c->stream, 16, mask) == hipSuccess)
        for (const unsigned m : mask) masked += __builtin_popcount(m);
    (void)hipGetLastError();
    if (masked > 0 && masked < units) units = masked;
    c->units = units > 0 ? units : 1;
    return c->units;
}

// Few queries over the bytes of the rows: two kernels, the second of which folds the hits if the caller is about to.  Its workgroups wait for
// each other, so it does that only where all of them fit on the chip at once, with the LDS that the gathered rows take (up to 146 KB: a compute
// unit each); otherwise the caller's update does.
static int few_lookup(siso_cache *c, const void *queries, long n, float theta, int count_index, int *out_idx, float *out_sim,
                      unsigned char *out_hit, int *folded) {
    const int units = c->opt_fold_units > 0 ? c->opt_fold_units : stream_units(c);
    const bool fold = folded && out_hit && n <= (long)units * ((160 * 1024) / (LISTED_LDS(c->dim) + LISTED_STATIC));
    const ByteView bytes = siso_byte_view(c);
    c->board_to_clear = fold ? c->counters + 4 : nullptr;
    siso_prof_begin(c);
    const int rc = siso_bytes_few_launch(c, queries, n, bytes);
    siso_prof_end(c);
    c->board_to_clear = nullptr;
    if (rc != SISO_OK) return rc;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_TRY(c, hipFuncSetAttribute((const void *)k_finalize_update<bf16_t, 4, FoldListed>, hipFuncAttributeMaxDynamicSharedMemorySize, LISTED_LDS(SISO_SCREEN_DIM)));
        attr_done = true;
    }
    hipLaunchKernelGGL((k_finalize_update<bf16_t, 4, FoldListed>), dim3((unsigned)n), dim3(256), LISTED_LDS(c->dim), c->stream, (const bf16_t *)queries, (const u64 *)nullptr, n,
                       c->count, c->dim, siso_bytes_few_workgroups(c), theta, 1, out_idx, out_sim, out_hit, count_index >= 0 ? c->access : nullptr,
                       (bf16_t *)c->cent, c->mean, c->size, c->invn, c->counters + 4,
                       c->opt_fold_spin_limit >= 0 ? c->opt_fold_spin_limit : 1 << 18, c->counters, (const float *)nullptr, (unsigned char *)nullptr,
                       (float *)nullptr, (float *)nullptr, (int *)nullptr, FoldListed{c->version, bytes, c->few, fold ? 1 : 0, c->few_flooded});
    if (fold) *folded = 1;
    return siso_check_hip(c, hipGetLastError(), "k_finalize_update");
}

int siso_lookup_impl(siso_cache *c, const void *queries, long n, const float *thetas, int m, int count_index,
                     int *out_idx, float *out_sim, unsigned char *out_hit, u64 *static_keys, long static_cap, int *folded, float floor) {
    if (folded) *folded = 0;
    if (n == 0) return SISO_OK;
    if (n > 2147483647L / 4) return siso_fail(c, SISO_EINVAL, "siso_lookup: batch of %ld is too large", n);
    ThetaList tl;
    tl.m = m;
    tl.count_at = count_index;
    for (int j = 0; j < SISO_MULTI_MAX; ++j) tl.v[j] = j < m ? thetas[j] : 0.f;
    // the notes of the update that follows are taken by whatever ends the lookup
    int *owner = nullptr, *members = nullptr;
    if (c->mark_in_finalize == 1 && m == 1 && c->upd_owner != nullptr) {
        owner = c->upd_owner;
        members = c->upd_members;
    }
    if (!static_keys && m == 1 && siso_mfma_aligned(queries) && siso_bytes_few_wanted(c, n) && siso_bytes_few_room(c, n))
        return few_lookup(c, queries, n, thetas[0], count_index, out_idx, out_sim, out_hit, folded);
    PlainLookup plain;
    // (not on the static keys: the bytes live in a workspace that other calls share and a larger one moves)
    const bool screen = siso_screen_above_wanted(c, n, floor);
    if (!static_keys && screen && siso_screen_room(c, n)) {
        // piece by piece: screened, then what that has left over.  Pieces of as many tiles of 256 queries each: a short last one
        // would go through the kernels for few queries, which do not know how many of them there are.
        const size_t row = (size_t)c->dim * elem_bytes(c->dtype);
        const long tiles = (n + 255) / 256, pieces = (n + SISO_SCREEN_PIECE - 1) / SISO_SCREEN_PIECE;
        int rc = SISO_OK;
        long off = 0, part = 0;
        for (long p = 0; p < pieces && rc == SISO_OK; ++p, off += part) {
            part = 256 * (tiles / pieces + (p < tiles % pieces ? 1 : 0));
            if (part > n - off) part = n - off;
            const char *q = (const char *)queries + (size_t)off * row;
            unsigned char *hit = out_hit ? out_hit + (size_t)off * m : nullptr;
            ScreenPlain left;
            rc = plan_plain(c, part, nullptr, 0, true, &plain);
            if (rc != SISO_OK) break;
            // (the gathered rows of left-over queries are aligned: a batch that those kernels refuse is refused here)
            if (plain.path != SISO_PATH_SCALAR && !siso_mfma_aligned(queries)) return siso_fail(c, SISO_EINVAL, SISO_MFMA_UNALIGNED);
            if (owner) c->mark_in_finalize = 2;
            rc = siso_screen_lookup(c, q, part, off == 0, pieces == 1, tl, off, out_idx + off, out_sim + off, hit,
                                    count_index >= 0 ? c->access : nullptr, owner, members, &left, floor);
            if (rc == SISO_OK)
                rc = plain_lookup(c, plain, left.rows, part, tl, off, out_idx + off, out_sim + off, hit, false, nullptr, owner, members, &left, true);
        }
        return rc;
    }
    int rc = plan_plain(c, n, static_keys, static_cap, false, &plain);
    if (rc == SISO_OK)
        rc = plain_lookup(c, plain, queries, n, tl, 0, out_idx, out_sim, out_hit, !static_keys, folded, owner, members, nullptr, screen);
    if (rc == SISO_OK && owner && !(folded && *folded)) c->mark_in_finalize = 2;  // done
    return rc;
}

#define UPDATE_CHUNK 32768L

// premarked: the notes of this batch (one chunk) have been taken already, by the finalize step of its lookup
static int update_hits_impl(siso_cache *c, const void *queries, const int *idx, const unsigned char *hit, long n,
                            bool premarked) {
    if (!c) return SISO_EINVAL;
    SISO_NOT_FP8(c, "siso_update");
    if (n < 0 || (n > 0 && (!queries || !idx))) return siso_fail(c, SISO_EINVAL, "siso_update: bad arguments");
    // A running mean folds chunk after chunk to the same mean as one big batch,
    // so very large batches are cut to bound the member scan of each block.
    for (long off = 0; off < n; off += UPDATE_CHUNK) {
        const long m = (n - off < UPDATE_CHUNK) ? n - off : UPDATE_CHUNK;
        const unsigned char *h = hit ? hit + off : nullptr;
        const float *qf = (const float *)queries + (size_t)off * c->dim;
        const bf16_t *qh = (const bf16_t *)queries + (size_t)off * c->dim;
        const dim3 grid((unsigned)m), block(256);
        int *owner = nullptr, *marked = nullptr;
        if (m > 256) {
            const int rc = ensure_update_notes(c);
            if (rc != SISO_OK) return rc;
            owner = c->upd_owner;
            marked = c->upd_members;
            if (!premarked)
                hipLaunchKernelGGL(k_update_mark, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, c->stream, idx + off, h,
                                   m, c->count, owner, marked);
        }
#define SISO_LAUNCH_UPDATE(T, E, QP)                                                                            \
    hipLaunchKernelGGL((k_update<T, E>), grid, block, 0, c->stream, QP, idx + off, h, m, (T *)c->cent, c->mean, \
                       c->size, c->invn, c->version, c->count, c->dim, c->counters, owner, marked)
        if (c->dtype == SISO_F32) {
            if (c->dim <= 1024) SISO_LAUNCH_UPDATE(float, 4, qf);
            else SISO_LAUNCH_UPDATE(float, 16, qf);
        } else {
            if (c->dim <= 1024) SISO_LAUNCH_UPDATE(bf16_t, 4, qh);
            else SISO_LAUNCH_UPDATE(bf16_t, 16, qh);
        }
#undef SISO_LAUNCH_UPDATE
        HIP_TRY(c, hipGetLastError());
        siso_bytes_behind(c, m);
    }
    return SISO_OK;
}

extern "C" int siso_update_hits(siso_cache *c, const void *queries, const int *idx, const unsigned char *hit, long n) {
    return update_hits_impl(c, queries, idx, hit, n, false);
}

extern "C" int siso_fp8_lookup_update(siso_cache *copy, siso_cache *master, const void *queries, long n, float threshold,
                                      int *out_idx, float *out_sim, unsigned char *out_hit) {
    if (!copy) return SISO_EINVAL;
    if (!master || n < 0 || (n > 0 && (!queries || !out_idx || !out_sim || !out_hit)))
        return siso_fail(copy, SISO_EINVAL, "siso_fp8_lookup_update: bad arguments");
    if (copy->dtype != SISO_FP8 || master->dtype != SISO_BF16 || copy->dim != master->dim || copy->count != master->count)
        return siso_fail(copy, SISO_EINVAL, "siso_fp8_lookup_update: an 8-bit cache and a bf16 cache with the same centroids");
    if (copy->stream != master->stream)
        return siso_fail(copy, SISO_EINVAL, "siso_fp8_lookup_update: both caches must work on the same stream");
    if (n == 0) return SISO_OK;
    int folded = 0;
    copy->fold_master = master;
    const int rc = siso_lookup_impl(copy, queries, n, &threshold, 1, 0, out_idx, out_sim, out_hit, nullptr, 0, &folded);
    copy->fold_master = nullptr;
    if (rc != SISO_OK || folded) return rc;
    const int rc2 = siso_update_hits(master, queries, out_idx, out_hit, n);
    return rc2 != SISO_OK ? rc2 : siso_fp8_follow(copy, master, out_idx, out_hit, n);
}

extern "C" int siso_update(siso_cache *c, const void *queries, const int *idx, long n) {
    return siso_update_hits(c, queries, idx, nullptr, n);
}

extern "C" int siso_lookup_update(siso_cache *c, const void *queries, long n, float threshold, int *out_idx, float *out_sim,
                                  unsigned char *out_hit) {
    if (!c) return SISO_EINVAL;
    SISO_NOT_FP8(c, "siso_lookup_update");
    if (n < 0 || (n > 0 && (!queries || !out_idx || !out_sim || !out_hit)))
        return siso_fail(c, SISO_EINVAL, "siso_lookup_update: bad arguments");
    int folded = 0;
    // a large batch (one chunk of the update): the end of the lookup takes the update's notes itself
    c->mark_in_finalize = 0;
    if (n > 256 && n <= UPDATE_CHUNK && ensure_update_notes(c) == SISO_OK) c->mark_in_finalize = 1;
    const int rc = siso_lookup_impl(c, queries, n, &threshold, 1, 0, out_idx, out_sim, out_hit, nullptr, 0, &folded);
    const bool premarked = c->mark_in_finalize == 2;
    c->mark_in_finalize = 0;
    if (rc != SISO_OK || folded || n == 0) {
        if (premarked) {  // (a failure behind the notes: leave them as a fresh cache has them)
            hipLaunchKernelGGL(k_update_mark_init, dim3((unsigned)((c->capacity + 255) / 256)), dim3(256), 0, c->stream,
                               c->upd_owner, c->upd_members, c->capacity);
            (void)hipGetLastError();
        }
        return rc;
    }
    return update_hits_impl(c, queries, out_idx, out_hit, n, premarked);
}

int siso_read_counter(siso_cache *c, int which, u64 *value) {
    HIP_TRY(c, hipMemcpyAsync(c->host_pin, c->counters, 4 * sizeof(u64), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    *value = c->host_pin[which];
    return SISO_OK;
}

__global__ void k_zero_counter(u64 *p) { *p = 0; }

// The tiled kernels read the inverse lengths of a whole last tile; the entries just past the
// live centroids hold NaN so that those rows never win.
__global__ void k_fill_nan(float *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = __uint_as_float(0x7FC00000u);
}

extern "C" int siso_export_meta(siso_cache *c, float *cluster_size, unsigned *access_count) {
    if (!c) return SISO_EINVAL;
    if (c->count == 0) return SISO_OK;
    if (cluster_size)
        HIP_TRY(c, hipMemcpyAsync(cluster_size, c->locality, (size_t)c->count * sizeof(float), hipMemcpyDeviceToDevice, c->stream));
    if (access_count)
        HIP_TRY(c, hipMemcpyAsync(access_count, c->access, (size_t)c->count * sizeof(unsigned), hipMemcpyDeviceToDevice, c->stream));
    return SISO_OK;
}

extern "C" long siso_bad_indices(siso_cache *c) {
    if (!c) return SISO_EINVAL;
    u64 v = 0;
    const int rc = siso_read_counter(c, 0, &v);
    return rc != SISO_OK ? (long)rc : (long)v;
}

int siso_pairs_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                      u64 *counter) {
    PairsRedo redo = {nullptr, 0};
    if (siso_screen_pairs_wanted(c, count, threshold) && siso_screen_pairs_room(c, count)) {
        const int rc = siso_screen_pairs_launch(c, rows, invn, count, threshold, out_pairs, cap, counter, &redo);
        if (rc != SISO_OK) return rc;
    }
    return siso_pairs_mfma_supported(c, count) ? siso_pairs_mfma_launch(c, rows, invn, count, threshold, out_pairs, cap, counter, redo)
                                               : siso_pairs_tile_launch(c, rows, invn, count, threshold, out_pairs, cap, counter, redo);
}

extern "C" long siso_merge(siso_cache *c, float threshold, int *out_pairs, long cap) {
    if (!c) return SISO_EINVAL;
    SISO_NOT_FP8(c, "siso_merge");
    if (cap < 0 || (cap > 0 && !out_pairs)) return siso_fail(c, SISO_EINVAL, "siso_merge: bad arguments");
    if (c->count < 2) return 0;
    hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, c->stream, c->counters + 1);
    int rc = siso_check_hip(c, hipGetLastError(), "k_zero_counter");
    if (rc != SISO_OK) return rc;
    siso_prof_begin(c);
    rc = siso_pairs_launch(c, c->cent, c->invn, c->count, threshold, out_pairs, cap, c->counters + 1);
    siso_prof_end(c);
    if (rc != SISO_OK) return rc;
    u64 total = 0;
    rc = siso_read_counter(c, 1, &total);
    siso_screen_done(c);
    return rc != SISO_OK ? (long)rc : (long)total;
}

extern "C" int siso_merge_apply(siso_cache *c, const int *pairs, long n_pairs, int *out_survivor) {
    if (!c) return SISO_EINVAL;
    SISO_NOT_FP8(c, "siso_merge_apply");
    if (n_pairs < 0 || (n_pairs > 0 && !pairs)) return siso_fail(c, SISO_EINVAL, "siso_merge_apply: bad arguments");
    const long K = c->count;
    if (K == 0) return SISO_OK;
    const int d = c->dim;
    const unsigned pb = (unsigned)((n_pairs + 255) / 256), kb = (unsigned)((K + 255) / 256);
    const unsigned sb = (unsigned)((K + SCAN_ROWS - 1) / SCAN_ROWS);
    int *parent, *root, *newpos, *members_of, *cursor, *first, *list;
    unsigned char *touched;
    int2 *sums;
    auto layout = [&](Carver a) {
        parent = a.take<int>(K);
        root = a.take<int>(K);
        newpos = a.take<int>(K);
        members_of = a.take<int>(K);
        cursor = a.take<int>(K);
        first = a.take<int>(K);
        list = a.take<int>(K);
        touched = a.take<unsigned char>(K);
        sums = a.take<int2>(sb);
        return a.used;
    };
    int rc = siso_arena(c, layout(Carver{nullptr}), 0);
    if (rc != SISO_OK) return rc;
    layout(Carver{c->arena});
    long live = K;
    if (rc == SISO_OK) {
        hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, c->stream, c->counters + 2);
        hipLaunchKernelGGL(k_uf_init, dim3(kb), dim3(256), 0, c->stream, parent, touched, members_of, cursor, K);
        // (us of 50,000 rows, with and without: 1,000 pairs in groups of eight 104.8 / 103.0, 10,000 104.9 / 112.0, in groups of three 106.5 / 105.5,
        // 60,000 127.4 / 132.6; of 5,000 rows 10,000 in groups of 32 95.4 / 111.3, 1,000 90.7 / 88.7)
        if (n_pairs >= 4096) hipLaunchKernelGGL(k_uf_first, dim3(pb), dim3(256), 0, c->stream, pairs, n_pairs, K, parent);
        if (n_pairs > 0)
            hipLaunchKernelGGL(k_uf_hook, dim3(pb), dim3(256), 0, c->stream, pairs, n_pairs, K, parent, touched, c->counters + 2);
        hipLaunchKernelGGL(k_uf_roots, dim3(kb), dim3(256), 0, c->stream, parent, touched, root, members_of, K);
        hipLaunchKernelGGL(k_scan_sums, dim3(sb), dim3(1024), 0, c->stream, members_of, root, K, sums);
        hipLaunchKernelGGL(k_scan_exclusive, dim3(sb), dim3(1024), 0, c->stream, members_of, root, K, sums, first, newpos,
                           c->counters + 3);
        hipLaunchKernelGGL(k_group_fill, dim3(kb), dim3(256), 0, c->stream, root, touched, K, first, cursor, list);
        rc = siso_check_hip(c, hipGetLastError(), "merge_apply kernels");
        u64 bad = 0;
        if (rc == SISO_OK) rc = siso_read_counter(c, 2, &bad);  // (all four counters come at once)
        live = (long)c->host_pin[3];
        if (rc == SISO_OK && bad != 0) rc = siso_fail(c, SISO_EINVAL, "siso_merge_apply: %llu invalid pairs", bad);
        // every valid pair joins two rows, so the survivors will be gathered into the second set of arrays: make
        // sure it exists before anything is changed in place (a failure here leaves the cache as it was)
        if (rc == SISO_OK && n_pairs > 0) rc = siso_second_set(c);
    }
    if (rc == SISO_OK && n_pairs > 0) {
        const int per = K <= 16384 ? 1 : K <= 65536 ? 4 : 16;
        const dim3 grid((unsigned)((K + per - 1) / per)), block(256);
#define SISO_LAUNCH_MEAN(T, E)                                                                                           \
    hipLaunchKernelGGL((k_group_mean<T, E>), grid, block, 0, c->stream, root, touched, K, members_of, first, list, (T *)c->cent, \
                       c->mean, c->size, c->invn, c->locality, c->access, c->version, d, per)
        if (c->dtype == SISO_F32) {
            if (d <= 1024) SISO_LAUNCH_MEAN(float, 4);
            else SISO_LAUNCH_MEAN(float, 16);
        } else {
            if (d <= 1024) SISO_LAUNCH_MEAN(bf16_t, 4);
            else SISO_LAUNCH_MEAN(bf16_t, 16);
        }
#undef SISO_LAUNCH_MEAN
        rc = siso_check_hip(c, hipGetLastError(), "k_group_mean");
    }
    if (rc == SISO_OK && out_survivor) {
        hipLaunchKernelGGL(k_survivor_map, dim3(kb), dim3(256), 0, c->stream, root, newpos, K, out_survivor);
        rc = siso_check_hip(c, hipGetLastError(), "k_survivor_map");
    }
    if (rc == SISO_OK && live < K) {
        // survivors packed to the front of the second set, which then becomes the cache
        if (c->dtype == SISO_F32)
            hipLaunchKernelGGL(k_gather_rows<float>, dim3((unsigned)K), dim3(256), 0, c->stream, root, newpos,
                               (const float *)c->cent, c->mean, c->size, c->invn, c->locality, c->access,
                               (float *)c->cent_b, c->mean_b, c->size_b, c->invn_b, c->locality_b, c->access_b, c->version_b, d);
        else
            hipLaunchKernelGGL(k_gather_rows<bf16_t>, dim3((unsigned)K), dim3(256), 0, c->stream, root, newpos,
                               (const bf16_t *)c->cent, c->mean, c->size, c->invn, c->locality, c->access,
                               (bf16_t *)c->cent_b, c->mean_b, c->size_b, c->invn_b, c->locality_b, c->access_b, c->version_b, d);
        rc = siso_check_hip(c, hipGetLastError(), "k_gather_rows");
        if (rc == SISO_OK) siso_swap_sets(c);
    }
    if (rc == SISO_OK) {
        hipLaunchKernelGGL(k_fill_nan, dim3(1), dim3(SISO_PAD_ROWS), 0, c->stream, c->invn + live, SISO_PAD_ROWS);
        rc = siso_check_hip(c, hipGetLastError(), "k_fill_nan");
    }
    (void)hipStreamSynchronize(c->stream);
    if (rc == SISO_OK) c->count = live;
    siso_arena_done(c);
    return rc;
}

extern "C" int siso_profile_enable(siso_cache *c, int on) {
    if (!c) return SISO_EINVAL;
    if (on < 0) return siso_fail(c, SISO_EINVAL, "siso_profile_enable: negative period");
    c->profile_on = on;
    c->prof_calls = 0;
    if (on > 0) {
        // A pair of events with nothing between them already measures some microseconds: the smallest of
        // a few such readings is taken off every bracket, so that short kernels are not overstated.
        hipEvent_t e[2] = {nullptr, nullptr};
        double least = -1.0;
        if (hipEventCreate(&e[0]) == hipSuccess && hipEventCreate(&e[1]) == hipSuccess) {
            for (int i = 0; i < 12; ++i) {
                float ms = 0.f;
                if (hipEventRecord(e[0], c->stream) != hipSuccess || hipEventRecord(e[1], c->stream) != hipSuccess) break;
                if (hipStreamSynchronize(c->stream) != hipSuccess) break;
                if (hipEventElapsedTime(&ms, e[0], e[1]) != hipSuccess) break;
                if (least < 0.0 || ms < least) least = ms;
            }
        }
        if (e[0]) (void)hipEventDestroy(e[0]);
        if (e[1]) (void)hipEventDestroy(e[1]);
        (void)hipGetLastError();
        c->prof_empty_ms = least > 0.0 ? least : 0.0;
    }
    return SISO_OK;
}

extern "C" int siso_profile_read(siso_cache *c, double *total_ms, long *launches) {
    if (!c) return SISO_EINVAL;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    double sum = 0.0;
    for (int i = 0; i < c->prof_count; ++i) {
        float ms = 0.f;
        hipEvent_t *e = c->prof_ev + 2 * i;
        if (hipEventElapsedTime(&ms, e[0], e[1]) == hipSuccess) sum += ms > c->prof_empty_ms ? ms - c->prof_empty_ms : 0.0;
        (void)hipEventDestroy(e[0]);
        (void)hipEventDestroy(e[1]);
        e[0] = e[1] = nullptr;
    }
    if (total_ms) *total_ms = sum;
    if (launches) *launches = c->prof_count;
    c->prof_count = 0;
    return SISO_OK;
}

extern "C" int siso_export(siso_cache *c, void *centroids, float *means, int *counts) {
    if (!c) return SISO_EINVAL;
    if (c->dtype == SISO_FP8 && means) return siso_fail(c, SISO_EINVAL, "siso_export: the 8-bit storage keeps no running means");
    const size_t cells = (size_t)c->count * c->dim;
    if (c->count == 0) return SISO_OK;
    if (centroids)
        HIP_TRY(c, hipMemcpyAsync(centroids, c->cent, cells * elem_bytes(c->dtype), hipMemcpyDeviceToDevice, c->stream));
    if (means) HIP_TRY(c, hipMemcpyAsync(means, c->mean, cells * sizeof(float), hipMemcpyDeviceToDevice, c->stream));
    if (counts)
        HIP_TRY(c, hipMemcpyAsync(counts, c->size, (size_t)c->count * sizeof(int), hipMemcpyDeviceToDevice, c->stream));
    return SISO_OK;
}

// ----------------------------------------------------------------------------
// Threshold-to-hit-ratio table and the SLO-aware choice of the retrieval threshold
// (section 4.3, "Adjusting theta_R to meet SLO")
// ----------------------------------------------------------------------------
#define SISO_T2H_MAX 1024

// hits[j] += number of queries of this block whose similarity exceeds thetas[j]
__global__ void k_t2h_count(const float *__restrict__ sim, long n, const float *__restrict__ thetas, int m,
                            u64 *__restrict__ hits) {
    __shared__ unsigned local[SISO_T2H_MAX];
    for (int j = threadIdx.x; j < m; j += blockDim.x) local[j] = 0;
    __syncthreads();
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const float s = i < n ? sim[i] : __uint_as_float(0x7FC00000u);  // NaN hits nothing
    for (int j = 0; j < m; ++j) {
        const u64 above = __ballot(s > thetas[j]);
        if ((threadIdx.x & 63) == 0 && above != 0) atomicAdd(&local[j], (unsigned)__popcll(above));
    }
    __syncthreads();
    for (int j = threadIdx.x; j < m; j += blockDim.x)
        if (local[j] != 0) atomicAdd(&hits[j], (u64)local[j]);
}

extern "C" int siso_t2h(siso_cache *c, const void *queries, long n, const float *thetas, int m, long *out_hits) {
    if (!c) return SISO_EINVAL;
    if (n < 0 || m < 0 || m > SISO_T2H_MAX || (m > 0 && (!thetas || !out_hits)) || (n > 0 && !queries))
        return siso_fail(c, SISO_EINVAL, "siso_t2h: bad arguments (at most %d thresholds)", SISO_T2H_MAX);
    for (int j = 0; j < m; ++j) out_hits[j] = 0;
    if (n == 0 || m == 0) return SISO_OK;
    // one lookup of the sample, then every threshold is a comparison against the same similarities
    int *idx;
    float *sim, *d_th;
    u64 *d_hits;
    auto layout = [&](Carver a) {
        idx = a.take<int>(n);
        sim = a.take<float>(n);
        d_th = a.take<float>(m);
        d_hits = a.take<u64>(m);
        return a.used;
    };
    int rc = siso_arena(c, layout(Carver{nullptr}), 0);
    if (rc != SISO_OK) return rc;
    layout(Carver{c->arena});
    hipError_t e = hipMemcpyAsync(d_th, thetas, (size_t)m * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(d_hits, 0, (size_t)m * sizeof(u64), c->stream);
    if (e != hipSuccess) rc = siso_check_hip(c, e, "siso_t2h: set-up");
    const float no_theta = 0.f;
    float floor = INFINITY;  // what does not exceed the lowest threshold is not told apart
    for (int j = 0; j < m; ++j) floor = thetas[j] < floor ? thetas[j] : floor;
    if (rc == SISO_OK)  // (test lookups are no references)
        rc = siso_lookup_impl(c, queries, n, &no_theta, 1, -1, idx, sim, nullptr, nullptr, 0, nullptr, floor);
    u64 host_hits[SISO_T2H_MAX];
    if (rc == SISO_OK) {
        hipLaunchKernelGGL(k_t2h_count, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, sim, n, d_th, m, d_hits);
        e = hipGetLastError();
        if (e == hipSuccess)
            e = hipMemcpyAsync(host_hits, d_hits, (size_t)m * sizeof(u64), hipMemcpyDeviceToHost, c->stream);
        if (e != hipSuccess) rc = siso_check_hip(c, e, "siso_t2h: count");
    }
    e = hipStreamSynchronize(c->stream);
    if (rc == SISO_OK && e != hipSuccess) rc = siso_check_hip(c, e, "siso_t2h: synchronize");
    siso_arena_done(c);
    if (rc == SISO_OK)
        for (int j = 0; j < m; ++j) out_hits[j] = (long)host_hits[j];
    return rc;
}

// Equation 2.  rho = lambda E is the load of the single server; the mean time in an M/D/1 system
// is the serving time plus rho E / (2 (1 - rho)) of queueing.
extern "C" double siso_md1_wait(double llm_time, double arrival_rate, double hit_ratio) {
    const double serve = llm_time * (1.0 - hit_ratio);
    const double load = arrival_rate * serve;
    if (load >= 1.0 || load != load) return HUGE_VAL;
    return serve + load * serve / (2.0 * (1.0 - load));
}

extern "C" int siso_pick_threshold(const float *thetas, const double *hit_ratio, int m, double llm_time,
                                   double arrival_rate, double slo, int *out_index) {
    if (!out_index) return SISO_EINVAL;
    *out_index = -1;
    if (m < 0 || (m > 0 && (!thetas || !hit_ratio))) return SISO_EINVAL;
    float chosen_theta = 0.f;
    for (int j = 0; j < m; ++j) {
        if (!(siso_md1_wait(llm_time, arrival_rate, hit_ratio[j]) < slo)) continue;
        if (*out_index < 0 || thetas[j] > chosen_theta) {
            *out_index = j;
            chosen_theta = thetas[j];
        }
    }
    return SISO_OK;
}

extern "C" int siso_adjust_threshold(const float *thetas, int m, int index, double wait_estimated, double wait_measured) {
    if (!thetas || index < 0 || index >= m) return index;
    const bool longer = wait_measured > 1.1 * wait_estimated, shorter = wait_measured < 0.9 * wait_estimated;
    if (!longer && !shorter) return index;
    // the neighbour in the order of the thresholds: the largest one below, or the smallest one above
    int neighbour = index;
    for (int j = 0; j < m; ++j) {
        const bool right_side = longer ? thetas[j] < thetas[index] : thetas[j] > thetas[index];
        if (!right_side) continue;
        if (neighbour == index || (longer ? thetas[j] > thetas[neighbour] : thetas[j] < thetas[neighbour])) neighbour = j;
    }
    return neighbour;
}
