// Phase 1 of a lookup of a few queries in single precision: every row of the cache passes through the chip once, and reading them
// is all that the time should go into.
//
// v_mfma_f32_16x16x4_f32 with the rows as A and the queries as B: lane l supplies row l % 16 and, of 64 bytes of it at a
// time (a step), the 16 bytes number l / 16, which come straight from memory in one load.  Nothing of the rows goes through LDS,
// so there is no barrier and no stage to wait for: a wave has AHEAD loads in flight, across the ends of its groups of 16
// rows.  The queries lie in LDS in the order in which the lanes ask for them (a step's fragments are 1 KiB in a row), and
// element k of a row meets element k of a query whatever order a step takes them in.
// D: lane l holds query l % 16, rows 4 * (l / 16) .. + 3 of the group: the running maximum is taken inside the lane.
// A sum depends on the row and the query alone, not on where they stand, so equal rows have equal products and the lowest
// index wins.
//
// The tiled kernel that served such batches (lookup_tile.hip) brings the rows through LDS, a barrier for each slab.  A batch with
// its update, us, tiled / here:
//   60,000 x 768   n 1  43.3 / 36.9   n 16  44.3 / 38.2   n 32  44.8 / 43.3       8,000 x 768   n 1  25.8 / 16.5   n 16  27.7 / 18.9
//   60,000 x 384   n 1  27.5 / 22.6   n 16  28.8 / 23.8   n 32  29.2 / 26.9       1,000 x 384   n 1  16.5 / 14.1   n 16  18.6 / 14.2
//   60,000 x 300   n 1  25.3 / 20.1   n 16  26.7 / 21.0   n 32  27.3 / 24.0       300,000 x 768  n 1  215 / 160    n 16  215 / 163
//   400,000 x 128  n 1  60.4 / 35.2   n 16  61.3 / 36.5   n 32  61.5 / 42.9       100,000 x 1,024  n 1  118 / 95   n 16  107 / 101
// Rows of bf16 and codes gain nothing here (60,000 x 768 22.7 / 22.8, 21.8 / 21.8; 300,000 x 768 75 / 83): their streaming kernel
// (PipeSmall) loads into LDS directly, three stages ahead.  Above 32 queries the matrix cores are the limit (n 64: 71.0 / 71.0).
#include <math.h>

#include "siso_internal.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

#define FEW_WORKGROUPS 256  // one for every compute unit

// one chunk of 16 bytes of either side; c[0], c[1] = two sums, added up at the end of a row
__device__ __forceinline__ void few_mma(u32x4_t a, u32x4_t b, f32x4 (&c)[2]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        c[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[j]), __uint_as_float(b[j]), c[j & 1], 0, 0, 0);
}

// steps of a row, a whole number of rounds of `ahead`
__host__ __device__ constexpr int few_steps(int row_bytes, int ahead) { return (row_bytes + 64 * ahead - 1) / (64 * ahead) * ahead; }
__host__ __device__ constexpr size_t few_lds(int nb, int waves, int row_bytes, int ahead) {
    return (size_t)nb * few_steps(row_bytes, ahead) * 1024 + (size_t)waves * nb * 16 * 8;
}

// NB blocks of 16 queries; row_bytes is a whole number of 16-byte chunks.  vec: the queries are aligned to them too.
// WHOLE: a row is a whole number of rounds; otherwise the steps beyond it read its last chunk, and the queries have zeros there.
template <int NB, int WAVES, int AHEAD, bool WHOLE>
__global__ __launch_bounds__(WAVES * 64) void k_lookup_few(const float *__restrict__ Q, const float *__restrict__ C,
                                                           const float *__restrict__ invn, int n, long K, int row_bytes, int vec,
                                                           u64 *__restrict__ keys, u64 *__restrict__ board) {
    extern __shared__ u32x4_t few_frags[];  // [NB][steps][64]
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int steps = few_steps(row_bytes, AHEAD), quarter = lane >> 4, col = lane & 15;
    u64(*red)[NB * 16] = (u64(*)[NB * 16])(few_frags + NB * steps * 64);  // [WAVES][NB * 16]
    if (board != nullptr && blockIdx.x == 0 && t < SISO_FOLD_BOARD) board[t] = 0;  // (see k_finalize_update)
    static_assert(SISO_FOLD_BOARD <= WAVES * 64, "a thread for every slot");

    // The loads walk through the groups of this wave one after the other, AHEAD steps ahead of the products; behind the last
    // one they fetch its group again.
    const int groups = (int)((K + 15) / 16), stride = (int)gridDim.x * WAVES;
    int g = (int)blockIdx.x * WAVES + wave;  // the group being multiplied
    int ld_g = g < groups ? g : groups - 1;
    int ld_s = 0;
    const unsigned row_off = (unsigned)(col * row_bytes), lane_off = row_off + (unsigned)quarter * 16;
    const char *ld = (const char *)C + (size_t)ld_g * 16 * row_bytes;
    auto load = [&](int i) __attribute__((always_inline)) {
        u32x4_t v;
        if constexpr (WHOLE) {
            v = *(const u32x4_t *)(ld + (size_t)ld_s * 64 + i * 64 + lane_off);
        } else {
            const int at = (ld_s + i) * 64 + quarter * 16;
            v = *(const u32x4_t *)(ld + (row_off + (unsigned)(at < row_bytes - 16 ? at : row_bytes - 16)));
        }
        return v;
    };
    auto loaded = [&]() __attribute__((always_inline)) {  // a round of them
        ld_s += AHEAD;
        if (ld_s == steps) {
            ld_s = 0;
            if (ld_g + stride < groups) ld_g += stride;
            ld = (const char *)C + (size_t)ld_g * 16 * row_bytes;
        }
    };
    u32x4_t a[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) a[i] = load(i);
    loaded();

    // the queries into LDS, zeros behind the last one
#pragma unroll 4
    for (int c = t; c < NB * steps * 64; c += WAVES * 64) {
        const int q = c / (steps * 64) * 16 + (c & 15), at = c / 64 % steps * 64 + (c >> 4 & 3) * 16;
        u32x4_t v = {0, 0, 0, 0};
        if (q < n && at < row_bytes) {
            const char *src = (const char *)Q + (size_t)q * row_bytes + at;
            if (vec) {
                v = *(const u32x4_t *)src;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = ((const unsigned *)src)[i];
            }
        }
        few_frags[c] = v;
    }
    __syncthreads();

    float bv[NB];
    unsigned bi[NB];
    f32x4 acc[NB][2];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        bv[b] = -INFINITY;
        bi[b] = 0xFFFFFFFFu;
        acc[b][0] = acc[b][1] = zero;
    }
    const u32x4_t *frag = few_frags + lane;
    u32x4_t next[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) next[b] = frag[b * steps * 64];
    for (; g < groups; g += stride) {
        // (asked for here, a round of loads and more before it is needed: waiting for it leaves the last round in flight)
        const f32x4 w = *(const f32x4 *)(invn + (size_t)g * 16 + quarter * 4);
        int s = 0;
        do {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                u32x4_t now[NB];
                const int s1 = s + i + 1 == steps ? 0 : s + i + 1;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    now[b] = next[b];
                    next[b] = frag[(b * steps + s1) * 64];
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) few_mma(a[i], now[b], acc[b]);
                a[i] = load(i);
                __builtin_amdgcn_sched_barrier(0);
            }
            loaded();
            s += AHEAD;
        } while (s < steps);
        const unsigned row0 = (unsigned)g * 16u + (unsigned)quarter * 4u;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = (acc[b][0][r] + acc[b][1][r]) * w[r];  // (rows past the end: NaN)
                if (v > bv[b]) {
                    bv[b] = v;
                    bi[b] = row0 + r;
                }
            }
            acc[b][0] = acc[b][1] = zero;
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        u64 key = bi[b] == 0xFFFFFFFFu ? 0ull : pack_key(bv[b], bi[b]);
        LanePair<u64> p = lane_pair<32>(key);
        key = p.b > p.a ? p.b : p.a;
        p = lane_pair<16>(key);
        key = p.b > p.a ? p.b : p.a;
        if (lane < 16) red[wave][b * 16 + lane] = key;
    }
    __syncthreads();
    if (t < NB * 16 && t < n) {
        u64 key = red[0][t];
#pragma unroll
        for (int v = 1; v < WAVES; ++v) key = red[v][t] > key ? red[v][t] : key;
        keys[(size_t)t * gridDim.x + blockIdx.x] = key;
    }
}

// ----------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------
// Workgroups of four waves for 16 queries, of eight for 32, whose products would otherwise hold up the loads (60,000 x 768, n 32:
// 48.2 with four, 43.3 with eight; n 1, 8,000 x 768, where half of the compute units would have no rows: 16.5 and 19.5).  Eight
// loads in flight where the rows come from beyond the 256 MB memory-side cache (300,000 x 768, n 1: 183 with four, 160 with
// eight; 60,000 x 768 37.3 and 38.5), and so where a row is a whole number of such rounds.
static int few_row_bytes(const siso_cache *c) { return c->dim * 4; }
static int few_waves(long n) { return n <= 16 ? 4 : 8; }
static bool few_far(const siso_cache *c, long n) {
    const int rb = few_row_bytes(c);
    return n <= 16 && rb % 512 == 0 && c->count * (long)rb > (256l << 20);
}

int siso_few_slices(const siso_cache *c, long n) {
    if (c->dtype != SISO_F32 || c->count < 1 || n < 1 || n > 32) return 0;
    if (c->opt_mfma_config != 0 || c->opt_tiles_per_slice != 0 || c->opt_mfma_qblock != 0) return 0;
    const int rb = few_row_bytes(c);
    // (with two blocks, rows of 4 KiB, 16 at a time, lose: 100,000 x 1,024, n 32: 107.8 / 120.8)
    if (rb % 16 != 0 || rb < 256 || (n > 16 && rb >= 4096) || few_lds(n <= 16 ? 1 : 2, few_waves(n), rb, few_far(c, n) ? 8 : 4) > 160 * 1024) return 0;
    // (rows about 8 KiB apart, 16 of them in a load, from beyond that cache: 52,000 x 1,984 and up to 131,072 x 2,112 take 4 to 20 % longer than
    // tiles, 60,000 x 2,112, n 16, 111 / 129; 48,000 x 2,000 106 / 101, 65,536 x 1,900 114 / 111, 57,444 x 2,176 112 / 115, 103,400 x 2,176 213 / 181)
    if (rb > 7700 && rb < 8600 && c->count * (long)rb > (384l << 20)) return 0;
    const long each = 16 * few_waves(n), want = (c->count + each - 1) / each;
    return (int)(want < FEW_WORKGROUPS ? want : FEW_WORKGROUPS);
}

template <int NB, int WAVES, int AHEAD, bool WHOLE>
static int few_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys) {
    const int rb = few_row_bytes(c);
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)k_lookup_few<NB, WAVES, AHEAD, WHOLE>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return siso_check_hip(c, e, "hipFuncSetAttribute(k_lookup_few)");
        attr_done = true;
    }
    hipLaunchKernelGGL((k_lookup_few<NB, WAVES, AHEAD, WHOLE>), dim3((unsigned)slices), dim3(WAVES * 64), few_lds(NB, WAVES, rb, AHEAD),
                       c->stream, (const float *)queries, (const float *)c->cent, c->invn, (int)n, c->count, rb,
                       ((uintptr_t)queries & 15) == 0 ? 1 : 0, keys, c->board_to_clear);
    c->board_to_clear = nullptr;  // taken
    return siso_check_hip(c, hipGetLastError(), "k_lookup_few");
}

int siso_few_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys) {
    if (siso_few_slices(c, n) != slices) return siso_fail(c, SISO_EINVAL, "lookup of few queries: plan mismatch");
    const bool whole = few_row_bytes(c) % 256 == 0;
    if (few_far(c, n)) return few_launch<1, 4, 8, true>(c, queries, n, slices, keys);
    if (n <= 16) return whole ? few_launch<1, 4, 4, true>(c, queries, n, slices, keys) : few_launch<1, 4, 4, false>(c, queries, n, slices, keys);
    return whole ? few_launch<2, 8, 4, true>(c, queries, n, slices, keys) : few_launch<2, 8, 4, false>(c, queries, n, slices, keys);
}
