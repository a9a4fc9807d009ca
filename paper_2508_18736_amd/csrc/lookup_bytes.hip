// Lookups of up to 64 queries against many bf16 rows, from the rows' bytes (screen.hip): such a lookup takes as long as reading the
// rows takes, and the bytes are half of them.  Two kernels: this one rules out every row whose cosine cannot be the largest, by the
// bound of screen.hip; k_finalize_update (siso.hip) forms the products of the few that are left from the stored rows, with
// the instruction and in the order of k_lookup_pipe: the results are that kernel's, bit for bit.
//
// The bytes lie in the order of the fragments of v_mfma_i32_32x32x32_i8, so a wave loads them from memory straight into the
// registers which that takes them from, one unbroken KiB an instruction, a block of 32 rows ahead: LDS holds the
// queries and nothing else passes through it.  A query is two bytes an element, in two products, 256 (hi . row) + lo . row: what is
// left of the bound's width is the error of the rows (0.0099 of 0.0176 for Gaussian directions of 768 elements), the lists are a
// fourth as long, and the matrix cores have nothing else to do.
//
// Rows that reach the largest lower end known so far (a low one lists more rows, never fewer) are collected in LDS, and what still does at the end
// goes to the query's slots of the workgroup, or behind them to the query's list.
//
// A block whose bytes are not those of its rows, or whose rows the bytes say nothing about, is multiplied as it is stored, with the sums of
// k_lookup_pipe, and so are all blocks of a workgroup that finds no room for what it would have to list (rows with a common direction),
// and all blocks where a query's length is near the ends of the range: the best row of such blocks goes to `best`.
//
// 262,144 x 768, n 64: 64 us by k_lookup_pipe (402 MB), 38 here (201 MB in 29, what a plain read of them takes, behind 7 of which the queries take
// half); the end of the step 7.7 and 12.  In those 29 it is bound by memory; a deeper ring of loads is no quicker.
#include "mfma_pipe.h"

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

#define FEW_WAVES 8
#define FEW_SLACK 2e-5f  // as SCREEN_SLACK
#define FEW_NOTES 4      // rounds whose rows are noted before they are collected
// The waves of a workgroup meet; LDS as the others have left it.  (__syncthreads() would wait for all the rows that are on their way.)
__device__ __forceinline__ void few_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
enum { QUERY_JUDGED, QUERY_ALONE /* not finite, or all zeros: no list needed */, QUERY_PLAIN /* length near the ends of the range */ };

// Bytes of LDS: the fragments of the queries; the rows collected; what is known of each query.
template <int NS, int WQ>
struct FewLds {
    static constexpr int FRAGS = NS * 4 * 2 * WQ * 1024;
    static constexpr int NOTES = FEW_WAVES * FEW_NOTES * WQ * 64 * 4;
    static constexpr int ROOM = (160 * 1024 - FRAGS - NOTES - 6144) / 4, STAGE = ROOM > 8192 ? 8192 : ROOM / 2 * 2;  // rows
    static constexpr int BYTES = FRAGS + STAGE * 4 + 64 * SISO_FEW_SLOTS * 4 + 64 * 8 + 4 * 64 * 4 + NOTES + 16;
    static_assert(STAGE >= 2048 && BYTES <= 160 * 1024, "fits in LDS");
};

// NS: slabs of 128 bytes a row; WQ: blocks of 32 queries; LANES: lanes that write a query as bytes.  Block b of 32 rows belongs to workgroup b % gridDim.x and there to wave (b / gridDim.x) % 8.
template <int NS, int WQ, int LANES>
__global__ __launch_bounds__(FEW_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_bytes_few(
    const bf16_t *__restrict__ Q, int n, const bf16_t *__restrict__ cent, const float *__restrict__ invn, long K, int d,
    const signed char *__restrict__ codes, const float4 *__restrict__ meta, const u64 *__restrict__ made,
    const unsigned *__restrict__ version, FewLists lists, u64 *__restrict__ board, int *flooded) {
    typedef FewLds<NS, WQ> Lds;
    constexpr int KS = NS * 4, STAGE = Lds::STAGE, QUERIES = LANES == 64 ? 8 : 32 * WQ, SLOTS = 64 * SISO_FEW_SLOTS / QUERIES;  // (words of LDS: the same)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned *stage = (unsigned *)(smem + Lds::FRAGS);
    u64 *best_s = (u64 *)(stage + STAGE);         // [64] of the blocks that were multiplied as they are stored
    unsigned *slot_s = (unsigned *)(best_s + 64);  // [QUERIES][SLOTS]: largest lower end, rows, rows ..
    unsigned *low_s = slot_s + 64 * SISO_FEW_SLOTS;         // [64] the largest lower end (nothing reaches +inf: no list)
    int *cnt_s = (int *)(low_s + 64);              // [64]
    float *scale_s = (float *)(cnt_s + 64), *err_s = scale_s + 64;  // [64] each
    unsigned *const notes = (unsigned *)(err_s + 64) + (threadIdx.x >> 6) * FEW_NOTES * WQ * 64 + (threadIdx.x & 63);  // each lane's own
    int *flags = (int *)((unsigned *)(err_s + 64) + FEW_WAVES * FEW_NOTES * WQ * 64);  // rows collected; a query whose length is near the ends of the range; no room
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const long blocks = (K + 31) / 32, stride = (long)gridDim.x * FEW_WAVES;
    constexpr int dp = NS * 128;

    if (board != nullptr && blockIdx.x == 0 && t < SISO_FOLD_BOARD) board[t] = 0;  // (see k_finalize_update)
    // the queries are asked for first, the first block of rows behind them
    constexpr int QCH = (dp + 8 * LANES - 1) / (8 * LANES);  // pieces of eight elements a lane
    const int mine = wave * (64 / LANES) + lane / LANES, part = lane % LANES;
    const bool quantise = wave * (64 / LANES) < n;
    u32x4_t raw[QCH];
    if (quantise) {
        const bf16_t *row = Q + (size_t)(mine < n ? mine : n - 1) * d;
#pragma unroll
        for (int c = 0; c < QCH; ++c) raw[c] = *(const u32x4_t *)(row + ((c * LANES + part) * 8 < d ? (c * LANES + part) * 8 : 0));
    }
    __builtin_amdgcn_sched_barrier(0);
    long b = (long)wave * gridDim.x + blockIdx.x;
    bool have = b < blocks;
    // what stands beside a block's bytes: asked for a round ahead, as the bytes are (by vector loads: the barriers wait for scalar ones)
    int none;
    asm volatile("v_mov_b32 %0, 0" : "=v"(none));
    float4 block_meta;
    u64 block_made;
    unsigned block_version;
    auto describe = [&](long blk) __attribute__((always_inline)) {
        block_meta = meta[blk + none];
        block_made = made[blk + none];
        block_version = version[blk + none];
    };
    const unsigned call = lists.call[none];
    describe(have ? b : 0);
    // steps on their way: a whole block of rows, or half of one where the registers end (128 KiB for a compute unit are enough)
    // (33 queries and more, 640 elements and more: five to fourteen registers that the products do not use wait in scratch memory, written once before the
    // rounds and read behind the products of one at most.)
    constexpr int R = KS <= (WQ == 1 ? 24 : 16) ? KS : KS / 2;
    i32x4 a[R];
    // Buffer loads: where there is no next block the lanes' offset lies behind all rows, and the instruction fetches nothing.  (A branch
    // around it would be two copies of the products, and of their registers.)
    const auto all = __builtin_amdgcn_make_buffer_rsrc((void *)codes, 0, (int)(unsigned)(blocks * 32 * dp), 0x00027000);
    auto fetch = [&](long blk, int s, unsigned at) __attribute__((always_inline)) {
        return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(all, at, (unsigned)blk * (32u * dp) + s * 1024, 0));
    };
    if (have) {
#pragma unroll
        for (int s = 0; s < R; ++s) a[s] = fetch(b, s, lane * 16);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int i = t; i < 64 * SISO_FEW_SLOTS; i += FEW_WAVES * 64) slot_s[i] = 0;
    if (t < 64) {
        best_s[t] = 0;
        low_s[t] = ordered_bits(INFINITY);
        cnt_s[t] = 0;
        scale_s[t] = err_s[t] = 0.f;  // (beyond the queries: no upper end reaches +inf)
    }
    if (t < 3) flags[t] = 0;
    few_barrier();
    if (quantise) {
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
        float ss = 0.f;
        u16x2 most = {0, 0};
#pragma unroll
        for (int c = 0; c < QCH; ++c) {
            if ((c * LANES + part) * 8 >= d) raw[c] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned two = raw[c][i];  // (a bit cast of the vector's element itself takes its first for each)
                ss = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b16x2, two), __builtin_bit_cast(b16x2, two), ss, false);
                most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, raw[c][i] & 0x7FFF7FFFu));
            }
        }
        ss = wave_fold<LANES / 2>(ss, [](float x, float y) __attribute__((always_inline)) { return x + y; });  // (over the lanes of a query)
        const unsigned top_bits = wave_fold<LANES / 2>((unsigned)max(most[0], most[1]) << 16,
                                                       [](unsigned x, unsigned y) __attribute__((always_inline)) { return max(x, y); });
        const float inv = inv_length(ss);
        const int kind = !(inv == inv) || top_bits == 0 ? QUERY_ALONE : inv == 0.f || inv > 1e15f || inv < 1e-15f ? QUERY_PLAIN : QUERY_JUDGED;
        // (whoever is not judged: zeros, or what a NaN leaves: nothing looks at it)
        const float top = kind == QUERY_JUDGED ? __uint_as_float(top_bits) * inv : 1.f, by = kind == QUERY_JUDGED ? inv * (32639.f / top) : 0.f;
        // element e of query q: step e / 32, lane 32 (e % 32 / 16) + q % 32, byte e % 16
        unsigned char *to = smem + (mine >> 5) * 1024 + (mine & 31) * 16;
#pragma unroll
        for (int c = 0; c < QCH; ++c) {
            const int e = (c * LANES + part) * 8;
            // a float near 1.5 * 2^23 holds its nearest integer v in its low bits; v = 256 hi + lo, a byte each (|v| <= 32639)
            unsigned v[8], u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = __uint_as_float(i % 2 == 0 ? raw[c][i / 2] << 16 : raw[c][i / 2] & 0xFFFF0000u);
                v[i] = __float_as_uint(fmaf(x, by, 12582912.f));
                u[i] = v[i] + 128u;
            }
            unsigned hi[2], lo[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {  // (the bytes 1 of four numbers, and the bytes 0)
                hi[i] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(u[4 * i + 3], u[4 * i + 2], 0x0C0C0501u), __builtin_amdgcn_perm(u[4 * i + 1], u[4 * i], 0x0C0C0501u), 0x05040100u);
                lo[i] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(v[4 * i + 3], v[4 * i + 2], 0x0C0C0400u), __builtin_amdgcn_perm(v[4 * i + 1], v[4 * i], 0x0C0C0400u), 0x05040100u);
            }
            if (e < dp) {
                unsigned char *at = to + (size_t)(e >> 5) * 2 * WQ * 1024 + ((e >> 4) & 1) * 512 + (e & 15);
                *(uint2 *)at = make_uint2(hi[0], hi[1]);
                *(uint2 *)(at + WQ * 1024) = make_uint2(lo[0], lo[1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (part == 0) {
            scale_s[mine] = top / 32639.f;
            err_s[mine] = top / 32639.f * 0.51f * sqrtf((float)d) + 1e-6f;  // (half a step an element, and what the product was rounded by)
            if (mine < n && kind == QUERY_JUDGED) low_s[mine] = ordered_bits(-INFINITY);
            if (mine < n && kind == QUERY_PLAIN) flags[1] = 1;
        }
    }
    few_barrier();
    const bool plain = flags[1] != 0;
    float scale[WQ], err[WQ];
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
        scale[q] = scale_s[q * 32 + l32];
        err[q] = err_s[q * 32 + l32];
    }

    unsigned as_stored = 0;  // bit r: the block of round r is multiplied as it is stored (at the end: its code takes other registers)
    for (int round = 0; have; ++round) {
        const long next = b + stride;
        const bool more = next < blocks;
        const long rows = K - b * 32;
        // What the workgroup has found, and heard, goes out once a round, and comes in from two others by each wave: in three rounds everyone has
        // heard of what anyone had found in the first, with plain stores and loads.  (By maxima in memory, 64 of each workgroup, the whole
        // kernel took 15 us longer.)  The number of the call tells what is left of an earlier one.
        u64 heard[2] = {0, 0};
        if (round > 0 && lane < n) {
            if (wave == 0 && low_s[lane] < ordered_bits(INFINITY))
                __hip_atomic_store(lists.table + blockIdx.x * SISO_FEW + lane, (u64)call << 32 | low_s[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const unsigned from = (blockIdx.x + 37u * (unsigned)(((round - 1) * FEW_WAVES + wave) * 2 + k + 1)) % gridDim.x;
                heard[k] = __hip_atomic_load(lists.table + from * SISO_FEW + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        i32x16 hi[WQ], lo[WQ];
#pragma unroll
        for (int q = 0; q < WQ; ++q) hi[q] = lo[q] = i32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        const i32x4 *frag = (const i32x4 *)smem + lane;
        i32x4 f[2][2 * WQ];  // the queries' fragments of this step and of the next: their upper bytes, their lower bytes
#pragma unroll
        for (int q = 0; q < 2 * WQ; ++q) f[0][q] = frag[q * 64];
        const unsigned at = more ? lane * 16 : 0xF0000000u;  // (and no block's offset on top, which could wrap)
        const long ahead = more ? next : 0;
        // (the products of a block that is multiplied as it is stored are formed, too: a branch would be a second copy of the registers)
        static_for<0, KS>([&](auto ss) __attribute__((always_inline)) {
            constexpr int s = decltype(ss)::value;
            if constexpr (s + 1 < KS) {
#pragma unroll
                for (int q = 0; q < 2 * WQ; ++q) f[(s + 1) & 1][q] = frag[((s + 1) * 2 * WQ + q) * 64];
            }
#pragma unroll
            for (int q = 0; q < WQ; ++q) {
                hi[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s % R], f[s & 1][q], hi[q], 0, 0, 0);
                lo[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s % R], f[s & 1][WQ + q], lo[q], 0, 0, 0);
            }
            if constexpr (s + R < KS) a[s % R] = fetch(b, s + R, lane * 16);
            else a[s % R] = fetch(ahead, s + R - KS, at);
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int q = 0; q < WQ; ++q) asm volatile("" : "+v"(hi[q]), "+v"(lo[q]));  // (here, not where a condition first asks for them)
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (round > 0 && lane < n && (unsigned)(heard[k] >> 32) == call && (unsigned)heard[k] > low_s[lane]) atomicMax(low_s + lane, (unsigned)heard[k]);
        const float4 m = block_meta;
        const bool judged = __builtin_amdgcn_readfirstlane(!plain && block_made == ((u64)block_version << 8) + (u64)(rows > 32 ? 32 : rows) && m.y < INFINITY) != 0;
        describe(more ? next : b);
        if (judged) {
            static_for<0, WQ>([&](auto qq) __attribute__((always_inline)) {
                constexpr int q = decltype(qq)::value;
                const unsigned col = (unsigned)(q * 32 + l32);
                float v[16], most = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    v[i] = fmaf((float)hi[q][i], 256.f, (float)lo[q][i]);  // (both below 2^24)
                    most = fmaxf(most, v[i]);
                }
                const float unit = scale[q] * m.x, width = fmaf(1.f + err[q], m.y, err[q]) + FEW_SLACK;
                float lower = fmaf(most, unit, -(fmaf(1.f + err[q], m.z, err[q]) + FEW_SLACK));
                lower = fmaxf(lower, __uint_as_float(other_half(__float_as_uint(lower))));
                float bound = unordered_bits(low_s[col]);
                if (h == 0 && lower > bound) atomicMax(low_s + col, ordered_bits(lower));
                bound = fmaxf(bound, lower);
                const float upper = fmaf(most, unit, width);
                unsigned note = 0;  // this lane's rows that reach it, and the upper end of the largest
                if (__ballot(upper >= bound) != 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) note |= fmaf(v[i], unit, width) >= bound ? 1u << i : 0u;
                    if (rows < 32) {
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            if (8 * (i >> 2) + 4 * h + (i & 3) >= rows) note &= ~(1u << i);
                    }
                    note = note == 0 ? 0 : note | few_upper_bits(upper) << 16;
                }
                notes[(round % FEW_NOTES * WQ + q) * 64] = note;
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            as_stored |= 1u << round;
#pragma unroll
            for (int q = 0; q < WQ; ++q) notes[(round % FEW_NOTES * WQ + q) * 64] = 0;
        }
        // The rows noted in the last rounds, by the bound as it has become: those that still reach it are collected.  (Listed as they are met, most
        // of them for want of a bound, they took as long as the products.)
        if (!more || round % FEW_NOTES == FEW_NOTES - 1) {
#pragma unroll
            for (int q = 0; q < WQ; ++q) {
                const unsigned col = (unsigned)(q * 32 + l32);
                const float bound = unordered_bits(low_s[col]);
                for (int k = 0; k <= round % FEW_NOTES; ++k) {
                    const unsigned note = notes[(k * WQ + q) * 64];
                    unsigned mask = note & 0xFFFFu;
                    if (mask == 0 || few_upper(note >> 16) < bound) continue;
                    int to = atomicAdd(flags, __popc(mask));
                    const unsigned entry = (col << 26) | ((unsigned)((round / FEW_NOTES * FEW_NOTES + k) * 256 + wave * 32 + 4 * h) << 13) | note >> 16;
                    for (; mask != 0 && to < STAGE; mask &= mask - 1, ++to) {
                        const unsigned i = (unsigned)__ffs((int)mask) - 1;
                        stage[to] = entry + ((8 * (i >> 2) + (i & 3)) << 13);
                    }
                }
            }
        }
        b = next;
        have = more;
    }
    few_barrier();
    // Places in a query's list are asked for once by a workgroup, for all of its rows that its slots have no room for.  (Asked for row by row, they were
    // additions to 64 words by everyone: 4.3 ms of a lookup of 32 queries against 131,072 x 768 rows with a mean cosine of 0.8.)
    const int collected = flags[0];
    int *place_s = (int *)scale_s, *far_s = (int *)err_s;  // (both are in registers)
    if (t < 64) far_s[t] = 0;
    if (collected > STAGE) {
        if (t == 0) flags[2] = 1;
    } else {
        for (int i = t; i < collected; i += FEW_WAVES * 64) {
            const unsigned e = stage[i], q = e >> 26;
            const bool reaches = few_upper(e) >= unordered_bits(low_s[q]);
            const int slot = reaches ? 2 + atomicAdd(cnt_s + q, 1) : 0;
            if (reaches && slot < SLOTS) slot_s[q * SLOTS + slot] = e;
            if (!reaches || slot < SLOTS) stage[i] = 0;  // (an upper end is never 0)
        }
        few_barrier();
        const int far = t < n ? cnt_s[t] - (SLOTS - 2) : 0;
        if (far > 0) {
            place_s[t] = atomicAdd(lists.cnt + t, far);
            if (place_s[t] + far > SISO_FEW_LIST) flags[2] = 1;
        }
        few_barrier();
        for (int i = t; i < collected; i += FEW_WAVES * 64) {
            const unsigned e = stage[i], q = e >> 26;
            if (e == 0) continue;
            const int at = place_s[q] + atomicAdd(far_s + q, 1);
            if (at < SISO_FEW_LIST) lists.rows[(size_t)q * SISO_FEW_LIST + at] = make_uint2(few_row(e, blockIdx.x, gridDim.x), e);
        }
    }
    __syncthreads();
    const bool flood = flags[2] != 0;  // (then all its rows are multiplied below, and it names none)
    for (int i = t; i < n * SLOTS; i += FEW_WAVES * 64)
        lists.slots[((size_t)(i / SLOTS) * gridDim.x + blockIdx.x) * SLOTS + i % SLOTS] = i % SLOTS == 0 ? low_s[i / SLOTS] : i % SLOTS == 1 ? (flood ? 0u : (unsigned)cnt_s[i / SLOTS]) : slot_s[i];
    if (flood) {
        as_stored = ~0u;
        if (t == 0 && flooded) __hip_atomic_store(flooded, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // the products of blocks as they are stored, with the sums of k_lookup_pipe; the best row of each query to best_s
    for (long blk = (long)wave * gridDim.x + blockIdx.x; as_stored != 0 && blk < blocks; blk += stride, as_stored >>= 1) {
        if ((as_stored & 1) == 0) continue;
        const bf16_t *row = cent + ((size_t)blk * 32 + l32) * d + h * 8;  // (rows past the end are readable, their weights NaN)
        const bf16_t *qrow[WQ];
        f32x16 acc[WQ];
#pragma unroll
        for (int q = 0; q < WQ; ++q) {
            const int at = q * 32 + l32;
            qrow[q] = Q + (size_t)(at < n ? at : n - 1) * d + h * 8;
            acc[q] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        }
        constexpr int AHEAD = 8 / WQ;  // steps on their way while as many are multiplied
        bf16x8 x[2][AHEAD], y[2][WQ][AHEAD];
        auto ask = [&](auto buf, int e0) __attribute__((always_inline)) {
            constexpr int U = decltype(buf)::value;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                const int e = e0 + i * 16 < d ? e0 + i * 16 : 0;
                x[U][i] = *(const bf16x8 *)(row + e);
#pragma unroll
                for (int q = 0; q < WQ; ++q) y[U][q][i] = *(const bf16x8 *)(qrow[q] + e);
            }
        };
        auto multiply = [&](auto buf, int e0) __attribute__((always_inline)) {
            constexpr int U = decltype(buf)::value;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (e0 + i * 16 >= d) break;
#pragma unroll
                for (int q = 0; q < WQ; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[U][i], y[U][q][i], acc[q], 0, 0, 0);
            }
        };
        ask(IC<0>{}, 0);
        for (int e = 0; e < d; e += 32 * AHEAD) {
            ask(IC<1>{}, e + 16 * AHEAD);
            multiply(IC<0>{}, e);
            ask(IC<0>{}, e + 32 * AHEAD);
            multiply(IC<1>{}, e + 16 * AHEAD);
        }
#pragma unroll
        for (int q = 0; q < WQ; ++q) {
            float m = -INFINITY;
            unsigned at = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const unsigned r = (unsigned)(blk * 32) + 8 * (i >> 2) + 4 * h + (i & 3);
                const float v = acc[q][i] * invn[r];
                if (v > m) {  // (ascending: the lowest among equal values)
                    m = v;
                    at = r;
                }
            }
            if (m > -INFINITY) atomicMax(best_s + q * 32 + l32, pack_key(m, at));
        }
    }
    __syncthreads();
    if (t < n && best_s[t] != 0) atomicMax(lists.best + t, best_s[t]);
}

// ----------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------
template <int NS, int WQ, int LANES>
static int few_bytes_launch(siso_cache *c, const void *queries, long n, const ByteView &v, int workgroups) {
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)k_bytes_few<NS, WQ, LANES>, hipFuncAttributeMaxDynamicSharedMemorySize, FewLds<NS, WQ>::BYTES);
        if (e != hipSuccess) return siso_check_hip(c, e, "hipFuncSetAttribute(k_bytes_few)");
        attr_done = true;
    }
    hipLaunchKernelGGL((k_bytes_few<NS, WQ, LANES>), dim3((unsigned)workgroups), dim3(FEW_WAVES * 64), (FewLds<NS, WQ>::BYTES), c->stream, (const bf16_t *)queries,
                       (int)n, (const bf16_t *)c->cent, c->invn, c->count, c->dim, v.codes, v.meta, v.made, c->version, c->few, c->board_to_clear,
                       c->few_flooded);
    c->board_to_clear = nullptr;  // taken
    return siso_check_hip(c, hipGetLastError(), "k_bytes_few");
}

int siso_bytes_few_workgroups(const siso_cache *c) {
    const long blocks = (c->count + 31) / 32;
    return (int)(blocks < SISO_FEW_WORKGROUPS ? blocks : SISO_FEW_WORKGROUPS);
}

int siso_bytes_few_launch(siso_cache *c, const void *queries, long n, const ByteView &v) {
    const int g = siso_bytes_few_workgroups(c);
#define SISO_FEW_CASE(NS) \
    case NS:                                                              \
        return n <= 8    ? few_bytes_launch<NS, 1, 64>(c, queries, n, v, g) \
               : n <= 32 ? few_bytes_launch<NS, 1, 16>(c, queries, n, v, g) \
                         : few_bytes_launch<NS, 2, 8>(c, queries, n, v, g)
    switch (v.dp / 128) {
        SISO_FEW_CASE(2);
        SISO_FEW_CASE(3);
        SISO_FEW_CASE(4);
        SISO_FEW_CASE(5);
        SISO_FEW_CASE(6);
        SISO_FEW_CASE(7);
        SISO_FEW_CASE(8);
    }
#undef SISO_FEW_CASE
    return siso_fail(c, SISO_EINVAL, "lookup of few queries: %d bytes a row", v.dp);
}
