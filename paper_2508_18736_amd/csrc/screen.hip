// Lookups and pair searches that form most products in eight bits.
//
// A large lookup is bound by the matrix cores and by the power they draw, and almost all of its products are of rows
// that are nowhere near the best.  So the rows and the queries, at unit length, are first written as signed bytes (the
// largest element of 32 rows, or of one query, becomes 127); v_mfma_i32_32x32x32_i8 forms the products of the bytes at
// twice the rate of bf16 from half the bytes, and exactly: sums of integers have no rounding.  What the bytes leave out
// is known: for unit vectors u, w and what their bytes stand for, u', w',
//     | u.w - u'.w' |  <=  |u - u'| |w| + |u'| |w - w'|  <=  e_u + (1 + e_u) e_w,     e = the length of the difference,
// and both lengths are measured when the bytes are written (Gaussian directions of 768 elements: 0.0077 for a query, 0.0099 for rows
// in blocks of 32).  A row is
// passed over only if the upper end of its cosine lies below the lower end of some other row's: what is left, some tens of
// rows a query, is multiplied again from the stored rows in single precision, as the end of a lookup does, and the
// largest of those cosines (lowest index among equal ones) is the result.  No result is made of bytes.
//
// Queries and rows for which the bound says nothing (no length, non-finite, more rows near the best than the list
// holds) are left to the kernels of lookup_mfma.hip and lookup_tile.hip: every call ends with a launch of those over the
// gathered rows of such queries, whose workgroups leave at once if there are none.
//
// Rows with a common direction (mean cosine 0.5 and more, as text embeddings have it) crowd together for queries that miss:
// the deviation of the cosines shrinks with the part that is not common while the error stays, and a list floods.  A query
// whose list is full lists nothing any more; k_screen_seed counts those whose lists can be foreseen to flood, from
// the sample and again from the lists of the first eighth; and if they are too many (lost, most_lost) the batch is given up:
// the rest of the products is not formed, and the other kernels do all of it, which by then has paid for little.  (No query
// is given up alone: for a few those kernels take a good part of the time that they take for all.)
//
// Rows are grouped by 32 (the rows of one MFMA): one scale and one error for each.  One outlier costs its 32 rows some
// precision and nobody else; and the end of a tile works on integers: a maximum of 16, one conversion, three operations
// in floating point for 16 products, against some two for each where every row has a weight.
#include <new>

#include "mfma_pipe.h"

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

typedef PipeCfg<4, 2, 2, 4, 2, 128, true, 1> ByteCfg;  // 256 x 256 tile, waves of 128 x 64, two stages of 128 bytes a row

#define SCREEN_LIST 1024          // rows a query's list holds
#define SCREEN_TILES 16           // tiles of a slice: a row of it is 12 bits
#define SCREEN_STAGE 896          // rows a wave collects in LDS before they are handed to the queries' lists
#define SCREEN_SLACK 2e-5f        // roundings of the lengths, of the unit rows and of the sums formed anew (about 4e-6 in all)
#define SCREEN_WHOLE 0x7FFFFFFF   // most_lost: never given up
#define SCREEN_COUNTED 8          // of so many queries one is looked at for `lost` (atomic additions to one address: 10 ns each)
#define SCREEN_LEAST_FLOOR 0.5f   // below it unrelated rows come near it, and it spares nothing
#define SCREEN_PLAIN (-2)         // instead of a list's length: this query is left to the other kernels
#define SCREEN_NAN (-1)           // and this one holds a NaN or an infinity

struct ScreenQuery {
    float scale, err;
};

// ---- bytes -------------------------------------------------------------------------------------------------------
// A float near 1.5 * 2^23 holds its nearest integer in its low bits, in two's complement.
#define SCREEN_ROUND 12582912.f
__device__ __forceinline__ unsigned pack_bytes(float a, float b, float c, float d) {  // the lowest bytes, a's first
    const unsigned ab = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x0C0C0400u);
    const unsigned cd = __builtin_amdgcn_perm(__float_as_uint(d), __float_as_uint(c), 0x04000C0Cu);
    return ab | cd;
}

// One workgroup per 32 rows, a wave for eight of them, which it holds in registers: NCH times four elements a lane.
// The bytes of 32 rows lie in the order in which the matrix cores take them: for every 32 elements of the dimension a KiB, 16 bytes
// for each lane of a wave (lane l: row l % 32, elements 16 (l / 32) to 16 (l / 32) + 15), so that whatever reads a fragment reads one
// unbroken KiB, from memory as well as from LDS.  They are put in that order in LDS (a pad of 128 bytes behind 512, of 16 more behind 1,024: all
// 64 banks for the 16 runs that a row's lanes write) and leave it 16 bytes a lane.
// ROWS: rows of the cache, meta = (scale, error, error for lower ends, 1 / scale); a block with a row that cannot be judged
// (past the end, non-finite, length near the ends of the range) has an infinite error for lower ends, and one with a
// length near the ends of the range is never ruled out.  Otherwise queries, each with its own scale.
#define BYTE_IMAGE_HALF (512 + 128)
#define BYTE_IMAGE_STEP (2 * BYTE_IMAGE_HALF - 128 + 16)
template <typename T, int NCH, bool ROWS>
__device__ __forceinline__ void write_bytes_block(unsigned char *image, long blk, const T *__restrict__ src, const float *__restrict__ invn, long have,
                                                  int vec, signed char *__restrict__ codes, float4 *__restrict__ meta,
                                                  ScreenQuery *__restrict__ qm, unsigned *__restrict__ low, u64 *__restrict__ seed,
                                                  int *__restrict__ cnt, int *__restrict__ near, float *__restrict__ largest,
                                                  int *__restrict__ totals, int d, int dp, float least) {
    constexpr int R = 8, STEP = BYTE_IMAGE_STEP, HALF = BYTE_IMAGE_HALF;
    __shared__ float sh[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long r0 = blk * 32 + wave * R;

    constexpr int W = (int)sizeof(T);  // words of four elements
    typedef unsigned chunk_t __attribute__((ext_vector_type(W)));
    unsigned v[R][NCH][W];
    float inv[R];
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int i = 0; i < W; ++i) v[j][c][i] = 0u;
    if (vec) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T *row = src + (size_t)(r0 + j < have ? r0 + j : 0) * d + lane * 4;
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                if (r0 + j < have && c * 256 + lane * 4 < d) {
                    const chunk_t x = *(const chunk_t *)(row + c * 256);
                    v[j][c][0] = x[0];
                    v[j][c][1] = x[1];
                    if constexpr (W == 4) {
                        v[j][c][2] = x[2];
                        v[j][c][3] = x[3];
                    }
                }
        }
    } else {
        for (int j = 0; j < R; ++j) {
            if (r0 + j >= have) break;
            const T *row = src + (size_t)(r0 + j) * d;
            unsigned x[NCH * 4];
#pragma unroll
            for (int i = 0; i < NCH * 4; ++i) {
                const int e = (i / 4) * 256 + lane * 4 + i % 4;
                const T y = row[e < d ? e : 0];
                if constexpr (sizeof(T) == 4) x[i] = e < d ? __float_as_uint(y) : 0u;
                else x[i] = e < d ? (unsigned)y : 0u;
            }
#pragma unroll
            for (int k = 0; k < R; ++k)  // (registers are not addressed by a variable)
#pragma unroll
                for (int i = 0; i < NCH * W; ++i) {
                    const unsigned word = sizeof(T) == 4 ? x[i] : x[(2 * i) % (NCH * 4)] | (x[(2 * i + 1) % (NCH * 4)] << 16);
                    v[k][i / W][i % W] = k == j ? word : v[k][i / W][i % W];
                }
        }
    }
    if constexpr (ROWS) {
#pragma unroll
        for (int j = 0; j < R; ++j) inv[j] = invn[r0 + j < have ? r0 + j : 0];
    }
    auto element = [&](int j, int c, int i) __attribute__((always_inline)) {
        if constexpr (sizeof(T) == 4) return __uint_as_float(v[j][c][i]);
        else return (i & 1) ? __uint_as_float(v[j][c][i >> 1] & 0xFFFF0000u) : __uint_as_float(v[j][c][i >> 1] << 16);
    };
    // largest element at unit length; what cannot be judged counts as zero.  (Magnitudes compare as integers, those of two
    // bf16 elements in one instruction; a NaN or an infinity shows in the inverse length.)
    float top[R], most = 0.f;
    int kind[R];  // 0 judged, SCREEN_PLAIN length near the ends of the range (or none, for a query), SCREEN_NAN
    bool all = true, plain = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        float a;
        if constexpr (sizeof(T) == 4) {
            unsigned m = 0;
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int i = 0; i < W; ++i) m = max(m, v[j][c][i] & 0x7FFFFFFFu);
            a = __uint_as_float(m);
        } else {
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            u16x2 m = {0, 0};
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int i = 0; i < W; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v[j][c][i] & 0x7FFF7FFFu));
            a = __uint_as_float((unsigned)max(m[0], m[1]) << 16);
        }
        if constexpr (!ROWS) {
            float ss = 0.f;
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) ss = fmaf(element(j, c, i), element(j, c, i), ss);
            inv[j] = inv_length(wave_sum(ss));
        }
        a = wave_max(a);
        kind[j] = !(inv[j] == inv[j]) ? SCREEN_NAN : inv[j] > 1e15f || (inv[j] != 0.f && inv[j] < 1e-15f) ? SCREEN_PLAIN : 0;
        // (an inverse length of 0 is that of a row without length, all of whose cosines are 0 - or of one whose squares vanish)
        if (inv[j] == 0.f && (!ROWS || a > 0.f)) kind[j] = SCREEN_PLAIN;
        if (r0 + j >= have) {
            kind[j] = 0;
            all = false;
            a = 0.f;
        }
        if (kind[j] != 0) {
            inv[j] = 0.f;
            a = 0.f;
            all = false;
            plain = plain || kind[j] == SCREEN_PLAIN;
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int i = 0; i < W; ++i) v[j][c][i] = 0u;
        }
        top[j] = a == 0.f ? 0.f : a * inv[j];
        most = fmaxf(most, top[j]);
    }
    float scale = 0.f, to = 0.f;
    if constexpr (ROWS) {
        if (lane == 0) sh[0][wave] = most;
        __syncthreads();
        most = fmaxf(fmaxf(sh[0][0], sh[0][1]), fmaxf(sh[0][2], sh[0][3]));
        scale = most / 127.f;
        to = most > 0.f ? 127.f / most : 0.f;
    }
    float err = 0.f;
    unsigned char *const dst = image + (lane >> 3) * STEP + (lane >> 2 & 1) * HALF + wave * R * 16 + (lane & 3) * 4;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if constexpr (!ROWS) {
            scale = top[j] / 127.f;
            to = top[j] > 0.f ? 127.f / top[j] : 0.f;
        }
        const float by = top[j] > 0.f ? inv[j] * to : 0.f;
        float off2 = 0.f;  // in steps
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            float f[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = element(j, c, i);
                f[i] = fmaf(x, by, SCREEN_ROUND);
                const float r = fmaf(x, by, SCREEN_ROUND - f[i]);
                off2 = fmaf(r, r, off2);
            }
            *(unsigned *)(dst + c * 8 * STEP + j * 16) = pack_bytes(f[0], f[1], f[2], f[3]);
        }
        const float e = scale * sqrtf(wave_sum(off2)) * 1.0005f + 1e-6f;
        err = fmaxf(err, e);
        if (!ROWS && lane == 0) {
            const long q = r0 + j;
            const bool ok = q < have && kind[j] == 0;
            qm[q] = ScreenQuery{ok ? scale : 1.f, ok ? e : -1.f};  // (grow = 0 in k_screen_lookup)
            low[q] = ordered_bits(ok ? least : INFINITY);  // (nothing reaches +inf: no list)
            seed[q] = 0;
            cnt[q] = kind[j];
            near[q] = 0;
            largest[q] = 0.f;
        }
    }
    if constexpr (!ROWS) {
        if (blk == 0 && threadIdx.x < 3) totals[threadIdx.x] = 0;
        __syncthreads();
    } else {
        if (lane == 0) {
            sh[1][wave] = err;
            sh[2][wave] = all ? 0.f : INFINITY;
            sh[3][wave] = plain ? INFINITY : 0.f;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            err = fmaxf(fmaxf(sh[1][0], sh[1][1]), fmaxf(sh[1][2], sh[1][3]));
            const float un = sh[2][0] + sh[2][1] + sh[2][2] + sh[2][3], pl = sh[3][0] + sh[3][1] + sh[3][2] + sh[3][3];
            meta[blk] = make_float4(scale, err + pl, err + un, 127.f / most);
        }
    }
    unsigned char *const out = (unsigned char *)codes + (size_t)blk * 32 * dp;
    for (int i = threadIdx.x; i < 2 * dp; i += 256)
        *(u32x4_t *)(out + 16 * i) = *(const u32x4_t *)(image + (i >> 6) * STEP + (i >> 5 & 1) * HALF + (i & 31) * 16);
}

// Which rows of the cache a launch of k_screen_bytes writes, in tiles of 256 (eight workgroups): all; those that are looked at
// before a batch may be given up (the tiles below `ahead` and the sample, `some` tiles every `stride`); or the others, and
// none if it has been.
struct ScreenTiles {
    int part, ahead, some, stride;  // part 0, 1, 2
};
// Blocks below row_blocks: rows of the cache; the others: queries.  PARTS: tiles.part is not 0.
// made (or NULL): what the bytes of 32 rows were made from, the count of ByteRows and the number of rows.  They are left as they are where
// that is still so: of 60,000 x 384 fp32 rows between two batches of 1,000 queries that move their centroids 16 us (the queries' bytes among them) instead of 28, of 1,048,576 x 1,024
// bf16 between two of 16,384 173 instead of 590.
template <typename T, int NCH, bool PARTS>
__global__ __launch_bounds__(256) void k_screen_bytes(const T *__restrict__ rows, const float *__restrict__ invn, long K,
                                                      unsigned row_blocks, int row_vec, signed char *__restrict__ codes,
                                                      float4 *__restrict__ meta, const T *__restrict__ queries, long n, int query_vec,
                                                      signed char *__restrict__ qcodes, ScreenQuery *__restrict__ qm,
                                                      unsigned *__restrict__ low, u64 *__restrict__ seed, int *__restrict__ cnt,
                                                      int *__restrict__ near, float *__restrict__ largest, int *__restrict__ totals,
                                                      int d, int dp, ScreenTiles tiles, int most_lost, float least,
                                                      const unsigned *__restrict__ version, u64 *__restrict__ made) {
    __shared__ __attribute__((aligned(16))) unsigned char image[NCH * 8 * BYTE_IMAGE_STEP];
    if (blockIdx.x < row_blocks) {
        long blk = blockIdx.x;
        if constexpr (PARTS) {
            if (tiles.part == 2) {
                blk += 8L * tiles.ahead;
                const long tile = blk / 8;
                if (totals[2] > most_lost || (tile % tiles.stride == 0 && tile / tiles.stride < tiles.some)) return;
            } else if (blk >= 8L * tiles.ahead) {
                const long tile = (blk / 8 - tiles.ahead) * tiles.stride;
                if (tile < tiles.ahead) return;
                blk = tile * 8 + blk % 8;
            }
        }
        if (made) {
            const long have = K - blk * 32;
            const u64 from = ((u64)version[blk] << 8) + (u64)(have < 0 ? 0 : have > 32 ? 32 : have);
            if (made[blk] == from) return;
            __syncthreads();  // (everyone has read it)
            if (threadIdx.x == 0) made[blk] = from;
        }
        write_bytes_block<T, NCH, true>(image, blk, rows, invn, K, row_vec, codes, meta, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                                        nullptr, d, dp, least);
    } else {
        write_bytes_block<T, NCH, false>(image, blockIdx.x - row_blocks, queries, nullptr, n, query_vec, qcodes, nullptr, qm, low, seed, cnt,
                                         near, largest, totals, d, dp, least);
    }
}

// ---- products of bytes --------------------------------------------------------------------------------------------
// The pipeline of k_pairs_stream over bytes: slab after slab of `pairs` pairs of tiles that `src` names, fold(acc) behind the
// last slab of each; src.side() is called with a pair's first slab and loads what its fold needs.
// The loads of a slab (64 wave instructions for a compute unit, which its texture unit takes a thousand cycles to work off)
// are dealt out, one behind every second of the 16 MFMAs that follow the barrier.  Issued at once they hold up the waves, and
// with them the MFMAs: 65,536 x 65,536 / 2 products of 768 bytes 1.47 -> 1.32 ms, of zeros, which the power limit does not
// slow down, 1.17 -> 0.90 (without any loads 1.15 and 0.87; behind 8 MFMAs 1.36 and 0.99, behind 32 1.39 and 1.10).  So
// nothing between the MFMAs may depend on a condition: behind the last slab the loads fetch it once more, into a stage nobody
// reads again, and the fragment reads find a slab that does not exist.  What bounds it now is the power limit: 2.5 PFLOP/s on
// random bytes, 3.7 on zeros.
template <class Src, class Fold>
__device__ __forceinline__ void byte_stream(unsigned char *smem, int dp, int pairs, Src &src, Fold &&fold) {
    typedef ByteCfg Cfg;
    constexpr int WC = Cfg::WC, WQ = Cfg::WQ, NWC = Cfg::NWC, BC = Cfg::BC, NW = Cfg::NW, STAGE = Cfg::STAGE, NLA = Cfg::NLA,
                  NL = Cfg::NL, RB = Cfg::RB, KK = Cfg::KK, SUB = 32 * Cfg::RB;
    static_assert(KK == 4 && SUB == KK * 1024, "a slab is four fragments deep");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wc = wave % NWC, wq = wave / NWC;
    const int nk = dp / RB, T = pairs * nk;
    // (a slab of 32 rows is four KiB in a row; load j of a wave takes KiB j * NW + wave of a tile)
    unsigned off[NLA];
#pragma unroll
    for (int j = 0; j < NLA; ++j) {
        const int kib = j * NW + wave;
        off[j] = (unsigned)(kib / KK * 32 * dp + kib % KK * 1024 + lane * 16);
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const unsigned row_a = lds0 + (unsigned)(wc * WC * SUB + lane * 16);
    const unsigned row_b = lds0 + (unsigned)(BC * RB + wq * WQ * SUB + lane * 16);
    constexpr unsigned so[KK] = {0, 1024, 2048, 3072};

    int ld_t = 0, ld_ks = 0;
    unsigned ld_off = 0;
    auto part = [&](auto jj) __attribute__((always_inline)) {
        constexpr int j = decltype(jj)::value;
        if constexpr (j == 0) {
            if (ld_ks == 0) src.side(wave, lane);
        }
        unsigned o = off[j % NLA];
        asm volatile("" : "+v"(o));
        unsigned char *sb = smem + ld_off + wave * 1024;
        const size_t k = (size_t)ld_ks * SUB;
        if constexpr (j < NLA) gload_lds16((const char *)src.c + k + o, sb + j * NW * 1024);
        else gload_lds16((const char *)src.q + k + o, sb + BC * RB + (j - NLA) * NW * 1024);
        if constexpr (j == NL - 1) {
            ld_off ^= STAGE;
            if (ld_t + 1 < T) {
                ++ld_t;
                if (++ld_ks == nk) {
                    ld_ks = 0;
                    src.advance();
                }
            }
        }
    };
    constexpr int NF = WC + WQ;
    bf16x8 af[2][WC], bf[2][WQ];
    i32x16 acc[WC][WQ];
    auto mac = [&](auto buf, auto firstc, auto &&extra) __attribute__((always_inline)) {
        constexpr int U = decltype(buf)::value;
        static_for<0, WC * WQ>([&](auto ii) __attribute__((always_inline)) {
            constexpr int i = decltype(ii)::value, A = i / WQ, B = i % WQ;
            const i32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            acc[A][B] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4, af[U][A]), __builtin_bit_cast(i32x4, bf[U][B]),
                                                              decltype(firstc)::value ? zero : acc[A][B], 0, 0, 0);
            extra(ii);
        });
    };
    // parts P .. P + 3, one behind every second MFMA
    auto deal = [&](auto p) __attribute__((always_inline)) {
        return [&](auto ii) __attribute__((always_inline)) {
            constexpr int i = decltype(ii)::value;
            if constexpr (i % 2 == 1) {
                __builtin_amdgcn_sched_barrier(0);
                part(IC<decltype(p)::value + i / 2>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        };
    };
    auto none = [](auto) __attribute__((always_inline)) {};
    static_assert(NL == 8 && WC * WQ == 8, "eight loads behind two steps of eight MFMAs");
    // slab 0 and the first half of slab 1, as if a slab had just gone by
    static_for<0, NL>(part);
    static_for<0, NL / 2>(part);
    if (src.leave()) {  // (looked up while the first loads are on their way; the same for all waves)
        vm_wait<0>();
        return;
    }
    vm_wait<NL / 2>();
    __syncthreads();
    lds_frags<SUB>(af[0], bf[0], row_a + so[0], row_b + so[0]);
    int ks = 0;
    unsigned sto = 0;
    for (int t = 0; t < T; ++t) {
        const unsigned sto_next = sto ^ STAGE;
        static_for<0, KK - 1>([&](auto kc) __attribute__((always_inline)) {
            constexpr int kk = decltype(kc)::value;
            lds_frags<SUB>(af[(kk + 1) & 1], bf[(kk + 1) & 1], row_a + sto + so[kk + 1], row_b + sto + so[kk + 1]);
            lds_wait<NF>(af[kk & 1], bf[kk & 1]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kk == 0) {
                if (ks == 0) mac(IC<0>{}, IC<1>{}, deal(IC<4>{}));
                else mac(IC<0>{}, IC<0>{}, deal(IC<4>{}));
            } else {
                mac(IC<kk & 1>{}, IC<0>{}, none);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        lds_wait<0>(af[1], bf[1]);
        vm_wait<0>();
        __syncthreads();
        lds_frags<SUB>(af[0], bf[0], row_a + sto_next + so[0], row_b + sto_next + so[0]);
        __builtin_amdgcn_sched_barrier(0);
        mac(IC<1>{}, IC<0>{}, deal(IC<0>{}));
        __builtin_amdgcn_sched_barrier(0);
        if (ks == nk - 1) {
            fold(acc);
            ks = 0;
        } else {
            ++ks;
        }
        sto = sto_next;
    }
    lds_wait<0>(af[0], bf[0]);
    vm_wait<0>();
    __syncthreads();
}

// direct load of four bytes per lane that other XCDs may have changed meanwhile (past the L2 of this one)
__device__ __forceinline__ void gload_lds4_fresh(const void *g, void *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 4, 0, 16);
}

__device__ __forceinline__ int max16(const i32x16 &a) {
    int m = a[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) m = a[i] > m ? a[i] : m;
    return m;
}

// Upper ends travel in LDS as twelve bits, rounded up; the largest of them stands for anything above.
__device__ __forceinline__ unsigned upper_bits(float v) {
    const float x = (v + 1.25f) * (4095.f / 2.5f);
    return x >= 4094.f ? 4095u : x <= 0.f ? 1u : (unsigned)x + 1u;
}
__device__ __forceinline__ float upper_value(unsigned b) { return b >= 4095u ? INFINITY : (float)b * (2.5f / 4095.f) - 1.25f + 1e-6f; }

__device__ __forceinline__ void list_row(uint2 *list, int *cnt, unsigned *low, long q, long row0, long row, long K, float upper) {
    if (row >= K) return;  // (rows past the end are zeros)
    const int slot = atomicAdd(cnt + q, 1);
    if (slot < SCREEN_LIST) list[(size_t)q * SCREEN_LIST + slot] = make_uint2((unsigned)(row0 + row), __float_as_uint(upper));
    else if (slot == SCREEN_LIST) atomicMax(low + q, ordered_bits(INFINITY));  // no list will do: no more of it
}

// Products of the queries of a tile with the rows of a slice.  low[q] = the largest lower end any workgroup has found for
// query q so far (to begin with, the cosine of the best row of a sample); a row whose upper end reaches it goes to the
// query's list.  low only grows, and a stale value lists more rows than needed, never fewer: nothing has to be ordered.
// Rows are collected in LDS and judged by the newest low once more when they are handed over.
// codes, meta and the K rows are a run of the cache's, from its row number row0 on.
// SAMPLE: one tile per workgroup, every `stride`-th of them, and only its best row counts: seed[q] = (product, row); and for
// k_screen_seed, of 128 rows of every tile, the largest cosine and how many come within the error of it (ScreenCrowd; every
// SCREEN_COUNTED-th query).
template <bool LEAVE>
struct LookupSrc {
    const signed char *c, *q;
    int ct, dp, buf;
    const int *lost;
    int most_lost;
    const float4 *meta;
    const unsigned *low;  // of the tile's queries
    float *meta_s;        // [2][64]
    unsigned *low_s;      // [2][256]
    __device__ __forceinline__ bool leave() const { return LEAVE && *lost > most_lost; }
    __device__ __forceinline__ void side(int wave, int lane) {
        if (wave < 4) gload_lds4_fresh(low + wave * 64 + lane, low_s + buf * 256 + wave * 64);
        else if (wave == 4) gload_lds4((const float *)(meta + (size_t)ct * 8) + lane, meta_s + buf * 64);  // (32 of them count)
    }
    __device__ __forceinline__ void advance() {
        c += 256 * (size_t)dp;
        buf ^= 1;
        ++ct;
    }
};
#define SCREEN_LDS (ByteCfg::NSTAGE * ByteCfg::STAGE + 2 * 256 * 4 + 2 * 64 * 4 + 8 * SCREEN_STAGE * 4)
static_assert(SCREEN_LDS <= 160 * 1024, "fits in LDS");

template <bool SAMPLE>
__global__ __launch_bounds__(ByteCfg::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_screen_lookup(
    const signed char *__restrict__ qcodes, const signed char *__restrict__ codes, const float4 *__restrict__ meta,
    const ScreenQuery *__restrict__ qm, unsigned *__restrict__ low, u64 *__restrict__ seed, int *__restrict__ cnt,
    int *__restrict__ near_, float *__restrict__ largest, uint2 *__restrict__ list, long row0, long K, int dp, int tiles_per_slice,
    int slices, int nqt, int qb, int stride, const int *__restrict__ lost, int most_lost) {
    typedef ByteCfg Cfg;
    constexpr int WC = Cfg::WC, WQ = Cfg::WQ, BC = Cfg::BC, BQ = Cfg::BQ;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned *low_s = (unsigned *)(smem + Cfg::NSTAGE * Cfg::STAGE);
    float *meta_s = (float *)(low_s + 2 * 256);
    unsigned *stages = (unsigned *)(meta_s + 2 * 64);  // [8][SCREEN_STAGE]
    int qt, s, ct_begin, ct_end;
    if constexpr (SAMPLE) {
        qt = blockIdx.x % nqt;
        ct_begin = (int)(blockIdx.x / nqt) * stride;
        ct_end = ct_begin + 1;
        if ((long)ct_begin * BC >= K) return;
    } else {
        if (!pipe_map_block<BC>(K, tiles_per_slice, slices, nqt, qb, qt, s, ct_begin, ct_end)) return;
        if (ct_end <= ct_begin) return;
    }
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wc = wave % Cfg::NWC, wq = wave / Cfg::NWC, h = lane >> 5, l32 = lane & 31;
    const long q0 = (long)qt * BQ;
    unsigned *stage = stages + wave * SCREEN_STAGE;
    int mine = 0;  // rows this wave has collected

    float scale[WQ], rscale[WQ], halfw[WQ], grow[WQ], best[WQ];  // per query: scale, 1 / scale, e + slack, (1 + e) / scale; a lower end
#pragma unroll
    for (int b = 0; b < WQ; ++b) {
        const ScreenQuery m = qm[q0 + (wq * WQ + b) * 32 + l32];
        scale[b] = m.scale;
        rscale[b] = 1.f / m.scale;
        halfw[b] = m.err + SCREEN_SLACK;
        grow[b] = (1.f + m.err) * rscale[b];
        best[b] = -INFINITY;
    }
    LookupSrc<!SAMPLE> src;
    src.lost = lost;
    src.most_lost = most_lost;
    src.c = codes + (size_t)ct_begin * BC * dp;
    src.q = qcodes + (size_t)q0 * dp;
    src.ct = ct_begin;
    src.dp = dp;
    src.buf = 0;
    src.meta = meta;
    src.low = low + q0;
    src.meta_s = meta_s;
    src.low_s = low_s;

    if constexpr (SAMPLE) {
        byte_stream(smem, dp, 1, src, [&](const i32x16(&acc)[WC][WQ]) __attribute__((always_inline)) {
            const float4 *mt = (const float4 *)meta_s + wc * WC;
            static_for<0, WQ>([&](auto ib) __attribute__((always_inline)) {
                constexpr int B = decltype(ib)::value;
                float top = -INFINITY;
                int row = 0;
                static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
                    constexpr int A = decltype(ia)::value;
                    const int m = max16(acc[A][B]);
                    const float p = (float)m * mt[A].x;
                    int at = 0;
                    static_for<0, 16>([&](auto ii) __attribute__((always_inline)) {
                        constexpr int I = decltype(ii)::value;
                        if (acc[A][B][I] == m) at = 8 * (I >> 2) + (I & 3);
                    });
                    if (p > top) {
                        top = p;
                        row = ct_begin * BC + (wc * WC + A) * 32 + 4 * h + at;
                    }
                });
                const float ov = __uint_as_float(other_half(__float_as_uint(top)));
                const int orow = (int)other_half((unsigned)row);
                if (ov > top) {
                    top = ov;
                    row = orow;
                }
                if (h == 0) atomicMax(seed + q0 + (wq * WQ + B) * 32 + l32, pack_key(top, (unsigned)row));
                if (wc != 0) return;  // (half of the rows will do for the rest)
                int near = 0;
                static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
                    constexpr int A = decltype(ia)::value;
                    // (as in a lookup's fold; a query that lists nothing has halfw < 0, and zeros for bytes: none of them counts)
                    const int least = (int)floorf((top - halfw[B] * rscale[B] - grow[B] * mt[A].y) * mt[A].w);
                    static_for<0, 16>([&](auto ii) __attribute__((always_inline)) { near += acc[A][B][decltype(ii)::value] >= least ? 1 : 0; });
                });
                near += (int)other_half((unsigned)near);
                if (h == 0 && l32 % SCREEN_COUNTED == 0) {
                    atomicAdd(near_ + q0 + (wq * WQ + B) * 32 + l32, near);
                    atomicAdd(largest + q0 + (wq * WQ + B) * 32 + l32, top * scale[B]);
                }
            });
        });
        return;
    }

    // the rows collected so far go to the lists of their queries (a wave's own: nothing to wait for)
    auto flush = [&]() __attribute__((always_inline)) {
        const int many = mine < SCREEN_STAGE ? mine : SCREEN_STAGE;
#pragma unroll 4
        for (int p = lane; p < many; p += 64) {
            const unsigned e = stage[p];
            const long q = q0 + (e >> 24);
            const float upper = upper_value(e & 0xFFFu);
            if (upper > unordered_bits(__hip_atomic_load(low + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
                list_row(list, cnt, low, q, row0, ct_begin * (long)BC + ((e >> 12) & 0xFFFu), K, upper);
        }
        mine = 0;
    };
    int tile = 0;
    byte_stream(smem, dp, ct_end - ct_begin, src, [&](const i32x16(&acc)[WC][WQ]) __attribute__((always_inline)) {
        const float4 *mt = (const float4 *)(meta_s + (tile & 1) * 64) + wc * WC;
        const unsigned *lt = low_s + (tile & 1) * 256;
        // Upper ends, over the scale of the query: the largest of a column against what it needs is all that most tiles get.
        // (the whole end of a tile with everything below for every block: 2.9 us of 11.4, 768 bytes a row)
        float4 m[WC];
#pragma unroll
        for (int a = 0; a < WC; ++a) m[a] = mt[a];
        float seen[WQ], need[WQ], up[WC][WQ], most[WQ];
        int top[WC][WQ];
        static_for<0, WQ>([&](auto ib) __attribute__((always_inline)) {
            constexpr int B = decltype(ib)::value;
            seen[B] = unordered_bits(lt[(wq * WQ + B) * 32 + l32]);
            need[B] = (fmaxf(seen[B], best[B]) - halfw[B]) * rscale[B];
            most[B] = -INFINITY;
            static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
                constexpr int A = decltype(ia)::value;
                top[A][B] = max16(acc[A][B]);
                // (a query that lists nothing needs +inf, and nothing is larger; where it never did, grow = 0 and the NaN of a
                // block never ruled out is no number to compare)
                up[A][B] = fmaf((float)top[A][B], m[A].x, grow[B] * m[A].y);
                most[B] = fmaxf(most[B], up[A][B]);
            });
        });
        static_for<0, WQ>([&](auto ib) __attribute__((always_inline)) {
            constexpr int B = decltype(ib)::value;
            if (__ballot(most[B] > need[B]) == 0) return;
            const unsigned col = (unsigned)((wq * WQ + B) * 32 + l32);
            float lo = -INFINITY;
            static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
                constexpr int A = decltype(ia)::value;
                lo = fmaxf(lo, fmaf(-grow[B], m[A].z, (float)top[A][B] * m[A].x));
            });
            lo = fmaxf(lo, __uint_as_float(other_half(__float_as_uint(lo))));
            lo = fmaf(scale[B], lo, -halfw[B]);
            if (lo > best[B] && seen[B] < INFINITY) best[B] = lo;
            need[B] = (fmaxf(seen[B], best[B]) - halfw[B]) * rscale[B];
            // (in steps of a thousandth: a bound that is a little low lists a few rows more)
            if (h == 0 && lo > seen[B] + 1e-3f) atomicMax(low + q0 + col, ordered_bits(lo));
            static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
                constexpr int A = decltype(ia)::value;
                if (__ballot(up[A][B] > need[B]) == 0) return;
                // the bound as an integer, rounded down: the three operations are off by some 2^-22 of the product that would
                // be needed, a cosine of at most about one, and the slack is 2e-5 of that whatever the scale.  No scale (rows of
                // zeros): plus or minus infinity, or a NaN, which converts to 0
                const int least = up[A][B] > need[B] ? (int)floorf((need[B] - grow[B] * m[A].y) * m[A].w) : 0x7FFFFFFF;
                // one upper end for the rows of a lane, mostly one: that of the largest
                const int rel0 = tile * BC + (wc * WC + A) * 32 + 4 * h;  // register I holds row rel0 + 8 * (I / 4) + I % 4
                const unsigned upper = upper_bits(fmaf(scale[B], up[A][B], halfw[B]));
                const unsigned entry = (col << 24) | ((unsigned)rel0 << 12) | upper;
                static_for<0, 16>([&](auto ii) __attribute__((always_inline)) {
                    constexpr int I = decltype(ii)::value, ROW = 8 * (I >> 2) + (I & 3);
                    const u64 mask = __ballot(acc[A][B][I] >= least);
                    if (mask == 0) return;
                    if (acc[A][B][I] >= least) {
                        const int pos = mine + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                        if (pos < SCREEN_STAGE) stage[pos] = entry + (ROW << 12);
                        else list_row(list, cnt, low, q0 + col, row0, ct_begin * (long)BC + rel0 + ROW, K, upper_value(upper));
                    }
                    mine += __popcll(mask);
                });
            });
        });
        ++tile;
        if (mine > SCREEN_STAGE / 2) flush();
    });
    flush();
}

// Queries of this wave: its row in LDS as chunks (or left where it is), and 1 / |q| with the sums of k_lookup_finalize (the
// squares as its four waves add them).
template <typename T>
__device__ __forceinline__ float stage_query(const T *qrow, int d, int vec, u32x4_t *sh_q) {
    constexpr int EPC = 16 / (int)sizeof(T), CH = (SISO_SCREEN_DIM / EPC + 255) / 256;  // chunks a thread of k_lookup_finalize takes
    const int lane = threadIdx.x & 63;
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        u32x4_t v[4][CH];
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int e = (w * 64 + lane + 256 * c) * EPC;
                v[w][c] = *(const u32x4_t *)(qrow + (e < d ? e : 0));
            }
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int e = (w * 64 + lane + 256 * c) * EPC;
                if (e < d) {
                    sh_q[e / EPC] = v[w][c];
                    ss[w] += chunk_dot(v[w][c], v[w][c], T());
                }
            }
    } else {
#pragma unroll
        for (int w = 0; w < 4; ++w)
            for (int e = w * 64 + lane; e < d; e += 256) ss[w] += widen(qrow[e]) * widen(qrow[e]);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) ss[w] = wave_sum(ss[w]);
    return inv_length((ss[0] + ss[1]) + (ss[2] + ss[3]));
}

// The deviations above the mean that a share p of a normal distribution exceeds (Abramowitz and Stegun, 26.2.23).
__device__ __forceinline__ float normal_above(float p) {
    const float t = sqrtf(-2.f * __logf(p < 0.5f ? p : 1.f - p));
    const float z = t - (2.515517f + t * (0.802853f + t * 0.010328f)) / (1.f + t * (1.432788f + t * (0.189269f + t * 0.001308f)));
    return p < 0.5f ? z : -z;
}

// The share of the rows that a query lists whose bound is `bound`, from what the sample has left of it: of 128 rows at a time
// the mean of the largest cosine, and how many came within the error of that (`near`).  The cosines of unrelated rows are near
// enough to normal, and only the time of a call depends on this: the largest of 128 lies where 0.56 / 128 of the
// distribution is above it (the median), and from there the number within the error gives the error in deviations.
__device__ __forceinline__ float listed_share(float bound, float largest, float near, float error) {
    const float z = normal_above(0.56f / 128.f);
    const float width = z - normal_above(fminf(near, 127.f) / 128.f);
    return 0.5f * erfcf((z + ((bound - largest) / error - 1.f) * width) * 0.70710678f);
}

// What k_screen_seed goes by to count a query as lost.
struct ScreenCrowd {
    const int *near;       // per query, over the `groups` of 128 rows of the sample: how many came within the error of the largest
    const float *largest;  // and the sum of the largest cosines
    float groups;
    float rows, most;      // of so many rows it may list so many
    int heavy;             // LISTED: rows that still count
    int *lost;
    int most_lost;
};

// A better bound, a wave for each query: the cosine with its best row of the sample (seed), or with the row of the highest
// upper end that is listed so far (the bound was short of it by the error).  And *lost counts the queries whose lists can be
// foreseen to flood, or to take more work than the products save.
template <typename T, bool LISTED>
__global__ __launch_bounds__(256) void k_screen_seed(const T *__restrict__ Q, const T *__restrict__ cent, const float *__restrict__ invn,
                                                     long n, long K, int d, int vec, const ScreenQuery *__restrict__ qm,
                                                     const float4 *__restrict__ meta, const u64 *__restrict__ seed,
                                                     const int *__restrict__ cnt, const uint2 *__restrict__ list,
                                                     unsigned *__restrict__ low, ScreenCrowd crowd) {
    __shared__ u32x4_t sh_q[4][SISO_SCREEN_DIM * sizeof(T) / 16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long q = (long)blockIdx.x * 4 + wave;
    if (q >= n || (LISTED && *crowd.lost > crowd.most_lost)) return;
    const float had = unordered_bits(low[q]);
    const int many = LISTED ? cnt[q] : 0, listed = many < SCREEN_LIST ? many : SCREEN_LIST;
    if (had == INFINITY && many <= SCREEN_LIST) return;  // (no list)
    bool lost = many > SCREEN_LIST;
    if (!lost) {
        long r = K;
        if constexpr (LISTED) {
            u64 high = 0;
            for (int i = lane; i < listed; i += 64) {
                const uint2 e = list[(size_t)q * SCREEN_LIST + i];
                const u64 key = pack_key(__uint_as_float(e.y), e.x);
                high = key > high ? key : high;
            }
            high = wave_max(high);
            if (high != 0) r = (long)(0xFFFFFFFFu - (unsigned)(high & 0xFFFFFFFFull));
        } else {
            if (seed[q] != 0) r = (long)(0xFFFFFFFFu - (unsigned)(seed[q] & 0xFFFFFFFFull));
        }
        float bound = had, error = INFINITY, largest = 0.f, near = 0.f;
        const bool counted = q % SCREEN_COUNTED == 0;
        if (!LISTED && r < K && counted) {
            const float e = qm[q].err;
            error = e + (1.f + e) * meta[r >> 5].y + SCREEN_SLACK;
            largest = crowd.largest[q] / crowd.groups;
            near = (float)crowd.near[q] / crowd.groups;
        }
        if (r < K) {
            const T *qrow = Q + (size_t)q * d;
            const float qi = stage_query(qrow, d, vec, sh_q[wave]);
            const float cosine = row_product<T>(qrow, sh_q[wave], vec, cent + (size_t)r * d, d, lane) * qi * invn[r];
            if (cosine == cosine) bound = fmaxf(bound, cosine - 5e-6f);
        }
        if constexpr (LISTED) {
            int left = 0;
            for (int i = lane; i < (counted ? listed : 0); i += 64)
                left += __popcll(__ballot(__uint_as_float(list[(size_t)q * SCREEN_LIST + i].y) > bound));
            left = __builtin_amdgcn_readfirstlane(left);  // (lane 0 has taken part in every round)
            lost = left > crowd.heavy;
        } else if (r < K && counted && crowd.most_lost != SCREEN_WHOLE) {
            lost = listed_share(bound, largest, near, error) * crowd.rows > crowd.most;
        }
        if (lane == 0 && bound > had) low[q] = ordered_bits(bound);
    }
    if (lane == 0 && lost && q % SCREEN_COUNTED == 0) atomicAdd(crowd.lost, 1);
}

// The end of a screened lookup in three steps, so that the long lists (a query that misses leaves up to some hundred rows, one
// that hits its 16 neighbours) are spread over the whole chip: with a workgroup for each query, or for four, the
// longest list decided (4,096 queries, 30 % misses: 65 to 78 us; so 48).
// First step, a wave for each query: the bound, with the cosine of the listed row of the highest upper end (the bound is
// then no longer short of the best by twice the error but by once); the listed rows that reach it go to one list of all
// queries.  Queries that are left to the other kernels are numbered and their rows gathered.  The queries of a workgroup take their room
// in the list together: the additions queue for one counter, 10 ns each (how many there are: screen_launch).
struct ScreenWork {
    int q, row;
};
#define PICK_WAVES 16  // at most
template <typename T>
__global__ __launch_bounds__(PICK_WAVES * 64) void k_screen_pick(const T *__restrict__ Q, const T *__restrict__ cent, const float *__restrict__ invn,
                                                     long n, int d, int vec, const unsigned *__restrict__ low,
                                                     const int *__restrict__ cnt, const uint2 *__restrict__ list,
                                                     int *__restrict__ totals, int most_lost, ScreenWork *__restrict__ work,
                                                     int work_room, u64 *__restrict__ best, float *__restrict__ qinv,
                                                     int *__restrict__ plain_of, T *__restrict__ plain_rows) {
    __shared__ u32x4_t sh_q[PICK_WAVES][SISO_SCREEN_DIM * sizeof(T) / 16];
    __shared__ int sh_n[PICK_WAVES];
    __shared__ int sh_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const long q = (long)blockIdx.x * waves + wave;
    const T *qrow = Q + (size_t)(q < n ? q : 0) * d;
    const uint2 *ql = list + (size_t)(q < n ? q : 0) * SCREEN_LIST;
    const uint2 e0 = ql[lane];  // (beyond the list: anything, not looked at)
    const int listed = q < n ? cnt[q] : 0;
    float bound = unordered_bits(low[q < n ? q : 0]);
    const float qi = stage_query(qrow, d, vec, sh_q[wave]);
    // (a bound of +inf: no list, or one that was given up)
    const bool all = totals[2] > most_lost;  // the whole batch was given up: it stays in its order
    bool leave = all || (listed != SCREEN_NAN && (listed == SCREEN_PLAIN || listed > SCREEN_LIST || bound == INFINITY));
    u64 mine = 0;
    int first = -1, some = 0;
    if (!leave && listed > 0) {
        u64 high = lane < listed ? pack_key(__uint_as_float(e0.y), e0.x) : 0;
        for (int i = lane + 64; i < listed; i += 64) {
            const uint2 e = ql[i];
            const u64 key = pack_key(__uint_as_float(e.y), e.x);
            high = key > high ? key : high;
        }
        high = wave_max(high);
        first = (int)(0xFFFFFFFFu - (unsigned)(high & 0xFFFFFFFFull));
        const float sv = row_product<T>(qrow, sh_q[wave], vec, cent + (size_t)first * d, d, lane) * qi * invn[first];
        if (sv == sv) {  // a NaN never wins
            bound = fmaxf(bound, sv - 5e-6f);
            mine = pack_key(sv, (unsigned)first);
        }
        for (int i = lane; i < listed; i += 64) {
            const uint2 e = i < 64 ? e0 : ql[i];
            some += __popcll(__ballot((int)e.x != first && __uint_as_float(e.y) > bound));
        }
        some = __builtin_amdgcn_readfirstlane(some);
    }
    if (lane == 0) sh_n[wave] = some;
    __syncthreads();
    if (threadIdx.x == 0) {
        int more = 0;
        for (int w = 0; w < waves; ++w) more += sh_n[w];
        sh_base = more > 0 ? atomicAdd(totals, more) : 0;
        if (all && blockIdx.x == 0) totals[1] = (int)n;
    }
    __syncthreads();
    if (q >= n) return;
    int at = sh_base;
    for (int w = 0; w < wave; ++w) at += sh_n[w];
    if (at + some > work_room) leave = true;  // (the entries behind work_room are not read)
    for (int i = lane; i < listed && some > 0; i += 64) {
        const uint2 e = i < 64 ? e0 : ql[i];
        const bool take = (int)e.x != first && __uint_as_float(e.y) > bound;
        const u64 mask = __ballot(take);
        const int to = at + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
        if (take && to < work_room) work[to] = ScreenWork{(int)q, (int)e.x};
        at += __popcll(mask);
    }
    int place = -1;
    if (leave) {
        if (lane == 0) place = all ? (int)q : atomicAdd(totals + 1, 1);
        place = __builtin_amdgcn_readfirstlane(place);
        T *to = plain_rows + (size_t)place * d;
        if (vec)
            for (int e = lane; e < d * (int)sizeof(T) / 16; e += 64) ((u32x4_t *)to)[e] = sh_q[wave][e];
        else
            for (int e = lane; e < d; e += 64) to[e] = qrow[e];
        if (lane == 0) plain_of[place] = (int)q;
    }
    if (lane == 0) {
        best[q] = leave ? ~0ull : mine;  // (nothing is larger, and no cosine)
        qinv[q] = qi;
    }
}

// Second step, a wave for four rows at a time: the cosines, with the sums of k_lookup_finalize; best[q] = (cosine, lowest row).
template <typename T>
__global__ __launch_bounds__(256) void k_screen_score(const T *__restrict__ Q, const T *__restrict__ cent, const float *__restrict__ invn,
                                                      int d, int vec, const int *__restrict__ totals,
                                                      const ScreenWork *__restrict__ work, int work_room,
                                                      const float *__restrict__ qinv, u64 *__restrict__ best) {
    constexpr int EPC = 16 / (int)sizeof(T), R = 4;
    const int lane = threadIdx.x & 63;
    const int many = totals[0] < work_room ? totals[0] : work_room;
    for (int i = (blockIdx.x * 4 + (threadIdx.x >> 6)) * R; i < many; i += gridDim.x * 4 * R) {
        const T *rows[R], *qrows[R];
        int row[R], q[R];
        float sum[R], by[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const ScreenWork w = work[i + r < many ? i + r : i];
            row[r] = __builtin_amdgcn_readfirstlane(w.row);
            q[r] = __builtin_amdgcn_readfirstlane(w.q);
            rows[r] = cent + (size_t)row[r] * d;
            qrows[r] = Q + (size_t)q[r] * d;
            by[r] = qinv[q[r]];
            sum[r] = 0.f;
        }
        if (vec) {  // as row_products, the query from memory too
            for (int e0 = lane * EPC; e0 < d; e0 += 2 * 64 * EPC) {
                const int e1 = e0 + 64 * EPC, f1 = e1 < d ? e1 : 0;
                u32x4_t c0[R], c1[R], q0[R], q1[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    c0[r] = *(const u32x4_t *)(rows[r] + e0);
                    c1[r] = *(const u32x4_t *)(rows[r] + f1);
                    q0[r] = *(const u32x4_t *)(qrows[r] + e0);
                    q1[r] = *(const u32x4_t *)(qrows[r] + f1);
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    sum[r] += chunk_dot(q0[r], c0[r], T());
                    const float part = chunk_dot(q1[r], c1[r], T());
                    sum[r] += e1 < d ? part : 0.f;
                }
            }
        } else {
            for (int e = lane; e < d; e += 64)
#pragma unroll
                for (int r = 0; r < R; ++r) sum[r] += widen(qrows[r][e]) * widen(rows[r][e]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float sv = wave_sum(sum[r]) * by[r] * invn[row[r]];
            if (lane == 0 && sv == sv) atomicMax(best + q[r], pack_key(sv, (unsigned)row[r]));
        }
    }
}

// Third step, a thread for each query.
__global__ __launch_bounds__(256) void k_screen_write(long n, long q_base, const int *__restrict__ cnt, const u64 *__restrict__ best,
                                                      ThetaList thetas, int *out_idx, float *out_sim, unsigned char *out_hit,
                                                      unsigned *access, int *upd_owner, int *upd_members) {
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q >= n) return;
    const u64 key = best[q];
    if (key == ~0ull) return;
    const long idx = key == 0 ? -1 : (long)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
    const float sim = cnt[q] == SCREEN_NAN ? __uint_as_float(0x7FC00000u) : key == 0 ? -INFINITY : unordered_bits((unsigned)(key >> 32));
    write_lookup(q, q_base, idx, sim, thetas, out_idx, out_sim, out_hit, access, upd_owner, upd_members);
}

// ---- pairs ---------------------------------------------------------------------------------------------------------
// All pairs i < j above a threshold, from bytes: a pair whose lower end exceeds it is a pair, one whose upper end does not
// is none, and the cosines of the few between are formed anew (k_screen_pairs_check).  Error and scale belong to the two
// blocks of 32 rows, so a block of 32 x 32 products is dismissed by one comparison of its largest integer.
struct PairSrc {
    const signed char *c, *q, *codes;
    const float4 *meta;
    float *meta_s;  // [2][2][64]: row tile, column tile
    PairItems items;
    int ct, qt, dp, buf;
    __device__ __forceinline__ bool leave() const { return false; }
    __device__ __forceinline__ void side(int wave, int lane) {
        if (wave < 2) gload_lds4((const float *)(meta + (size_t)(wave == 0 ? ct : qt) * 8) + lane, meta_s + (buf * 2 + wave) * 64);
    }
    __device__ __forceinline__ void take() {
        c = codes + (size_t)ct * 256 * dp;
        q = codes + (size_t)qt * 256 * dp;
    }
    __device__ __forceinline__ void advance() {
        buf ^= 1;
        items.next(qt, ct);
        take();
    }
};
#define SCREEN_PAIR_STAGE 224  // pairs a wave collects in LDS, and as many in doubt
#define SCREEN_PAIR_LDS (ByteCfg::NSTAGE * ByteCfg::STAGE + 4 * 64 * 4 + 8 * 2 * SCREEN_PAIR_STAGE * 8)
static_assert(SCREEN_PAIR_LDS <= 160 * 1024, "fits in LDS");
enum { PAIRS_ALL, PAIRS_FIRST, PAIRS_REST };  // what a launch takes of every workgroup's pairs of tiles

__global__ __launch_bounds__(ByteCfg::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_screen_pairs(
    const signed char *__restrict__ codes, const float4 *__restrict__ meta, long K, int dp, int qb, int part, float threshold,
    int *__restrict__ out_pairs, long cap, u64 *__restrict__ counter, int *__restrict__ maybe, u64 maybe_room,
    u64 *__restrict__ maybe_count) {
    if (part == PAIRS_REST && *maybe_count > maybe_room) return;  // (they will all be searched for anew)
    typedef ByteCfg Cfg;
    constexpr int WC = Cfg::WC, WQ = Cfg::WQ, BC = Cfg::BC;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *meta_s = (float *)(smem + Cfg::NSTAGE * Cfg::STAGE);
    const int tiles = (int)((K + BC - 1) / BC);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wc = wave % Cfg::NWC, wq = wave / Cfg::NWC, h = lane >> 5, l32 = lane & 31;
    PairSrc src;
    PairItems done;
    src.items.init(tiles, qb);
    done.init(tiles, qb);
    src.codes = codes;
    src.meta = meta;
    src.meta_s = meta_s;
    src.dp = dp;
    src.buf = 0;
    src.qt = src.ct = 0;
    int qt = 0, ct = 0, seq = 0, pairs = src.items.count();
    if (part != PAIRS_ALL) {
        const int first = (pairs + 7) / 8;
        if (part == PAIRS_FIRST) {
            pairs = first;
        } else {
            pairs -= first;
            src.items.skip(first);
            done.skip(first);
        }
    }
    if (pairs == 0) return;
    src.items.next(src.qt, src.ct);
    done.next(qt, ct);
    src.take();
    // the pairs this wave has found, and those in doubt, handed over when they may not hold those of another instruction (a wave's
    // own: nothing to wait for, which a buffer of the workgroup would at the end of every tile; and one atomic addition for some
    // hundred pairs: they all go to one address, 10 ns each)
    int2 *stage = (int2 *)(meta_s + 4 * 64) + wave * 2 * SCREEN_PAIR_STAGE, *doubt = stage + SCREEN_PAIR_STAGE;
    int mine = 0, doubts = 0;
    int over = 0;  // more in doubt than there is room for: all of this is searched for anew
    auto put = [&](u64 base) __attribute__((always_inline)) {
        for (int p = lane; p < mine; p += 64)
            if (base + (u64)p < (u64)cap) {  // (the caller's array: aligned to an int)
                const int2 e = stage[p];
                out_pairs[2 * (base + p)] = e.x;
                out_pairs[2 * (base + p) + 1] = e.y;
            }
    };
    auto put_doubts = [&](u64 base) __attribute__((always_inline)) {
        for (int p = lane; p < doubts; p += 64)
            if (base + (u64)p < maybe_room) ((int2 *)maybe)[base + p] = doubt[p];
    };
    auto flush = [&]() __attribute__((always_inline)) {
        u64 base = 0;
        if (lane == 0 && mine > 0) base = atomicAdd(counter, (u64)mine);
        put(__shfl(base, 0));
        mine = 0;
    };
    auto flush_doubts = [&]() __attribute__((always_inline)) {
        u64 base = 0;
        if (lane == 0 && doubts > 0) base = atomicAdd(maybe_count, (u64)doubts);
        base = __shfl(base, 0);
        put_doubts(base);
        over = __builtin_amdgcn_readfirstlane(base + (u64)doubts > maybe_room ? 1 : 0);
        doubts = 0;
    };
    byte_stream(smem, dp, pairs, src, [&](const i32x16(&acc)[WC][WQ]) __attribute__((always_inline)) {
        const float4 *ma = (const float4 *)(meta_s + (seq & 1) * 128) + wc * WC;
        const float4 *mb = (const float4 *)(meta_s + (seq & 1) * 128 + 64) + wq * WQ;
        float4 a[WC], b[WQ];
#pragma unroll
        for (int x = 0; x < WC; ++x) a[x] = ma[x];
#pragma unroll
        for (int x = 0; x < WQ; ++x) b[x] = mb[x];
        float up[WC][WQ], most = -INFINITY;
        static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
            constexpr int A = decltype(ia)::value;
            static_for<0, WQ>([&](auto ib) __attribute__((always_inline)) {
                constexpr int B = decltype(ib)::value;
                up[A][B] = fmaf((float)max16(acc[A][B]), a[A].x * b[B].x, fmaf(1.f + a[A].y, b[B].y, a[A].y) + SCREEN_SLACK);
                most = fmaxf(most, up[A][B]);
            });
        });
        if (over == 0 && __ballot(most > threshold) != 0) static_for<0, WC>([&](auto ia) __attribute__((always_inline)) {
            constexpr int A = decltype(ia)::value;
            static_for<0, WQ>([&](auto ib) __attribute__((always_inline)) {
                constexpr int B = decltype(ib)::value;
                if (__ballot(up[A][B] > threshold) == 0) return;
                const float scale = a[A].x * b[B].x, err = fmaf(1.f + a[A].y, b[B].y, a[A].y) + SCREEN_SLACK;
                // as an integer (see k_screen_lookup); without a scale the products are zeros, below any threshold but for a block
                // that is never ruled out
                const int least = scale > 0.f ? (int)floorf((threshold - err) / scale) : err > threshold ? 0 : 1;
                const int icol = qt * BC + (wq * WQ + B) * 32 + l32;
                const int jrow0 = ct * BC + (wc * WC + A) * 32 + 4 * h;  // register I holds row jrow0 + 8 * (I / 4) + I % 4
                static_for<0, 16>([&](auto ii) __attribute__((always_inline)) {
                    constexpr int I = decltype(ii)::value;
                    const bool near = acc[A][B][I] >= least;
                    if (__ballot(near) == 0) return;
                    const int j = jrow0 + 8 * (I >> 2) + (I & 3);
                    const float p = (float)acc[A][B][I] * scale;
                    const bool sure = near && icol < j && j < K && p - err > threshold, open = near && icol < j && j < K && !sure;
                    const u64 yes = __ballot(sure), maybe_so = __ballot(open);
                    auto before = [&](u64 mask) { return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u)); };
                    if (mine > SCREEN_PAIR_STAGE - 64) flush();
                    if (sure) stage[mine + before(yes)] = make_int2(icol, j);
                    mine += __popcll(yes);
                    if (doubts > SCREEN_PAIR_STAGE - 64) {
                        if (over == 0) flush_doubts();
                        else doubts = 0;
                    }
                    if (open) doubt[doubts + before(maybe_so)] = make_int2(icol, j);
                    doubts += __popcll(maybe_so);
                });
            });
        });
        ++seq;
        done.next(qt, ct);
    });
    // What is left goes out together: every wave for itself, 2,048 additions would queue for either counter behind shares that all
    // end at the same time (rows in groups of eight, us: 12,000 x 768 122.5 -> 115.7, 20,000 x 256 171 -> 146).  (The stages hold nothing
    // any more.)
    int *const ends = (int *)smem;           // [2][8]
    u64 *const bases = (u64 *)(smem + 64);
    if (lane == 0) {
        ends[wave] = mine;
        ends[8 + wave] = doubts;
    }
    __syncthreads();
    if (const int tid = threadIdx.x; tid < 2) {
        int all = 0;
        for (int w = 0; w < 8; ++w) all += ends[8 * tid + w];
        bases[tid] = all > 0 ? atomicAdd(tid == 0 ? counter : maybe_count, (u64)all) : 0;
    }
    __syncthreads();
    u64 base = bases[0], base_doubt = bases[1];
    for (int w = 0; w < wave; ++w) {
        base += (u64)ends[w];
        base_doubt += (u64)ends[8 + w];
    }
    put(base);
    put_doubts(base_doubt);
}

__global__ void k_screen_clear(u64 *maybe_count) { *maybe_count = 0; }

// Behind the first eighth: more in doubt already than their share of the room: the list will not hold.
__global__ void k_screen_pairs_judge(u64 *maybe_count, u64 most, u64 room) {
    if (*maybe_count > most) *maybe_count = room + 1;
}

// The pairs in doubt, a wave for four at a time.  More of them than the list holds: nothing is kept, and the kernels of all pairs
// (which look at the same count) do the search.  The pairs that are found are collected in LDS: additions to the one counter
// take 10 ns each (16,000 x 768, rows in groups of eight around the threshold: 518 -> 191 us).
template <typename T>
__global__ __launch_bounds__(256) void k_screen_pairs_check(const T *__restrict__ rows, const float *__restrict__ invn, int d, int vec,
                                                            float threshold, const int *__restrict__ maybe, u64 maybe_room,
                                                            const u64 *__restrict__ maybe_count, int *__restrict__ out_pairs, long cap,
                                                            u64 *__restrict__ counter) {
    constexpr int R = 4, EPC = 16 / (int)sizeof(T);
    __shared__ int2 found[4][64];
    __shared__ int sh_n[4];
    __shared__ u64 sh_base;
    const u64 many = *maybe_count;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (many > maybe_room) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *counter = 0;
        return;
    }
    int mine = 0;  // pairs this wave has found: at most 64
    auto hand_over = [&](u64 base) {
        if (lane < mine && base + (u64)lane < (u64)cap) {  // (the caller's array: aligned to an int)
            out_pairs[2 * (base + lane)] = found[wave][lane].x;
            out_pairs[2 * (base + lane) + 1] = found[wave][lane].y;
        }
    };
    for (u64 p = ((u64)blockIdx.x * 4 + wave) * R; p < many; p += (u64)gridDim.x * 4 * R) {
        int i[R], j[R];
        const T *a[R], *b[R];
        float s[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const u64 at = p + r < many ? p + r : p;
            i[r] = maybe[2 * at];
            j[r] = maybe[2 * at + 1];
            a[r] = rows + (size_t)i[r] * d;
            b[r] = rows + (size_t)j[r] * d;
            s[r] = 0.f;
        }
        if (vec) {
            for (int e = lane * EPC; e < d; e += 64 * EPC) {
                u32x4_t x[R], y[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    x[r] = *(const u32x4_t *)(a[r] + e);
                    y[r] = *(const u32x4_t *)(b[r] + e);
                }
#pragma unroll
                for (int r = 0; r < R; ++r) s[r] += chunk_dot(x[r], y[r], T());
            }
        } else {
            for (int e = lane; e < d; e += 64)
#pragma unroll
                for (int r = 0; r < R; ++r) s[r] += widen(a[r][e]) * widen(b[r][e]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float cosine = wave_sum(s[r]) * invn[i[r]] * invn[j[r]];
            if (__builtin_amdgcn_readfirstlane(cosine > threshold && p + r < many ? 1 : 0) != 0) {
                if (lane == 0) found[wave][mine] = make_int2(i[r], j[r]);
                ++mine;
            }
        }
        if (mine > 64 - R) {
            u64 base = 0;
            if (lane == 0) base = atomicAdd(counter, (u64)mine);
            hand_over(__shfl(base, 0));
            mine = 0;
        }
    }
    if (lane == 0) sh_n[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int all = sh_n[0] + sh_n[1] + sh_n[2] + sh_n[3];
        sh_base = all > 0 ? atomicAdd(counter, (u64)all) : 0;
    }
    __syncthreads();
    u64 base = sh_base;
    for (int w = 0; w < wave; ++w) base += (u64)sh_n[w];
    hand_over(base);
}

// ---------------------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------------------
namespace {

struct ByteStore {  // see ByteRows
    signed char *codes;
    float4 *meta;
    u64 *made;
    size_t bytes;
};

struct ScreenRoom {
    signed char *codes, *qcodes;
    float4 *meta;
    ScreenQuery *qm;
    unsigned *low;
    u64 *seed, *best;
    int *cnt, *near, *totals, *plain_of, *maybe;
    float *qinv, *largest;
    uint2 *list;
    ScreenWork *work;
    int work_room;
    void *plain_rows;
    u64 *maybe_count, maybe_room;
    size_t bytes;
};

int byte_dim(int d) { return d <= 256 ? 256 : (d + 127) / 128 * 128; }
long up256(long x) { return (x + 255) / 256 * 256; }
// of a bf16 product: bytes are multiplied twice as fast, but in rows of 256 bytes and whole multiples of 128
double saved_dim(int d) { return d - byte_dim(d) / 2.0; }

// Rows that a query on average can have multiplied again before the kernels of all products are the better way.
// One row takes about a nanosecond (0.1 ms for 96,000 of 768 bf16 elements), all products of a query 150 ns for 131,072 of
// them, and 393 for 60,000 of 384 in single precision, whose matrix cores are a sixteenth as fast (1,000 such queries that miss,
// mean cosine 0.7: 484 us with 96 rows each, 264 with 312).
int again_per_query(const siso_cache *c, long rows) {
    const long most = rows / (c->dtype == SISO_F32 ? 192 : 1024);
    return (int)(most < 96 ? 96 : most > SCREEN_LIST ? SCREEN_LIST : most);
}

// Pairs that can be in doubt before the search of all pairs is the better way: half of what that takes, at 0.6 ns for a pair of
// bf16 rows of 768 elements (65,536 of them in groups of 32 around the threshold, a million pairs in doubt: 1,495 -> 2,025 us,
// all pairs 3,121).
long pairs_in_doubt(const siso_cache *c, long rows) {
    const bool f32 = c->dtype == SISO_F32;
    const double all = (double)rows * (double)rows * c->dim / (f32 ? 1.13e5 : 1.25e6);  // ns
    const double most = all / 2 / (0.6 * c->dim * (f32 ? 4.0 : 2.0) / 1536);
    return most < 65536 ? 65536 : most > 16777216 ? 16777216 : (long)most;
}

ByteStore byte_store(char *base, const siso_cache *c, long rows) {
    Carver a{base};
    ByteStore s;
    s.made = a.take<u64>((size_t)up256(rows) / 32);
    s.meta = a.take<float4>((size_t)up256(rows) / 32 + 8);
    s.codes = a.take<signed char>((size_t)up256(rows) * byte_dim(c->dim));
    s.bytes = a.used;
    return s;
}

// for lookups of up to n queries (n = 0: for a pair search, with the bytes of its rows)
ScreenRoom screen_room(char *base, const siso_cache *c, long rows, long n) {
    const int d = c->dim;
    const int dp = byte_dim(d);
    const long q = up256(n < SISO_SCREEN_PIECE ? n : SISO_SCREEN_PIECE);
    Carver a{base};
    ScreenRoom r;
    const size_t pair_rows = n == 0 ? (size_t)up256(rows) : 0;
    r.codes = a.take<signed char>(pair_rows * dp);
    r.meta = a.take<float4>(pair_rows / 32 + 8);
    r.qcodes = a.take<signed char>((size_t)q * dp);
    r.qm = a.take<ScreenQuery>(q);
    r.low = a.take<unsigned>(q);
    r.seed = a.take<u64>(q);
    r.best = a.take<u64>(q);
    r.cnt = a.take<int>(q);
    r.near = a.take<int>(q);
    r.largest = a.take<float>(q);
    r.totals = a.take<int>(3);  // rows to be multiplied again, queries left to the other kernels, queries counted as lost
    r.plain_of = a.take<int>(q);
    r.plain_rows = a.take<char>((size_t)q * d * (c->dtype == SISO_F32 ? 4 : 2));
    r.qinv = a.take<float>(q);
    r.work_room = (int)q * again_per_query(c, rows);
    r.work = a.take<ScreenWork>((size_t)r.work_room);
    r.list = a.take<uint2>((size_t)q * SCREEN_LIST);
    r.maybe_count = a.take<u64>(1);
    r.maybe_room = n == 0 ? (u64)pairs_in_doubt(c, rows) : 0;
    r.maybe = a.take<int>(2 * (size_t)r.maybe_room);
    r.bytes = a.used;
    return r;
}

bool capturing(const siso_cache *c) {
    if (c->stream == nullptr) return false;  // (the null stream cannot be captured, and to ask takes 0.2 us)
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
}

bool take(char **at, size_t bytes) {
    if (hipMalloc((void **)at, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *at = nullptr;
    return false;
}

// Room for `bytes`; false = there is none, which no caller needs to fail for.  keep: where the old room goes if it must stay
// (NULL: it is freed).  The old room is given up only for the new one: a call that cannot have more leaves what smaller ones use.
bool make_room(siso_cache *c, ScreenSpace &room, size_t bytes, std::vector<char *> *keep) {
    if (bytes <= room.cap) return true;
    if (capturing(c) || (room.refused != 0 && bytes >= room.refused)) return false;
    if (c->opt_screen_room > 0 && bytes > (size_t)c->opt_screen_room << 10) {
        room.refused = bytes;
        return false;
    }
    char *larger = nullptr;
    bool have = take(&larger, bytes);
    if (room.at && (have || !keep)) {
        if (have && keep) {
            keep->push_back(room.at);  // (room for it: siso_screen_lookup)
        } else {
            if (hipStreamSynchronize(c->stream) != hipSuccess) {
                (void)hipGetLastError();
                if (larger) (void)hipFree(larger);
                return false;
            }
            (void)hipFree(room.at);
        }
        room.at = nullptr;
        if (!have) {  // perhaps with what it had
            have = take(&larger, bytes);
            if (!have && !take(&room.at, room.cap)) room.cap = 0;
        }
    }
    if (!have) {
        room.refused = bytes;
        return false;
    }
    room.at = larger;
    room.cap = bytes;
    return true;
}

// rows (those of `tiles`, if with_rows) and n queries to bytes
template <typename T>
int write_bytes(siso_cache *c, const ScreenRoom &r, const ByteStore &s, const unsigned *version, const T *rows, const float *invn, long count,
                bool with_rows, const T *queries, long n, const ScreenTiles &tiles, int most_lost, float least) {
    const int d = c->dim, dp = byte_dim(d);
    const long all = up256(count) / 256;
    const unsigned row_blocks = !with_rows ? 0u : 8u * (unsigned)(tiles.part == 0 ? all : tiles.part == 1 ? tiles.ahead + tiles.some : all - tiles.ahead);
    const dim3 grid(row_blocks + (unsigned)(up256(n) / 32)), block(256);
    if (s.made && with_rows) c->bytes.written = 1;
    const size_t four = 4 * sizeof(T);  // rows that are whole runs of four elements, aligned to them
    const int rv = d % 4 == 0 && (uintptr_t)rows % four == 0 ? 1 : 0, qv = d % 4 == 0 && (uintptr_t)queries % four == 0 ? 1 : 0;
#define SISO_LAUNCH_BYTES2(NCH, PARTS)                                                                                        \
    hipLaunchKernelGGL((k_screen_bytes<T, NCH, PARTS>), grid, block, 0, c->stream, rows, invn, count, row_blocks, rv, s.codes, s.meta, \
                       queries, n, qv, r.qcodes, r.qm, r.low, r.seed, r.cnt, r.near, r.largest, r.totals, d, dp, tiles, most_lost, least, \
                       version, s.made)
#define SISO_LAUNCH_BYTES(NCH)                      \
    if (tiles.part == 0) SISO_LAUNCH_BYTES2(NCH, false); \
    else SISO_LAUNCH_BYTES2(NCH, true)
    if (dp <= 256) {
        SISO_LAUNCH_BYTES(1);
    } else if (dp <= 512) {
        SISO_LAUNCH_BYTES(2);
    } else if (dp <= 768) {
        SISO_LAUNCH_BYTES(3);
    } else {
        SISO_LAUNCH_BYTES(4);
    }
#undef SISO_LAUNCH_BYTES
#undef SISO_LAUNCH_BYTES2
    return siso_check_hip(c, hipGetLastError(), "k_screen_bytes");
}

template <typename T>
int screen_launch(siso_cache *c, const T *queries, long n, bool with_rows, bool whole, const ThetaList &tl, long q_base, int *out_idx,
                  float *out_sim, unsigned char *out_hit, unsigned *access, int *owner, int *members, ScreenPlain *plain, float floor) {
    const ScreenRoom r = screen_room(c->screen.at, c, c->count, n);
    const ByteStore s = byte_store(c->bytes.at, c, c->bytes.rows);
    const unsigned *version = c->version;
    const int d = c->dim, dp = byte_dim(d);
    const long tiles = up256(c->count) / 256, nqt = up256(n) / 256;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void *)k_screen_lookup<true>, hipFuncAttributeMaxDynamicSharedMemorySize, SCREEN_LDS);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)k_screen_lookup<false>, hipFuncAttributeMaxDynamicSharedMemorySize, SCREEN_LDS);
        if (e != hipSuccess) return siso_check_hip(c, e, "hipFuncSetAttribute(k_screen_lookup)");
        attr_done = true;
    }
    const T *cent = (const T *)c->cent;
    const int vec = (size_t)d * sizeof(T) % 16 == 0 && ((uintptr_t)queries & 15) == 0 ? 1 : 0;
    const dim3 fours((unsigned)((n + 3) / 4)), block(256);
    // A sample of the tiles supplies the first bounds: one for every compute unit, or a 128th of them, whichever is more, but no
    // more than a quarter.
    long some = 256 / nqt > tiles / 128 ? 256 / nqt : tiles / 128;
    if (some > tiles / 4) some = tiles / 4;
    // Much work: an eighth of the tiles first, and better bounds from what it has listed, for queries that are near nothing (a
    // bound from 2,000 rows lets some 700 of 131,072 pass, one from 16,000 some 200).
    const long ahead = tiles * nqt >= 32 * 256 ? tiles / 8 : 0;
    // Given up (see above): never where the option asks for the bytes.
    // A batch of which a part f is lost costs its bytes and f of all products (more, as fewer do not fill the chip): in bf16 the bytes
    // are more than half of it, in single precision a quarter to a tenth, and some 75 us stand around them: `share` is where the two
    // ways meet.  Rows of mean cosine m, sixteen near each other, all products / screened to the end / as it is here, us:
    //   no query misses, m 0.5   bf16  4,096 x 131,072 x 768   623 / 489 / 500     fp32  1,000 x 60,000 x 384   393 / 103 / 106
    //   30 % miss, m 0.5         bf16  4,096 x 131,072 x 768   621 / 788 / 790     fp32  1,000 x 60,000 x 384   393 / 119 / 123
    //   all miss, m 0.5          bf16  4,096 x 131,072 x 768   621 / 1,094 / 750   fp32  1,000 x 60,000 x 384   393 / 158 / 163
    //   30 % miss, m 0.7         bf16  4,096 x 131,072 x 768   617 / 1,097 / 770   fp32  1,000 x 16,000 x 384   118 / 116 / 150
    //   all miss, m 0.7          bf16  8,192 x 131,072 x 1,024  1,639 / 4,460 / 1,663   fp32  4,096 x 60,000 x 768  2,968 / 3,772 / 3,058
    //   all miss, m 0.9          bf16  4,096 x 131,072 x 768   612 / 10,899 / 657  fp32  1,000 x 60,000 x 384   393 / 1,232 / 460
    const bool stay = c->opt_screen == 1, f32 = c->dtype == SISO_F32;
    const double products = 2.0 * (double)n * (double)c->count * d / (f32 ? 1.13e8 : 1.25e9);  // us
    double share = f32 ? 0.9 - 75 / products : 0.55 - 150 / products;
    share = share < 0.1 ? 0.1 : share > 0.75 ? 0.75 : share;
    const int most_lost = stay ? SCREEN_WHOLE : (int)(share * (double)n / SCREEN_COUNTED);
    ScreenCrowd crowd = {r.near, r.largest, (float)some, (float)c->count, SCREEN_LIST / 2, 0, r.totals + 2, most_lost};
    if (ahead > 0) {
        const long flood = SCREEN_LIST * ahead / tiles, worth = c->count / (f32 ? 800 : 6500);
        crowd.rows = ahead * 256.f;
        crowd.heavy = (int)(worth < flood ? worth : flood);
    } else if (2 * again_per_query(c, c->count) < SCREEN_LIST) {  // (the bound gets better yet: half as many will count)
        crowd.most = 1.25f * again_per_query(c, c->count);
    }
    int *lost = r.totals + 2;
    // (cosines are rounded: a row that exceeds the floor by the least bit is listed whatever its bytes)
    const float least = floor >= SCREEN_LEAST_FLOOR ? floor - 1e-5f : -INFINITY;
    // The bytes of the rows that are looked at first, and the others only once the batch is not given up (of more queries they are
    // the smaller part: 500 / n of the time that all products take in bf16).
    ScreenTiles which = {with_rows && whole && ahead > 0 && n <= 8192 ? 1 : 0, (int)ahead, (int)some, some > 0 ? (int)(tiles / some) : 1};
    int rc = write_bytes<T>(c, r, s, version, cent, c->invn, c->count, with_rows, queries, n, which, most_lost, least);
    if (rc != SISO_OK) return rc;
    if (with_rows && which.part == 0 && !capturing(c)) siso_bytes_current(c);
    if (some > 0) {
        hipLaunchKernelGGL(k_screen_lookup<true>, dim3((unsigned)(some * nqt)), dim3(ByteCfg::NT), SCREEN_LDS, c->stream, r.qcodes, s.codes,
                           s.meta, r.qm, r.low, r.seed, r.cnt, r.near, r.largest, r.list, 0L, c->count, dp, 1, (int)some, (int)nqt, 1, which.stride,
                           lost, most_lost);
        hipLaunchKernelGGL((k_screen_seed<T, false>), fours, block, 0, c->stream, queries, cent, c->invn, n, c->count, d, vec, r.qm,
                           s.meta, r.seed, r.cnt, r.list, r.low, crowd);
    }
    siso_prof_begin(c);
    for (int part = ahead > 0 ? 0 : 1; part < 2; ++part) {
        const long t0 = part == 0 ? 0 : ahead, row0 = t0 * 256;
        const long rows = part == 0 ? ahead * 256 : c->count - row0;
        BytePlan p;
        if (!siso_byte_plan(c, rows, n, dp, SCREEN_TILES, &p)) return siso_fail(c, SISO_EINVAL, "screened lookup: no plan");
        hipLaunchKernelGGL(k_screen_lookup<false>, dim3((unsigned)p.grid), dim3(ByteCfg::NT), SCREEN_LDS, c->stream, r.qcodes,
                           s.codes + (size_t)row0 * dp, s.meta + t0 * 8, r.qm, r.low, r.seed, r.cnt, r.near, r.largest, r.list, row0, rows,
                           dp,
                           p.tiles_per_slice, p.slices, p.nqt, p.qb, 1, lost, most_lost);
        if (part == 0) {
            hipLaunchKernelGGL((k_screen_seed<T, true>), fours, block, 0, c->stream, queries, cent, c->invn, n, c->count, d, vec, r.qm,
                               s.meta, r.seed, r.cnt, r.list, r.low, crowd);
            if (which.part == 1) {
                which.part = 2;
                rc = write_bytes<T>(c, r, s, version, cent, c->invn, c->count, true, queries, 0, which, most_lost, least);
                if (rc != SISO_OK) return rc;
            }
        }
    }
    siso_prof_end(c);
    // Sixteen queries to a workgroup, of few queries four: those are as many workgroups as the chip has work for (lookups of queries that mostly hit, us,
    // four / sixteen: 60,000 x 384 fp32 n 200 65.1 / 66.6, 300 70.6 / 72.6, 700 80.6 / 82.3, 1,000 90.8 / 91.9; a third of them
    // misses: 300 74.2 / 74.8, 1,000 96.5 / 95.6, 8,192 310.9 / 305.7; the step alone for 6,553 rows of a refresh, 65,536 x 768 bf16, 23.0 / 10.7)
    const unsigned pick_waves = n < 1000 ? 4u : PICK_WAVES;
    hipLaunchKernelGGL(k_screen_pick<T>, dim3((unsigned)((n + pick_waves - 1) / pick_waves)), dim3(pick_waves * 64), 0, c->stream,
                       queries, cent, c->invn, n, d, vec, r.low, r.cnt, r.list, r.totals,
                       most_lost, r.work, r.work_room, r.best, r.qinv, r.plain_of, (T *)r.plain_rows);
    hipLaunchKernelGGL(k_screen_score<T>, dim3((unsigned)(n < 4096 ? (n + 1) / 2 : 2048)), block, 0, c->stream, queries, cent, c->invn, d, vec,
                       r.totals, r.work, r.work_room, r.qinv, r.best);
    hipLaunchKernelGGL(k_screen_write, dim3((unsigned)((n + 255) / 256)), block, 0, c->stream, n, q_base, r.cnt, r.best, tl, out_idx, out_sim,
                       out_hit, access, owner, members);
    *plain = ScreenPlain{r.totals + 1, r.plain_of, r.plain_rows, vec};
    return siso_check_hip(c, hipGetLastError(), "k_screen_lookup, k_screen_pick, k_screen_score");
}

template <typename T>
int pairs_launch(siso_cache *c, const T *rows, const float *invn, long count, float threshold, int *out_pairs, long cap, u64 *counter,
                 PairsRedo *redo) {
    const ScreenRoom r = screen_room(c->screen_pairs.at, c, count, 0);
    const int d = c->dim, dp = byte_dim(d);
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t e = hipFuncSetAttribute((const void *)k_screen_pairs, hipFuncAttributeMaxDynamicSharedMemorySize, SCREEN_PAIR_LDS);
        if (e != hipSuccess) return siso_check_hip(c, e, "hipFuncSetAttribute(k_screen_pairs)");
        attr_done = true;
    }
    hipLaunchKernelGGL(k_screen_clear, dim3(1), dim3(1), 0, c->stream, r.maybe_count);
    const ByteStore s{r.codes, r.meta, nullptr, 0};  // (rows of any origin: their bytes serve this search alone)
    const int rc = write_bytes<T>(c, r, s, nullptr, rows, invn, count, true, rows, 0, ScreenTiles{0, 0, 0, 1}, SCREEN_WHOLE, 0.f);
    if (rc != SISO_OK) return rc;
    int qb = 8;
    while (qb > 1 && qb > up256(count) / 256) qb >>= 1;
    // Where a workgroup has eight pairs of tiles and more, an eighth of them goes first and tells whether those in doubt will be too
    // many (half as many again as their share, so that an uneven order of the rows does not decide).  It takes some 15 us more,
    // and saves half of what all pairs take in bf16, a fifth in single precision: there, and below, the list decides when it is
    // full.  Rows of mean cosine 0.88 at a threshold of 0.9, all pairs / before / now, us: bf16 131,072 x 768 11,512 / 1,623,000 /
    // 12,779, 16,000 x 768 232 / 24,300 / 385; fp32 8,000 x 768 503 / 6,554 / 573.
    const long tiles = up256(count) / 256, all = tiles * (tiles + 1) / 2;
    auto search = [&](int part) {
        hipLaunchKernelGGL(k_screen_pairs, dim3(256), dim3(ByteCfg::NT), SCREEN_PAIR_LDS, c->stream, r.codes, r.meta, count, dp, qb, part, threshold,
                           out_pairs, cap, counter, r.maybe, r.maybe_room, r.maybe_count);
    };
    if (all >= 8 * 256 && c->dtype != SISO_F32) {
        search(PAIRS_FIRST);
        hipLaunchKernelGGL(k_screen_pairs_judge, dim3(1), dim3(1), 0, c->stream, r.maybe_count,
                           (u64)(1.5 * (0.125 + 128.0 / (double)all) * (double)r.maybe_room), r.maybe_room);
        search(PAIRS_REST);
    } else {
        search(PAIRS_ALL);
    }
    const int vec = (size_t)d * sizeof(T) % 16 == 0 && ((uintptr_t)rows & 15) == 0 ? 1 : 0;
    hipLaunchKernelGGL(k_screen_pairs_check<T>, dim3(512), dim3(256), 0, c->stream, rows, invn, d, vec, threshold, r.maybe, r.maybe_room,
                       r.maybe_count,                       out_pairs, cap, counter);
    *redo = PairsRedo{r.maybe_count, r.maybe_room};
    return siso_check_hip(c, hipGetLastError(), "k_screen_pairs");
}

}  // namespace

// Is a lookup worth it?  The bytes of rows that have changed are written (here: of all), and six small kernels
// stand around the products.  Lookups alone, no misses / 30 % / 60 % misses, us, without -> with:
//   fp32  1,000 x 8,000 x 384      75 -> 69 / 72 -> 73 / 73 -> 75          300 x 16,000 x 384     54 -> 64 / 54 -> 69 / 54 -> 72
//         1,000 x 16,000 x 384    118 -> 72 / 118 -> 77                    2,000 x 2,000 x 768    77 -> 88 / 75 -> 101 / 75 -> 111
//         1,000 x 30,000 x 384    209 -> 80 / 209 -> 87 / 210 -> 91        200 x 60,000 x 384    114 -> 78 / 110 -> 84 / 110 -> 89
//         4,096 x 60,000 x 768    2,964 -> 300 / 2,969 -> 351              130 x 100,000 x 384   185 -> 94 / 185 -> 99 / 184 -> 105
//   bf16  4,096 x 65,536 x 768    336 -> 298 / 333 -> 338 / 334 -> 367     1,000 x 400,000 x 768  532 -> 513 / 531 -> 542 / 527 -> 567
//         6,553 x 65,536 x 768    563 -> 467 / 562 -> 545 / 561 -> 595     4,096 x 131,072 x 768  648 -> 514 / 649 -> 556 / 648 -> 594
//         8,192 x 131,072 x 1,024 1,679 -> 1,150 / 1,677 -> 1,437 / 1,678 -> 1,528
// The lines lie where batches of which more than half misses are ahead, too.  A query costs its candidates, whatever the products
// take, so a small cache is better off without at any batch, and so are bf16 rows of 128 elements, whose bytes have to be filled up:
//   fp32  8,192 x 1,000 x 768     127 -> 146 / 134 -> 177        8,192 x 2,000 x 768    232 -> 147 / 225 -> 177 / 222 -> 202
//         32,768 x 8,000 x 128    610 -> 426 / 608 -> 435        16,384 x 4,000 x 384   432 -> 211 / 430 -> 236 / 428 -> 255
//   bf16  65,536 x 50,000 x 128   845 -> 1,671 / 844 -> 1,713    16,384 x 30,000 x 768  797 -> 555 / 794 -> 665 / 791 -> 763
//         32,768 x 16,000 x 1,024 852 -> 904 / 847 -> 1,203      16,384 x 100,000 x 256 886 -> 670 / 885 -> 705 / 884 -> 729
//         8,192 x 200,000 x 192   571 -> 601 / 570 -> 624        8,192 x 200,000 x 320  870 -> 775 / 870 -> 810 / 870 -> 840
// Up to 256 queries of single precision would end
// in one kernel with their update (k_finalize_update), which a screened batch does not: with the update, 256 x 42,000 x 384
// 93 -> 81 / 94 -> 88 / 94 -> 90, 256 x 100,000 x 384 192 -> 102 / 191 -> 109 / 190 -> 114.  Rows with a common direction: see
// screen_launch.  Longer rows than SISO_SCREEN_DIM: the error stays what it is while the cosines of unrelated rows crowd
// together (deviation d^-1/2), and ever more rows are near the best.
int siso_screen_wanted(const siso_cache *c, long n) {
    if (c->dtype == SISO_FP8 || c->opt_screen == 2 || c->count < 1 || n < 1 || c->dim > SISO_SCREEN_DIM) return 0;
    if (c->opt_screen == 1 || c->opt_screen == 3) return 1;
    if (c->path != SISO_PATH_AUTO || c->opt_mfma_config != 0 || c->opt_tiles_per_slice != 0 || c->opt_mfma_qblock != 0) return 0;
    const double elements = (double)c->count * c->dim, saved = (double)c->count * saved_dim(c->dim);
    if (c->dim < 128) return 0;
    if (c->dtype == SISO_F32) return n > 128 && 2.0 * (double)n * elements >= 8e9 && elements >= 1e6;
    return n >= 768 && 2.0 * (double)n * saved >= 3.75e11 && saved >= 1.1e7;  // (both lines: half of the bf16 work, mostly)
}

// A floor leaves queries that miss without candidates, so smaller lookups are ahead (bf16; a lookup with the rest of its call, us,
// without -> with): a refresh of 40,000 x 768 by 5,000 rows 656 -> 639, of 100,000 x 1,024 by 2,500 912 -> 811, of 200,000 x 256 by 5,000
// 1,041 -> 973, of 65,536 x 768 by 6,553 (553 us of it all products) 140 less; 3,276 samples of a table against 65,536 x 768
// 372 -> 357; whole tables right above the line, without -> with: 40,000 x 768 by 4,964 326 -> 263, 65,536 x 384 by 6,059 309 -> 246, 100,000 x
// 1,024 by 1,489 305 -> 282, 200,000 x 256 by 2,978 325 -> 293; behind the line 1,638 rows against 65,536 x 768 432 -> 445, 3,276 against 65,536 x 384 220 -> 262.
int siso_screen_above_wanted(const siso_cache *c, long n, float floor) {
    if (siso_screen_wanted(c, n)) return 1;
    if (!(floor >= SCREEN_LEAST_FLOOR) || c->dtype != SISO_BF16 || c->opt_screen == 2 || c->dim > SISO_SCREEN_DIM || c->dim < 128) return 0;
    if (c->path != SISO_PATH_AUTO || c->opt_mfma_config != 0 || c->opt_tiles_per_slice != 0 || c->opt_mfma_qblock != 0) return 0;
    const double saved = (double)c->count * saved_dim(c->dim);
    return n >= 768 && 2.0 * (double)n * saved >= 1.5e11 && saved >= 1.1e7;
}

extern "C" int siso_screened(const siso_cache *c, long n) {
    if (!c || n < 0) return SISO_EINVAL;
    return n == 0 ? siso_screen_pairs_wanted(c, c->count, 1.f) : siso_screen_wanted(c, n) || siso_bytes_few_wanted(c, n);
}

// Room for the bytes of `rows` rows of the cache, which are then made by the next lookup (nothing made from is recorded there).  Of a cache that
// is nearly full: for all it can hold, if that is to be had, so that the last eighth does not move them once more (a first refresh of 65,536
// rows x 768 by 6,553, 1.87 ms, was 0.09 of it longer than with one room for bytes and workspace).
static bool byte_room(siso_cache *c, long rows) {
    ByteRows &b = c->bytes;
    if (rows <= b.rows) return true;
    if (capturing(c) || (b.refused != 0 && rows >= b.refused)) return false;
    const size_t room = (size_t)c->opt_screen_room << 10;  // (0: as there is)
    auto take_rows = [&](long count, size_t beside) {
        const size_t bytes = byte_store(nullptr, c, count).bytes;
        char *at = nullptr;
        if ((room > 0 && bytes + beside > room) || !take(&at, bytes)) return (char *)nullptr;
        if (hipMemsetAsync(at, 0, (size_t)up256(count) / 32 * sizeof(u64), c->stream) == hipSuccess) return at;
        (void)hipGetLastError();
        (void)hipFree(at);
        return (char *)nullptr;
    };
    const long had = b.rows, full = c->capacity - rows <= rows / 8 ? c->capacity : rows;
    long count = full;
    char *larger = nullptr;
    if (room == 0 || byte_store(nullptr, c, rows).bytes <= room) {
        const size_t beside = b.at ? byte_store(nullptr, c, had).bytes : 0;
        larger = take_rows(full, beside);
        if (!larger && full > rows) larger = take_rows(count = rows, beside);
        // (the old ones go: nothing but their recorded launches needs them)
        if (b.at && larger && b.recorded) {
            c->screen_kept->push_back(b.at);  // (room for it: note_recorded)
        } else if (b.at && !b.recorded) {
            if (hipStreamSynchronize(c->stream) != hipSuccess) {
                (void)hipGetLastError();
                if (larger) (void)hipFree(larger);
                return false;
            }
            (void)hipFree(b.at);
            if (!larger) {  // not beside them: perhaps in their place
                larger = take_rows(count = rows, 0);
                b.at = larger ? nullptr : take_rows(had, 0);
                b.rows = b.at ? had : 0;
                siso_bytes_all_behind(c);
            }
        }
    }
    if (!larger) {
        b.refused = rows;
        return false;
    }
    b.at = larger;
    b.rows = count;
    b.recorded = 0;
    siso_bytes_all_behind(c);
    return true;
}

ByteView siso_byte_view(const siso_cache *c) {
    if (!c->bytes.at || c->bytes.rows < c->count) return ByteView{nullptr, nullptr, nullptr, 0};  // (rows that they have no room for are not written to them)
    const ByteStore s = byte_store(c->bytes.at, c, c->bytes.rows);
    return ByteView{s.codes, s.meta, s.made, byte_dim(c->dim)};
}

unsigned *siso_counted(const siso_cache *c) { return c->bytes.written || capturing(c) ? c->version : nullptr; }

// A graph that records launches over the bytes or the workspace goes on using them when a larger call has outgrown them.
static int note_recorded(siso_cache *c, bool workspace) {
    if ((!workspace || c->screen_recorded) && c->bytes.recorded) return SISO_OK;
    try {
        if (!c->screen_kept) c->screen_kept = new std::vector<char *>;
        c->screen_kept->reserve(c->screen_kept->size() + 2);  // (the bytes, and what stands around them)
    } catch (const std::bad_alloc &) {
        return siso_fail(c, SISO_ENOMEM, "siso_lookup: note of a recorded workspace");
    }
    if (workspace) c->screen_recorded = 1;
    c->bytes.recorded = 1;
    return SISO_OK;
}

bool siso_bytes_may_record(siso_cache *c) { return !capturing(c) || note_recorded(c, false) == SISO_OK; }

// ---- few queries over the bytes (lookup_bytes.hip)
static bool few_lists_room(siso_cache *c) {
    if (c->few.best) return true;
    if (capturing(c) || c->few_refused) return false;
    FewLists f;
    auto layout = [&](Carver a) {
        f.best = a.take<u64>(SISO_FEW);
        f.table = a.take<u64>(SISO_FEW_WORKGROUPS * SISO_FEW);
        f.call = a.take<unsigned>(1);
        f.cnt = a.take<int>(SISO_FEW);
        f.rows = a.take<uint2>((size_t)SISO_FEW * SISO_FEW_LIST);
        f.slots = a.take<unsigned>((size_t)SISO_FEW * SISO_FEW_WORKGROUPS * SISO_FEW_SLOTS);
        return a.used;
    };
    const size_t bytes = layout(Carver{nullptr});
    char *at = nullptr;
    int *flooded = nullptr;
    if ((c->opt_screen_room > 0 && bytes > (size_t)c->opt_screen_room << 10) || !take(&at, bytes)) {
        c->few_refused = 1;
        return false;
    }
    bool ok = hipHostMalloc((void **)&flooded, sizeof(int), hipHostMallocDefault) == hipSuccess;
    ok = ok && hipMemsetAsync(at, 0, bytes, c->stream) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (flooded) (void)hipHostFree(flooded);
        (void)hipFree(at);
        c->few_refused = 1;
        return false;
    }
    *flooded = 0;
    layout(Carver{at});
    c->few = f;
    c->few_flooded = flooded;
    return true;
}

// Steps of n queries (lookup and fold), the rows as they are stored / the bytes, us, if none, 30 % and 60 % of the queries miss:
//   768:   30,000 (60 %) n 1 19 / 17, n 8 22 / 27, n 64 23 / 35;  60,000 (60 %) n 1 21 / 24, n 8 23 / 31, n 64 24 / 41
//          88,000 n 8 36 / 29, 33, 32;  132,000 n 9 49 / 33, 35, 35, n 32 49 / 35, 38, 41, n 64 50 / 38, 43, 45;  196,608 n 64 54 / 43, 49, 49;  400,000 n 1 102 / 60, n 64 109 / 77
//   896:   115,000 n 16 42 / 32, 36, 43, n 32 42 / 34, 44, 40;  132,000 n 32 55 / 36, 41, 43;  196,608 n 33 59 / 48, 54, 60, n 64 60 / 49, 57, 59
//   960:   105,000 n 9 43 / 34, 38, 40, n 32 43 / 36, 44, 45;  140,000 n 64 60 / 48, 63, 62;  196,608 n 64 63 / 57, 70, 80;  198,000 n 64 75 / 58, 75, 73
//   1,024: 64,000 n 1 26 / 26, 26, 26, n 8 28 / 27, 31, 35;  66,000 n 8 44 / 29, 32, 35;  131,072 n 16 47 / 37, 44, 46, n 32 47 / 39, 44, 52;  131,073 n 32 63 / 39, 47, 49
//          140,000 n 64 64 / 48, 64, 65;  180,000 n 64 66 / 59, 73, 77;  198,000 n 64 81 / 58, 74, 78;  262,144 n 64 87 / 72, 87, 88;  400,000 n 1 138 / 84, n 64 140 / 115
//   512:   131,000 n 1 27 / 24, 24, 23, n 8 28 / 26, 27, 28;  197,000 n 9 46 / 31, 32, 32, n 64 45 / 36, 39, 39
//   384:   176,000 n 8 29 / 26, 27, 27;  264,000 n 64 43 / 36, 39, 38.     256: 266,000 n 8 33 / 26, 27, 27;  394,000 n 64 43 / 35, 36, 36.     128: 2,000,000 n 64 96 / 115
// Two kernels with longer chains of round trips stand against half of the reading; and with few rows a workgroup has
// little to go by: with one or two blocks for each wave the bounds of 33 queries and more come too late for its lists.  Over the stored rows a
// step takes as long as 256 workgroups with whole tiles of 256 rows do: up to 65,536 rows the time of one tile, up to 131,072 of two, and so on.  The lines lie
// where such a tile is added: 65,536 rows of 1,024, 131,072 of 768.  Beyond 896 elements the lists of 33 queries and more have the least room (LDS holds the
// queries), and one tile more is needed.
int siso_bytes_few_wanted(const siso_cache *c, long n) {
    if (c->dtype != SISO_BF16 || n < 1 || n > SISO_FEW || c->count < 1 || c->count > SISO_FEW_MOST_ROWS) return 0;
    if (c->dim % 64 != 0 || c->dim < 128 || c->dim > SISO_SCREEN_DIM) return 0;
    if (c->opt_screen == 4) return 1;
    if (c->opt_screen != 0 || c->path != SISO_PATH_AUTO || c->opt_mfma_config != 0 || c->opt_tiles_per_slice != 0 || c->opt_mfma_qblock != 0) return 0;
    const double elements = (double)c->count * c->dim;
    if (c->dim < 256) return 0;
    if (n <= 8) return elements > 65536. * 1024;
    return elements > 131072. * 768 && (n <= 16 || c->count > (n > 32 && c->dim > 896 ? 196608 : 131072));
}

int siso_bytes_few_room(siso_cache *c, long n) {
    const bool forced = c->opt_screen == 4, recording = capturing(c);
    // A graph holds one way for good: over the bytes every replay would write changed rows as bytes (8 to 18 us), and could not turn back on rows that lists
    // flood on (3 to 13 times the time).  Replays of a step of 64 against 262,144 x 768 75 us as they are stored, 66 over the bytes; of 64 against 140,001 x 1,024
    // 60 and 74, of eight against 64,000 x 1,024 33 and 39.
    if (recording && !forced) return 0;
    // Lists that found no room, or that were too long to be worth it (LISTED_MANY), of some call since the last one that was looked at: the next 64 lookups go over
    // the rows as they are stored, twice as many whenever that is seen again before 4,096 have gone over the bytes.  (Rows with a common direction give the same
    // results at up to eight times the time: mean cosine 0.8, 32 queries against 131,073 x 768 161 us, 46 over the stored rows and by this rule; eight against
    // 66,000 x 1,024 155 and 41; 0.6 65 and 41.  Below that it turns over gradually: 0.4, 64 against 140,001 x 768 52 and 47, against 262,144 x 768 61 and 69.)
    if (!forced && c->few_flooded && *(volatile int *)c->few_flooded != 0) {
        *(volatile int *)c->few_flooded = 0;
        c->few_rests = c->few_rests == 0 || c->few_went >= 4096 ? 64 : c->few_rests < 4096 ? 2 * c->few_rests : c->few_rests;
        c->few_rest = c->few_rests;
        c->few_went = 0;
    }
    if (!forced && c->few_rest > 0) {
        --c->few_rest;
        return 0;
    }
    ByteRows &b = c->bytes;
    // (what siso_reserve was asked for does not allocate afterwards, with or without room)
    if (n <= c->few_reserved ? b.rows < c->count || !c->few.best : !byte_room(c, c->count) || !few_lists_room(c)) return 0;
    if (b.behind > 0 || recording || b.served >= 64) {  // (single rows that a fold could not bring up to date stay behind for 64 lookups at most)
        // Rows that have changed are written as bytes once lookups have read as much for want of that: a lookup over the bytes reads one byte an
        // element less, and to write them takes three, and 8 to 18 us however few they are.  So if fewer than 16 lookups went over what was written
        // last (an update behind each, say), twice as many go over the stored rows before the next time: a lookup and its update, 64 queries against
        // 262,144 x 768 as they are stored 73 us, with the bytes written each time 76; against 140,001 x 1,024 57 and 82.
        // (A graph, where it is told to go this way, may be replayed behind any change, and records it always.)
        const double elements = (double)c->count * c->dim, blocks = (double)b.behind * 32 < (double)c->count ? (double)b.behind * 32 * c->dim : elements;
        if (!forced && !recording && b.behind > 0) {
            b.forgone += elements;
            ++b.waited;
            if (b.forgone < 2 * blocks || b.waited < b.wait) return 0;
        }
        if (recording && note_recorded(c, false) != SISO_OK) return 0;
        const ScreenRoom none = screen_room(nullptr, c, c->count, 0);
        const ByteStore s = byte_store(b.at, c, b.rows);
        const int rc = write_bytes<bf16_t>(c, none, s, c->version, (const bf16_t *)c->cent, c->invn, c->count, true, (const bf16_t *)c->cent, 0,
                                           ScreenTiles{0, 0, 0, 1}, SCREEN_WHOLE, 0.f);
        if (rc != SISO_OK) return 0;
        if (!recording) {
            b.wait = b.served >= 16 ? 0 : b.wait == 0 ? 8 : b.wait < 512 ? 2 * b.wait : b.wait;
            b.served = 0;
            siso_bytes_current(c);
        }
    }
    ++b.served;
    ++c->few_went;
    return 1;
}

static bool lookup_room(siso_cache *c, long rows, long n) {
    if (!byte_room(c, rows)) return false;
    const char *before = c->screen.at;
    const bool room = make_room(c, c->screen, screen_room(nullptr, c, rows, n).bytes, c->screen_recorded ? c->screen_kept : nullptr);
    if (c->screen.at != before) c->screen_recorded = 0;
    return room;
}

int siso_screen_room(siso_cache *c, long n) {
    // (what siso_reserve was asked for does not allocate afterwards, with or without room)
    if (n <= c->screen_reserved) return c->count <= c->bytes.rows && screen_room(nullptr, c, c->count, n).bytes <= c->screen.cap;
    return lookup_room(c, c->count, n);
}

void siso_screen_reserve(siso_cache *c, long n) {
    c->screen.refused = c->screen_pairs.refused = c->bytes.refused = 0;
    (void)lookup_room(c, c->capacity, n);
    if (n > c->screen_reserved) c->screen_reserved = n;
}

void siso_bytes_few_reserve(siso_cache *c, long n) {
    siso_cache full = *c;
    full.count = c->capacity < SISO_FEW_MOST_ROWS ? c->capacity : SISO_FEW_MOST_ROWS;
    bool wanted = false;  // (by any batch of up to n: the rule asks for more rows from nine, 17 and 33 queries on)
    for (const long least : {1L, 9L, 17L, 33L}) wanted = wanted || (least <= n && siso_bytes_few_wanted(&full, least));
    if (!wanted) return;
    c->bytes.refused = 0;
    c->few_refused = 0;
    if (byte_room(c, full.count)) (void)few_lists_room(c);
    if (n > c->few_reserved) c->few_reserved = n;
}

int siso_screen_pairs_room(siso_cache *c, long rows) {
    return make_room(c, c->screen_pairs, screen_room(nullptr, c, rows, 0).bytes, nullptr);
}

void siso_screen_done(siso_cache *c) {
    if (c->screen_pairs.cap <= (size_t)SISO_ARENA_KEEP) return;
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(c->screen_pairs.at);
    c->screen_pairs = ScreenSpace{nullptr, 0, 0};
    c->screen.refused = c->bytes.refused = 0;
    c->few_refused = 0;
}

void siso_screen_release(siso_cache *c) {
    if (c->screen.at) (void)hipFree(c->screen.at);
    if (c->screen_pairs.at) (void)hipFree(c->screen_pairs.at);
    if (c->bytes.at) (void)hipFree(c->bytes.at);
    if (c->few.best) (void)hipFree(c->few.best);
    if (c->few_flooded) (void)hipHostFree(c->few_flooded);
    if (c->screen_kept)
        for (char *room : *c->screen_kept) (void)hipFree(room);
    delete c->screen_kept;
}

int siso_screen_lookup(siso_cache *c, const void *queries, long n, bool with_rows, bool whole, const ThetaList &tl, long q_base, int *out_idx,
                       float *out_sim, unsigned char *out_hit, unsigned *access, int *owner, int *members, ScreenPlain *plain, float floor) {
    if (capturing(c)) {
        const int rc = note_recorded(c, true);
        if (rc != SISO_OK) return rc;
    }
    return c->dtype == SISO_F32 ? screen_launch<float>(c, (const float *)queries, n, with_rows, whole, tl, q_base, out_idx, out_sim, out_hit,
                                                       access, owner, members, plain, floor)
                                : screen_launch<bf16_t>(c, (const bf16_t *)queries, n, with_rows, whole, tl, q_base, out_idx, out_sim, out_hit,
                                                        access, owner, members, plain, floor);
}

// Searches with their read-back, rows in groups of four, us, without and with: fp32 1,000 x 384 39 -> 52, 1,500 x 768 61 -> 55
// (no pairs 55 -> 50), 2,000 x 256 53 -> 49 (39 -> 45), 2,000 x 768 81 -> 56, 4,000 x 256 130 -> 60, 8,000 x 768 500 -> 97; bf16 8,000 x 256 62 -> 71, 6,000 x 768 94 -> 86, 16,000 x 256 101 -> 99, 16,000 x 768
// 229 -> 151, 50,000 x 768 1,666 -> 886; where it does not pay: fp32 1,250 x 1,000 62 -> 87, bf16 14,000 x 128 80 -> 108, 20,000 x 128
// 129 -> 178, 10,000 x 256 80 -> 90.  Below a threshold of 0.25 rows of zeros and the many pairs of unrelated rows would come
// near it.
int siso_screen_pairs_wanted(const siso_cache *c, long count, float threshold) {
    if (c->dtype == SISO_FP8 || c->opt_screen == 2 || c->opt_merge_config != 0 || count < 2 || c->dim > SISO_SCREEN_DIM) return 0;
    if (!(threshold >= 0.25f)) return 0;
    if (c->opt_screen == 1 || c->opt_screen == 3) return 1;
    const double squared = (double)count * (double)count;
    if (c->dim < 128) return 0;
    return c->dtype == SISO_F32 ? count >= 1500 && squared * c->dim >= 1.5e9 : squared * saved_dim(c->dim) >= 1.3e10;
}

int siso_screen_pairs_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                             u64 *counter, PairsRedo *redo) {
    return c->dtype == SISO_F32 ? pairs_launch<float>(c, (const float *)rows, invn, count, threshold, out_pairs, cap, counter, redo)
                                : pairs_launch<bf16_t>(c, (const bf16_t *)rows, invn, count, threshold, out_pairs, cap, counter, redo);
}
