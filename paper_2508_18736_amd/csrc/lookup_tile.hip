// Lookup and pair search for what the pipelined bf16 and 8-bit kernels do not take: single-precision caches, bf16
// caches whose dimension is not a multiple of 64, rows and queries at any alignment.  A tiled GEMM on the matrix
// cores in the element type itself (v_mfma_f32_32x32x2_f32: 157 TFLOP/s dense, twice what single-precision multiply-adds
// reach; v_mfma_f32_32x32x16_bf16), products and sums in single precision.
//
// A = centroid rows, B = query rows (D: lane l holds query l % 32; its 16 registers are the centroid rows
// 8 * (i / 4) + 4 * (l / 32) + i % 4 of a run of 32).  Four waves share a tile of BC x BQ rows; the dimension passes
// in slabs of 128 bytes per row.  Rows go global -> registers -> LDS, because a slab may end inside a row (the rest is
// zero on both sides, so it adds nothing and a non-finite neighbour cannot leak in) and rows may be misaligned: two
// slabs are on their way in registers and one in LDS while a fourth is being multiplied.  A 32 x 32 x 2 product takes
// 64 cycles for the 8 bytes a lane supplies, eight times as long per byte as in bf16: neither LDS nor memory is near
// its limit on the single-precision tiles, and what is left to lose is latency on small problems: hence three tiles.
//
// LDS: row r of the tile is 128 bytes = 8 chunks of 16 bytes, chunk c in slot c ^ ((r >> 1) & 7) (the 16 rows x
// 16 bytes that a fragment read serves at a time then cover all banks).  Lane half h reads chunk 2 s + h in step s,
// on both sides alike, which is all that a sum asks of the order of its terms.
#include <math.h>

#include "siso_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int WC_, int WQ_, int NWC_, int NWQ_, int DEPTH_, int CHAINS_>
struct TileCfg {
    static constexpr int WC = WC_, WQ = WQ_, NWC = NWC_, NWQ = NWQ_;  // 32-row blocks per wave, waves, on either side
    static constexpr int BC = 32 * WC * NWC, BQ = 32 * WQ * NWQ;
    static constexpr int JC = BC / 32, JQ = BQ / 32;                  // 16-byte chunks per thread and slab
    static constexpr int STAGE = (BC + BQ) * 128;
    static constexpr int DEPTH = DEPTH_;                              // slabs on their way in registers
    // Partial sums of a product, added at the end: two (half as many roundings in a row) where the registers allow it and
    // the sums need not be those of the pipelined kernels.  With one the products are added in their order, and bf16 batches
    // of at most 64 give the same bits whichever kernel a cache's size sends them to.  (Codes do not: the pipelined
    // kernels take 64 to an instruction, these 16.)
    static constexpr int CHAINS = CHAINS_;
    static_assert(DEPTH % 2 == 0, "slab number i of a round goes to stage i % 2");
    static_assert(NWC * NWQ == 4, "four waves");
    static_assert(BC <= SISO_PAD_ROWS, "the inverse lengths of a whole last tile are readable");
    static_assert(NWC * BQ * 8 <= 2 * STAGE, "the reduction fits in the stages");
};
typedef TileCfg<2, 2, 2, 2, 2, 1> TileLarge;  // 128 x 128
typedef TileCfg<1, 1, 2, 2, 4, 2> TileSmall;  // 64 x 64
typedef TileCfg<1, 1, 4, 1, 4, 1> TileFew;    // 128 centroids x 32 queries

// One 16-byte chunk of a row at element k; W = bytes every row is aligned to (16, 8, or the element).  Elements at
// d and beyond are read from the row's start and zeroed later (zero_tail), so that nothing waits here.
template <int W, typename T>
__device__ __forceinline__ u32x4_t load_chunk(const T *row, int k, int d) {
    constexpr int EPC = 16 / (int)sizeof(T);
    if constexpr (W == 16) {
        return *(const u32x4_t *)(row + (k < d ? k : 0));
    } else if constexpr (W == 8) {
        const uint2 lo = *(const uint2 *)(row + (k < d ? k : 0));
        const uint2 hi = *(const uint2 *)(row + (k + EPC / 2 < d ? k + EPC / 2 : 0));
        return u32x4_t{lo.x, lo.y, hi.x, hi.y};
    } else {
        T x[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) x[e] = row[k + e < d ? k + e : 0];
        u32x4_t v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (sizeof(T) == 4) v[i] = __float_as_uint(x[i]);
            else if constexpr (sizeof(T) == 2) v[i] = (unsigned)x[2 * i] | ((unsigned)x[2 * i + 1] << 16);
        }
        return v;
    }
}
template <int W, typename T>
__device__ __forceinline__ u32x4_t zero_tail(u32x4_t v, int k, int d) {
    constexpr int EPC = 16 / (int)sizeof(T);
    if constexpr (W == 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = k < d ? v[i] : 0u;
    } else if constexpr (W == 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = k + (i >= 2 ? EPC / 2 : 0) < d ? v[i] : 0u;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (sizeof(T) == 4) v[i] = k + i < d ? v[i] : 0u;
            else v[i] = k + 2 * i + 1 < d ? v[i] : k + 2 * i < d ? v[i] & 0xFFFFu : 0u;
        }
    }
    return v;
}

__device__ __forceinline__ f32x16 product(u32x4_t a, u32x4_t b, f32x16 acc, float) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j]), __uint_as_float(b[j]), acc, 0, 0, 0);
    return acc;
}
__device__ __forceinline__ f32x16 product(u32x4_t a, u32x4_t b, f32x16 acc, bf16_t) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// (codes: the 16-deep form takes the two halves of a chunk one after the other, on both sides alike)
__device__ __forceinline__ f32x16 product(u32x4_t a, u32x4_t b, f32x16 acc, fp8_t) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < 4; j += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(__builtin_bit_cast(long, u32x2{a[j], a[j + 1]}),
                                                         __builtin_bit_cast(long, u32x2{b[j], b[j + 1]}), acc, 0, 0, 0);
    return acc;
}

// Everything the wave holds in LDS is written or read before the workgroup goes on; loads from memory stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Streams `tiles` tiles of A (rows a0 .. of `a_rows`) past one tile of B (rows b0 ..): after the last slab of each
// tile, done(first row of the tile, acc) is called by all threads with the finished products.  Rows past the end are
// read from the last row; the caller discards them.
template <class Cfg, int W, typename T, class Done>
__device__ __forceinline__ void tile_stream(const T *__restrict__ A, long a_rows, long a0, int tiles, const T *__restrict__ B,
                                            long b_rows, long b0, int d, char *lds, Done done) {
    constexpr int EPC = 16 / (int)sizeof(T), SLAB = 8 * EPC;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wc = wave / Cfg::NWQ, wq = wave % Cfg::NWQ;
    const int row = t >> 3, chunk = t & 7;
    const int nslab = (d + SLAB - 1) / SLAB;
    const long total = (long)tiles * nslab;
    const T *bp[Cfg::JQ];
#pragma unroll
    for (int j = 0; j < Cfg::JQ; ++j) {
        const long r = b0 + row + 32 * j;
        bp[j] = B + (size_t)(r < b_rows ? r : b_rows - 1) * d;
    }
    const T *ap[Cfg::JC];
    long la = a0;   // first row of the tile being loaded
    int ls = 0;     // its slab
    u32x4_t reg[Cfg::DEPTH][Cfg::JC + Cfg::JQ];
    auto load = [&](u32x4_t(&r)[Cfg::JC + Cfg::JQ]) __attribute__((always_inline)) {
        if (ls == 0) {
#pragma unroll
            for (int j = 0; j < Cfg::JC; ++j) {
                const long x = la + row + 32 * j;
                ap[j] = A + (size_t)(x < a_rows ? x : a_rows - 1) * d;
            }
        }
        const int k = ls * SLAB + chunk * EPC;
#pragma unroll
        for (int j = 0; j < Cfg::JC; ++j) r[j] = load_chunk<W>(ap[j], k, d);
#pragma unroll
        for (int j = 0; j < Cfg::JQ; ++j) r[Cfg::JC + j] = load_chunk<W>(bp[j], k, d);
        if (++ls == nslab) {
            ls = 0;
            la += Cfg::BC;
        }
    };
    const int put = row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4);
    const int swz = (lane >> 1) & 7, h = lane >> 5;
    const int get_a = (wc * 32 * Cfg::WC + (lane & 31)) * 128, get_b = (Cfg::BC + wq * 32 * Cfg::WQ + (lane & 31)) * 128;
    f32x16 acc[Cfg::CHAINS][Cfg::WC][Cfg::WQ];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h2 = 0; h2 < Cfg::CHAINS; ++h2)
#pragma unroll
            for (int i = 0; i < Cfg::WC; ++i)
#pragma unroll
                for (int j = 0; j < Cfg::WQ; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[h2][i][j][e] = 0.f;
    };
    clear();
    long ca = a0;  // first row of the tile being multiplied
    int cs = 0;    // its slab
    // one slab: out of the registers into LDS, the load after next on its way, multiply.  One barrier: a stage is
    // written again two slabs later, when every wave has passed the barrier of the slab between.
    auto step = [&](u32x4_t(&r)[Cfg::JC + Cfg::JQ], char *stage, bool more) __attribute__((always_inline)) {
        const int k = cs * SLAB + chunk * EPC;
        if ((cs + 1) * SLAB > d) {  // uniform: the last slab of a row, if the row ends inside it
#pragma unroll
            for (int j = 0; j < Cfg::JC + Cfg::JQ; ++j) r[j] = zero_tail<W, T>(r[j], k, d);
        }
#pragma unroll
        for (int j = 0; j < Cfg::JC + Cfg::JQ; ++j) *(u32x4_t *)(stage + put + 4096 * j) = r[j];
        if (more) load(r);
        lds_barrier();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int c = ((2 * s + h) ^ swz) << 4;
            u32x4_t a[Cfg::WC], b[Cfg::WQ];
#pragma unroll
            for (int i = 0; i < Cfg::WC; ++i) a[i] = *(const u32x4_t *)(stage + get_a + 4096 * i + c);
#pragma unroll
            for (int j = 0; j < Cfg::WQ; ++j) b[j] = *(const u32x4_t *)(stage + get_b + 4096 * j + c);
#pragma unroll
            for (int i = 0; i < Cfg::WC; ++i)
#pragma unroll
                for (int j = 0; j < Cfg::WQ; ++j)
                    acc[s % Cfg::CHAINS][i][j] = product(a[i], b[j], acc[s % Cfg::CHAINS][i][j], T());
        }
        if (++cs == nslab) {
            if constexpr (Cfg::CHAINS == 2) acc[0][0][0] += acc[1][0][0];
            done(ca, acc[0]);
            cs = 0;
            ca += Cfg::BC;
            clear();
        }
    };
#pragma unroll
    for (int i = 0; i < Cfg::DEPTH; ++i)
        if (i < total) load(reg[i]);
    for (long it = 0; it < total; it += Cfg::DEPTH) {
#pragma unroll
        for (int i = 0; i < Cfg::DEPTH; ++i)
            if (it + i < total) step(reg[i], lds + (i & 1) * Cfg::STAGE, it + i + Cfg::DEPTH < total);
    }
}

// The eight workgroups b, b + 1, .. land on the eight XCDs: each XCD gets a run of consecutive pieces of work, so that
// what neighbours share (the centroids of a slice, for all query tiles) is fetched into one L2.
__device__ __forceinline__ long xcd_run(long total) {
    const long per = (total + 7) / 8;
    const long id = (long)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    return id < total ? id : -1;
}
inline unsigned xcd_grid(long total) { return (unsigned)((total + 7) / 8 * 8); }

// Phase 1 of a lookup: the best scaled product of every query of a tile with the rows of a slice, as a key that names
// the row.  GROUPS: of a top-k lookup: the two largest products of every group of 16 rows instead (see siso_internal.h).
template <class Cfg, int W, typename T, bool GROUPS, bool LEFT>  // LEFT: *many of the n queries
__global__ __launch_bounds__(256, Cfg::WC * Cfg::WQ == 1 ? 3 : 2) void k_lookup_tile(const T *__restrict__ Q, const T *__restrict__ cent,
                                                      const float *__restrict__ invn, long n, long K, int d,
                                                      int tiles_per_slice, int slices, int qtiles, u64 *keys, u64 *board,
                                                      float2 *groups, int ng, const int *__restrict__ many) {
    __shared__ __align__(16) char lds[2 * Cfg::STAGE];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wc = wave / Cfg::NWQ, wq = wave % Cfg::NWQ, h = lane >> 5;
    // (a step that ends in k_finalize_update: the slots of its board are emptied here, a kernel ahead)
    if (board != nullptr && blockIdx.x == 0 && t < SISO_FOLD_BOARD) board[t] = 0;
    const long id = xcd_run((long)qtiles * slices);
    if (id < 0) return;
    const long q0 = id % qtiles * Cfg::BQ;
    if constexpr (LEFT)
        if (q0 >= *many) return;
    const int s = (int)(id / qtiles);
    const long ctiles = (K + Cfg::BC - 1) / Cfg::BC;
    const long first = (long)s * tiles_per_slice;
    const int tiles = (int)(ctiles - first < tiles_per_slice ? ctiles - first : tiles_per_slice);
    float best[Cfg::WQ];
    int at[Cfg::WQ];
#pragma unroll
    for (int j = 0; j < Cfg::WQ; ++j) {
        best[j] = -INFINITY;
        at[j] = -1;
    }
    tile_stream<Cfg, W>(cent, K, first * Cfg::BC, tiles, Q, n, q0, d, lds,
                        [&](long c0, const f32x16(&acc)[Cfg::WC][Cfg::WQ]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < Cfg::WC; ++i) {
            const long r0 = c0 + (wc * Cfg::WC + i) * 32 + 4 * h;
            if constexpr (GROUPS) {
                TwoLargest most[Cfg::WQ];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 w4 = *(const float4 *)(invn + r0 + 8 * g);  // (NaN behind the live rows)
                    const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int j = 0; j < Cfg::WQ; ++j) most[j].take(acc[i][j][4 * g + e] * w[e], (unsigned)(4 * g + e));
                }
                const int grp = (int)(r0 >> 5) * 2 + h;
#pragma unroll
                for (int j = 0; j < Cfg::WQ; ++j) {
                    const long q = q0 + (wq * Cfg::WQ + j) * 32 + (lane & 31);
                    if (q < n && grp < ng) groups[(size_t)q * ng + grp] = make_float2(most[j].first, most[j].second);
                }
                continue;
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 w4 = *(const float4 *)(invn + r0 + 8 * g);  // (NaN behind the live rows: those never win)
                const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < Cfg::WQ; ++j) {
                        const float v = acc[i][j][4 * g + e] * w[e];
                        if (v > best[j]) {  // rows ascend: the lowest index keeps a tie
                            best[j] = v;
                            at[j] = (int)(r0 + 8 * g + e);
                        }
                    }
            }
        }
    });
    if constexpr (GROUPS) return;
    lds_barrier();  // everyone is done with the stages: the keys of the waves that share a query meet there
    u64(*red)[Cfg::BQ] = (u64(*)[Cfg::BQ])lds;
#pragma unroll
    for (int j = 0; j < Cfg::WQ; ++j) {
        u64 key = at[j] < 0 ? 0ull : pack_key(best[j], (unsigned)at[j]);
        const LanePair<u64> both = lane_pair<32>(key);
        key = both.b > both.a ? both.b : both.a;
        if (h == 0) red[wc][(wq * Cfg::WQ + j) * 32 + lane] = key;
    }
    __syncthreads();
    if (t < Cfg::BQ && q0 + t < n) {
        u64 key = red[0][t];
#pragma unroll
        for (int w = 1; w < Cfg::NWC; ++w) key = red[w][t] > key ? red[w][t] : key;
        keys[(size_t)(q0 + t) * slices + s] = key;
    }
}

// Small single-precision lookups: a tile of 32 x 32 per workgroup, and the dimension split among its four waves, whose sums meet
// in LDS.  Such a problem does not fill the chip with larger tiles, and then takes as long as one of their waves takes for
// the whole dimension, slab by slab: 256 queries x 1,024 rows x 384 in 64 x 64 tiles are 64 workgroups for 256 compute
// units and 192 instructions of 64 cycles in a row for each wave; here 256 workgroups and 48.  Fragments come from memory
// straight into registers (what the workgroups share is in L2), a group of steps ahead of the one being multiplied.
template <int W, bool LEFT>
__global__ __launch_bounds__(256) void k_lookup_split(const float *__restrict__ Q, const float *__restrict__ cent,
                                                      const float *__restrict__ invn, long n, long K, int d, int slices, int qtiles,
                                                      u64 *keys, u64 *board, const int *__restrict__ many) {
    constexpr int G = 6;  // steps of eight elements whose fragments are under way together
    __shared__ float red[4][16][64];
    __shared__ u64 best_s[4][32];
    const int t = threadIdx.x, lane = t & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (board != nullptr && blockIdx.x == 0 && t < SISO_FOLD_BOARD) board[t] = 0;  // (see k_lookup_tile)
    const long id = xcd_run((long)qtiles * slices);
    if (id < 0) return;
    const long q0 = id % qtiles * 32, c0 = id / qtiles * 32;
    if constexpr (LEFT)
        if (q0 >= *many) return;
    const long cr = c0 + (lane & 31), qr = q0 + (lane & 31);
    const float *a_row = cent + (size_t)(cr < K ? cr : K - 1) * d, *b_row = Q + (size_t)(qr < n ? qr : n - 1) * d;
    const int steps = (d + 31) / 32;  // of every wave; wave w has the elements from 8 * steps * w on
    const int k0 = 8 * steps * wave + 4 * h;
    const float4 w4 = *(const float4 *)(invn + c0 + 8 * wave + 4 * h);  // (NaN behind the live rows: those never win)
    u32x4_t a[2][G], b[2][G];
    auto load = [&](int buf_, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int buf = 0; buf < 2; ++buf)
            if (buf == buf_) {
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    const int k = first + s < steps ? k0 + 8 * (first + s) : d;  // (from d on: zeros, see zero_tail)
                    a[buf][s] = load_chunk<W>(a_row, k, d);
                    b[buf][s] = load_chunk<W>(b_row, k, d);
                }
            }
    };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    auto multiply = [&](int buf_, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int buf = 0; buf < 2; ++buf)
            if (buf == buf_) {
#pragma unroll
                for (int s = 0; s < G; ++s) {
                    const int k = first + s < steps ? k0 + 8 * (first + s) : d;
                    acc = product(zero_tail<W, float>(a[buf][s], k, d), zero_tail<W, float>(b[buf][s], k, d), acc, 0.f);
                }
            }
    };
    load(0, 0);
    load(1, G);
    for (int first = 0; first < steps; first += 2 * G) {
        multiply(0, first);
        if (first + 2 * G < steps) load(0, first + 2 * G);
        if (first + G < steps) multiply(1, first + G);
        if (first + 3 * G < steps) load(1, first + 3 * G);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][e][lane] = acc[e];
    __syncthreads();
    // wave w sums registers 4 w .. 4 w + 3: rows c0 + 8 w + 4 h + e of column lane % 32
    const float w[4] = {w4.x, w4.y, w4.z, w4.w};
    float best = -INFINITY;
    int at = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int r = 4 * wave + e;
        const float v = ((red[0][r][lane] + red[1][r][lane]) + (red[2][r][lane] + red[3][r][lane])) * w[e];
        if (v > best) {  // rows ascend: the lowest index keeps a tie
            best = v;
            at = (int)(c0 + 8 * wave + 4 * h + e);
        }
    }
    u64 key = at < 0 ? 0ull : pack_key(best, (unsigned)at);
    const LanePair<u64> both = lane_pair<32>(key);
    key = both.b > both.a ? both.b : both.a;
    if (h == 0) best_s[wave][lane] = key;
    __syncthreads();
    if (t < 32 && q0 + t < n) {
#pragma unroll
        for (int x = 0; x < 4; ++x) key = best_s[x][t] > key ? best_s[x][t] : key;
        keys[(size_t)(q0 + t) * slices + id / qtiles] = key;
    }
}

// Pairs (i, j), i < j, of rows whose cosine exceeds the threshold: one pair of tiles per workgroup, upper triangle
// only; the rows j are A, the rows i are B (a lane holds one i and 16 rows j of every block).  A launch takes the `pairs`
// pairs of tiles from number `first` on.
template <class Cfg, int W, typename T>
__global__ __launch_bounds__(256, 2) void k_pairs_tile(const T *__restrict__ rows, const float *__restrict__ invn, long K, int d,
                                                     float threshold, long first, long pairs, int *out_pairs, long cap,
                                                     u64 *counter, PairsRedo redo) {
    if (redo.count != nullptr && *redo.count <= redo.above) return;  // (a screened search has found them all)
    static_assert(Cfg::BC == Cfg::BQ, "square tiles");
    __shared__ __align__(16) char lds[2 * Cfg::STAGE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wc = wave / Cfg::NWQ, wq = wave % Cfg::NWQ, h = lane >> 5;
    const long run = xcd_run(pairs);
    if (run < 0) return;
    const long id = first + run;
    // id = y (y + 1) / 2 + x, x <= y
    long y = (long)((sqrt(8.0 * (double)id + 1.0) - 1.0) * 0.5);
    while (y * (y + 1) / 2 > id) --y;
    while ((y + 1) * (y + 2) / 2 <= id) ++y;
    const long i0 = (id - y * (y + 1) / 2) * Cfg::BC, j0 = y * Cfg::BC;
    tile_stream<Cfg, W>(rows, K, j0, 1, rows, K, i0, d, lds,
                        [&](long, const f32x16(&acc)[Cfg::WC][Cfg::WQ]) __attribute__((always_inline)) {
#pragma unroll
        for (int jj = 0; jj < Cfg::WQ; ++jj) {
            const long i = i0 + (wq * Cfg::WQ + jj) * 32 + (lane & 31);
            const float wi = invn[i];  // (NaN behind the last row)
#pragma unroll
            for (int ii = 0; ii < Cfg::WC; ++ii) {
                const long r0 = j0 + (wc * Cfg::WC + ii) * 32 + 4 * h;
                unsigned mask = 0;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 w4 = *(const float4 *)(invn + r0 + 8 * g);
                    const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const long j = r0 + 8 * g + e;
                        if (i < j && j < K && acc[ii][jj][4 * g + e] * wi * w[e] > threshold) mask |= 1u << (4 * g + e);
                    }
                }
                if (__ballot(mask != 0) != 0)
                    emit_pairs(mask, (int)i, [&](int I) { return (int)(r0 + 8 * (I >> 2) + (I & 3)); }, out_pairs, cap, counter);
            }
        }
    });
}

// bytes that every row of the two arrays is aligned to (16, 8, or the element's size)
template <typename T>
int row_alignment(const void *a, const void *b, int d) {
    const uintptr_t x = (uintptr_t)a | (uintptr_t)b | (uintptr_t)((size_t)d * sizeof(T));
    return (x & 15) == 0 ? 16 : (x & 7) == 0 ? 8 : (int)sizeof(T);
}

struct TilePlan {
    int cfg;  // 0 = TileFew, 1 = TileSmall, 2 = TileLarge, 3 = k_lookup_split
    int tiles_per_slice, slices, qtiles;
};

// left: for what a screened lookup leaves over of n queries.  Mostly they are few, and their tiles have the chip to themselves:
// shorter slices give each tile more workgroups, where one walked through a seventh of the rows for a single query (4,096
// queries, 60,000 x 768, some hundreds of them left over: 3,360 -> 825 us; all of them: 3,058 -> 3,020).  Four tiles long: a
// launch that finds nothing to do has to get rid of its workgroups (3,752 of them instead of 472: 2 us).
TilePlan tile_plan(const siso_cache *c, long n, bool groups, bool left) {
    TilePlan p;
    auto tiles = [](long rows, int per) { return (rows + per - 1) / per; };
    // the large tile needs at least two of them per compute unit to be worth its fewer reads
    // (few queries: up to 64 in bf16, see TileCfg, and in codes, where a second tile of them finds the rows in L2)
    p.cfg = n <= (c->dtype == SISO_F32 ? 32 : 64) ? 0 : tiles(c->count, 128) * tiles(n, 128) >= 512 ? 2 : 1;
    // One workgroup of k_lookup_split for every compute unit, or two of long rows; beyond that the larger tiles read less.  Lookup
    // alone, 64 x 64 tiles / split, us: 1,024 rows x 256 queries x 384 14.8 / 11.3, 4,000 x 64 x 768 23.6 / 14.9, 300 x 300 x
    // 2,048 52.0 / 23.9; 504 workgroups: 2,000 x 256 x 768 24.0 / 20.8, 4,000 x 128 x 128 9.0 / 12.4; 1,000 of them: 4,000 x
    // 256 x 768 25.1 / 33.0, 16,000 x 64 x 384 15.1 / 20.7.
    const long split = tiles(c->count, 32) * tiles(n, 32);
    if (p.cfg == 1 && c->dtype == SISO_F32 && !groups && split <= (c->dim >= 512 ? 512 : 256)) {
        p.cfg = 3;
        p.tiles_per_slice = 1;
        p.slices = (int)tiles(c->count, 32);
        p.qtiles = (int)tiles(n, 32);
        return p;
    }
    const int bc = p.cfg == 1 ? 64 : 128, bq = p.cfg == 0 ? 32 : p.cfg == 1 ? 64 : 128;
    const long resident = p.cfg == 2 ? 512 : 1024;  // workgroups the chip holds at a time
    const long ct = tiles(c->count, bc), qt = tiles(n, bq);
    long tps = (ct * qt + resident - 1) / resident;
    if (tps > ct) tps = ct;
    if (tps < 1) tps = 1;
    if (p.cfg == 2) {
        // The large tiles keep the matrix cores of a compute unit busy two at a time, so what counts is the number of tiles
        // the busiest unit gets: among the slice lengths, the one with the least of them, a workgroup counted as its
        // tiles and a fifth for getting started (8 query tiles x 469 centroid tiles: 94 slices of 5 leave the busiest
        // unit 15 tiles, 59 of 8 leave it 16: 844 -> 814 us for two batches of 1,000 x 60,000 x 384 floats).
        double least = 1e30;
        for (long t = 1; t <= ct && t <= 64; ++t) {
            const long groups = tiles(ct, (int)t) * qt;
            if (groups < 512 && t > 1) break;
            if (groups > 4096) continue;  // (the keys of a lookup stay within half of the library's static workspace)
            const double cost = (double)tiles(groups, 256) * ((double)t + 0.2);
            if (cost < least) {
                least = cost;
                tps = t;
            }
        }
    }
    if (left && tps > 4) {
        const long most = (ct * qt + 4095) / 4096;
        tps = most > 4 ? most : 4;
    }
    p.tiles_per_slice = (int)tps;
    p.slices = (int)tiles(ct, (int)tps);
    p.qtiles = (int)qt;
    return p;
}

template <typename T, int W, bool GROUPS, bool LEFT>
int lookup_launch(siso_cache *c, const void *queries, long n, const TilePlan &p, u64 *keys, float2 *groups, int ng, const int *many) {
    const dim3 grid(xcd_grid((long)p.qtiles * p.slices)), block(256);
#define SISO_LAUNCH_TILE(Cfg)                                                                                            \
    hipLaunchKernelGGL((k_lookup_tile<Cfg, W, T, GROUPS, LEFT>), grid, block, 0, c->stream, (const T *)queries, (const T *)c->cent, c->invn, \
                       n, c->count, c->dim, p.tiles_per_slice, p.slices, p.qtiles, keys, c->board_to_clear, \
                       groups, ng, many)
    if (p.cfg == 0) SISO_LAUNCH_TILE(TileFew);
    else if (p.cfg == 1) SISO_LAUNCH_TILE(TileSmall);
    else SISO_LAUNCH_TILE(TileLarge);
#undef SISO_LAUNCH_TILE
    c->board_to_clear = nullptr;  // taken
    return siso_check_hip(c, hipGetLastError(), "k_lookup_tile");
}

template <int W, bool LEFT>
int split_launch(siso_cache *c, const void *queries, long n, const TilePlan &p, u64 *keys, const int *many) {
    hipLaunchKernelGGL((k_lookup_split<W, LEFT>), dim3(xcd_grid((long)p.qtiles * p.slices)), dim3(256), 0, c->stream, (const float *)queries,
                       (const float *)c->cent, c->invn, n, c->count, c->dim, p.slices, p.qtiles, keys, c->board_to_clear, many);
    c->board_to_clear = nullptr;  // taken
    return siso_check_hip(c, hipGetLastError(), "k_lookup_split");
}

template <typename T, bool GROUPS, bool LEFT = false>
int lookup_launch_t(siso_cache *c, const void *queries, long n, const TilePlan &p, u64 *keys, float2 *groups, int ng,
                    const int *many = nullptr) {
    if (p.cfg == 3) switch (row_alignment<T>(queries, c->cent, c->dim)) {
            case 16: return split_launch<16, LEFT>(c, queries, n, p, keys, many);
            case 8: return split_launch<8, LEFT>(c, queries, n, p, keys, many);
            default: return split_launch<4, LEFT>(c, queries, n, p, keys, many);
        }
    switch (row_alignment<T>(queries, c->cent, c->dim)) {
        case 16: return lookup_launch<T, 16, GROUPS, LEFT>(c, queries, n, p, keys, groups, ng, many);
        case 8: return lookup_launch<T, 8, GROUPS, LEFT>(c, queries, n, p, keys, groups, ng, many);
        default: return lookup_launch<T, (int)sizeof(T), GROUPS, LEFT>(c, queries, n, p, keys, groups, ng, many);
    }
}

#define PAIR_TILES_PER_LAUNCH (1L << 22)
template <typename T, int W>
int pairs_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                 u64 *counter, PairsRedo redo) {
    // small sets: more and smaller tiles, so that every compute unit has one
    const long large = (count + TileLarge::BC - 1) / TileLarge::BC, small = (count + TileSmall::BC - 1) / TileSmall::BC;
    const bool few = large * (large + 1) / 2 < 512;
    const long tiles = few ? small : large, pairs = tiles * (tiles + 1) / 2;
    // a launch holds fewer than 2^32 threads: 128-row tiles of more than 741,000 rows are more workgroups than that
    for (long first = 0; first < pairs; first += PAIR_TILES_PER_LAUNCH) {
        const long many = pairs - first < PAIR_TILES_PER_LAUNCH ? pairs - first : PAIR_TILES_PER_LAUNCH;
        const dim3 grid(xcd_grid(many)), block(256);
        if (few)
            hipLaunchKernelGGL((k_pairs_tile<TileSmall, W, T>), grid, block, 0, c->stream, (const T *)rows, invn, count, c->dim,
                               threshold, first, many, out_pairs, cap, counter, redo);
        else
            hipLaunchKernelGGL((k_pairs_tile<TileLarge, W, T>), grid, block, 0, c->stream, (const T *)rows, invn, count, c->dim,
                               threshold, first, many, out_pairs, cap, counter, redo);
        const int rc = siso_check_hip(c, hipGetLastError(), "k_pairs_tile");
        if (rc != SISO_OK) return rc;
    }
    return SISO_OK;
}

template <typename T>
int pairs_launch_t(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs, long cap,
                   u64 *counter, PairsRedo redo) {
    switch (row_alignment<T>(rows, rows, c->dim)) {
        case 16: return pairs_launch<T, 16>(c, rows, invn, count, threshold, out_pairs, cap, counter, redo);
        case 8: return pairs_launch<T, 8>(c, rows, invn, count, threshold, out_pairs, cap, counter, redo);
        default: return pairs_launch<T, (int)sizeof(T)>(c, rows, invn, count, threshold, out_pairs, cap, counter, redo);
    }
}

}  // namespace

// Is a bf16 batch that the pipelined kernels could take better off here?  Their workgroups have tiles of 256 rows x up to
// 256 queries, one per compute unit: a small problem leaves most units without one, and the few that work pass through
// the whole dimension at the pace of a single workgroup.  Measured, lookup of n queries among K rows of 768 elements, pipelined
// against tiled, us: K 1,000: n 1 13.5 / 11.5, n 64 14.7 / 12.0, n 256 26.3 / 11.6, n 1,024 28.7 / 12.5; K 16,000:
// n 32 18.6 / 12.1, n 128 21.1 / 13.7, n 256 31.8 / 19.7, n 1,024 32.3 / 35.3; K 64,000: n 64 22.0 / 25.1, n 256 33.2 / 35.7.
// With about half the units busy (126 such tiles: 31.8 against 32.3; of 256 elements 17.9 against 16.5) the two meet.
int siso_tile_preferred(const siso_cache *c, long n) {
    const long tiles = (c->count + 255) / 256 * ((n + 255) / 256);
    // Codes (twice the rate of the matrix cores in the pipelined kernels): n 64, K 32,000: 19.4 / 16.7; n 256, K 16,000:
    // 23.5 / 20.6, K 32,000: 24.2 / 28.7; n 512, K 16,000: 23.5 / 29.0; n 1,024, K 4,000: 24.2 / 21.5.
    const long limit = c->dtype == SISO_FP8 && n > 128 ? 70 : 112;
    return c->dtype != SISO_F32 && c->opt_mfma_config == 0 && tiles < limit;
}

int siso_tile_slices(const siso_cache *c, long n, bool left) { return c->count < 1 || n < 1 ? 1 : tile_plan(c, n, false, left).slices; }

// No more keys than this, for n queries and any number of rows up to the capacity (the slices are not monotone in it): the
// slices of a query tile are at most 4,096 workgroups' worth (tile_plan), and no more than there are tiles.
long siso_tile_keys_bound(const siso_cache *c, long n) {
    const long all = (c->capacity + 31) / 32, most = 4096 / ((n + 127) / 128) + 1;
    return n * (all < most ? all : most);
}

int siso_tile_launch(siso_cache *c, const void *queries, long n, int slices, u64 *keys, const int *many) {
    const TilePlan p = tile_plan(c, n, false, many != nullptr);
    if (p.slices != slices) return siso_fail(c, SISO_EINVAL, "tiled lookup: plan mismatch");
    if (c->dtype == SISO_FP8) return lookup_launch<fp8_t, 16, false, false>(c, queries, n, p, keys, nullptr, 0, nullptr);  // (whole slabs)
    if (many != nullptr)
        return c->dtype == SISO_F32 ? lookup_launch_t<float, false, true>(c, queries, n, p, keys, nullptr, 0, many)
                                    : lookup_launch_t<bf16_t, false, true>(c, queries, n, p, keys, nullptr, 0, many);
    return c->dtype == SISO_F32 ? lookup_launch_t<float, false>(c, queries, n, p, keys, nullptr, 0)
                                : lookup_launch_t<bf16_t, false>(c, queries, n, p, keys, nullptr, 0);
}

int siso_tile_groups_launch(siso_cache *c, const void *queries, long n, float2 *groups, int ng) {
    const TilePlan p = tile_plan(c, n, true, false);
    if (c->dtype == SISO_FP8) return lookup_launch<fp8_t, 16, true, false>(c, queries, n, p, nullptr, groups, ng, nullptr);
    return c->dtype == SISO_F32 ? lookup_launch_t<float, true>(c, queries, n, p, nullptr, groups, ng)
                                : lookup_launch_t<bf16_t, true>(c, queries, n, p, nullptr, groups, ng);
}

int siso_pairs_tile_launch(siso_cache *c, const void *rows, const float *invn, long count, float threshold, int *out_pairs,
                           long cap, u64 *counter, PairsRedo redo) {
    if (count < 2) return SISO_OK;
    if (count > 65535L * 64) return siso_fail(c, SISO_EINVAL, "tiled pair search handles at most %d rows", 65535 * 64);
    return c->dtype == SISO_F32 ? pairs_launch_t<float>(c, rows, invn, count, threshold, out_pairs, cap, counter, redo)
                                : pairs_launch_t<bf16_t>(c, rows, invn, count, threshold, out_pairs, cap, counter, redo);
}
