// What the pipelined kernels share (lookup_mfma.hip, screen.hip): tile configurations, direct loads into LDS, fragment
// reads and their waits, accumulators, the map from workgroups to tiles.  lookup_mfma.hip describes the pipeline.
#pragma once

#include "siso_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ROWS: the keys of the lookup carry the winning row itself instead of its group of four rows (more
// compares per product, affordable where the kernel waits for memory anyway; the finalize step then
// has no centroid rows to read)
// ES: bytes per element: 2 = bf16; 1 = the 8-bit storage variant (E4M3 codes: a slab then holds 128 elements
// in the same 128 bytes per row, and a 16-byte fragment feeds two v_mfma_f32_32x32x16_fp8_fp8, one per half)
template <int WC_, int WQ_, int NWC_, int NWQ_, int NSTAGE_, int BK_ = 64, bool ROWS_ = false, int ES_ = 2, bool K64_ = false>
struct PipeCfg {
    static constexpr int WC = WC_, WQ = WQ_, NWC = NWC_, NWQ = NWQ_, NSTAGE = NSTAGE_;
    static constexpr bool ROWS = ROWS_;
    static constexpr int ES = ES_;
    static constexpr bool K64 = K64_;  // codes only: 64-deep MFMAs, 32 bytes per lane and operand (see k_lookup_pipe)
    static_assert(!K64_ || ES_ == 1, "the 64-deep form is for one-byte elements");
    static constexpr int BK = BK_;            // elements of the dimension per slab (64; or 32: half lines; 128 codes)
    static constexpr int RB = BK * ES;        // bytes of a tile row in a stage
    static constexpr int CPR = RB / 16;       // 16-byte chunks per tile row
    static constexpr int RPI = 64 / CPR;      // tile rows one direct load of a wave fills
    static constexpr int RP = 256 / RB;       // tile rows per 256 bytes (all 64 banks)
    static constexpr int KK = RB / 32;        // fragment steps per slab (a step = one 16-byte chunk per lane half)
    static constexpr int BC = 32 * WC * NWC;  // centroid rows per tile
    static constexpr int BQ = 32 * WQ * NWQ;  // query rows per tile
    static constexpr int NW = NWC * NWQ, NT = 64 * NW;
    static constexpr int STAGE = (BC + BQ) * RB;
    static constexpr int NLA = BC / RPI / NW, NLB = BQ / RPI / NW;  // direct loads per wave and slab
    static_assert((ES == 2 && (BK == 64 || BK == 32)) || (ES == 1 && BK == 128), "slab of 64 or 32 bf16 elements, or 128 codes");
    static constexpr int NL = NLA + NLB;
    static constexpr int NINV = 3;  // tiles whose inverse lengths are kept at a time (see k_lookup_pipe)
    static constexpr int LDS_BYTES = NSTAGE * STAGE + NINV * BC * 4;
    static_assert((BC / RPI) % NW == 0 && (BQ / RPI) % NW == 0, "whole row groups per wave");
    static_assert(BC <= SISO_PAD_ROWS && BC <= NT && BC % 64 == 0, "tile of inverse lengths: one direct load per wave");
    static_assert(BQ * NWC * 8 <= NSTAGE * STAGE, "reduction scratch fits in the stage buffers");
    static_assert(NSTAGE >= 2 && LDS_BYTES <= 160 * 1024, "stages fit in LDS");
    static_assert((NSTAGE - 1) * NL <= 63, "wait count fits the counter");
};

// direct global -> LDS loads: lane i of the wave writes its 16 (4) bytes at lds_wave_base + 16 (4) * i
__device__ __forceinline__ void gload_lds16(const void *g, void *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 0);
}
// the same with the non-temporal hint: data that is read once should not push reusable lines out of L2
__device__ __forceinline__ void gload_lds16_nt(const void *g, void *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 2);
}
__device__ __forceinline__ void gload_lds4(const void *g, void *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 4, 0, 0);
}

// LDS fragment reads and their waits are written out by hand: while direct loads are in
// flight the compiler waits for *all* outstanding LDS reads before every use, which would
// serialise the fragment double buffering.  LDS operations complete in order, so
// "lgkmcnt(N)" = everything but the newest N reads has arrived.  Each read and its wait sit
// in the same straight-line stretch of code.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_frag(unsigned addr) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2 ; hand-scheduled" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return __builtin_bit_cast(bf16x8, v);
}
template <int N, int NA, int NB>
__device__ __forceinline__ void lds_wait(bf16x8 (&a)[NA], bf16x8 (&b)[NB]) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a[0]) : "n"(N));
#pragma unroll
    for (int i = 1; i < NA; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(b[i]));
}
// the same for the fragments of the 64-deep form (two chunks per block row; B in two buffers)
template <int N, int NA, int NB>
__device__ __forceinline__ void lds_wait64(bf16x8 (&al)[NA], bf16x8 (&ah)[NA], bf16x8 (&bl)[2][NB], bf16x8 (&bh)[2][NB]) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(al[0]) : "n"(N));
#pragma unroll
    for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(al[i]), "+v"(ah[i]));
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(bl[0][i]), "+v"(bh[0][i]), "+v"(bl[1][i]), "+v"(bh[1][i]));
}
// SUB = bytes between the 32-row blocks of a wave's tile (32 tile rows)
template <int SUB, int NA, int NB>
__device__ __forceinline__ void lds_frags(bf16x8 (&a)[NA], bf16x8 (&b)[NB], unsigned addr_a, unsigned addr_b) {
    static_assert(NA <= 4 && NB <= 4, "fragment offsets are spelled out up to four");
    a[0] = lds_frag<0>(addr_a);
    if constexpr (NA > 1) a[1] = lds_frag<SUB>(addr_a);
    if constexpr (NA > 2) a[2] = lds_frag<2 * SUB>(addr_a);
    if constexpr (NA > 3) a[3] = lds_frag<3 * SUB>(addr_a);
    b[0] = lds_frag<0>(addr_b);
    if constexpr (NB > 1) b[1] = lds_frag<SUB>(addr_b);
    if constexpr (NB > 2) b[2] = lds_frag<2 * SUB>(addr_b);
    if constexpr (NB > 3) b[3] = lds_frag<3 * SUB>(addr_b);
}
template <int N>
__device__ __forceinline__ void vm_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The barrier between slabs.  Every wave has waited for its own LDS reads and for the loads that must have landed;
// __syncthreads() would wait for all other direct loads as well, those of the slabs further ahead (one query against 60,000 x
// 768 bf16 rows, sixteen steps: 378 -> 371 us; 64 against 262,144: 1,159 -> 1,146).
__device__ __forceinline__ void slab_barrier() { asm volatile("s_barrier" ::: "memory"); }

// compile-time loop: f(IC<0>{}), f(IC<1>{}), ...
template <int I>
struct IC {
    static constexpr int value = I;
};
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(IC<I>{});
        static_for<I + 1, N>(f);
    }
}

// The accumulator blocks of a wave: WC x WQ blocks of 32 x 32, 16 registers per lane each.
// Up to 8 blocks they are ordinary values and the compiler places them.
// One fragment step: 16 bytes per lane of either operand.  bf16: one MFMA over 16 elements (8 per lane half);
// E4M3 codes: two MFMAs over 16 codes each (the low and the high 8 bytes of both fragments: both operands
// split their bytes the same way, which is all a dot product asks of the order of its terms).
template <bool F8>
__device__ __forceinline__ f32x16 frag_mma(bf16x8 a, bf16x8 b, f32x16 c) {
    if constexpr (F8) {
        typedef long l2 __attribute__((ext_vector_type(2)));
        const l2 a2 = __builtin_bit_cast(l2, a), b2 = __builtin_bit_cast(l2, b);
        c = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a2[0], b2[0], c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a2[1], b2[1], c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
}

// The 64-deep form over E4M3 codes: 32 bytes per lane of either operand = two 16-byte chunks (scales of 2^0).
__device__ __forceinline__ f32x16 frag_mma64(bf16x8 a_lo, bf16x8 a_hi, bf16x8 b_lo, bf16x8 b_hi, f32x16 c) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    typedef int i8 __attribute__((ext_vector_type(8)));
    const i8 a = __builtin_shufflevector(__builtin_bit_cast(i4, a_lo), __builtin_bit_cast(i4, a_hi), 0, 1, 2, 3, 4, 5, 6, 7);
    const i8 b = __builtin_shufflevector(__builtin_bit_cast(i4, b_lo), __builtin_bit_cast(i4, b_hi), 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
}

template <bool FIXED, int WC, int WQ, bool F8 = false>
struct Acc {
    f32x16 v[WC][WQ];
    template <int A, int B>
    __device__ __forceinline__ void first(bf16x8 a, bf16x8 b) {  // start from zero
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        v[A][B] = frag_mma<F8>(a, b, zero);
    }
    template <int A, int B>
    __device__ __forceinline__ void mac(bf16x8 a, bf16x8 b) {
        v[A][B] = frag_mma<F8>(a, b, v[A][B]);
    }
    template <int A, int B, int I>
    __device__ __forceinline__ float get() const {
        return v[A][B][I];
    }
    __device__ __forceinline__ void reserve() {}
};
// With 16 blocks the accumulators fill the AGPR half of the register file exactly, which the
// register allocator cannot pack (it spills).  So block (A, B) sits in a[16*(A*WQ+B) .. +15] by
// hand: the MFMAs and the reads are written out, and the compiler only learns that those
// registers are taken.  It knows of no dependence between these statements, so all of them are
// volatile (kept in program order), and the hardware's rules are kept by construction: a block
// is read back only after 15 more MFMAs have been issued behind the one that wrote it (or, for
// the last blocks, after the whole scaling of the blocks before them), far beyond the 8 passes
// such an MFMA takes; and a block is overwritten only by an MFMA issued after it was read.
template <int WC, int WQ>
struct Acc<true, WC, WQ, false> {
    template <int A, int B>
    __device__ __forceinline__ void first(bf16x8 a, bf16x8 b) {
        constexpr int R = 16 * (A * WQ + B);
        asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, 0 ; hand-placed" ::"v"(a), "v"(b), "n"(R), "n"(R + 15));
    }
    template <int A, int B>
    __device__ __forceinline__ void mac(bf16x8 a, bf16x8 b) {
        constexpr int R = 16 * (A * WQ + B);
        asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3] ; hand-placed" ::"v"(a), "v"(b), "n"(R),
                     "n"(R + 15));
    }
    template <int A, int B, int I>
    __device__ __forceinline__ float get() const {
        float x;
        asm volatile("v_accvgpr_read_b32 %0, a[%1] ; hand-placed" : "=v"(x) : "n"(16 * (A * WQ + B) + I));
        return x;
    }
    // tells the compiler (and through it the kernel descriptor) that a0 .. a255 and the fragment
    // registers are in use (it warns that some of them are not its to hand out anyway)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    __device__ __forceinline__ void reserve() {
        static_assert(WC * WQ == 16, "all 256 AGPRs");
        asm volatile("; fragments: v[208:255]" ::: "v208", "v255");
        asm volatile("; accumulators: a[0:255]" ::: "a0", "a15", "a16", "a31", "a32", "a47", "a48", "a63", "a64", "a79", "a80",
                     "a95", "a96", "a111", "a112", "a127", "a128", "a143", "a144", "a159", "a160", "a175", "a176", "a191",
                     "a192", "a207", "a208", "a223", "a224", "a239", "a240", "a255");
    }
#pragma clang diagnostic pop
};

// Block -> (query tile qt, slice s of the centroid tiles).  Workgroups are handed to the 8 XCDs
// round robin and every XCD has its own L2.  The 32 workgroups that run together on one XCD are
// made a unit of qb query tiles x 32/qb slices, so that a centroid tile fetched into that L2
// serves qb workgroups and qb query tiles stay resident in it.  With many groups of 32/qb slices
// an XCD owns every eighth group and walks through all blocks of query tiles for it before moving
// on (the same slices again and again: repeats come from the caches); with at most four groups
// the XCDs also split the blocks of query tiles among them, so that none stays idle.
// False = nothing to do for this block.
__host__ __device__ __forceinline__ int pipe_group_split(int groups) { return groups <= 1 ? 1 : groups == 2 ? 2 : 4; }
static long pipe_grid(long slices, long nqt, int qb) {
    const long sb = 32 / qb, groups = (slices + sb - 1) / sb, nqb = (nqt + qb - 1) / qb;
    if (groups > 4) return 8 * ((groups + 7) / 8) * nqb * 32;
    const long r = 8 / pipe_group_split((int)groups);  // XCDs per group of slices
    return 8 * ((nqb + r - 1) / r) * 32;
}
// Rounds of 32 workgroups that the busiest XCD goes through.
static long pipe_rounds(long slices, long nqt, int qb) {
    const long sb = 32 / qb, groups = (slices + sb - 1) / sb, nqb = (nqt + qb - 1) / qb;
    if (groups <= 4) {
        const long r = 8 / pipe_group_split((int)groups);
        return (nqb + r - 1) / r;
    }
    long busiest = 0;
    for (long x = 0; x < 8 && x < groups; ++x) {  // XCD x owns the groups x, x + 8, ...
        long mine = 0;
        for (long g = x; g < groups; g += 8) mine += (g + 1) * sb <= slices ? sb : slices - g * sb;
        if (mine > busiest) busiest = mine;
    }
    return (busiest * nqt + 31) / 32;
}
template <int BC>
__device__ __forceinline__ bool pipe_map_block(long K, int tiles_per_slice, int slices, int nqt, int qb, int &qt, int &s,
                                               int &ct_begin, int &ct_end) {
    const int total_ct = (int)((K + BC - 1) / BC);
    const int sb = 32 / qb, groups = (slices + sb - 1) / sb, nqb = (nqt + qb - 1) / qb;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int i = local & 31, u = local >> 5;  // place in the unit, number of the unit on this XCD
    int g, b;
    if (groups > 4) {
        g = (u / nqb) * 8 + xcd;
        b = u % nqb;
    } else {
        const int gp = pipe_group_split(groups);
        g = xcd % gp;
        b = xcd / gp + (8 / gp) * u;
    }
    if (g >= groups || b >= nqb || i >= qb * sb) return false;  // (qb need not divide 32: the last places stay empty)
    qt = b * qb + i % qb;
    s = g * sb + i / qb;
    if (qt >= nqt || s >= slices) return false;
    ct_begin = s * tiles_per_slice;
    ct_end = (ct_begin + tiles_per_slice < total_ct) ? ct_begin + tiles_per_slice : total_ct;
    return true;
}

// The value lane l ^ 32 holds: v_permlane32_swap exchanges the upper half of its first register with the
// lower half of its second; given the same value twice, the first then holds the lower half in both halves
// and the second the upper half in both.  One instruction, no LDS crossbar.
__device__ __forceinline__ unsigned other_half(unsigned v) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
}

// The tile pairs of a pair search (see k_pairs_stream): the sequence that one workgroup walks through.  All pairs of tiles stand
// in one order: groups of sb row tiles, in a group column after column, in a column row after row, and behind the columns
// that all rows of the group have the few on the diagonal.  32 pairs in a row are a block of sb rows and 32 / sb columns.  An XCD
// has an eighth of them, and its 32 workgroups take one of 32 each: every share is as large as the next, but for one pair.
// (Whole groups were dealt out to the XCDs before: the busiest workgroup of 196 row tiles had 79 pairs, 75.4 on average; of
// 137 row tiles 42 and 36.9; of 20, one group for each of five XCDs, 3 and 0.8.  With the searches' ends, us: 5,000 x 768 93 -> 49, 24,576
// 326 -> 289, 35,001 542 -> 497, 50,001 946 -> 915.)
struct PairItems {
    long p, end;  // this workgroup's next place in the order; where its XCD's share ends
    int sb, tiles, group, at;  // the group of place p, and p's number in it
    __device__ __forceinline__ void init(int tiles_, int qb) {
        const long xcd = blockIdx.x & 7, total = (long)tiles_ * (tiles_ + 1) / 2;
        tiles = tiles_;
        sb = 32 / qb;
        p = total * xcd / 8 + ((blockIdx.x >> 3) & 31);
        end = total * (xcd + 1) / 8;
        find();
    }
    __device__ __forceinline__ void find() {  // (row r begins at r (r + 1) / 2, and so does a group that begins with it)
        int r = (int)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
        while ((long)r * (r + 1) / 2 > p) --r;
        while ((long)(r + 1) * (r + 2) / 2 <= p) ++r;
        group = __builtin_amdgcn_readfirstlane(r / sb);
        const long r0 = (long)group * sb;
        at = __builtin_amdgcn_readfirstlane((int)(p - r0 * (r0 + 1) / 2));
    }
    __device__ __forceinline__ int count() const { return p < end ? (int)((end - p + 31) / 32) : 0; }
    __device__ __forceinline__ void skip(int n) {
        p += 32L * n;
        find();
    }
    // next tile pair (column tile qt <= row tile ct) of this workgroup; false = none left
    __device__ __forceinline__ bool next(int &qt, int &ct) {
        if (p >= end) return false;
        int r0, rows, all;
        for (;;) {
            r0 = group * sb;
            rows = tiles - r0 < sb ? tiles - r0 : sb;
            all = rows * (r0 + 1);
            const int here = all + rows * (rows - 1) / 2;
            if (at < here) break;
            at -= here;
            ++group;
        }
        if (at < all) {
            qt = at / rows;
            ct = r0 + at - qt * rows;
        } else {
            int e = at - all, r = 1;
            for (; e >= r; ++r) e -= r;
            qt = r0 + 1 + e;
            ct = r0 + r;
        }
        p += 32;
        at += 32;
        return true;
    }
};
