// oz2h_kernels.hpp -- gfx950 kernels of the Ozaki-II pipeline (device code).
//
//   k_exp_*      stage 1: shared exponents e_i / f_j (Eq. 1)
//   k_residues   stage 2: integerization (Eq. 1) + centred residues per modulus,
//                balanced base-128 halves for two-limb moduli (VALU, fp64-exact sums)
//   k_resgemm    stage 3: INT8 MFMA residue GEMMs (LDS-staged tiles) with the
//                mod-m_l reduction and Karatsuba recombination fused in the epilogue
//   k_crt        stage 4+5: direct CRT, symmetric lift, rescale and one RNE rounding
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "oz2h_plan.hpp"

namespace oz2h {

// lambdas of kernels that must be inlined whatever their size (their captures live in registers)
#define OZ2H_INL __attribute__((always_inline))

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- stage 1

constexpr int kExpChunk = 1024;   // contraction entries per wave (contiguous rows)
constexpr int kExpRowsK = 16;     // contraction entries per thread (other layouts)

__global__ void k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Largest exponent of the nonzero entries of one contiguous stretch [k0, k1) of a row (base
// offset rb), over a wave: lane reads k0 + lane + 64 u.  Every load is issued before any is
// used: entries past k1 read entry k0 (always in range) and are ignored, and the exponent is
// read whatever the sign.  INT_MIN when the stretch has no nonzero entry.
__device__ __forceinline__ int exp_max_wave(const int8_t *__restrict__ sign, const int32_t *__restrict__ exps,
                                            const int32_t *__restrict__ koff, int64_t rb, int64_t k0,
                                            int64_t k1, int lane) {
    constexpr int U = kExpChunk / 64;
    int sg[U], ex[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t k = k0 + lane + 64 * u;
        const int64_t kk = k < k1 ? k : k0;
        sg[u] = k < k1 ? sign[rb + kk] : 0;
        ex[u] = exps[rb + kk] + (koff ? koff[kk] : 0);
    }
    int m = INT_MIN;
#pragma unroll
    for (int u = 0; u < U; ++u) m = sg[u] ? max(m, ex[u]) : m;
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
    return m;
}

// The same for one thread over kExpRowsK entries k0 .. of a row with entry stride cs.
__device__ __forceinline__ int exp_max_thread(const int8_t *__restrict__ sign, const int32_t *__restrict__ exps,
                                              const int32_t *__restrict__ koff, int64_t rb, int64_t cs,
                                              int64_t k0, int64_t count) {
    int sg[kExpRowsK], ex[kExpRowsK];
#pragma unroll
    for (int u = 0; u < kExpRowsK; ++u) {
        const int64_t k = k0 + u;
        const int64_t kk = k < count ? k : k0;
        sg[u] = k < count ? sign[rb + kk * cs] : 0;
        ex[u] = exps[rb + kk * cs] + (koff ? koff[kk] : 0);
    }
    int m = INT_MIN;
#pragma unroll
    for (int u = 0; u < kExpRowsK; ++u) m = sg[u] ? max(m, ex[u]) : m;
    return m;
}

// rows whose entries are contiguous along the contraction (cs == 1): one wave
// per (row, kExpChunk-entry chunk), lanes stride 1, partial maxima combined by atomicMax
// koff (nullable): a per-contraction-index exponent offset added before the max
// (the exponent folding of the backward products)
__global__ __launch_bounds__(256) void k_exp_kcontig(const int8_t *__restrict__ sign,
                                                     const int32_t *__restrict__ exps,
                                                     int64_t rows, int64_t count, int64_t rs,
                                                     const int32_t *__restrict__ koff,
                                                     int32_t *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int64_t k0 = (int64_t)blockIdx.y * kExpChunk;
    int m = exp_max_wave(sign, exps, koff, r * rs, k0, min(count, k0 + kExpChunk), lane);
    if (lane == 0 && m != INT_MIN) atomicMax(out + r, m);
}

// any other layout: one thread per row, kExpRowsK entries of the contraction per block
// row (loads unrolled, so that they are all in flight at once)
__global__ __launch_bounds__(256) void k_exp_generic(const int8_t *__restrict__ sign,
                                                     const int32_t *__restrict__ exps,
                                                     int64_t rows, int64_t count, int64_t rs,
                                                     int64_t cs, const int32_t *__restrict__ koff,
                                                     int32_t *__restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    const int m = exp_max_thread(sign, exps, koff, r * rs, cs, (int64_t)blockIdx.y * kExpRowsK, count);
    if (m != INT_MIN) atomicMax(out + r, m);
}

// all-zero rows get exponent 0
__global__ void k_exp_fix(int32_t *__restrict__ p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && p[i] == INT_MIN) p[i] = 0;
}

// One launch for both sides (and both parts of complex operands): a block of 1024 threads owns
// 2^lr rows over the whole contraction, 1024 >> lr threads per row, and writes their exponents
// (0 for all-zero rows), so that nothing is filled before or mended after.  Consecutive lanes
// take consecutive entries of the part's contiguous direction.
//
// What bounds it: launches and the latency of a few loads for small sides (16^3 19 to 7 us,
// 256^3 22 to 7, against fill, scan and fix per side), the reads of signs and exponents for
// large ones (8192^2 on both sides 223 to 147 us, 4.6 TB/s; 4096^2 70 to 49).
struct ExpPart {
    const int8_t *sign;
    const int32_t *exps;
    int64_t rs, cs;
};
struct ExpSide {
    ExpPart part[2];
    int64_t rows, nb;        // nb: blocks of this side
    const int32_t *koff;
    int32_t *out;
    int32_t lr, nparts;
};
struct ExpArgs {
    ExpSide side[2];
    int64_t count;
};
constexpr int kExpThreads = 1024;

__global__ __launch_bounds__(kExpThreads) void k_exponents(ExpArgs a) {
    __shared__ int32_t red[kExpThreads];
    constexpr int U = 8;
    const bool second = blockIdx.x >= a.side[0].nb;
    const ExpSide &s = a.side[second];
    const int tid = threadIdx.x, lr = s.lr, R = 1 << lr, S = kExpThreads >> lr;
    const int64_t r0 = ((int64_t)blockIdx.x - (second ? a.side[0].nb : 0)) << lr, count = a.count;
    if (tid < R) red[tid] = INT_MIN;
    __syncthreads();
    for (int q = 0; q < s.nparts; ++q) {
        const ExpPart p = s.part[q];
        const bool contig = p.cs == 1;
        const int rl = contig ? tid >> (10 - lr) : tid & (R - 1);
        const int sl = contig ? tid & (S - 1) : tid >> lr;
        const int64_t rb = min(r0 + rl, s.rows - 1) * p.rs;   // a dead row reads the last one
        int m = INT_MIN;
        for (int64_t k0 = sl; k0 < count; k0 += (int64_t)S * U) {
            int sg[U], ex[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {   // every load issued before any is used, as above
                const int64_t k = k0 + (int64_t)u * S;
                const int64_t kk = k < count ? k : k0;
                sg[u] = p.sign[rb + kk * p.cs];
                ex[u] = p.exps[rb + kk * p.cs] + (s.koff ? s.koff[kk] : 0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) m = sg[u] ? max(m, ex[u]) : m;   // a repeated entry changes nothing
        }
        if (contig && S >= 64) {   // one row per wave
            for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
            if ((tid & 63) == 0) atomicMax(red + rl, m);
        } else {
            atomicMax(red + rl, m);
        }
    }
    __syncthreads();
    if (tid < R && r0 + tid < s.rows) s.out[r0 + tid] = red[tid] == INT_MIN ? 0 : red[tid];
}

// ---------------------------------------------------------------- stage 2

// global-memory views of pointers (pointers read from a descriptor are generic;
// the casts let the compiler use global and scalar loads)
#define OZ2H_G(T) const __attribute__((address_space(1))) T
typedef __attribute__((address_space(1))) int8_t g_i8;
typedef __attribute__((address_space(1))) uint32_t g_u32;
typedef __attribute__((address_space(1))) uint16_t g_u16;
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) v4u g_v4u;

// a ModInfo record read through a global-memory pointer (field by field: the
// implicit copy constructor does not bind to an address-space-qualified object)
__device__ __forceinline__ ModInfo load_info(OZ2H_G(ModInfo) *p) {
    ModInfo r;
    r.m = p->m;
    r.g0 = p->g0;
    r.nprod = p->nprod;
    r.minv = p->minv;
    r.inv_m = p->inv_m;
    r.kc[0] = p->kc[0];
    r.kc[1] = p->kc[1];
    r.kc[2] = p->kc[2];
    r.pad = 0;
    return r;
}

// The (t+1)-bit integer a^ = RNE(mant * 2^sh) of one entry as nw 32-bit words
// col[w * st] (zero above the value); returns the sign after rounding (0 if a^ = 0).
// sh = t - p + exp - e <= t - p (Eq. 1); mant is p bits in 64-bit limbs (bits at or
// above p ignored).  One pass over the significand's 32-bit words: with sh = 32 q + r,
// r in [1, 32], word j lands in output word q + j as the funnel shift
// alignbit(m_j, m_{j-1}, 32 - r); for sh < 0 the same pass collects the round bit
// (position -sh - 1) and the sticky bits below it, and a round-up carries through the
// words.  A shift below -(32 nd + 2) drops every bit, the round bit included (a^ = 0).
// The significand is read through feed(limb), which calls limb(x) for each limb in turn from
// the lowest (limbs at and above nlimb may be anything).
template <class Feed>
__device__ __forceinline__ int build_words_from(Feed feed, int s, int64_t sh, int p, int nw, uint32_t *col,
                                                int st) {
    for (int w = 0; w < nw; ++w) col[w * st] = 0u;
    if (s == 0) return 0;
    const int nlimb = (p + 63) >> 6;
    const int nd = (p + 31) >> 5;
    const uint64_t topm = (p & 63) ? (1ull << (p & 63)) - 1ull : ~0ull;
    const int shc = (int)max(sh, (int64_t)-(32 * nd + 2));
    const int q = (shc - 1) >> 5;        // floor((sh - 1) / 32)
    const int sa = 32 * (q + 1) - shc;   // 32 - r, in [0, 31]
    const int rp = -shc - 1;             // round bit position (sh < 0)
    uint32_t prev = 0u, nz = 0u;
    bool rbit = false, sticky = false;
    auto word = [&](int j, uint32_t cur) {   // word j of the significand (0 above it)
        const int w = q + j;
        if (w >= 0 && w < nw) {
            const uint32_t v = __builtin_amdgcn_alignbit(cur, prev, sa);
            col[w * st] = v;
            nz |= v;
        }
        if (shc < 0) {
            const int b = rp - 32 * j;   // the round bit's position within word j
            if (b >= 32) {
                sticky |= cur != 0u;
            } else if (b >= 0) {
                rbit = (cur >> b) & 1u;
                sticky |= (cur & ((1u << b) - 1u)) != 0u;
            }
        }
        prev = cur;
    };
    int l = 0;
    feed([&](uint64_t x) {
        if (l >= nlimb) x = 0ull;
        if (l == nlimb - 1) x &= topm;
        word(2 * l, (uint32_t)x);
        word(2 * l + 1, (uint32_t)(x >> 32));
        ++l;
    });
    word(2 * l, 0u);   // one more word of zeros for the carry-out of the shift
    if (rbit && (sticky || (col[0] & 1u))) {   // round half to even: add one
        for (int w = 0; w < nw; ++w) {
            const uint32_t v = col[w * st] + 1u;
            col[w * st] = v;
            if (v) break;
        }
        nz = 1u;
    }
    return nz ? s : 0;
}

// The limbs from memory: a ring of two registers, loaded two limbs ahead with clamped
// unconditional loads, so that the loads of one entry overlap.
__device__ __forceinline__ int build_words(OZ2H_G(uint64_t) *__restrict__ sl, int s, int64_t sh,
                                           int p, int nw, uint32_t *col, int st) {
    const int nlimb = (p + 63) >> 6;
    return build_words_from(
        [&](auto limb) {
            auto ld = [&](int l) { return sl[min(l, nlimb - 1)]; };
            uint64_t r0 = ld(0), r1 = ld(1);
            for (int l = 0; l < nlimb; l += 2) {
                const uint64_t x0 = r0, x1 = r1;
                r0 = ld(l + 2);
                limb(x0);
                r1 = ld(l + 3);
                limb(x1);
            }
        },
        s, sh, p, nw, col, st);
}

// One operand side as the residue kernels read it: logical rows x count entries, entry (r, k)
// at r rs + k cs; planes of rpad x kpad bytes.
struct ResSide {
    const uint64_t *limbs;
    const int32_t *exps;
    const int8_t *signs;
    int64_t rs, cs, rows, count, kpad, plane_stride;
    const int32_t *erow;
    const int32_t *koff;   // nullable per-contraction exponent offsets (exponent folding)
    int8_t *planes;
};

// The plan's part of the entry kernel's arguments.
struct ResTab {
    const double *tab;          // [passes][nw32][res_pass_units]
    const ResUnitGroup *grp;    // [groups]
    int p, nl, t, nw32, groups;
};

// a wave-uniform plane pointer held in scalar registers, so that a store through it with a
// 32-bit lane offset takes the scalar-base form
__device__ __forceinline__ g_i8 *uniform_ptr(g_i8 *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (g_i8 *)(((uint64_t)hi << 32) | lo);
}

// Low bytes of four ints in one dword, byte i from b[i].
__device__ __forceinline__ uint32_t pack_bytes(int b0, int b1, int b2, int b3) {
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b1, (uint32_t)b0, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)b3, (uint32_t)b2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// 4 x 4 byte transpose within each quad of lanes: lane 4 a + q enters holding byte i of
// row q and leaves holding byte q of rows 0..3 (byte j from row j).  Two exchanges (with
// lane ^ 2, then lane ^ 1) of DPP quad permutes, each followed by a byte select whose
// selector depends on the lane's place in the quad (v_perm_b32: selector values 0-3 take
// the bytes of the second operand, 4-7 those of the first).
struct QuadSel {
    uint32_t a, b;
};
__device__ __forceinline__ QuadSel quad_sel(int lane) {
    const int q = lane & 3;
    return QuadSel{q < 2 ? 0x05040100u : 0x03020706u, (q & 1) ? 0x03070105u : 0x06020400u};
}
__device__ __forceinline__ uint32_t quad_transpose_bytes(uint32_t w, QuadSel sel) {
    const uint32_t p2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, false);
    w = __builtin_amdgcn_perm(p2, w, sel.a);
    const uint32_t p1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, false);
    return __builtin_amdgcn_perm(p1, w, sel.b);
}

// Waves of a residue block along k: two when the block has at least two, so that a block
// covers 128 consecutive entries of RB / 2 rows.  Blocks are dealt to the XCDs round-robin,
// so with one wave per row the two 64-byte halves of a plane line would be written from two
// different L2s.  Grids: (kpad / (64 KW)) x (rpad / (RB / KW)) blocks, launched as a 1-D grid
// with the k blocks fastest (no 65535 limit on the rows).
__host__ __device__ constexpr int res_waves_k(int rb) { return rb >= 2 ? 2 : 1; }
// lanes of one wave hand data over through LDS: keep the compiler from moving LDS
// accesses across this point (LDS itself serves a wave's instructions in order)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Residues of a^ (stage 2), integers of up to kResMaxWords words.  The words of an entry are
// dotted with centred 2^(32 w) mod M weights by exact fp64 FMAs (every partial sum an integer
// below 2^53).  M is one two-limb modulus, or the PRODUCT of two one-limb moduli: the sum is
// then reduced by either, so that a pair costs the multiply-adds of one modulus.
// Reduction: r = x - rint(x / m) m.  For the one-limb moduli |x| < 2^51 (integers of up to 16
// words; wider ones are first reduced by the pair's product), so x / m is at least 1 / (2 m)
// away from a half-integer and its rounding error below that: the quotient is exact, up to
// either tie of the even modulus 128, and |r| <= 127.  For a two-limb modulus it is at worst off
// by one, |r| <= (m + 3) / 2, whose balanced base-128 split r = r0 + 128 r1 has |r0|, |r1|,
// |r0 + r1| <= 127.  Any representative of a^ mod m within these bounds gives the same exact
// GEMM result mod m.  x is added to 1.5 2^52, so that r is the low word of the last FMA.
//
// A wave takes RW rows x 128 consecutive k (RW = EPT / 2).  Its entries' words are built with
// one lane per entry (so that the operand is read along its rows) into LDS, word-major; then
// each lane takes EPT consecutive k: one LDS read gives a word of all of them, and a residue's
// EPT bytes leave as one store, 128 bytes per row of a plane.  The weights and moduli are
// wave-uniform scalar loads; units go in groups of four of one kind.  NW > 0 (integers of
// exactly NW words): EPT = 4, the words stay in registers, as signed doubles, for every group.
// NW = 0 (wider ones): EPT = 2, which leaves LDS for three waves per SIMD at 23 words where 4
// would leave one; the words are read again for every four groups.
//
// What bounds it: up to 12 words the plane stores and operand reads (8192^3, p = 113: 8.4 GB,
// 1.8 ms at the rate of a copy) and VALU issue about as much, above that issue and LDS.
// Against one entry per lane and every modulus on its own, bytes exchanged between lanes:
// both sides 3.62 to 2.65 ms at 8192^3, p = 113; 1.95 to 1.42 ms at 4096^3, p = 256; 1.24 to
// 1.08 ms at 2048^3, p = 512.
constexpr int kResWaves = 4;   // waves per block
__host__ __device__ constexpr int res_ept(int nw) { return nw <= kResRegWords ? 4 : 2; }
__host__ __device__ constexpr int res_block_rows(int nw) { return kResWaves * res_ept(nw) / 2; }
__host__ __device__ constexpr size_t res_wave_lds(int nw) { return (size_t)64 * res_ept(nw) * 4 * (nw + 1); }

template <int NW>
__device__ __forceinline__ void residue_wave(const ResSide &a, const ResTab &tb, int64_t bx, int64_t by,
                                             uint32_t *words, int part = 0, int parts = 1) {
    constexpr int EPT = NW > 0 ? 4 : 2, NE = 64 * EPT;
    constexpr int NG = NW > 0 ? 1 : 4;   // groups per pass over the words
    typedef uint32_t vEu __attribute__((ext_vector_type(EPT)));
    typedef typename std::conditional<EPT == 4, uint32_t, uint16_t>::type bytes_t;
    typedef __attribute__((address_space(1))) bytes_t g_bytes;
    const int lane = threadIdx.x & 63;
    const int nw = NW > 0 ? NW : tb.nw32;
    const int64_t r0 = by, k0 = bx * 128;   // the wave's first row and k
    uint32_t *sgn = words + (size_t)nw * NE;   // sign bits of the entries
    g_i8 *planes = (g_i8 *)a.planes + r0 * a.kpad + k0;
    const uint32_t loff =
        EPT == 4 ? (uint32_t)((lane >> 5) * a.kpad + 4 * (lane & 31)) : (uint32_t)(2 * lane);
    // the tables are read-only for the launch: scalar loads whatever is stored in between
    typedef const __attribute__((address_space(4))) ResUnitGroup cgrp;
    typedef const __attribute__((address_space(4))) double cdouble;
    cgrp *grec = (cgrp *)tb.grp;
    if (r0 >= a.rows || k0 >= a.count) {   // padding only
        if (part) return;
        const int64_t G = grec[tb.groups - 1].g0 + grec[tb.groups - 1].nplanes;
        for (int64_t g = 0; g < G; ++g) *(g_bytes *)(planes + g * a.plane_stride + loff) = 0;
        return;
    }

    // the words of the wave's entries: pass e, lane -> row r0 + e / 2, k = k0 + 64 (e % 2) + lane
    OZ2H_G(int8_t) *gsigns = (OZ2H_G(int8_t) *)a.signs;
    OZ2H_G(int32_t) *gexps = (OZ2H_G(int32_t) *)a.exps;
    OZ2H_G(int32_t) *gerow = (OZ2H_G(int32_t) *)a.erow;
    OZ2H_G(int32_t) *gkoff = (OZ2H_G(int32_t) *)a.koff;
    OZ2H_G(uint64_t) *glimbs = (OZ2H_G(uint64_t) *)a.limbs;
    int s[EPT];
    int64_t sh[EPT], idx[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {   // an entry outside the operand reads entry (r0, k0), as 0
        const int64_t r = r0 + (e >> 1), k = k0 + 64 * (e & 1) + lane;
        const bool in = r < a.rows && k < a.count;
        const int64_t rr = in ? r : r0, kk = in ? k : k0;
        idx[e] = rr * a.rs + kk * a.cs;
        s[e] = in ? gsigns[idx[e]] : 0;
        sh[e] = (int64_t)tb.t - tb.p + gexps[idx[e]] + (a.koff ? gkoff[kk] : 0) - gerow[rr];
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int ent = 64 * e + lane;
        const int sg = build_words(glimbs + idx[e] * tb.nl, s[e], sh[e], tb.p, nw, words + ent, NE);
        sgn[ent] = sg < 0 ? 0x80000000u : 0u;
    }
    wave_lds_sync();

    // lane: entries EPT lane .. (EPT = 4: row lane / 32, k = 4 (lane % 32) ..; 2: k = 2 lane ..)
    const vEu *wrow = (const vEu *)words + lane;
    const vEu sb = *((const vEu *)sgn + lane);
    auto signed_word = [&](uint32_t w, uint32_t sbit) {
        const uint64_t d = __builtin_bit_cast(uint64_t, (double)w);
        return __builtin_bit_cast(double, d ^ ((uint64_t)sbit << 32));
    };
    double xw[NW > 0 ? NW : 1][EPT];
    if constexpr (NW > 0) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const vEu q = wrow[w * 64];
#pragma unroll
            for (int i = 0; i < EPT; ++i) xw[w][i] = signed_word(q[i], sb[i]);
        }
    }
    constexpr double kMagic = 6755399441055744.0;   // 1.5 2^52
    auto low = [](double v) { return (uint32_t)__builtin_bit_cast(uint64_t, v); };
    cdouble *gtab = (cdouble *)tb.tab;
    const int passes = (tb.groups + NG - 1) / NG;   // this part's share of them
    const int gend = min((part + 1) * passes / parts * NG, tb.groups);
    for (int g = part * passes / parts * NG; g < gend; g += NG) {
        double acc[NG][kResUnits][EPT];
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int u = 0; u < kResUnits; ++u)
#pragma unroll
                for (int i = 0; i < EPT; ++i) acc[n][u][i] = 0.0;
        cdouble *cg = gtab + (size_t)g * nw * kResUnits;   // [nw][NG groups][units]
        if constexpr (NW > 0) {
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int u = 0; u < kResUnits; ++u) {
                    const double c = cg[w * kResUnits + u];
#pragma unroll
                    for (int i = 0; i < EPT; ++i) acc[0][u][i] = fma(xw[w][i], c, acc[0][u][i]);
                }
        } else {
            // the next word and its weights load while one is multiplied
            constexpr int NU = NG * kResUnits;
            struct Word {
                vEu q;
                double c[NU];
            };
            auto load = [&](int w, Word &o) OZ2H_INL {
                o.q = wrow[w * 64];
#pragma unroll
                for (int u = 0; u < NU; ++u) o.c[u] = cg[w * NU + u];
            };
            auto mult = [&](const Word &o) OZ2H_INL {
                double x[EPT];
#pragma unroll
                for (int i = 0; i < EPT; ++i) x[i] = signed_word(o.q[i], sb[i]);
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int i = 0; i < EPT; ++i)
                        acc[u / kResUnits][u % kResUnits][i] = fma(x[i], o.c[u], acc[u / kResUnits][u % kResUnits][i]);
            };
            Word wa, wb;
            load(0, wa);
            for (int w = 0; w < nw; w += 2) {
                load(min(w + 1, nw - 1), wb);
                __builtin_amdgcn_sched_barrier(0);
                mult(wa);
                __builtin_amdgcn_sched_barrier(0);
                if (w + 1 >= nw) break;
                load(min(w + 2, nw - 1), wa);
                __builtin_amdgcn_sched_barrier(0);
                mult(wb);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            if (n && g + n >= gend) break;
            cgrp *R = grec + g + n;
            g_i8 *pb = uniform_ptr(planes + (int64_t)R->g0 * a.plane_stride);
            const int np = R->nplanes;
            // a full group without guards, so that its constants load at once
            auto pairs = [&](auto full_) OZ2H_INL {
                constexpr bool FULL = decltype(full_)::value;
#pragma unroll
                for (int u = 0; u < kResUnits; ++u) {
                    double y[EPT];
#pragma unroll
                    for (int i = 0; i < EPT; ++i) {
                        double &x = acc[n][u][i];
                        if (NW == 0 && nw > kResExactWords) x = fma(-rint(x * R->inv2[u]), R->m2[u], x);
                        y[i] = x + kMagic;
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if (!FULL && 2 * u + j >= np) break;
                        uint32_t b[EPT];
#pragma unroll
                        for (int i = 0; i < EPT; ++i)
                            b[i] = low(fma(-rint(acc[n][u][i] * R->inv[2 * u + j]), R->md[2 * u + j], y[i]));
                        uint32_t v = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u);
                        if constexpr (EPT == 4)
                            v = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u), v, 0x05040100u);
                        *(g_bytes *)(pb + (int64_t)(2 * u + j) * a.plane_stride + loff) = (bytes_t)v;
                    }
                }
            };
            auto twos = [&](auto full_) OZ2H_INL {
                constexpr bool FULL = decltype(full_)::value;
                typedef short s2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int u = 0; u < kResUnits; ++u) {
                    if (!FULL && 3 * u >= np) break;
                    uint32_t r[EPT];
#pragma unroll
                    for (int i = 0; i < EPT; ++i) {
                        const double x = acc[n][u][i];
                        r[i] = low(fma(-rint(x * R->inv[u]), R->md[u], x + kMagic));
                    }
                    // the residues as packed pairs: r1 = (r + 64) >> 7, r0 = r - 128 r1
                    uint32_t q0[EPT / 2], q1[EPT / 2], qs[EPT / 2];
#pragma unroll
                    for (int h = 0; h < EPT / 2; ++h) {
                        const s2 v = __builtin_bit_cast(
                            s2, (uint32_t)__builtin_amdgcn_perm(r[2 * h + 1], r[2 * h], 0x05040100u));
                        const s2 v1 = (v + (short)64) >> (short)7;
                        q1[h] = __builtin_bit_cast(uint32_t, v1);
                        q0[h] = __builtin_bit_cast(uint32_t, (s2)(v - v1 * (short)128));
                        qs[h] = __builtin_bit_cast(uint32_t, (s2)(v - v1 * (short)127));
                    }
                    auto put = [&](int pl, const uint32_t (&q)[EPT / 2]) OZ2H_INL {
                        *(g_bytes *)(pb + (int64_t)(3 * u + pl) * a.plane_stride + loff) =
                            (bytes_t)__builtin_amdgcn_perm(q[EPT / 2 - 1], q[0], 0x06040200u);
                    };
                    put(0, q0);
                    put(1, q1);
                    put(2, qs);
                }
            };
            if (!R->two) {
                if (np == 2 * kResUnits) pairs(std::true_type{});
                else pairs(std::false_type{});
            } else {
                if (np == 3 * kResUnits) twos(std::true_type{});
                else twos(std::false_type{});
            }
        }
    }
}

// both sides of a product (or one: blocks0 = all) in one launch: the first blocks0 blocks are
// side 0's; a side is a 1-D grid of kpad / 128 (fastest) x rpad / res_block_rows blocks
struct ResArgs {
    ResSide side[2];
    int64_t blocks0;
    int parts;   // grid.y: blocks sharing the unit groups
    ResTab tab;
};

template <int NW>
__global__ __launch_bounds__(64 * kResWaves) void k_residues(ResArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t words[];
    const int sd = (int64_t)blockIdx.x >= a.blocks0;
    const ResSide sa = a.side[sd];
    const int64_t lb = (int64_t)blockIdx.x - (sd ? a.blocks0 : 0), nbx = sa.kpad / 128;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    residue_wave<NW>(sa, a.tab, lb % nbx, (lb / nbx * kResWaves + wave) * (res_ept(NW ? NW : kResMaxWords) / 2),
                     words + wave * (res_wave_lds(NW ? NW : a.tab.nw32) / 4), blockIdx.y, a.parts);
}

// Residues of a^ on the vector ALUs with row broadcasts (stage 2, no MFMA; wide integers).  The
// residue of a^ = sum_w x_w 2^(32 w) modulo m is sum_w x_w c_w with the centred
// c_w = 2^(32 w) mod M (an exact fp64 integer, |sum| < 2^53), reduced by m.  M is one two-limb
// modulus, or the product of two one-limb moduli, whose sum is first reduced by M and then by
// either: a unit.  The x_w are signed base-2^32 digits of the signed integer (|x_w| <= 2^31:
// half the bound of magnitude words, and no sign left to apply).  Each lane of a 16-lane row
// owns one unit of a group of 16 and keeps that unit's weights c_w in registers; the row works
// on one entry at a time, its digits spread over the row's lanes (lane j holds digit 16 c + j
// of chunk c), and each multiply-add takes the digit from lane w % 16 by a DPP row broadcast
// (v_fmac_f64 with row_newbcast): no constant loads in the inner loop.
// A block of four waves covers 128 consecutive k of one row of the operand side:
//   phase 1: threads 0-127 build their entry's digits into LDS (digit w of entry e at
//            words[w * kResRowS + e]: a row of 16 lanes reading 16 digits of one entry, and
//            the four rows four entries 16 apart, hit 64 different banks);
//   phase 2: wave v takes the groups v, v + 4, .. for all 128 entries; row q of the wave takes
//            entries 64 s + 16 q + i (i < 16, s = 0, 1), eight at a time;
//   stores:  a lane holds its unit's residues of 16 consecutive entries, packs their bytes
//            in registers and stores 16 bytes per plane.
constexpr int kResRowS = 129;   // LDS word stride of the row-broadcast residue kernel

// v_fmac_f64 with its first source broadcast from lane LANE of each row of 16 lanes (DPP
// row_newbcast).  The DPP source must not be written by a VALU instruction in the two
// instructions before; the words come from asm blocks that end with s_nop 1.
template <int LANE>
__device__ __forceinline__ void fmac_rowbcast(double &acc, double x, double c) {
    asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(x), "v"(c), "n"(LANE));
}

// four signed digits as doubles, followed by the two wait states a DPP read of them needs
__device__ __forceinline__ void cvt4_digits(uint32_t a, uint32_t b, uint32_t c, uint32_t d, double &x0,
                                           double &x1, double &x2, double &x3) {
    asm volatile(
        "v_cvt_f64_i32 %0, %4\n\t"
        "v_cvt_f64_i32 %1, %5\n\t"
        "v_cvt_f64_i32 %2, %6\n\t"
        "v_cvt_f64_i32 %3, %7\n\t"
        "s_nop 1"
        : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3)
        : "v"(a), "v"(b), "v"(c), "v"(d));
}

// an NC-word chunk (NC = 16, 4 or 2) into NE accumulators: lane j's weights c[i] are word
// w0 + i's; word w0 + i of entry u comes from lane i of the row.  For each broadcast lane the
// NE entries follow each other, so that consecutive multiply-adds are independent.
template <int NC, int NE, int I = 0>
__device__ __forceinline__ void row_fmas(double (&a)[NE], const double (&x)[NE], const double *c) {
    if constexpr (I < NC) {
#pragma unroll
        for (int u = 0; u < NE; ++u) fmac_rowbcast<I>(a[u], x[u], c[I]);
        row_fmas<NC, NE, I + 1>(a, x, c);
    }
}

struct ResRowArgs {
    ResSide d;
    int p, nl, t, nw, nwp, groups;   // digits; padded to a multiple of 4 (the weights' stride)
    const double *tab;               // [16 groups][nwp]
    const ResRowUnit *units;         // [16 groups]
};

__host__ __device__ constexpr size_t res_row_lds(int nwp) { return (size_t)nwp * kResRowS * 4; }

// WIDE: more than kResRowDigits digits.  Units are single moduli, and a two-limb modulus's sum is
// reduced before it meets 1.5 2^52 too.
template <bool WIDE>
__device__ __forceinline__ void residues_row_block(const ResRowArgs &a, int64_t bx, int64_t r, uint32_t *words) {
    const ResSide &d = a.d;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t k0 = bx * 128;
    int8_t *prow = d.planes + r * d.kpad + k0;   // the block's segment of plane 0
    if (r >= d.rows || k0 >= d.count) {          // padding only
        const ResRowUnit *last = a.units + 16 * a.groups - 1;
        const int64_t G = (int64_t)last->g0 + last->nplanes;
        for (int64_t g = wv; g < G; g += 4) *(g_u16 *)((g_i8 *)prow + g * d.plane_stride + 2 * lane) = 0;
        return;
    }

    // phase 1: the signed digits of the block's 128 entries
    if (tid < 128) {
        OZ2H_G(int8_t) *gsigns = (OZ2H_G(int8_t) *)d.signs;
        OZ2H_G(int32_t) *gexps = (OZ2H_G(int32_t) *)d.exps;
        const int64_t k = k0 + tid;
        int s = 0;
        int64_t sh = 0, idx = 0;
        if (k < d.count) {
            idx = r * d.rs + k * d.cs;
            s = gsigns[idx];
            sh = (int64_t)a.t - a.p + gexps[idx] + (d.koff ? d.koff[k] : 0) - d.erow[r];
        }
        uint32_t *col = words + tid;
        s = build_words((OZ2H_G(uint64_t) *)d.limbs + idx * a.nl, s, sh, a.p, a.nwp, col, kResRowS);
        // sum of +-w 2^(32 i) in digits of [-2^31, 2^31): the top digit has room (|a^| < 2^(32 nw - 1))
        int64_t cy = 0;
        for (int w = 0; w < a.nw; ++w) {
            const int64_t m = (int64_t)col[w * kResRowS];
            const int64_t v = (s < 0 ? -m : m) + cy;
            const int32_t x = (int32_t)v;
            col[w * kResRowS] = (uint32_t)x;
            cy = (v - x) >> 32;
        }
    }
    __syncthreads();

    // phase 2
    const int j = lane & 15, q = lane >> 4;
    // digits past the full 16-digit chunks: chunks of 4, and a last chunk of 2 when at most two
    // digits remain (the digits past nw are zero in LDS)
    const int nfull = a.nw >> 4, nrem = a.nw & 15;
    const int ntail = (nrem & 3) == 3 ? (nrem >> 2) + 1 : nrem >> 2;
    const bool tail2 = (nrem & 3) == 1 || (nrem & 3) == 2;
    constexpr double kMagic = 6755399441055744.0;   // 1.5 2^52: an integer added to it is its low word
    auto low = [](double v) { return (uint32_t)__builtin_bit_cast(uint64_t, v); };
    for (int g = wv; g < a.groups; g += 4) {
        const ResRowUnit *gu = a.units + 16 * g + j;
        const double *crow = a.tab + ((size_t)g * 16 + j) * a.nwp;
        double acc[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[i] = 0.0;
        // one NC-digit chunk (NC = 16, 4 or 2) from digit w0 with the weights c
        auto chunk = [&](auto nc_, int w0, const double *c) {
            constexpr int NC = decltype(nc_)::value;
            const uint32_t *wr = words + (size_t)(w0 + (j & (NC - 1))) * kResRowS + 16 * q;
#pragma unroll
            for (int eb = 0; eb < 4; ++eb) {
                const int e = 64 * (eb / 2) + 8 * (eb % 2);   // + 16 q, entries e .. e + 7
                double x[8], a8[8];
                cvt4_digits(wr[e], wr[e + 1], wr[e + 2], wr[e + 3], x[0], x[1], x[2], x[3]);
                cvt4_digits(wr[e + 4], wr[e + 5], wr[e + 6], wr[e + 7], x[4], x[5], x[6], x[7]);
#pragma unroll
                for (int u = 0; u < 8; ++u) a8[u] = acc[8 * eb + u];
                row_fmas<NC, 8>(a8, x, c);
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[8 * eb + u] = a8[u];
            }
        };
        for (int c = 0; c < nfull; ++c) {
            double cc[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) cc[i] = crow[16 * c + i];
            chunk(std::integral_constant<int, 16>{}, 16 * c, cc);
        }
        for (int c = 0; c < ntail; ++c) {
            double c4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) c4[i] = crow[16 * nfull + 4 * c + i];
            chunk(std::integral_constant<int, 4>{}, 16 * nfull + 4 * c, c4);
        }
        if (tail2) {
            double c2[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) c2[i] = crow[16 * nfull + 4 * ntail + i];
            chunk(std::integral_constant<int, 2>{}, 16 * nfull + 4 * ntail, c2);
        }

        // per entry half: lane (q, j) holds its unit's sums for the 16 consecutive entries
        // 64 hs + 16 q + i; the residues' bytes are packed in registers and leave as one 16-byte
        // store per plane (the four rows of a wave write 64 contiguous bytes of each plane).
        // (Split and packed two residues to a register: 14 instead of 21 instructions per
        // modulus and entry with the sign and the conversion the digits and kMagic save.)
        const ResRowUnit ru = *gu;
        typedef short s2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int hs = 0; hs < 2; ++hs) {
            g_i8 *dst = (g_i8 *)prow + (int64_t)ru.g0 * d.plane_stride + 64 * hs + 16 * q;
            if (ru.nplanes == 3) {
                v4u b0, b1, b2;
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    uint32_t q0[2], q1[2], qs[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint32_t rr[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            double x = acc[16 * hs + 4 * i4 + 2 * h + u];
                            if constexpr (WIDE) x = fma(-rint(x * ru.inv2), ru.m2, x);
                            rr[u] = low(fma(-rint(x * ru.inv[0]), ru.md[0], x + kMagic));
                        }
                        // r = r0 + 128 r1, balanced
                        const s2 v = __builtin_bit_cast(s2, (uint32_t)__builtin_amdgcn_perm(rr[1], rr[0], 0x05040100u));
                        const s2 v1 = (v + (short)64) >> (short)7;
                        q1[h] = __builtin_bit_cast(uint32_t, v1);
                        q0[h] = __builtin_bit_cast(uint32_t, (s2)(v - v1 * (short)128));
                        qs[h] = __builtin_bit_cast(uint32_t, (s2)(v - v1 * (short)127));
                    }
                    b0[i4] = __builtin_amdgcn_perm(q0[1], q0[0], 0x06040200u);
                    b1[i4] = __builtin_amdgcn_perm(q1[1], q1[0], 0x06040200u);
                    b2[i4] = __builtin_amdgcn_perm(qs[1], qs[0], 0x06040200u);
                }
                *(g_v4u *)dst = b0;
                *(g_v4u *)(dst + d.plane_stride) = b1;
                *(g_v4u *)(dst + 2 * d.plane_stride) = b2;
            } else if (ru.nplanes) {
                v4u b0, b1;
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    uint32_t r0[4], r1[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        double x = acc[16 * hs + 4 * i4 + u];
                        x = fma(-rint(x * ru.inv2), ru.m2, x);
                        const double y = x + kMagic;
                        r0[u] = low(fma(-rint(x * ru.inv[0]), ru.md[0], y));
                        r1[u] = low(fma(-rint(x * ru.inv[1]), ru.md[1], y));
                    }
                    b0[i4] = pack_bytes((int)r0[0], (int)r0[1], (int)r0[2], (int)r0[3]);
                    b1[i4] = pack_bytes((int)r1[0], (int)r1[1], (int)r1[2], (int)r1[3]);
                }
                *(g_v4u *)dst = b0;
                if (ru.nplanes == 2) *(g_v4u *)(dst + d.plane_stride) = b1;
            }
        }
    }
}

template <bool WIDE>
__global__ __launch_bounds__(256) void k_residues_row(ResRowArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t smem_rr[];
    const int64_t nbx = a.d.kpad / 128;
    residues_row_block<WIDE>(a, (int64_t)blockIdx.x % nbx, (int64_t)blockIdx.x / nbx, smem_rr);
}

// Residues of a^ on the matrix cores (stage 2).  For every modulus the residue of an
// entry is a dot product of its magnitude's bytes with the weights 256^j mod m, so a
// wave computes a (weight rows) x (64 entries) int8 product with
// v_mfma_i32_32x32x32_i8 and then reduces each exact int32 sum x to the centred
// x - rint(x/m) m (exact in fp64, |x| < 2^31): no per-modulus pass over the words.
// The weight rows, the correction bytes that carry the sign, and the row layout are
// described with build_residue_mma_tables.  One wave per (row r, 64 consecutive k):
//   phase 0: lane k writes its entry's bytes to LDS (entry-major, stride es words),
//            complemented if negative, already offset by -128 (xor 0x80);
//   phase 1: per block of 32 weight rows, rnq k-steps of two MFMAs (entries 0-31 and
//            32-63) with A = weight fragments (global), B = entry bytes (read from LDS
//            into registers once);
//   phase 2: the 32 x 64 sums go through an LDS scratch (entry-major, 144-byte rows) so
//            that lane k reduces its own entry for every modulus of the block with
//            wave-uniform modulus data, and stores 64 contiguous bytes per plane.
// Bank layout: es = 4 (2 i + 1) words and the 144-byte scratch rows put the 16 lanes a
// 16-byte LDS access serves per cycle on 16 different bank groups.
struct ResMmaArgs {
    const uint64_t *limbs;
    const int32_t *exps;
    const int8_t *signs;
    int64_t rs, cs, rows, count, kpad, plane_stride;
    const int32_t *erow;
    const int32_t *koff;
    int p, nl, t, nw32, nq, nrb, es;
    const int8_t *wfrag;
    const ResRowBlock *rblk;
    int8_t *planes;
};

static_assert(offsetof(ResRowBlock, md) == 256 && offsetof(ResRowBlock, g0) == 512 &&
                  offsetof(ResRowBlock, n1) == 640 && offsetof(ResRowBlock, p0) == 644 &&
                  offsetof(ResRowBlock, n2) == 648,
              "byte offsets the MFMA residue kernel reads the row block record at");
constexpr int kResScratchRow = 144;   // bytes per entry in the sums scratch (32 rows + 16)
constexpr int kResMmaMaxQ = 16;       // k-steps of the widest integer (t < 3400 bits: 14)
constexpr int kResMmaPfQ = 8;         // up to this many k-steps the next weights are prefetched

__host__ __device__ constexpr int res_mma_es(int nq) { return 8 * nq + 4; }
// LDS per wave: the entry bytes, later reused by the sums scratch
__host__ __device__ constexpr int res_mma_wave_lds(int nq) {
    return 64 * res_mma_es(nq) * 4 > 64 * kResScratchRow ? 64 * res_mma_es(nq) * 4 : 64 * kResScratchRow;
}


// At most NQ k-steps: entry and weight fragments live in registers (up to kResMmaPfQ
// k-steps the weights of the next block of rows are prefetched while one block is
// reduced), and the sums scratch reuses the entry bytes' LDS.
template <int RB, int NQ>
__device__ __forceinline__ void residue_block_mma_r(
    const uint64_t *__restrict__ limbs, const int32_t *__restrict__ exps,
    const int8_t *__restrict__ signs, const int32_t *__restrict__ erow,
    const int32_t *__restrict__ koff, const int8_t *__restrict__ wfrag,
    const ResRowBlock *__restrict__ rblk, int8_t *__restrict__ planes, int64_t rs, int64_t cs,
    int64_t rows, int64_t count, int64_t kpad, int64_t plane_stride, int p, int nl, int t,
    int nw32, int nq, int nrb, int64_t bx, int64_t by, uint32_t *smem) {
    static_assert(NQ >= 1 && NQ <= kResMmaMaxQ, "k-steps");
    constexpr bool PF = NQ <= kResMmaPfQ;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int es = res_mma_es(nq);
    uint32_t *ent = smem + (size_t)wv * (res_mma_wave_lds(nq) / 4);
    uint8_t *scr = (uint8_t *)ent;
    constexpr int KW = res_waves_k(RB);   // waves side by side along k, as in residue_block_r
    const int64_t k = (bx * KW + wv % KW) * 64 + lane;
    const int64_t r = by * (RB / KW) + wv / KW;

    typedef const __attribute__((address_space(1))) v4i gv4i;
    gv4i *wf = (gv4i *)wfrag + lane;
    v4i wa[NQ], wn[PF ? NQ : 1];
#pragma unroll
    for (int q = 0; q < NQ; ++q)   // the first block's weights load while the entry is built
        if (q < nq) wa[q] = wf[q * 64];

    // phase 0: this lane's entry, bytes offset by -128
    OZ2H_G(int8_t) *gsigns = (OZ2H_G(int8_t) *)signs;
    OZ2H_G(int32_t) *gexps = (OZ2H_G(int32_t) *)exps;
    OZ2H_G(int32_t) *gerow = (OZ2H_G(int32_t) *)erow;
    OZ2H_G(int32_t) *gkoff = (OZ2H_G(int32_t) *)koff;
    int s = 0;
    int64_t sh = 0, idx = 0;
    if (r < rows && k < count) {
        idx = r * rs + k * cs;
        s = gsigns[idx];
        sh = (int64_t)t - p + gexps[idx] + (koff ? gkoff[k] : 0) - gerow[r];
    }
    uint32_t *ew = ent + lane * es;
    s = build_words((OZ2H_G(uint64_t) *)limbs + idx * nl, s, sh, p, nw32, ew, 1);
    const uint32_t cmask = s < 0 ? 0xFFFFFFFFu : 0u;
    for (int w = 0; w < nw32; ++w) ew[w] = (s == 0 ? 0u : ew[w] ^ cmask) ^ 0x80808080u;
    ew[nw32] = (s < 0 ? 0x100u : 0u) ^ 0x80808080u;   // correction bytes nb, nb + 1
    for (int w = nw32 + 1; w < 8 * nq; ++w) ew[w] = 0x80808080u;

    // read-only for the whole launch: the constant address space keeps these wave-uniform
    // reads on the scalar unit across the LDS hand-over fences
    typedef const __attribute__((address_space(4))) ResRowBlock crb_t;
    crb_t *grb = (crb_t *)rblk;
    const int h = lane >> 5, c = lane & 31;
    const v4i *b0p = (const v4i *)(ent + c * es + 4 * h);          // entries 0-31
    const v4i *b1p = (const v4i *)(ent + (32 + c) * es + 4 * h);   // entries 32-63
    v4i bf0[NQ], bf1[NQ];
    wave_lds_sync();   // entry bytes written
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (q < nq) {
            bf0[q] = b0p[2 * q];
            bf1[q] = b1p[2 * q];
        }
    // the block's region of every plane (uniform 64-bit base) and a 32-bit lane offset in it
    const int64_t r0b = by * (RB / KW), k0b = bx * KW * 64;
    planes += r0b * kpad + k0b;
    const uint32_t loff = (uint32_t)((r - r0b) * kpad + (k - k0b));
    // stores: after a quad byte transpose, lane 4 a + q writes entries 4 a .. 4 a + 3 of
    // plane q of a group of four (a dword at the quad's first entry)
    const QuadSel qsel = quad_sel(lane);
    const int64_t qoff = (int64_t)(lane & 3) * plane_stride + (int64_t)(loff & ~3u);
    const uint32_t *xrow = (const uint32_t *)(scr + lane * kResScratchRow);
    for (int rb = 0; rb < nrb; ++rb) {
        wave_lds_sync();   // entry bytes read; the previous block's sums read
        v16i acc0 = v16i{}, acc1 = v16i{};
        if constexpr (PF) {
            if (rb + 1 < nrb) {
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (q < nq) wn[q] = wf[((size_t)(rb + 1) * nq + q) * 64];
            }
        } else if (rb > 0) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (q < nq) wa[q] = wf[((size_t)rb * nq + q) * 64];
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (q < nq) {
                acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa[q], bf0[q], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa[q], bf1[q], acc1, 0, 0, 0);
            }
        // sums element e: row 8 (e / 4) + 4 h + e % 4, entry c (acc0) or 32 + c (acc1)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            const int ro = (8 * a4 + 4 * h) * 4;
            *(v4i *)(scr + c * kResScratchRow + ro) =
                v4i{acc0[4 * a4], acc0[4 * a4 + 1], acc0[4 * a4 + 2], acc0[4 * a4 + 3]};
            *(v4i *)(scr + (32 + c) * kResScratchRow + ro) =
                v4i{acc1[4 * a4], acc1[4 * a4 + 1], acc1[4 * a4 + 2], acc1[4 * a4 + 3]};
        }
        wave_lds_sync();   // sums written
        // lane k reduces its own entry: four rows per 16-byte read (two-limb pairs start
        // on a multiple of 4), the modulus data of four rows per scalar load, every row of
        // the four computed (rows past the moduli hold zeros).  The sums and modulus data of
        // the next four rows load while four rows are reduced (scheduling fences keep those
        // loads behind the first use of the current ones, whose wait covers every scalar and
        // LDS load in flight); reads up to row 35 stay inside the block record and the
        // scratch row.  Only the last group of a kind guards its stores.
        typedef double d4 __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(4))) d4 cd4;
        typedef const __attribute__((address_space(4))) char cch;
        typedef const __attribute__((address_space(4))) uint32_t cu32;
        cch *B = (cch *)(grb + rb);
        const int n1 = (int)((cu32 *)(B + 640))[0], p0 = (int)((cu32 *)(B + 640))[1],
                  n2 = (int)((cu32 *)(B + 640))[2];
        // row data of rows i .. i + 3: fl(1/m) at byte 8 i, m at 256 + 8 i
        v4i xn;
        d4 imn, mmn;
        auto fetch = [&](uint32_t i) {
            xn = *(const v4i *)(xrow + i);
            imn = *(cd4 *)(B + 8u * i);
            mmn = *(cd4 *)(B + (256u + 8u * i));
        };
        // first planes (byte 512 + 4 i): the one-limb rows of a block own consecutive planes
        // from that of row 0, and its two-limb pairs consecutive triples from that of row p0
        const uint32_t g1 = *(cu32 *)(B + 512);
        int i4 = 0;
        fetch(0);
        auto group1 = [&](auto full_) {   // one-limb rows i4 .. i4 + 3
            constexpr bool FULL = decltype(full_)::value;
            const d4 mm = mmn;
            double x[4], q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = (double)xn[e];
                q[e] = rint(x[e] * imn[e]);
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(i4 + 4);
            __builtin_amdgcn_sched_barrier(0);
            g_i8 *pb = uniform_ptr((g_i8 *)planes + (int64_t)(g1 + i4) * plane_stride);
            int ri[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) ri[e] = (int)fma(-q[e], mm[e], x[e]);
            const uint32_t w = quad_transpose_bytes(pack_bytes(ri[0], ri[1], ri[2], ri[3]), qsel);
            if (FULL || (lane & 3) < n1 - i4) *(g_u32 *)(pb + qoff) = w;
        };
        for (; i4 + 4 <= n1; i4 += 4) group1(std::true_type{});
        if (i4 < n1) group1(std::false_type{});
        if (n2 > 0) {
            const uint32_t g2 = *(cu32 *)(B + (512u + 4u * (uint32_t)p0));
            // only the first row of a pair holds modulus data: load those two of four rows
            // (loading all four would leave half of the destination registers dead, free for
            // reuse while the load is still in flight)
            typedef const __attribute__((address_space(4))) double cdbl;
            double im0, im2, mm0, mm2;
            auto fetch2 = [&](uint32_t i) {
                xn = *(const v4i *)(xrow + i);
                im0 = *(cdbl *)(B + 8u * i);
                im2 = *(cdbl *)(B + (16u + 8u * i));
                mm0 = *(cdbl *)(B + (256u + 8u * i));
                mm2 = *(cdbl *)(B + (272u + 8u * i));
            };
            int j2 = 0;
            fetch2((uint32_t)p0);
            auto group2 = [&](auto full_) {   // two-limb pairs j2, j2 + 1 (rows p0 + 2 j2 ..)
                constexpr bool FULL = decltype(full_)::value;
                const uint32_t i4 = (uint32_t)(p0 + 2 * j2);
                const double mm[2] = {mm0, mm2};
                double x[2], q[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) x[e] = (double)(xn[2 * e] + 128 * xn[2 * e + 1]);
                q[0] = rint(x[0] * im0);
                q[1] = rint(x[1] * im2);
                __builtin_amdgcn_sched_barrier(0);
                fetch2(i4 + 4);
                __builtin_amdgcn_sched_barrier(0);
                g_i8 *pb = uniform_ptr((g_i8 *)planes + (int64_t)(g2 + 3u * (uint32_t)j2) * plane_stride);
                int r0[2], r1[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int ri = (int)fma(-q[e], mm[e], x[e]);
                    r0[e] = ((ri + 64) & 127) - 64;   // balanced base-128 split
                    r1[e] = (ri - r0[e]) >> 7;
                }
                // planes 0-5 of the two pairs: (r0, r1, r0 + r1) of the first, then the second
                const uint32_t wa = quad_transpose_bytes(pack_bytes(r0[0], r1[0], r0[0] + r1[0], r0[1]), qsel);
                const uint32_t wb = quad_transpose_bytes(pack_bytes(r1[1], r0[1] + r1[1], 0, 0), qsel);
                const int nv = FULL ? 6 : 3 * (n2 - j2);   // planes to write
                if ((lane & 3) < nv) *(g_u32 *)(pb + qoff) = wa;
                if ((lane & 3) + 4 < nv) *(g_u32 *)(pb + 4 * plane_stride + qoff) = wb;
            };
            for (; j2 + 2 <= n2; j2 += 2) group2(std::true_type{});
            if (j2 < n2) group2(std::false_type{});
        }
        if constexpr (PF) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) wa[q] = wn[q];
        }
    }
}

template <int RB, int NQ>
__global__ __launch_bounds__(64 * RB) void k_residues_mma(ResMmaArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t smem_res[];
    const int64_t nbx = a.kpad / (64 * res_waves_k(RB));
    residue_block_mma_r<RB, NQ>(a.limbs, a.exps, a.signs, a.erow, a.koff, a.wfrag, a.rblk, a.planes,
                            a.rs, a.cs, a.rows, a.count, a.kpad, a.plane_stride, a.p, a.nl, a.t,
                            a.nw32, a.nq, a.nrb, (int64_t)blockIdx.x % nbx, (int64_t)blockIdx.x / nbx,
                            smem_res);
}

// ---------------------------------------------------------------- stage 3

constexpr int GBK = 128;   // k padding granule of the residue planes = the GEMM k-tile
constexpr int TBK = 128;   // k-tile of the GEMM kernel: one 128-byte LDS row per output row

// centred residue x - rint(x/m) m of an exact fp64 integer x (|x| < 2^52)
__device__ __forceinline__ int32_t centred_mod(double x, double md, double inv_m) {
    return (int32_t)fma(-rint(x * inv_m), md, x);
}

// chunk swizzle of LDS tile row r: distinct over the rows of equal parity among any 16
// aligned rows, and over any 8 aligned rows
__device__ __forceinline__ int lds_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// One (64 WR) x (64 WC) output tile of one modulus per block; WR x WC waves, each a 64 x 64
// sub-tile of v_mfma_i32_16x16x64_i8 blocks (exact int32 sums, K * 127^2 < 2^31).  B's fragment
// is the first operand and its rows are taken as 8 a + 4 y + b, so a lane ends with runs of eight
// consecutive columns of one row: a wave's 16-byte stores fill 64-byte pieces.
// k-tiles of 64 bytes move global -> LDS by direct loads (no register staging) into ST stages:
// two, one tile ahead of the multiplies, or four, three ahead, for blocks alone on their compute
// unit.  Planes are padded to 128 bytes, so every product has an even number of k-tiles and
// starts in stage 0 (with four stages and an odd number of pairs, two steps of the last round
// only load).  The products of a modulus and their k-tiles are
// plain loops with no branch around the accumulators (a branch at a product's end inside the
// k-loop moved all of them between the register files every k-tile).
//
// What bounds it: latency and the work per product (fold, stores).  Three blocks per compute
// unit (146 registers, 32 KiB of LDS each) cover one block's loads, folds and stores with the
// others' products.  Against one block per unit with 128-byte k-tiles, three stages and 2-byte
// stores: 3328 x 3072 x 384, p = 256 1060 to 812 us; 2048 x 2048 x 128, p = 512 540 to 361;
// 1024 x 1024 x 384, p = 256 112 to 82; 517 x 389 x 1003, p = 113 41 to 38.  Four blocks (128
// registers, spills in the fold) 1111 us on the first, a 256 x 128 tile of eight waves 1061.
//
// An LDS row is four 16-byte chunks, chunk c of row r stored at c ^ swz(r): the 16 rows a
// ds_read_b128 serves per LDS cycle (64 banks of 4 bytes, four 64-byte rows per bank period) then
// hit 16 different 16-byte bank groups.  The lane order of a direct load fixes the LDS side (16
// bytes per lane, consecutive), so the swizzle is applied to the global addresses.
// The output is v_l = c_l (P/m_l)^-1 mod m_l as a centred int16: the reduction
// mod m_l and the first step of the direct CRT are fused here.
// A two-limb modulus runs its three Karatsuba products (planes r0, r1, r0 + r1:
// P0, P2, Ps) as one continuous k-loop into the SAME accumulators: we want
// c0 P0 + c2 P2 + cs Ps mod m with the weighted coefficients
// (c0, c2, cs) = (-127, 16256, 128) (P/m)^-1, and fold in place at the end of
// each product with w0 = c2^-1 c0, w1 = cs^-1 c2, w2 = cs (m is prime, so the
// inverses exist): acc = P0 w0 -> + P2 -> * w1 -> + Ps -> * w2.  Between the
// products |acc| <= m/2, so acc + K 127^2 < 2^31 stays exact.
// Blocks run the two-limb moduli first (they are three times longer).
// RAW = true: plain int32 output of a single plane (the stage call's longer products).
struct GemmArgs {
    const int8_t *A, *B;
    int64_t kpad, a_ps, b_ps;
    const ModInfo *mi;
    int16_t *V;
    int64_t v_ps, ldv;
    int32_t *Craw;
};

// LDS stage S of the direct-load GEMM: one object per stage, so that the compiler can
// tell a read of one stage from a load still filling another
constexpr int SBK = 64;   // k-tile of the four-wave kernels
template <int WR, int WC, int S>
__device__ __forceinline__ int8_t *gemm_stage() {
    __shared__ __attribute__((aligned(1024))) int8_t st[64 * (WR + WC) * SBK];
    return st;
}

// s_waitcnt immediate: wait until at most `vm` vector-memory loads are outstanding
// (LDS/scalar and export counters left at their maximum)
constexpr int vmcnt_imm(int vm) { return (vm & 0xF) | (((vm >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8); }

// Arguments of the products that combine into an existing output (complex products):
// V2 is a second output set with the same strides as V.
struct GemmArgsZ : GemmArgs {
    int16_t *V2;
};

// output combination of a complex product's residue GEMMs (x = this product's weighted
// residue, all values centred mod m_l):
//   ZSTORE  V = x;   ZADD  V = V + x;   ZSUB  V = V - x;
//   ZGAUSS  (t1, t2) = (V, V2);  V = t1 - t2;  V2 = x - t1 - t2   (3M's last product)
enum GemmMode { ZSTORE = 0, ZADD = 1, ZSUB = 2, ZGAUSS = 3 };

// 16 bytes per lane from base + voff + soff (of the wave-uniform range base .. base + bytes) into
// the wave's 1 KiB of LDS at dst
__device__ __forceinline__ void load_lds(const int8_t *base, int bytes, int8_t *dst, uint32_t voff, int soff) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, bytes, 0x00020000),
                                             (__attribute__((address_space(3))) void *)dst, 16, voff, soff, 0, 0);
#endif
}

// waves per SIMD the register allocation aims at
constexpr int gemm_waves(int nw, int st) { return nw == 4 && st == 2 ? 3 : 2; }

// one output tile (mt, nt) of modulus l
template <int WR, int WC, int ST, bool RAW, int MODE = ZSTORE, class Args = GemmArgs>
__device__ __forceinline__ void gemm_tile(const Args &args, int64_t mt, int64_t nt, int l) {
    constexpr int NW = WR * WC, BM = 64 * WR, BN = 64 * WC;
    constexpr int FM = 4, FN = 2;                           // 16-row fragments, groups of 32 columns
    constexpr int NLA = 4 / WC, NL = NLA + 4 / WR;          // direct loads per wave per k-tile
    const int8_t *__restrict__ A = args.A;
    const int8_t *__restrict__ B = args.B;
    const int64_t kpad = args.kpad, a_ps = args.a_ps, b_ps = args.b_ps, ldv = args.ldv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int64_t m0 = mt * BM, n0 = nt * BN;

    uint32_t g0 = 0, nprod = 1;
    double md = 1.0, inv_m = 1.0;
    int32_t kc[3] = {1, 1, 1};
    if (!RAW) {
        const ModInfo info = args.mi[l];
        g0 = info.g0;
        nprod = info.nprod;
        md = (double)info.m;
        inv_m = info.inv_m;
        kc[0] = info.kc[0];
        kc[1] = info.kc[1];
        kc[2] = info.kc[2];
    }
    // kpad is a multiple of 128: an even number of k-tiles

    // load i of wave w fills 16 rows of A or B, lane -> row lane / 4, chunk lane % 4
    auto swz_a = [](int r) OZ2H_INL { return (r >> 2) & 3; };
    auto swz_b = [](int r) OZ2H_INL { return (r >> 3) & 3; };
    uint32_t goff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int R = 16 * (NW * (i < NLA ? i : i - NLA) + wave) + (lane >> 2);
        goff[i] = (uint32_t)(R * kpad) + (((lane & 3) ^ (i < NLA ? swz_a(R) : swz_b(R))) << 4);
    }
    const int8_t *la = A + m0 * kpad + (int64_t)g0 * a_ps, *lb = B + n0 * kpad + (int64_t)g0 * b_ps;
    auto issue = [&](auto s_, int ko) OZ2H_INL {
        int8_t *dst = gemm_stage<WR, WC, decltype(s_)::value>();
#pragma unroll
        for (int i = 0; i < NL; ++i)
            load_lds(i < NLA ? la : lb, (i < NLA ? BM : BN) * (int)kpad, dst + (NW * i + wave) * 1024, goff[i], ko);
    };

    v4i acc[FN][FM][2];
#pragma unroll
    for (int c = 0; c < FN; ++c)
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[c][x][y] = v4i{};

    const int fr = lane & 15, frb = (fr >> 2) * 8 + (fr & 3);
    const int fo = (wr * 64 + fr) * SBK + (((lane >> 4) ^ swz_a(fr)) << 4);
    const int go = (wc * 64 + frb) * SBK + (((lane >> 4) ^ swz_b(frb)) << 4);   // y = 1: 4 rows on
    // (acc w) mod m, centred, as in the 256 x 256 kernel
    auto fold = [&](int prod) OZ2H_INL {
        constexpr double kMagic = 6755399441055744.0;
        const double w = (double)(prod == 0 ? kc[0] : prod == 1 ? kc[1] : kc[2]), wi = w * inv_m;
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int x = 0; x < FM; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double v = (double)acc[c][x][y][e];
                        acc[c][x][y][e] =
                            (int32_t)(uint32_t)__builtin_bit_cast(uint64_t, fma(-rint(v * wi), md, fma(v, w, kMagic)));
                    }
                    __builtin_amdgcn_sched_barrier(0);   // four at a time: few registers
                }
    };
    // one k-tile from stage S; the one ST - 1 ahead (k offset ko) goes into the stage before S,
    // which every wave finished reading before the barrier
    constexpr int FS = ST == 4 ? 2 : 1;   // fragment sets
    v4i fa[FS][FM], fb[FS][FN][2];
    auto fetch = [&](auto s_) OZ2H_INL {
        constexpr int S = decltype(s_)::value, F = S % FS;
        const int8_t *cA = gemm_stage<WR, WC, S>(), *cB = cA + BM * SBK;
#pragma unroll
        for (int x = 0; x < FM; ++x) fa[F][x] = *(const v4i *)(cA + x * 16 * SBK + fo);
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int y = 0; y < 2; ++y) fb[F][c][y] = *(const v4i *)(cB + (c * 32 + 4 * y) * SBK + go);
    };
    // two stages: wait for this k-tile and read it.  Four: wait for the next one and read that
    // (the fragments of this one are there), so that a block alone on its unit multiplies while
    // it reads
    auto step = [&](auto s_, int ko) OZ2H_INL {
        constexpr int S = decltype(s_)::value;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(ST == 4 ? NL : 0));   // own loads of that tile landed
        __builtin_amdgcn_s_barrier();                              // everyone's did
        issue(std::integral_constant<int, (S + ST - 1) % ST>{}, ko);
        __builtin_amdgcn_sched_barrier(0);
        fetch(std::integral_constant<int, ST == 4 ? (S + 1) % ST : S>{});
    };
    auto multiply = [&](auto s_) OZ2H_INL {
        constexpr int F = decltype(s_)::value % FS;
#pragma unroll
        for (int c = 0; c < FN; ++c)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < FM; ++x)
                    acc[c][x][y] =
                        __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[F][c][y], fa[F][x], acc[c][x][y], 0, 0, 0);
        if constexpr (ST == 4) {   // one read ahead of every two products
#pragma unroll
            for (int u = 0; u < FM + 2 * FN; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2 % ST>;
    using I3 = std::integral_constant<int, 3 % ST>;
    const int kp = (int)kpad;
    issue(I0{}, 0);
    if constexpr (ST == 4) {
        issue(I1{}, SBK);
        issue(I2{}, min(2 * SBK, kp - SBK));
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * NL));
        __builtin_amdgcn_s_barrier();
        fetch(I0{});
    }
    int prod = 0;
    do {
        int ko = 0;
        do {
            // the next ST k-tiles: of this product, or the next one's first (after the last
            // product any, not read); an offset past the end reads the last k-tile instead
            const int nko = ko + ST * SBK;
            const bool wrap = nko >= kp, more = wrap && prod + 1 < (int)nprod;
            const int n0 = wrap ? 0 : nko;
            if constexpr (ST == 2) {
                step(I0{}, ko + SBK);
                multiply(I0{});
                la += more ? a_ps : 0;
                lb += more ? b_ps : 0;
                step(I1{}, n0);
                multiply(I1{});
            } else {
                const bool full = nko <= kp;   // else two of the four k-tiles are none
                step(I0{}, min(ko + 3 * SBK, kp - SBK));
                multiply(I0{});
                la += more ? a_ps : 0;
                lb += more ? b_ps : 0;
                step(I1{}, n0);
                multiply(I1{});
                step(I2{}, n0 + SBK);
                if (full) multiply(I2{});
                step(I3{}, min(n0 + 2 * SBK, kp - SBK));
                if (full) multiply(I3{});
            }
            ko = nko;
        } while (ko < kp);
        if (!RAW) fold(prod);
    } while (++prod < (int)nprod);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no load still writing LDS past the block's end

    // a lane's runs: row m0 + .. + 16 x + lane % 16, columns n0 + .. + 32 c + 8 (lane / 16) ..
    const int64_t lane_off = (m0 + wr * 64 + fr) * ldv + n0 + wc * 64 + (lane >> 4) * 8;
    if (RAW) {
        int32_t *base = args.Craw + lane_off;
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int c = 0; c < FN; ++c)
#pragma unroll
                for (int y = 0; y < 2; ++y) *(v4i *)(base + (int64_t)(x * 16) * ldv + c * 32 + 4 * y) = acc[c][x][y];
        return;
    }
    auto pack = [](const int32_t (&t)[8]) OZ2H_INL {
        v4i o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = (int)__builtin_amdgcn_perm((uint32_t)t[2 * i + 1], (uint32_t)t[2 * i], 0x05040100u);
        return o;
    };
    int16_t *base = args.V + (int64_t)l * args.v_ps + lane_off;
#pragma unroll
    for (int x = 0; x < FM; ++x) {
        // complex products: every old value of a row group is loaded before its first store, so
        // the group waits once (stores count against the same counter as loads)
        v4i p1[FN], p2[FN];
        if constexpr (MODE != ZSTORE) {
#pragma unroll
            for (int c = 0; c < FN; ++c) {
                int16_t *dst = base + (int64_t)(x * 16) * ldv + c * 32;
                p1[c] = *(const v4i *)dst;
                if constexpr (MODE == ZGAUSS) p2[c] = *(const v4i *)(dst + (args.V2 - args.V));
            }
        }
#pragma unroll
        for (int c = 0; c < FN; ++c) {
            int16_t *dst = base + (int64_t)(x * 16) * ldv + c * 32;
            int32_t r[8];
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int e = 0; e < 4; ++e) r[4 * y + e] = acc[c][x][y][e];
            if constexpr (MODE != ZSTORE) {
                int32_t r2[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int32_t t1 = (int16_t)((uint32_t)p1[c][i / 2] >> (16 * (i % 2)));
                    if constexpr (MODE == ZADD) r[i] = centred_mod((double)(t1 + r[i]), md, inv_m);
                    if constexpr (MODE == ZSUB) r[i] = centred_mod((double)(t1 - r[i]), md, inv_m);
                    if constexpr (MODE == ZGAUSS) {
                        const int32_t t2 = (int16_t)((uint32_t)p2[c][i / 2] >> (16 * (i % 2)));
                        r2[i] = centred_mod((double)(r[i] - t1 - t2), md, inv_m);
                        r[i] = centred_mod((double)(t1 - t2), md, inv_m);
                    }
                }
                if constexpr (MODE == ZGAUSS) *(v4i *)(dst + (args.V2 - args.V)) = pack(r2);
            }
            *(v4i *)dst = pack(r);
        }
    }
}

// XCD-aware block order of the plain launch.  Blocks are dealt to the 8 XCDs round-robin
// (block b runs on XCD b % 8, as its (b / 8)-th block there), and each XCD has its own L2.
// With `on`, XCD x covers one rectangle of h x w tiles (rectangle row x / rx, column x % rx)
// of every modulus, moduli in launch order: all XCDs still share each modulus's work
// evenly, but an XCD reads h tile rows of A and w tile columns of B instead of all of A.
struct XcdMap {
    uint32_t on, rx, h, w;   // h * w tiles per XCD and modulus
};

// plain launch: two-limb moduli (listed last) first; grid (N tiles, M tiles, moduli), or
// with an XCD map a 1-D grid of the same blocks
template <int WR, int WC, int ST, bool RAW>
__global__ __launch_bounds__(64 * WR * WC, gemm_waves(WR * WC, ST)) void k_resgemm(GemmArgs args, int L, XcdMap xm) {
    uint32_t mt = blockIdx.y, nt = blockIdx.x, zi = blockIdx.z;
    if (xm.on) {
        const uint32_t b = blockIdx.x, x = b & 7u, s = b >> 3, t8 = xm.h * xm.w;
        zi = s / t8;
        const uint32_t u = s - zi * t8;
        mt = (x / xm.rx) * xm.h + u / xm.w;
        nt = (x % xm.rx) * xm.w + u % xm.w;
    }
    const int l = RAW ? 0 : L - 1 - (int)zi;
    gemm_tile<WR, WC, ST, RAW>(args, mt, nt, l);
}

// Plain int32 product C = A B^T of one plane (the stage call), (2 WM) x (2 WN) tiles of four waves
// in 2 x 2, each WM x WN of v_mfma_i32_32x32x32_i8 blocks.  k-tiles of 128 bytes move global ->
// LDS by direct loads into three stages, two tiles ahead of the multiplies; chunk c of LDS row r
// is stored at c ^ lds_swz(r), applied to the global addresses.
//
// What bounds it: one block per compute unit, so the k-loop itself, without a fold or reduction
// that other blocks could cover: half the barriers per byte of k_resgemm's 64-byte k-tiles
// (k_resgemm / this one, 128 x 128: 4096^3 94 / 88 us, 2048^3 16.3 / 14.6, 2048 x 2048 x 512
// 10.0 / 8.9; 256 x 128: 8192^3 590 / 570, 2048 x 2048 x 512 10.8 / 10.2).
template <int WM, int WN, int S>
__device__ __forceinline__ int8_t *i8_stage() {
    __shared__ __attribute__((aligned(1024))) int8_t st[(2 * WM + 2 * WN) * TBK];
    return st;
}

template <int WM, int WN>
__global__ __launch_bounds__(256) void k_i8gemm(const int8_t *__restrict__ A, const int8_t *__restrict__ B,
                                                int64_t K, int32_t *__restrict__ C, int64_t ldc, XcdMap xm) {
    constexpr int BM = 2 * WM, BN = 2 * WN, FM = WM / 32, FN = WN / 32;
    constexpr int NLA = BM / 32, NL = (BM + BN) / 32;   // direct loads per wave per k-tile
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    uint32_t mt = blockIdx.y, nt = blockIdx.x;
    if (xm.on) {
        const uint32_t x = blockIdx.x & 7u, u = blockIdx.x >> 3;
        mt = (x / xm.rx) * xm.h + u / xm.w;
        nt = (x % xm.rx) * xm.w + u % xm.w;
    }
    const int64_t m0 = (int64_t)mt * BM, n0 = (int64_t)nt * BN;
    const int nk = (int)(K / TBK);

    uint32_t goff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int R = 32 * i + 8 * wave + (lane >> 3);
        goff[i] = (uint32_t)((i < NLA ? R : R - BM) * K) + (((lane & 7) ^ lds_swz(R)) << 4);
    }
    const int8_t *Ab = A + m0 * K, *Bb = B + n0 * K;
    // the next k-tile; near the end the last one again, so that the number of loads in flight
    // behind a tile is always the same
    int lk = 0;
    auto issue = [&](auto s_) OZ2H_INL {
        int8_t *dst = i8_stage<WM, WN, decltype(s_)::value>();
        const int8_t *a = Ab + (int64_t)lk * TBK, *b = Bb + (int64_t)lk * TBK;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            __builtin_amdgcn_global_load_lds((const void *)((i < NLA ? a : b) + goff[i]),
                                             (__attribute__((address_space(3))) void *)(dst + (4 * i + wave) * 1024),
                                             16, 0, 0);
        lk = min(lk + 1, nk - 1);
    };

    v16i acc[FM][FN];
#pragma unroll
    for (int x = 0; x < FM; ++x)
#pragma unroll
        for (int y = 0; y < FN; ++y) acc[x][y] = v16i{};
    const int frow = lane & 31;
    v4i fa[2][FM], fb[2][FN];
    auto fetch = [&](int set, int ks, const int8_t *cA, const int8_t *cB) OZ2H_INL {
        const int fo = frow * TBK + (((2 * ks + (lane >> 5)) ^ lds_swz(frow)) << 4);
#pragma unroll
        for (int x = 0; x < FM; ++x) fa[set][x] = *(const v4i *)(cA + (wr * WM + x * 32) * TBK + fo);
#pragma unroll
        for (int y = 0; y < FN; ++y) fb[set][y] = *(const v4i *)(cB + (wc * WN + y * 32) * TBK + fo);
    };
    // one k-tile from stage S; the one two ahead goes into the stage before S, which every wave
    // finished reading before the barrier
    auto body = [&](auto s_) OZ2H_INL {
        constexpr int S = decltype(s_)::value;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(NL));   // own loads of this tile landed
        __builtin_amdgcn_s_barrier();                // everyone's did
        issue(std::integral_constant<int, (S + 2) % 3>{});
        const int8_t *cA = i8_stage<WM, WN, S>(), *cB = cA + BM * TBK;
        fetch(0, 0, cA, cB);
        auto kstep = [&](auto k_) OZ2H_INL {
            constexpr int ks = decltype(k_)::value;
            if constexpr (ks + 1 < 4) fetch((ks + 1) & 1, ks + 1, cA, cB);
#pragma unroll
            for (int x = 0; x < FM; ++x)
#pragma unroll
                for (int y = 0; y < FN; ++y)
                    acc[x][y] =
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks & 1][x], fb[ks & 1][y], acc[x][y], 0, 0, 0);
            if constexpr (ks + 1 < 4) __builtin_amdgcn_sched_group_barrier(0x100, FM + FN, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, FM * FN, 0);
        };
        kstep(std::integral_constant<int, 0>{});
        kstep(std::integral_constant<int, 1>{});
        kstep(std::integral_constant<int, 2>{});
        kstep(std::integral_constant<int, 3>{});
    };
    issue(std::integral_constant<int, 0>{});
    issue(std::integral_constant<int, 1>{});
    int t = 0;
    for (; t + 3 <= nk; t += 3) {
        body(std::integral_constant<int, 0>{});
        body(std::integral_constant<int, 1>{});
        body(std::integral_constant<int, 2>{});
    }
    if (t < nk) body(std::integral_constant<int, 0>{});
    if (t + 1 < nk) body(std::integral_constant<int, 1>{});
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no load still writing LDS past the block's end

    int32_t *base = C + (m0 + wr * WM + 4 * (lane >> 5)) * ldc + n0 + wc * WN + (lane & 31);
#pragma unroll
    for (int x = 0; x < FM; ++x)
#pragma unroll
        for (int y = 0; y < FN; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                base[(int64_t)(x * 32 + 8 * (e >> 2) + (e & 3)) * ldc + y * 32] = acc[x][y][e];
}

// one residue GEMM of a complex product (the 3M / 4M schemes): the plain launch's block
// order and tiles, the output combined into V (and V2) by MODE
template <int WR, int WC, int ST, int MODE>
__global__ __launch_bounds__(64 * WR * WC, gemm_waves(WR * WC, ST)) void k_resgemm_z(GemmArgsZ args, int L, XcdMap xm) {
    uint32_t mt = blockIdx.y, nt = blockIdx.x, zi = blockIdx.z;
    if (xm.on) {
        const uint32_t b = blockIdx.x, x = b & 7u, s = b >> 3, t8 = xm.h * xm.w;
        zi = s / t8;
        const uint32_t u = s - zi * t8;
        mt = (x / xm.rx) * xm.h + u / xm.w;
        nt = (x % xm.rx) * xm.w + u % xm.w;
    }
    gemm_tile<WR, WC, ST, false, MODE, GemmArgsZ>(args, mt, nt, L - 1 - (int)zi);
}

// ---- 256 x 256 tiles

// LDS of the 256 x 256 kernel: two stages of four 16 KiB parts (128 rows of one 128-byte
// k-tile), one object per part so that the compiler can tell a read of one part from a load
// still filling another
template <int S, int P>
__device__ __forceinline__ int8_t *gemm8_part() {
    __shared__ __attribute__((aligned(1024))) int8_t st[128 * TBK];
    return st;
}

// chunk swizzle of a B part: the 16 rows of a fragment are 8 a + 4 y + b (a, b < 4; y fixed)
__device__ __forceinline__ int lds_swz_b(int r) { return ((r >> 1) & 1) | (((r >> 3) & 3) << 1); }

// s_waitcnt immediate: at most `vm` vector-memory operations outstanding, no LDS operation
constexpr int vmlgkm_imm(int vm) { return (vm & 0xF) | (((vm >> 4) & 3) << 14) | (0x7 << 4); }

// Arguments of the 256 x 256 kernel: GemmArgsZ's fields plus the moduli split (one-limb moduli
// 0 .. L1 - 1 own planes 0 .. L1 - 1, two-limb ones three planes each after them) and the
// work list: tiles tm x tn of each modulus, dealt by XCD rectangle when xm.on.
struct Gemm8Args {
    GemmArgsZ g;
    int L, L1, tm, tn;
    XcdMap xm;
};

// Residue GEMM with 256 x 256 tiles: eight waves, two per SIMD, each 128 x 64 of the tile
// (wave (wr, wc): rows 64 wr .. of both 128-row halves of A, columns 64 wc .. in two 32-column
// groups of B), as 16 x 16 x 64 int8 products (one lane: one output row, four consecutive
// columns of B's fragment).
//
// The k-loop alternates two phases per 128-byte k-tile T:
//   phase 0: read A0(T), B1(T) from LDS;        multiply A0 by B0, B1
//   phase 1: read A1(T), B0(T + 1) from LDS;    multiply A1 by B1, B0
// (B0(T + 1) is read one phase early, which makes every phase 12 LDS reads and 32 products.)
// The waves of a SIMD run half a phase apart: while one reads, the other multiplies; a barrier
// ends each half phase.  A part's LDS slot is free once both wave groups have read it, so its
// next load goes out a phase later, after that phase's LDS reads (before them the LDS reads
// wait behind the loads' issue: 2.70 against 2.91 POP/s raw at 8192^3), and is waited for two
// phases after that, just before the barrier in front of its first reader.
//
// What bounds it: the power limit.  On operands of zeros the loop runs at 4.34 POP/s (88 % of
// the 4.95 of a loop of products alone), on random ones at 2.91, where products alone reach
// 4.05 (3.35 with 32 x 32 x 32 products, whose accumulators move twice as often).
//
// A block walks its share of the (modulus, tile) list as one stream of k-tiles: the loads run
// two k-tiles ahead across products, tiles and moduli, so nothing drains between tiles.  At
// the end of a product the two accumulator halves are folded (or reduced and stored) in the
// read halves of the next two phases, beside the other group's multiplies.
template <int MODE>
__global__ __launch_bounds__(512, 2) void k_resgemm8(Gemm8Args) {
    // The arguments are read where they are used, mostly between products, through a pointer
    // the compiler cannot see behind: kept in registers they and what follows from them would
    // spill (the k-loop holds 230 of 256 vector registers).
    typedef const __attribute__((address_space(4))) Gemm8Args cargs;
    auto kargs = []() OZ2H_INL {
        cargs *p = (cargs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return p;
    };
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3;
    const int kpad = (int)kargs()->g.kpad;
    const int nk = kpad / TBK;

    // item: tile u of modulus L - 1 - zi; a block's items go on by its XCD's (or the whole)
    // number of blocks.  All of it is uniform and kept in scalar registers.
    struct Item {
        uint32_t zi, u;
    };
    auto uni = [](uint32_t v) OZ2H_INL { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    auto unip = [&](const int8_t *p) OZ2H_INL {
        const uint64_t v = (uint64_t)p;
        return (const int8_t *)(((uint64_t)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v));
    };
    auto step = [&](Item it, uint32_t by) OZ2H_INL {
        cargs *ka = kargs();
        const uint32_t t8 = ka->xm.on ? ka->xm.h * ka->xm.w : (uint32_t)(ka->tm * ka->tn);
        const uint32_t u = it.u + by, q = uni(u / t8);
        return Item{uni(it.zi + q), uni(u - q * t8)};
    };
    auto next = [&](Item it) OZ2H_INL { return step(it, kargs()->xm.on ? gridDim.x >> 3 : gridDim.x); };
    auto tile_of = [&](Item it, int &mt, int &nt) OZ2H_INL {
        cargs *ka = kargs();
        const uint32_t on = ka->xm.on, x8 = blockIdx.x & 7u, cols = on ? ka->xm.w : (uint32_t)ka->tn;
        const uint32_t r = uni(it.u / cols), c = it.u - r * cols, q = uni(x8 / ka->xm.rx);
        mt = (int)uni(on ? q * ka->xm.h + r : r);
        nt = (int)uni(on ? (x8 - q * ka->xm.rx) * ka->xm.w + c : c);
    };
    Item item = step(Item{0, 0}, kargs()->xm.on ? blockIdx.x >> 3 : blockIdx.x);
    if (item.zi >= (uint32_t)kargs()->L) return;   // no work: the whole block leaves

    // loads: load i of wave w fills LDS rows 64 i + 8 w .. + 7 of a part (lane -> row lane / 8,
    // physical chunk lane % 8); row R of part Bh is column 64 (R / 32) + 32 h + R % 32
    uint32_t va[2], vb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int R = 64 * i + 8 * wave + (lane >> 3);
        va[i] = (uint32_t)(R * kpad) + (((lane & 7) ^ lds_swz(R)) << 4);
        vb[i] = (uint32_t)(((R >> 5) * 64 + (R & 31)) * kpad) + (((lane & 7) ^ lds_swz_b(R)) << 4);
    }
    // load cursor: the k-tile loaded next (two ahead of the multiplies); the A rows and k
    // offset of the one before it
    struct Cursor {
        Item it;
        const int8_t *a, *b;   // the product's tile rows and columns in its planes
        int prods, ko;         // products left in the item (this one included), k offset
    };
    auto open = [&](Item it) OZ2H_INL {
        cargs *ka = kargs();
        const int l = ka->L - 1 - (int)it.zi, l1 = ka->L1;
        const int g0 = l < l1 ? l : l1 + 3 * (l - l1);
        int mt, nt;
        tile_of(it, mt, nt);
        return Cursor{it, unip(ka->g.A + g0 * ka->g.a_ps + (int64_t)mt * 256 * kpad),
                      unip(ka->g.B + g0 * ka->g.b_ps + (int64_t)nt * 256 * kpad), l < l1 ? 1 : 3, 0};
    };
    Cursor cur = open(item);
    const int8_t *pa = cur.a;
    int pko = 0;
    auto advance = [&]() OZ2H_INL {   // at the end of the list the last k-tile repeats
        pa = cur.a;
        pko = cur.ko;
        if (cur.ko + TBK < kpad) {
            cur.ko += TBK;
        } else if (cur.prods > 1) {
            cargs *ka = kargs();
            --cur.prods;
            cur.ko = 0;
            cur.a = unip(cur.a + ka->g.a_ps);
            cur.b = unip(cur.b + ka->g.b_ps);
        } else {
            const Item n = next(cur.it);
            if (n.zi < (uint32_t)kargs()->L) cur = open(n);
        }
    };
    // parts: 0 A0, 1 B0, 2 B1, 3 A1 of the tile rows or columns at p, k offset ko
    auto issue = [&](auto s_, auto p_, const int8_t *p, int ko) OZ2H_INL {
        constexpr int S = decltype(s_)::value, P = decltype(p_)::value;
        int8_t *dst = gemm8_part<S, P>();
        const auto rs = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 256 * kpad, 0x00020000);
        const int so = ko + (P == 3 ? 128 * kpad : P == 2 ? 32 * kpad : 0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void *)(dst + (8 * i + wave) * 1024), 16,
                P == 0 || P == 3 ? va[i] : vb[i], so, 0, 0);
    };

    v4i acc[2][2][4][2];   // [A half][B group][16-row block][fragment y]
    auto clear = [&](v4i (&h)[2][4][2]) OZ2H_INL {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) h[c][x][y] = v4i{};
    };
    clear(acc[0]);
    clear(acc[1]);

    v4i fa[4][2], fb0[2][2], fb1[2][2], fb2[2][2];
    const int fr = lane & 15, frb = (fr >> 2) * 8 + (fr & 3);
    int foa[2], fob[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        foa[ks] = (wr * 64 + fr) * TBK + (((4 * ks + (lane >> 4)) ^ lds_swz(fr)) << 4);
#pragma unroll
        for (int y = 0; y < 2; ++y)
            fob[y][ks] = (wc * 32 + frb + 4 * y) * TBK + (((4 * ks + (lane >> 4)) ^ lds_swz_b(frb + 4 * y)) << 4);
    }
    auto read_a = [&](const int8_t *p) OZ2H_INL {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int x = 0; x < 4; ++x) fa[x][ks] = *(const v4i *)(p + x * 16 * TBK + foa[ks]);
    };
    auto read_b = [&](const int8_t *p, v4i (&f)[2][2]) OZ2H_INL {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int y = 0; y < 2; ++y) f[y][ks] = *(const v4i *)(p + fob[y][ks]);
    };
    auto mult = [&](v4i (&c)[4][2], v4i (&f)[2][2]) OZ2H_INL {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    c[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[y][ks], fa[x][ks], c[x][y], 0, 0, 0);
    };
    auto fence = [&]() OZ2H_INL {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto barrier = [&]() OZ2H_INL {
        fence();
        __builtin_amdgcn_s_barrier();
        fence();
    };

    // the product being multiplied
    auto products = [&](Item it) OZ2H_INL { return kargs()->L - 1 - (int)it.zi < kargs()->L1 ? 1 : 3; };
    int prod = 0, nprod = products(item);

    // (acc w) mod m, centred: x w is exact (x < 2^31, w < 2^13) and x (w / m) off by less than
    // 2^-20, which is inside 1 / (2 m), the least distance of the quotient from a half-integer
    // for odd m (for m = 128 it is exact); added to 1.5 2^52 the residue is in the low word
    constexpr double kMagic = 6755399441055744.0;
    // the end of a product for one accumulator half (rows 128 H ..): folded in place, or after
    // the last product reduced, stored as 16-byte runs of eight columns and cleared
    auto finish = [&](auto h_) OZ2H_INL {
        constexpr int H = decltype(h_)::value;
        v4i (&h)[2][4][2] = acc[H];
        cargs *ka = kargs();
        const int l = ka->L - 1 - (int)item.zi;
        typedef const __attribute__((address_space(4))) ModInfo cinfo;
        cinfo *mi = (cinfo *)ka->g.mi + l;
        const double md = (double)mi->m, inv_m = mi->inv_m;
        const double w = (double)mi->kc[prod], wi = w * inv_m;
        auto residue = [&](int32_t a) OZ2H_INL {
            const double x = (double)a;
            const double q = rint(x * wi);
            return (int32_t)(uint32_t)__builtin_bit_cast(uint64_t, fma(-q, md, fma(x, w, kMagic)));
        };
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[c][x][y][e] = residue(h[c][x][y][e]);
                __builtin_amdgcn_sched_barrier(0);   // eight at a time: few registers
            }
        if (prod + 1 < nprod) return;
        int mt, nt, ln = lane;
        asm volatile("" : "+v"(ln));   // nothing of this address lives through the k-loop
        tile_of(item, mt, nt);
        const int64_t ldv = ka->g.ldv;
        int16_t *base = ka->g.V + (int64_t)l * ka->g.v_ps +
                        ((int64_t)mt * 256 + 128 * H + wr * 64 + (ln & 15)) * ldv + nt * 256 + wc * 64 +
                        (ln >> 4) * 8;
        int64_t o2 = 0;
        if constexpr (MODE == ZGAUSS) o2 = ka->g.V2 - ka->g.V;
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                int16_t *dst = base + (int64_t)(16 * x) * ldv + 32 * c;
                int32_t r[8];
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[4 * y + e] = h[c][x][y][e];
                auto pack = [&](const int32_t (&t)[8]) OZ2H_INL {
                    v4i o;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        o[i] = (int)__builtin_amdgcn_perm((uint32_t)t[2 * i + 1], (uint32_t)t[2 * i], 0x05040100u);
                    return o;
                };
                if constexpr (MODE == ZSTORE) {
                    *(v4i *)dst = pack(r);
                } else {
                    const v4i p1 = *(const v4i *)dst;
                    v4i p2 = v4i{};
                    if constexpr (MODE == ZGAUSS) p2 = *(const v4i *)(dst + o2);
                    int32_t s1[8], s2[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int32_t t1 = (int16_t)((uint32_t)p1[i / 2] >> (16 * (i % 2)));
                        const int32_t t2 = (int16_t)((uint32_t)p2[i / 2] >> (16 * (i % 2)));
                        if constexpr (MODE == ZADD) s1[i] = centred_mod((double)(t1 + r[i]), md, inv_m);
                        if constexpr (MODE == ZSUB) s1[i] = centred_mod((double)(t1 - r[i]), md, inv_m);
                        if constexpr (MODE == ZGAUSS) {
                            s1[i] = centred_mod((double)(t1 - t2), md, inv_m);
                            s2[i] = centred_mod((double)(r[i] - t1 - t2), md, inv_m);
                        }
                    }
                    *(v4i *)dst = pack(s1);
                    if constexpr (MODE == ZGAUSS) *(v4i *)(dst + o2) = pack(s2);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        clear(h);
    };
    // the operations the schedule below is written in; waits of half_end: every LDS read, and all
    // but the newest vector-memory operations, 8 loads and the stores (8 each) of `stores` halves
    constexpr int kSt = MODE == ZSTORE ? 8 : 0;   // (the other modes wait for theirs)
    auto half_end = [&](int stores) OZ2H_INL {
        fence();
        if (stores == 2) __builtin_amdgcn_s_waitcnt(vmlgkm_imm(8 + 2 * kSt));
        else if (stores == 1) __builtin_amdgcn_s_waitcnt(vmlgkm_imm(8 + kSt));
        else __builtin_amdgcn_s_waitcnt(vmlgkm_imm(8));
        barrier();
    };
    auto wait_vm = [&](auto n_) OZ2H_INL { __builtin_amdgcn_s_waitcnt(vmcnt_imm(decltype(n_)::value)); };
    auto next_item = [&]() OZ2H_INL {
        item = next(item);
        nprod = products(item);
        return item.zi < (uint32_t)kargs()->L;
    };
#include "oz2h_gemm8_schedule.inc"
}

// Residue planes of a sum of two operands (3M: Ar + Ai, Br + Bi) from the planes of
// each: per modulus l, s = x + y reduced to the centred residue s - rint(s/m) m (the
// quotient in fp32 is exact: |s| <= m + 3 < 2^15 and s/m is at least 1/(2m) from a
// half-integer for odd m; for the even one-limb modulus 128 either tie is a valid
// representative with |r| <= 64), then split like the residue kernels (one byte, or
// the balanced base-128 limbs (r0, r1, r0 + r1)).  One thread per 16 bytes of a plane;
// grid (ps / 4096 blocks of 256 threads, L).  ps is a multiple of 4096.
__global__ __launch_bounds__(256) void k_plane_sum(const int8_t *__restrict__ X,
                                                   const int8_t *__restrict__ Y,
                                                   int8_t *__restrict__ S, int64_t ps,
                                                   const ModInfo *__restrict__ mi) {
    const ModInfo info = load_info((OZ2H_G(ModInfo) *)(mi + blockIdx.y));
    const int64_t o = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 16;
    if (o >= ps) return;
    const float inv_m = (float)info.inv_m;
    const int64_t b0 = (int64_t)info.g0 * ps + o;
    auto reduce = [&](int sv) { return sv - (int)rintf((float)sv * inv_m) * (int)info.m; };
    if (info.nprod == 1) {
        const int4 xa = *(const int4 *)(X + b0), ya = *(const int4 *)(Y + b0);
        const int8_t *xb = (const int8_t *)&xa, *yb = (const int8_t *)&ya;
        int4 out;
        int8_t *ob = (int8_t *)&out;
#pragma unroll
        for (int i = 0; i < 16; ++i) ob[i] = (int8_t)reduce((int)xb[i] + (int)yb[i]);
        *(int4 *)(S + b0) = out;
        return;
    }
    const int4 x0 = *(const int4 *)(X + b0), x1 = *(const int4 *)(X + b0 + ps);
    const int4 y0 = *(const int4 *)(Y + b0), y1 = *(const int4 *)(Y + b0 + ps);
    const int8_t *x0b = (const int8_t *)&x0, *x1b = (const int8_t *)&x1;
    const int8_t *y0b = (const int8_t *)&y0, *y1b = (const int8_t *)&y1;
    int4 o0, o1, o2;
    int8_t *o0b = (int8_t *)&o0, *o1b = (int8_t *)&o1, *o2b = (int8_t *)&o2;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int r = reduce((int)x0b[i] + 128 * (int)x1b[i] + (int)y0b[i] + 128 * (int)y1b[i]);
        const int r0 = ((r + 64) & 127) - 64;   // balanced base-128 split
        const int r1 = (r - r0) >> 7;
        o0b[i] = (int8_t)r0;
        o1b[i] = (int8_t)r1;
        o2b[i] = (int8_t)(r0 + r1);
    }
    *(int4 *)(S + b0) = o0;
    *(int4 *)(S + b0 + ps) = o1;
    *(int4 *)(S + b0 + 2 * ps) = o2;
}

// ---------------------------------------------------------------- stage 4 + 5

// multi-digit helpers on an LDS digit column (stride `st` words between digits)
__device__ __forceinline__ bool dig_ge(const uint32_t *sd, int64_t st, const uint32_t *__restrict__ Q,
                                       int nd) {   // column >= Q ?
    int64_t br = 0;
    for (int k = 0; k < nd; ++k) br = ((int64_t)sd[k * st] - (int64_t)Q[k] - br) < 0;
    return br == 0;
}
__device__ __forceinline__ void dig_sub(uint32_t *sd, int64_t st, const uint32_t *__restrict__ Q,
                                        int nd) {   // column -= Q
    int64_t br = 0;
    for (int k = 0; k < nd; ++k) {
        const int64_t d = (int64_t)sd[k * st] - (int64_t)Q[k] - br;
        sd[k * st] = (uint32_t)d;
        br = d < 0;
    }
}
__device__ __forceinline__ void dig_rsub(uint32_t *sd, int64_t st, const uint32_t *__restrict__ Q,
                                         int nd) {   // column = Q - column
    int64_t br = 0;
    for (int k = 0; k < nd; ++k) {
        const int64_t d = (int64_t)Q[k] - (int64_t)sd[k * st] - br;
        sd[k * st] = (uint32_t)d;
        br = d < 0;
    }
}
__device__ __forceinline__ void dig_add(uint32_t *sd, int64_t st, const uint32_t *__restrict__ Q,
                                        int nd) {   // column += Q (mod 2^(32 nd))
    uint64_t cy = 0;
    for (int k = 0; k < nd; ++k) {
        const uint64_t d = (uint64_t)sd[k * st] + Q[k] + cy;
        sd[k * st] = (uint32_t)d;
        cy = d >> 32;
    }
}
// The magnitude digits of c^ read from its digit column.  On the fast path the
// column holds c^ in two's complement; for c^ < 0, |c^| = ~X + 1, so with z the
// lowest nonzero digit of X: digit k of |c^| is ~X_k above z, -X_z at z and 0
// below (no negation pass over the column).  Digits outside [0, nd) read as 0.
struct MagView {
    const uint32_t *sd;
    int64_t st;
    int nd, z;
    bool inv;
    __device__ __forceinline__ uint32_t operator()(int64_t k) const {
        if (k < 0 || k >= nd) return 0u;
        const uint32_t x = sd[k * st];
        if (!inv) return x;
        return k > z ? ~x : (k == z ? 0u - x : 0u);
    }
    // bits [pos, pos + 32)
    __device__ __forceinline__ uint32_t bits32(int64_t pos) const {
        const int64_t q = pos >> 5;
        const int r = (int)(pos & 31);
        const uint64_t lo = (*this)(q), hi = (*this)(q + 1);
        return (uint32_t)(((hi << 32) | lo) >> r);
    }
    // any nonzero bit below position pos
    __device__ __forceinline__ bool any_below(int64_t pos) const {
        const int64_t full = pos >> 5;
        const int rr = (int)(pos & 31);
        if (rr && ((*this)(full) & ((1u << rr) - 1)) != 0) return true;
        if (inv) return z < full;   // digit z is nonzero, everything below it is zero
        for (int64_t k = min(full, (int64_t)nd) - 1; k >= 0; --k)
            if (sd[k * st] != 0) return true;
        return false;
    }
};

// Direct CRT (subsection "Direct CRT without multiple-precision division").
// Each thread reconstructs EPT output entries (entries tid + q*blockDim of the
// block's range, so every load is coalesced).  Pass c accumulates digits
// [c*DC, (c+1)*DC) of S = sum_l v_l M_l over all moduli: v_l centred, M_l in
// balanced base-2^32 digits, so each column sum is an exact fp64 integer and
// the DC digit constants of modulus l are shared by the EPT entries.  Pass 0
// also forms sum_l v_l / m_l in binary64, an estimate of S/P = n + c^/P.
// Since |c^| < P/2, the nearest integer beta of that estimate is n unless the
// estimate lies within 2^-30 of a half-integer (never, when the CRT margin is
// at least 2, because then |c^| < P/4); in that case c^ = S - beta P comes out
// of one signed carry pass, already lifted.  Otherwise the paper's sequence is
// used: R = S - (alpha - 1) P with alpha = floor(estimate), R in [0, 3P), at
// most two subtractions of P, and the symmetric lift against floor(P/2).
// The magnitude digits sit in an LDS column; (ROUND) they are rounded once,
// nearest-even, to p bits with the scale 2^(e_i + f_j - 2t).
// The planes hold v_l = u_l (P/m_l)^-1 mod m_l as centred int16 (the residue
// GEMM applies the weight); WEIGHT = true takes plain residues u_l instead.
// The digit constants (and 1/m_l) are wave-uniform: scalar loads (SGPR operands of the
// FMAs) with LDS digit columns, LDS-staged slices of LB moduli with global ones.
struct CrtArgs {
    const int16_t *V;
    int64_t v_ps, ldv, M, N;
    const ModInfo *mi;
    int L;
    const double *dig;
    int ndpad, nc, nd32;
    const uint32_t *Pd, *Phd;
    const int32_t *erow, *fcol;   // nullable (0)
    int tsum, p;                  // value = c^ 2^(erow + fcol - tsum); tsum = 2t in the forward
    int8_t *osign;
    int32_t *oexp;
    uint64_t *olimbs;
    int64_t ldc;
    uint64_t *chat_mag;
    int nlc, LB;
    uint32_t *gdig;    // GDIG: digit columns in global memory, digit k of entry e at
    int64_t gstride;   // gdig[k * gstride + e] (gstride >= all entries the grid covers)
    // matrix-core CRT (k_crt_mma): A fragments, row blocks, contraction steps, top digits
    const int8_t *afr;
    int nbk, kq, nt;
    double inv_ptop;
    // unit CRT (k_crt_units): units, their digits, pairs among them (an even number)
    const CrtUnit *units;
    const double *udig;   // [units][ND]
    int npair;
};

// Lift and (ROUND) rounding of output entry (i, j) from its digit column sd (stride
// cst): on the fast path the column holds c^ in two's complement over nd32 digits
// (sign = carry < 0); on the slow path it holds R = S - (alpha - 1) P in [0, 3P).
// STASH: the limbs go into the column (limb w in its digits 2 w and 2 w + 1) where no later one
// reads them, and the result is true; else they are stored.
template <bool ROUND, bool STASH = false>
__device__ __forceinline__ bool crt_finish(const CrtArgs &a, int64_t i, int64_t j, uint32_t *sd, int64_t cst,
                                           bool slow, int64_t carry) {
    const int nd32 = a.nd32, p = a.p;
    const uint32_t *__restrict__ Phd = a.Phd;
    const int nl = (p + 63) / 64;
    bool neg;
    MagView mag{sd, cst, nd32, 0, false};
    if (!slow) {
        neg = carry < 0;   // two's complement c^ over nd32 digits
        if (neg) {
            int z = 0;
            while (z < nd32 - 1 && sd[z * cst] == 0) ++z;
            mag.z = z;
            mag.inv = true;
        }
    } else {
        // R in [0, 3P): at most two subtractions of P, then the symmetric lift
        if (dig_ge(sd, cst, a.Pd, nd32)) dig_sub(sd, cst, a.Pd, nd32);
        if (dig_ge(sd, cst, a.Pd, nd32)) dig_sub(sd, cst, a.Pd, nd32);
        neg = !dig_ge(sd, cst, Phd, nd32) ? false : true;   // x0 >= floor(P/2) ...
        if (neg) {                                          // ... and x0 != floor(P/2)
            dig_sub(sd, cst, Phd, nd32);
            bool eq = true;
            for (int k = 0; k < nd32 && eq; ++k) eq = sd[k * cst] == 0;
            dig_add(sd, cst, Phd, nd32);
            neg = !eq;
        }
        if (neg) dig_rsub(sd, cst, a.Pd, nd32);   // |c^| = P - x0
    }
    int top = nd32 - 1;
    while (top >= 0 && mag(top) == 0) --top;

    if (!ROUND) {
        const int64_t e = i * a.N + j;
        __attribute__((address_space(1))) uint64_t *o =
            (__attribute__((address_space(1))) uint64_t *)a.chat_mag + e * a.nlc;
        for (int w = 0; w < a.nlc; ++w)
            o[w] = (uint64_t)mag(2 * w) | ((uint64_t)mag(2 * w + 1) << 32);
        a.osign[e] = top < 0 ? 0 : (neg ? -1 : 1);
        return false;
    }
    const int64_t oi = i * a.ldc + j;
    __attribute__((address_space(1))) uint64_t *o =
        (__attribute__((address_space(1))) uint64_t *)a.olimbs + oi * nl;
    if (top < 0) {
        for (int w = 0; w < nl; ++w) o[w] = 0;
        a.osign[oi] = 0;
        a.oexp[oi] = 0;
        return false;
    }
    int64_t nb = 32 * (int64_t)top + (32 - __builtin_clz(mag(top)));
    const int64_t sh = nb - p;   // mant = RNE(mag / 2^sh)
    bool inc = false;
    if (sh > 0) {
        const int64_t rpos = sh - 1;
        if ((mag.bits32(rpos) & 1u) != 0)   // round bit set: up unless an exact tie to even
            inc = mag.any_below(rpos) || (mag.bits32(sh) & 1u);
    }
    // mant = mag / 2^sh (+ 1): limb w is bits [sh + 64 w, sh + 64 w + 64) of mag, formed from
    // three consecutive digits by funnel shifts, one pass from the bottom
    const int64_t q0 = sh >> 5;   // floor: sh < 0 reads zero digits below the column
    const int rsh = (int)(sh & 31);
    const bool stash = STASH && q0 >= 0;   // limb w + 1 reads from digit q0 + 2 w + 3 on
    auto put = [&](int w, uint64_t v) {
        if (stash) {
            sd[2 * w * cst] = (uint32_t)v;
            sd[(2 * w + 1) * cst] = (uint32_t)(v >> 32);
        } else {
            o[w] = v;
        }
    };
    uint32_t prev = mag(q0);
    bool cy = inc;
    uint64_t last = 0;
    for (int w = 0; w < nl; ++w) {
        const uint32_t d1 = mag(q0 + 2 * w + 1), d2 = mag(q0 + 2 * w + 2);
        const uint64_t v = ((uint64_t)__builtin_amdgcn_alignbit(d2, d1, rsh) << 32) |
                           __builtin_amdgcn_alignbit(d1, prev, rsh);
        last = v + (cy ? 1u : 0u);
        cy = cy && last == 0;
        put(w, last);
        prev = d2;
    }
    const int pb = p - 64 * (nl - 1);   // bits of the top limb
    if (pb < 64 ? (last >> pb) != 0 : cy) {   // mant = 2^p - 1 rounded up to 2^p: renormalise
        for (int w = 0; w < nl; ++w) put(w, w == (p - 1) >> 6 ? 1ull << ((p - 1) & 63) : 0);
        nb += 1;
    }
    a.osign[oi] = neg ? -1 : 1;
    a.oexp[oi] = (int32_t)(nb + (int64_t)(a.erow ? a.erow[i] : 0) + (a.fcol ? a.fcol[j] : 0) -
                           (int64_t)a.tsum);
    return stash;
}

// A wave whose lanes hold stashed limbs (crt_finish; columns kCrtFinS words apart, lane e's at
// sdig + e; oi: its output entry) stores them with consecutive lanes at consecutive limbs: a lane
// storing its own entry's limbs touches 64 lines with every store (CRT at 2048^2, row kernels,
// p = 1024 3.03 to 2.83 ms, p = 800 2.19 to 2.05).  Records of 30 limbs and more nearly fill their
// lines with each entry's own stores, and the wider columns cost a wave of LDS; few entries stay
// in the caches (finish kernel, stashed / not: 24 limbs 214 / 256 us at 1000^2, 29 282 / 311, 30
// 345 / 309, 40 537 / 457; 24 limbs 93 / 100 at 620^2, 27 109 / 109; at 300^2 19 31 / 24, 25 40 / 35,
// 29 45 / 42).
constexpr int kCrtFinS = 65;   // LDS words between the digits of a column
constexpr int kCrtStashLimbs = 29;
constexpr int64_t kCrtStashEntries = 262144;
__device__ __forceinline__ void store_limbs(const CrtArgs &a, const uint32_t *sdig, bool stashed, int64_t oi) {
    const uint64_t mask = __ballot(stashed);
    if (!mask) return;
    wave_lds_sync();
    const int lane = threadIdx.x & 63, nl = (a.p + 63) / 64, q = 64 / nl, rm = 64 - q * nl;
    int e = lane / nl, w = lane - e * nl;
    for (int it = 0; it < nl; ++it) {   // limb w of the wave's entry e
        const int64_t oe = __shfl(oi, e);
        const uint32_t lo = sdig[2 * w * kCrtFinS + e], hi = sdig[(2 * w + 1) * kCrtFinS + e];
        if ((mask >> e) & 1)
            ((__attribute__((address_space(1))) uint64_t *)a.olimbs)[oe * nl + w] = (uint64_t)hi << 32 | lo;
        e += q;
        w += rm;
        if (w >= nl) {
            w -= nl;
            ++e;
        }
    }
}

// LDS of a CRT block: bd * EPT digit columns of nd32 words (GDIG = false), or the
// LB x (DC + 1) doubles of a constant slice (GDIG = true: the digit columns of large
// nd32 sit in global memory).
template <int DC, int EPT, bool ROUND, bool WEIGHT, bool GDIG = false>
__device__ __forceinline__ void crt_block(const CrtArgs &a, int64_t blk, uint32_t *sdig) {
    const int tid = threadIdx.x, bd = blockDim.x, st = bd * EPT;
    const int64_t cst = GDIG ? a.gstride : (int64_t)st;   // digit stride of a column
    const int nd32 = a.nd32, L = a.L, LB = a.LB, ndpad = a.ndpad;
    const int64_t N = a.N, v_ps = a.v_ps;
    // global-memory views (pointers from a descriptor are generic otherwise)
    OZ2H_G(uint32_t) *Pd = (OZ2H_G(uint32_t) *)a.Pd;
    OZ2H_G(ModInfo) *mi = (OZ2H_G(ModInfo) *)a.mi;
    // digit constants and 1/m: read-only for the launch and wave-uniform.  With LDS digit
    // columns (two entries per thread) the constant address space puts them on the scalar
    // unit (SGPR operands of the FMAs); with global columns (GDIG) a slice of LB moduli is
    // staged in LDS and read as broadcasts, two constants per ds_read_b128.
    typedef const __attribute__((address_space(4))) double cdouble;
    typedef const __attribute__((address_space(4))) ModInfo cmodinfo;
    cdouble *cdig = (cdouble *)a.dig;
    cmodinfo *cmi = (cmodinfo *)a.mi;
    double *stab = (double *)sdig;               // GDIG: LB x DC digits
    double *sinv = stab + (size_t)LB * DC;       // GDIG: LB x 1/m
    const int64_t MN = a.M * N;
    int64_t idx[EPT];
    OZ2H_G(int16_t) *vp[EPT];
    bool live[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        idx[q] = blk * st + q * bd + tid;
        live[q] = idx[q] < MN;
        // a dead lane reads entry 0 (always valid) and writes nothing: no branch around loads
        const int64_t ii = live[q] ? idx[q] / N : 0, jj = live[q] ? idx[q] - ii * N : 0;
        vp[q] = (OZ2H_G(int16_t) *)a.V + ii * a.ldv + jj;
    }
    auto col = [&](int q) -> uint32_t * { return GDIG ? a.gdig + idx[q] : sdig + q * bd + tid; };

    int64_t beta[EPT], carry[EPT];
    bool slow[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        beta[q] = 0;
        carry[q] = 0;
        slow[q] = false;
    }
    for (int c = 0; c < a.nc; ++c) {
        double acc[EPT][DC], asum[EPT];
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            asum[q] = 0.0;
#pragma unroll
            for (int d = 0; d < DC; ++d) acc[q][d] = 0.0;
        }
        for (int l0 = 0; l0 < L; l0 += LB) {
            const int nlb = min(LB, L - l0);
            if constexpr (GDIG) {
                OZ2H_G(double) *dc = (OZ2H_G(double) *)a.dig + c * DC;
                __syncthreads();   // the previous slice has been consumed by every thread
                for (int e = tid; e < nlb * DC; e += bd) {
                    const int ll = e / DC, d = e - ll * DC;
                    stab[e] = dc[(size_t)(l0 + ll) * ndpad + d];
                }
                for (int e = tid; e < nlb; e += bd) sinv[e] = mi[l0 + e].inv_m;
                __syncthreads();
            }
            // v_l of the next PF moduli are loaded ahead (unconditional, clamped at the end)
            constexpr int PF = 4;
            int ring[PF][EPT];
#pragma unroll
            for (int f = 0; f < PF; ++f)
#pragma unroll
                for (int q = 0; q < EPT; ++q) ring[f][q] = vp[q][(int64_t)(l0 + min(f, nlb - 1)) * v_ps];
            // one modulus: its v values (one per entry of the thread) into the digit sums
            auto inv_of = [&](int ll) { return GDIG ? sinv[ll] : cmi[l0 + ll].inv_m; };
            auto modulus = [&](int ll, const int *cur, double inv_m) {
                const int l = l0 + ll;
                double vd[EPT];
#pragma unroll
                for (int q = 0; q < EPT; ++q) {
                    const int raw = cur[q];
                    if (WEIGHT) {
                        const ModInfo info = load_info(mi + l);
                        vd[q] = (double)centred_mod((double)raw * (double)info.minv, (double)info.m, inv_m);
                    } else {
                        vd[q] = (double)raw;
                    }
                    if (c == 0) asum[q] = fma(vd[q], inv_m, asum[q]);
                }
                if constexpr (GDIG) {
                    const double *dl = stab + (size_t)ll * DC;
#pragma unroll
                    for (int d = 0; d < DC; d += 2) {
                        const double2 w = *(const double2 *)(dl + d);
#pragma unroll
                        for (int q = 0; q < EPT; ++q) {
                            acc[q][d] = fma(vd[q], w.x, acc[q][d]);
                            acc[q][d + 1] = fma(vd[q], w.y, acc[q][d + 1]);
                        }
                    }
                } else {
                    cdouble *dl = cdig + (size_t)l * ndpad + c * DC;
#pragma unroll
                    for (int d = 0; d < DC; ++d) {
                        const double w = dl[d];
#pragma unroll
                        for (int q = 0; q < EPT; ++q) acc[q][d] = fma(vd[q], w, acc[q][d]);
                    }
                }
            };
            // full groups of PF moduli: straight-line code, so that the scalar constants of a
            // modulus can load while the previous one multiplies (measured faster from 16
            // digits per pass on with LDS columns; narrower passes and global columns, whose
            // constants come from the LDS slice, keep one guarded loop, which measured 2x
            // faster there at 4096^3 and p = 2048); the v ring runs PF moduli ahead
            constexpr bool SL = DC >= 16 && !GDIG;
            const int nfull = SL ? nlb - nlb % PF : 0;
            for (int lb = 0; lb < nfull; lb += PF) {
#pragma unroll
                for (int f = 0; f < PF; ++f) {
                    const int ll = lb + f;
                    int cur[EPT];
#pragma unroll
                    for (int q = 0; q < EPT; ++q) {
                        cur[q] = ring[f][q];
                        ring[f][q] = vp[q][(int64_t)(l0 + min(ll + PF, nlb - 1)) * v_ps];
                    }
                    modulus(ll, cur, inv_of(ll));
                }
            }
            if constexpr (SL) {
                for (int ll = nfull; ll < nlb; ++ll) {   // the last nlb % PF moduli
                    int cur[EPT];
#pragma unroll
                    for (int q = 0; q < EPT; ++q) cur[q] = vp[q][(int64_t)(l0 + ll) * v_ps];
                    modulus(ll, cur, inv_of(ll));
                }
            } else {
                for (int lb = 0; lb < nlb; lb += PF) {
#pragma unroll
                    for (int f = 0; f < PF; ++f) {
                        const int ll = lb + f;
                        if (ll >= nlb) break;
                        // 1/m is read before the next v load is issued: with global columns
                        // (1/m from LDS) the other order measured 1.4x slower at p = 2048
                        const double inv_m = inv_of(ll);
                        int cur[EPT];
#pragma unroll
                        for (int q = 0; q < EPT; ++q) {
                            cur[q] = ring[f][q];
                            ring[f][q] = vp[q][(int64_t)(l0 + min(ll + PF, nlb - 1)) * v_ps];
                        }
                        modulus(ll, cur, inv_m);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            if (c == 0) {
                const double r = rint(asum[q]);
                slow[q] = fabs(asum[q] - r) > 0.5 - 0x1p-30;
                beta[q] = slow[q] ? (int64_t)floor(asum[q]) - 1 : (int64_t)r;   // alpha - 1 when slow
            }
            // digit k of S - beta P in binary64, exact: |acc| <= L 8095 2^31 < 2^53 - 2^46 for
            // L <= 512, |beta P_k| < 2^42 and the carry is below 2^22
            uint32_t *sd = col(q);
            double cy = (double)carry[q];
            const double bq = (double)beta[q];
#pragma unroll
            for (int d = 0; d < DC; ++d) {
                const int k = c * DC + d;
                if (k < nd32) {
                    const double x = fma(-bq, (double)Pd[k], acc[q][d] + cy);
                    const double hi = floor(x * 0x1p-32);
                    sd[k * cst] = (uint32_t)fma(-hi, 0x1p32, x);
                    cy = hi;
                }
            }
            carry[q] = (int64_t)cy;
        }
    }

#pragma unroll
    for (int q = 0; q < EPT; ++q)
        if (live[q]) crt_finish<ROUND>(a, idx[q] / N, idx[q] % N, col(q), cst, slow[q], carry[q]);
}

template <int DC, int EPT, bool ROUND, bool WEIGHT, bool GDIG>
__global__ __launch_bounds__(256) void k_crt(CrtArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t sdig[];
    crt_block<DC, EPT, ROUND, WEIGHT, GDIG>(a, blockIdx.x, sdig);
}

// The same by units, for digit sums that fit one pass (nd32 <= 48, digit columns in LDS).  Two
// one-limb moduli a, b enter as one term: v_a (P / m_a) + v_b (P / m_b) = V P / (m_a m_b) with
// V = v_a m_b + v_b m_a, which takes the multiply-adds of one modulus.  The sums stay exact:
// the plan takes pairs while sum_u max |V_u| < 2^22 - 2^15, the bound crt_block's carry pass
// needs.  A thread takes EPT adjacent columns of a row; V of a pair is one v_dot2_i32_i16 per
// entry.  The digit constants are wave-uniform scalar loads (SGPR operands of the FMAs), ND
// (crt_unit_digits) per unit; v planes are read four moduli ahead.
//
// What bounds it: VALU issue (FMAs with a scalar operand issue at 50 to 60 TFLOP/s at the two
// to four waves per SIMD that registers and digit columns leave), at 8192^2, p = 113 the v
// planes as much (7 GB).  Against single moduli in blocks of 512 entries: 2.76 to 1.74 ms at
// 8192^2, p = 113; 1.76 to 0.95 ms at 4096^2, p = 256; 25 to 11 us at 256^2, p = 128.
template <int ND, int EPT, bool ROUND>
__device__ __forceinline__ void crt_units_block(const CrtArgs &a, int64_t blk, uint32_t *sdig) {
    static_assert(EPT == 1 || EPT == 2, "one column or two adjacent ones");
    const int tid = threadIdx.x, bd = blockDim.x, cst = bd * EPT;
    const int nd32 = a.nd32, L = a.L, npair = a.npair;
    const int64_t v_ps = a.v_ps, cols = (a.N + EPT - 1) / EPT;
    typedef const __attribute__((address_space(4))) double cdouble;
    typedef const __attribute__((address_space(4))) CrtUnit cunit;
    typedef const __attribute__((address_space(4))) uint32_t cu32;
    typedef typename std::conditional<EPT == 2, int32_t, int16_t>::type raw_t;
    cdouble *ud = (cdouble *)a.udig;
    cunit *cu = (cunit *)a.units;

    const int64_t idx = blk * bd + tid, total = a.M * cols;
    const bool live = idx < total;   // a dead thread reads entry (0, 0) and writes nothing
    int64_t i = 0, j = 0;
    if (live) {
        i = total >> 32 ? idx / cols : (int64_t)((uint32_t)idx / (uint32_t)cols);
        j = (idx - i * cols) * EPT;
    }
    OZ2H_G(int16_t) *vp = (OZ2H_G(int16_t) *)a.V + i * a.ldv + j;
    auto load = [&](int l) OZ2H_INL { return (int)*(OZ2H_G(raw_t) *)(vp + (int64_t)l * v_ps); };

    double acc[EPT][ND], asum[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        asum[q] = 0.0;
#pragma unroll
        for (int d = 0; d < ND; ++d) acc[q][d] = 0.0;
    }
    // unit u with the terms x of the thread's entries
    auto unit = [&](int u, const double (&x)[EPT]) OZ2H_INL {
        cdouble *dl = ud + (size_t)u * ND;
        const double inv = cu[u].inv;
#pragma unroll
        for (int q = 0; q < EPT; ++q) asum[q] = fma(x[q], inv, asum[q]);
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            const double w = dl[d];
#pragma unroll
            for (int q = 0; q < EPT; ++q) acc[q][d] = fma(x[q], w, acc[q][d]);
        }
    };
    auto pair = [&](int u, int ra, int rb) OZ2H_INL {
        typedef short s2 __attribute__((ext_vector_type(2)));
        const s2 mm = __builtin_bit_cast(s2, cu[u].mm);   // (m_b, m_a)
        double x[EPT];
#pragma unroll
        for (int q = 0; q < EPT; ++q) {
            const uint32_t w = __builtin_amdgcn_perm((uint32_t)rb, (uint32_t)ra, q ? 0x07060302u : 0x05040100u);
            x[q] = (double)__builtin_amdgcn_sdot2(__builtin_bit_cast(s2, w), mm, 0, false);
        }
        unit(u, x);
    };
    auto single = [&](int u, int r) OZ2H_INL {
        double x[EPT];
        x[0] = (double)(int16_t)r;
        if constexpr (EPT == 2) x[1] = (double)(r >> 16);
        unit(u, x);
    };
    int ring[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) ring[f] = load(min(f, L - 1));
    int l = 0, u = 0;   // next modulus and unit
    for (; u < npair; u += 2, l += 4) {
        const int r0 = ring[0], r1 = ring[1], r2 = ring[2], r3 = ring[3];
#pragma unroll
        for (int f = 0; f < 4; ++f) ring[f] = load(min(l + 4 + f, L - 1));
        pair(u, r0, r1);
        pair(u + 1, r2, r3);
    }
    for (; l + 4 <= L; l += 4, u += 4) {
        int r[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            r[f] = ring[f];
            ring[f] = load(min(l + 4 + f, L - 1));
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) single(u + f, r[f]);
    }
#pragma unroll
    for (int f = 0; f < 3; ++f)
        if (l + f < L) single(u + f, ring[f]);

    // beta and S - beta P, as in crt_block
    cu32 *Pd = (cu32 *)a.Pd;
    bool slow[EPT];
    double cy[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const double r = rint(asum[q]);
        slow[q] = fabs(asum[q] - r) > 0.5 - 0x1p-30;
        const double beta = slow[q] ? floor(asum[q]) - 1.0 : r;   // alpha - 1 when slow
        uint32_t *sd = sdig + q * bd + tid;
        cy[q] = 0.0;
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            if (k < nd32) {
                const double x = fma(-beta, (double)Pd[k], acc[q][k] + cy[q]);
                const double hi = floor(x * 0x1p-32);
                sd[k * cst] = (uint32_t)fma(-hi, 0x1p32, x);
                cy[q] = hi;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q)
        if (live && j + q < a.N)
            crt_finish<ROUND>(a, i, j + q, sdig + q * bd + tid, cst, slow[q], cy[q] < 0.0 ? -1 : 0);
}

template <int ND, int EPT, bool ROUND>
__global__ __launch_bounds__(256) void k_crt_units(CrtArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t sdig[];
    crt_units_block<ND, EPT, ROUND>(a, blockIdx.x, sdig);
}

// Direct CRT on the matrix cores (digit columns in LDS: nd32 <= 32, L <= 127, blocks of 256
// entries; wider sets, up to nd32 <= kCrtMmaMaxDigits and L <= 255, blocks of 64).  The
// digit sums S = sum_l v_l M_l are formed as the int8 product (byte rows of S) x
// (entries) of the tables of build_crt_mma_tables with each v_l's two bytes; one wave
// covers 64 consecutive entries as two 32-entry column blocks.
//   B fragments: lane (h, c) holds, per 32-byte step q, the words of moduli
//     16 q + 8 h .. + 7 of entries c and 32 + c, each xor 0x0080 (low byte - 128).
//   Output element 4 a + i of a 32 x 32 block is byte row 8 a + 4 h + i, i.e. byte i of
//     digit 2 a + h: a lane assembles four digit partials per block; one ds_bpermute
//     hand-over then gives lane (0, c) all digits of entry c and lane (1, c) all digits of
//     entry 32 + c, which it carries into its LDS column.
//   S / P is estimated from the top nt digits (error below 2^-40); the nearest integer
//   beta is exact unless the estimate lies within 2^-30 of a half-integer, else the
//   paper's alpha - 1 (at most two subtractions of P follow in crt_finish).  Then the
//   column receives S - beta P and crt_finish lifts and rounds as in k_crt.
constexpr int kCrtMmaMaxQ = 8;   // contraction steps of the matrix-core CRT (2 L + 1 <= 256)
constexpr int kCrtMmaWideQ = 16; // ... of the wide form (2 L + 1 <= 512), in steps of two from 6 on
// below this many digits (p <~ 180) the fp64 CRT is faster: the matrix-core kernel's
// per-entry carry and subtraction passes outweigh its L x nd32 multiply-adds
constexpr int kCrtMmaMinDigits = 16;

// WEIGHT = true: the planes hold plain residues u_l (any representative, |u_l| < m_l),
// weighted here to v_l = u_l (P/m_l)^-1 mod m_l (the stage-4 parity entry point).
// BT: threads of the block.  BT = 64 (the wide form): the tables have exactly KQ steps, so the
// step loop has no guards and its loads go out together.  What bounds the wide form: the carries
// and the subtraction per digit and the fragment reads (108 KiB per wave at 70 digits and 182
// moduli); its products alone take 0.5 of 3.2 ms at 3072^2, p = 1024.
template <int KQ, bool ROUND, bool WEIGHT = false, int BT = 256>
__device__ __forceinline__ void crt_mma_block(const CrtArgs &a, int64_t blk, uint32_t *sdig) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int h = lane >> 5, c = lane & 31;
    const int nd32 = a.nd32, L = a.L, kq = a.kq, nbk = a.nbk;
    const int64_t N = a.N, MN = a.M * N, v_ps = a.v_ps;
    constexpr bool EXACT = BT == 64;   // kq == KQ
    constexpr int CS = BT == 64 ? kCrtFinS : BT;   // LDS words between the digits of a column
    const int64_t e0 = blk * BT + wv * 64;
    typedef const __attribute__((address_space(1))) uint16_t gu16;
    typedef const __attribute__((address_space(1))) v4i gv4i;
    typedef const __attribute__((address_space(4))) uint32_t cu32;

    // B fragments (a dead entry reads entry 0, always valid, and writes nothing).  Steps
    // with all 16 moduli present load unguarded (a lane base plus a wave-uniform offset);
    // the last step clamps the modulus and feeds 0 past L.
    v4i bf0[KQ], bf1[KQ];
    {
        gu16 *vb[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t e = e0 + 32 * b + c, ee = e < MN ? e : 0;
            const int64_t i = ee / N, j = ee - i * N;
            vb[b] = (gu16 *)a.V + i * a.ldv + j + (int64_t)(8 * h) * v_ps;
        }
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            if (EXACT || q < kq) {
                const bool full = 16 * q + 16 <= L;   // wave-uniform
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    uint32_t w[8];
                    if (full) {
#pragma unroll
                        for (int t = 0; t < 8; ++t) w[t] = vb[b][(int64_t)(16 * q + t) * v_ps];
                    } else {
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            const int l = 16 * q + 8 * h + t;
                            const int lc = min(l, L - 1) - 8 * h;   // relative to the lane base
                            const uint32_t x = vb[b][(int64_t)lc * v_ps];
                            w[t] = l < L ? x : 0u;
                        }
                    }
                    if constexpr (WEIGHT) {
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            const int l = 16 * q + 8 * h + t;
                            if (l < L) {
                                const ModInfo info = load_info((OZ2H_G(ModInfo) *)a.mi + l);
                                const int32_t v = centred_mod((double)(int16_t)w[t] * (double)info.minv,
                                                              (double)info.m, info.inv_m);
                                w[t] = (uint32_t)(uint16_t)(int16_t)v;
                            }
                        }
                    }
                    const v4i f = v4i{(int)((w[0] | (w[1] << 16)) ^ 0x00800080u),
                                      (int)((w[2] | (w[3] << 16)) ^ 0x00800080u),
                                      (int)((w[4] | (w[5] << 16)) ^ 0x00800080u),
                                      (int)((w[6] | (w[7] << 16)) ^ 0x00800080u)};
                    if (b == 0) bf0[q] = f;
                    else bf1[q] = f;
                }
            }
        }
    }

    // S: eight digits per block of 32 byte rows, carried into this lane's LDS column
    gv4i *af = (gv4i *)a.afr + lane;
    uint32_t *col = sdig + tid;   // digit k at col[CS k]
    int64_t carry = 0;
    for (int nb = 0; nb < nbk; ++nb) {
        v16i acc0 = v16i{}, acc1 = v16i{};
#pragma unroll
        for (int q = 0; q < KQ; ++q)
            if (EXACT || q < kq) {
                const v4i f = af[((size_t)nb * (EXACT ? KQ : kq) + q) * 64];
                acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f, bf0[q], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f, bf1[q], acc1, 0, 0, 0);
            }
        int64_t mine[4], got[4];
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            const int64_t d0 = (int64_t)acc0[4 * a4] + (int64_t)acc0[4 * a4 + 1] * 256 +
                               (int64_t)acc0[4 * a4 + 2] * 65536 + (int64_t)acc0[4 * a4 + 3] * 16777216;
            const int64_t d1 = (int64_t)acc1[4 * a4] + (int64_t)acc1[4 * a4 + 1] * 256 +
                               (int64_t)acc1[4 * a4 + 2] * 65536 + (int64_t)acc1[4 * a4 + 3] * 16777216;
            const int64_t send = h ? d0 : d1;   // the partner's entry
            mine[a4] = h ? d1 : d0;
            const int plo = __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(uint32_t)send);
            const int phi = __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(send >> 32));
            got[a4] = (int64_t)(((uint64_t)(uint32_t)phi << 32) | (uint32_t)plo);
        }
#pragma unroll
        for (int dk = 0; dk < 8; ++dk) {
            const int k = 8 * nb + dk;
            const int64_t D = (dk & 1) == h ? mine[dk >> 1] : got[dk >> 1];
            if (k < nd32) {
                const int64_t x = D + carry;
                col[CS * k] = (uint32_t)x;
                carry = x >> 32;
            }
        }
    }

    // beta from S / P, then S - beta P into the column
    double val = (double)(int32_t)col[CS * (nd32 - 1)];
    for (int k = nd32 - 2; k >= nd32 - a.nt; --k) val = val * 4294967296.0 + (double)col[CS * k];
    const double est = val * a.inv_ptop, r = rint(est);
    const bool slow = fabs(est - r) > 0.5 - 0x1p-30;
    const int64_t beta = slow ? (int64_t)floor(est) - 1 : (int64_t)r;
    cu32 *Pd = (cu32 *)a.Pd;
    int64_t cy = 0;
    for (int k = 0; k < nd32; ++k) {
        const int64_t x = (int64_t)col[CS * k] - beta * (int64_t)Pd[k] + cy;
        col[CS * k] = (uint32_t)x;
        cy = x >> 32;
    }
    const int64_t e = e0 + lane;
    bool stashed = false;
    if (e < MN) stashed = crt_finish<ROUND, ROUND && BT == 64>(a, e / N, e % N, col, CS, slow, cy + carry);
    if constexpr (ROUND && BT == 64) store_limbs(a, sdig, stashed, e / N * a.ldc + e % N);
}

template <int KQ, bool ROUND, bool WEIGHT, int BT>
__global__ __launch_bounds__(BT, BT == 64 ? 2 : 1) void k_crt_mma(CrtArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint32_t sdig[];
    crt_mma_block<KQ, ROUND, WEIGHT, BT>(a, blockIdx.x, sdig);
}

// Direct CRT for wide moduli sets on the vector ALUs with row broadcasts (no MFMA), in two
// kernels.  S = sum_l v_l M_l, M_l = P / m_l in balanced base-2^32 digits D[d][l]: each digit
// sum S_d = sum_l v_l D[d][l] is an exact fp64 integer (|S_d| < L 2^44 < 2^53).  Two one-limb
// moduli enter as one unit, V = v_a m_b + v_b m_a against the digits of P / (m_a m_b), as in the
// unit CRT and under the same bound (both kernels at 2048^2, p = 1024 3.33 to 3.09 ms, 4096^2,
// p = 2048 36.1 to 34.4).
//   k_crt_row_sums: a wave takes 64 consecutive entries and one group of 16 digits.  Lane j
//     of row q owns digit 16 dg + j of the row's entries 16 q + i (i < 16) and keeps, per
//     chunk of 16 units, their 16 digit constants in registers; lane m of the row loads v of
//     unit 16 c + m for the row's 16 entries, and each multiply-add takes v from lane m by
//     a DPP row broadcast.  The 16 sums of an entry then go through LDS to one lane, which
//     carries them into 16 digits in [0, 2^32) and a carry-out (digit-major in the
//     workspace: digit k of entry e at dig[k * estride + e]).  Blocks are four waves, four
//     consecutive tiles of one digit group; the digit groups of a tile run on one XCD (block b
//     goes to XCD b mod 8), so that its v planes are read from HBM once and then from that
//     XCD's L2.
//   k_crt_row_finish: one entry per thread: the groups' carry-outs are added in, S's nd32
//     digits land in an LDS column, and from there as in the matrix-core CRT: beta from the
//     top digits (the paper's alpha - 1 when the estimate is within 2^-30 of a half-integer),
//     S - beta P, and crt_finish (symmetric lift, one rounding).
struct CrtRowArgs {
    const int16_t *V;
    int64_t v_ps;       // plane stride of v; entry e' = i * ldv + j of a plane is at V + e'
    int64_t nent;       // entries e' covered: M * ldv
    int64_t ldv;
    int nu, npair;        // units; the first npair are pairs of one-limb moduli (2 u, 2 u + 1)
    int lpad, ndg, nd32;
    const double *drow;   // [16 ndg][lpad]
    const ModInfo *mi;    // WEIGHT: plain residues u_l, weighted here
    uint32_t *dig;        // [16 ndg][estride]
    int32_t *cout;        // [ndg][estride]
    int64_t estride;      // >= 64 * ntiles
    int ntiles;           // tiles of 64 entries (a multiple of 32: four per block, one block
                          // per XCD)
};

// 16 values as doubles, followed by the two wait states a DPP read of them needs
__device__ __forceinline__ void dpp_ready16(double (&x)[16]) {
    asm volatile("s_nop 1"
                 : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]),
                   "+v"(x[6]), "+v"(x[7]), "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]),
                   "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), "+v"(x[15]));
}

// 16 x 16 multiply-adds: for each broadcast lane m (modulus 16 c + m), the 16 entries'
// accumulators in turn, so that consecutive multiply-adds are independent
template <int M = 0>
__device__ __forceinline__ void crt_row_fmas(double (&acc)[16], const double (&x)[16], const double (&c)[16]) {
    if constexpr (M < 16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) fmac_rowbcast<M>(acc[i], x[i], c[M]);
        crt_row_fmas<M + 1>(acc, x, c);
    }
}

// The digit constants of the block's digit group are staged in LDS kCrtRowStage moduli at a
// time (row jj = digit 16 dg + jj), with a row stride = 2 mod 32 doubles, so that the 16 rows
// a ds_read_b128 of 16 lanes touches start on 16 different 4-bank groups.
constexpr int kCrtRowStage = 192;
constexpr int kCrtRowDStride = kCrtRowStage + 2;
constexpr int kCrtRowPairs = kCrtRowStage / 32;   // 16-byte pairs per thread and stage
static_assert(kCrtRowStage % 32 == 0 && kCrtRowDStride % 2 == 0, "stage rows of whole pairs");
constexpr size_t kCrtRowSumsLds = (size_t)16 * kCrtRowDStride * 8 + (size_t)4 * 32 * 17 * 8;

// blocks of four waves: four consecutive tiles of 64 entries, one digit group; block b runs
// on XCD b mod 8 and the digit groups of a tile quad go to one XCD.  Every wave takes part
// in the staging barriers; a wave past the last tile computes on tile 0 and stores nothing.
template <bool WEIGHT>
__global__ __launch_bounds__(256) void k_crt_row_sums(CrtRowArgs a) {
    extern __shared__ __attribute__((aligned(16))) double smem_crs[];
    double *Dl = smem_crs;   // [16][kCrtRowDStride]
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double *T = smem_crs + (size_t)16 * kCrtRowDStride + (size_t)wv * 32 * 17;   // transpose
    const uint32_t b = blockIdx.x, x8 = b & 7u, s = b >> 3;
    const int dg = (int)(s % (uint32_t)a.ndg);
    const int64_t tile0 = ((int64_t)(s / (uint32_t)a.ndg) * 8 + x8) * 4 + wv;
    const bool live = tile0 * 64 < a.nent;
    const int64_t tile = live ? tile0 : 0;
    const int q = lane >> 4, j = lane & 15;
    const int64_t e_row = crt_row_first(a.nent, tile, q);   // this row's entries e_row + i
    typedef const __attribute__((address_space(1))) v4i gv4i;
    typedef double d2 __attribute__((ext_vector_type(2)));
    const double *gsrc = a.drow + (size_t)16 * dg * a.lpad;
    double acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0;
    const int nch = a.lpad >> 4;
    // chunk c of 16 units: v of unit min(16 c + j, nu - 1) for the row's 16 entries (32
    // bytes; nent is a multiple of 16 and the launch checks that every plane holds nent
    // entries), loaded one chunk ahead; the 16 digit constants of this lane's digit from LDS
    // (zero past the last unit)
    // plane addresses: the chunk's offset 16 c v_ps is wave-uniform (scalar arithmetic); a lane
    // past the last unit reads the last plane
    const int16_t *vj = a.V + (int64_t)(a.npair + j) * a.v_ps + e_row;
    const int16_t *vlast = a.V + (int64_t)(a.npair + a.nu - 1) * a.v_ps + e_row;
    auto loadv = [&](int c, v4i &w0, v4i &w1) {
        gv4i *src = (gv4i *)(16 * c + j < a.nu ? vj + (int64_t)(16 * c) * a.v_ps : vlast);
        w0 = src[0];
        w1 = src[1];
    };
    auto fmas = [&](int c, int l0, double (&vd)[16]) OZ2H_INL {
        const double *drow = Dl + j * kCrtRowDStride + (16 * c - l0);
        double dc[16];
#pragma unroll
        for (int m = 0; m < 16; m += 2) {
            const d2 t = *(const d2 *)(drow + m);
            dc[m] = t.x;
            dc[m + 1] = t.y;
        }
        dpp_ready16(vd);
        crt_row_fmas(acc, vd, dc);
    };
    // a lane's 16 values of modulus l, weighted here where the planes hold plain residues
    auto values = [&](int l, const v4i &w0, const v4i &w1, int (&v)[16]) OZ2H_INL {
        const int raw[8] = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3]};
        ModInfo mi{};
        if constexpr (WEIGHT) mi = load_info((OZ2H_G(ModInfo) *)a.mi + l);
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            v[t] = t & 1 ? raw[t / 2] >> 16 : (raw[t / 2] << 16) >> 16;
            if constexpr (WEIGHT) v[t] = centred_mod((double)v[t] * (double)mi.minv, (double)mi.m, mi.inv_m);
        }
    };
    auto mult = [&](int c, int l0, const v4i &w0, const v4i &w1) OZ2H_INL {
        int v[16];
        double vd[16];
        values(min(16 * c + j, a.nu - 1) + a.npair, w0, w1, v);
#pragma unroll
        for (int t = 0; t < 16; ++t) vd[t] = (double)v[t];
        fmas(c, l0, vd);
    };
    // the first chunks hold the pairs (and, in the last of them, single moduli as pairs with
    // factors 1 and 0); their planes load where they are used
    auto mult_pairs = [&](int c, int l0) OZ2H_INL {
        const int u = min(16 * c + j, a.nu - 1);
        const bool pair = u < a.npair;
        const int la = pair ? 2 * u : u + a.npair, lb = pair ? la + 1 : la;
        OZ2H_G(ModInfo) *mi = (OZ2H_G(ModInfo) *)a.mi;
        const int ka = pair ? (int)mi[lb].m : 1, kb = pair ? (int)mi[la].m : 0;
        gv4i *sa = (gv4i *)(a.V + (int64_t)la * a.v_ps + e_row), *sb = (gv4i *)(a.V + (int64_t)lb * a.v_ps + e_row);
        const v4i wa0 = sa[0], wa1 = sa[1], wb0 = sb[0], wb1 = sb[1];
        int va[16], vb[16];
        double vd[16];
        values(la, wa0, wa1, va);
        values(lb, wb0, wb1, vb);
#pragma unroll
        for (int t = 0; t < 16; ++t) vd[t] = (double)(__mul24(va[t], ka) + __mul24(vb[t], kb));
        fmas(c, l0, vd);
    };
    // a stage's constants: thread t moves pairs (t & 15) + 16 i of row t >> 4 (lpad and the
    // stage are multiples of 16, so a row of a stage is a whole number of 16-byte pairs); the
    // next stage's pairs load into registers while the current stage is multiplied
    const int srow = threadIdx.x >> 4, spair = threadIdx.x & 15;
    d2 pre[kCrtRowPairs];
    auto stage_load = [&](int l0) {
        const int nl = min(kCrtRowStage, a.lpad - l0);
        const double *src = gsrc + (size_t)srow * a.lpad + l0;
#pragma unroll
        for (int i = 0; i < kCrtRowPairs; ++i) {
            const int l = 2 * (spair + 16 * i);
            if (l < nl) pre[i] = *(const d2 *)(src + l);
        }
    };
    auto stage_store = [&](int l0) {
        const int nl = min(kCrtRowStage, a.lpad - l0);
        double *dst = Dl + srow * kCrtRowDStride;
#pragma unroll
        for (int i = 0; i < kCrtRowPairs; ++i) {
            const int l = 2 * (spair + 16 * i);
            if (l < nl) *(d2 *)(dst + l) = pre[i];
        }
    };
    v4i aw0, aw1, bw0, bw1;
    stage_load(0);
    const int pch = (a.npair + 15) >> 4;   // at most two: within the first stage
    loadv(min(pch, nch - 1), aw0, aw1);
    for (int l0 = 0; l0 < a.lpad; l0 += kCrtRowStage) {
        const int nl = min(kCrtRowStage, a.lpad - l0);
        __syncthreads();   // the previous stage has been read by every wave
        stage_store(l0);
        if (l0 + kCrtRowStage < a.lpad) stage_load(l0 + kCrtRowStage);
        __syncthreads();
        const int c1 = (l0 + nl) >> 4;
        int c = l0 >> 4;
        for (; c < pch; ++c) mult_pairs(c, l0);
        for (; c + 2 <= c1; c += 2) {
            loadv(min(c + 1, nch - 1), bw0, bw1);
            mult(c, l0, aw0, aw1);
            loadv(min(c + 2, nch - 1), aw0, aw1);
            mult(c + 1, l0, bw0, bw1);
        }
        if (c < c1) {
            mult(c, l0, aw0, aw1);
            loadv(min(c + 1, nch - 1), aw0, aw1);
        }
    }
    // two halves of 32 entries: entry 16 q + i of the half's rows gets digit sum j at
    // T[(16 (q & 1) + i) * 17 + j]; lane 32 h + e then carries entry 32 h + e's 16 sums into
    // digits in [0, 2^32) and a carry-out
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        wave_lds_sync();
        if ((q >> 1) == h) {
#pragma unroll
            for (int i = 0; i < 16; ++i) T[(16 * (q & 1) + i) * 17 + j] = acc[i];
        }
        wave_lds_sync();
        if ((lane >> 5) == h) {
            const int el = lane & 31;
            const int64_t e = tile * 64 + lane;
            double cy = 0.0;
            uint32_t dv[16];
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) {
                const double xv = T[el * 17 + jj] + cy;
                cy = floor(xv * 0x1p-32);
                dv[jj] = (uint32_t)(xv - cy * 0x1p32);
            }
            if (live) {
#pragma unroll
                for (int jj = 0; jj < 16; ++jj) a.dig[(int64_t)(16 * dg + jj) * a.estride + e] = dv[jj];
                a.cout[(int64_t)dg * a.estride + e] = (int32_t)cy;
            }
        }
    }
}

// N columns of valid entries per row of ldv: entry e' = i * ldv + j, output (i, j) if j < N.
// beta comes first, from S's top digits: an exact carry pass over the top two digit groups
// (their digit sums and carry-outs) leaves out only the carry into them from the groups
// below, at most one unit at a digit 12 or more places below the top nt, far inside the
// 2^-30 margin of the half-integer test.  One carry pass from the bottom then forms
// c^ = S - beta P digit by digit in binary64 (every term an integer below 2^43: exact) and
// keeps its low nd32 digits in an LDS column, c^ in two's complement (|c^| < P/2, so the
// top digit is sign extension); on the paper's alpha - 1 path the column holds R in [0, 3P).
// STASH: limbs stored together (columns kCrtFinS words apart, 64 without)
template <bool ROUND, bool STASH>
__global__ __launch_bounds__(64) void k_crt_row_finish(CrtArgs a, CrtRowArgs r) {
    extern __shared__ __attribute__((aligned(16))) uint32_t sdig[];
    constexpr int CS = STASH ? kCrtFinS : 64;
    const int tid = threadIdx.x;
    const int64_t ep = (int64_t)blockIdx.x * 64 + tid;
    const int64_t i = ep / r.ldv, jj = ep - i * r.ldv;
    const bool live = ep < r.nent && jj < a.N;
    bool stashed = false;
    if (live) {
        const int nd32 = a.nd32, nt = a.nt;
        uint32_t *col = sdig + tid;   // digit k at col[CS k]
        // groups holding digits below nd32 (at least three: this kernel runs for nd32 > 32)
        const int ng = min(r.ndg, (nd32 + 15) / 16);
        auto ldg = [&](int g, uint32_t (&dv)[16], int32_t &co) {
            const int gc = min(g, ng - 1);
#pragma unroll
            for (int u = 0; u < 16; ++u) dv[u] = r.dig[(int64_t)(16 * gc + u) * r.estride + ep];
            co = gc > 0 ? r.cout[(int64_t)(gc - 1) * r.estride + ep] : 0;
        };
        uint32_t da[16], db[16];
        int32_t ca, cb;

        // S's top nt digits (the highest as a signed digit) as one binary64 value
        ldg(ng - 2, da, ca);
        ldg(ng - 1, db, cb);
        double val = 0.0;
        {
            const int base = 16 * (ng - 2), kb = nd32 - nt;
            uint32_t top[32];
            int64_t cy = ca;
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int64_t x = (int64_t)(u < 16 ? da[u] : db[u - 16]) + (u == 16 ? (int64_t)cb : 0) + cy;
                top[u] = (uint32_t)x;
                cy = x >> 32;
            }
            // Horner from the signed top digit down: the sign-extension digits cancel exactly
#pragma unroll
            for (int u = 31; u >= 0; --u) {
                const int k = base + u;
                if (k == nd32 - 1) val = (double)(int32_t)top[u];
                else if (k >= kb && k < nd32) val = fma(val, 0x1p32, (double)top[u]);
            }
        }
        const double est = val * a.inv_ptop, rr = rint(est);
        const bool slow = fabs(est - rr) > 0.5 - 0x1p-30;
        const double beta = slow ? floor(est) - 1.0 : rr;   // |beta| <= L + 2

        // c^ = S - beta P from the bottom, the next group's digits loading during a group
        typedef const __attribute__((address_space(4))) uint32_t cu32;
        cu32 *Pd = (cu32 *)a.Pd;
        double cy = 0.0;
        auto digit = [&](int k, uint32_t d, double add, uint32_t pk) {
            const double x = fma(-beta, (double)pk, (double)d + add + cy);
            const double hi = floor(x * 0x1p-32);
            col[CS * k] = (uint32_t)fma(-hi, 0x1p32, x);
            cy = hi;
        };
        auto pass = [&](int g, const uint32_t (&dv)[16], int32_t co) {
            if (16 * g + 16 <= nd32) {   // a whole group: its 16 digits of P in one scalar load
                uint32_t pk[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) pk[u] = Pd[16 * g + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) digit(16 * g + u, dv[u], u == 0 ? (double)co : 0.0, pk[u]);
            } else {
                for (int u = 0; u < 16 && 16 * g + u < nd32; ++u)
                    digit(16 * g + u, dv[u], u == 0 ? (double)co : 0.0, Pd[16 * g + u]);
            }
        };
        ldg(0, da, ca);
        int g = 0;
        for (; g + 2 <= ng; g += 2) {
            ldg(g + 1, db, cb);
            pass(g, da, ca);
            ldg(g + 2, da, ca);
            pass(g + 1, db, cb);
        }
        if (g < ng) pass(g, da, ca);
        const int64_t sgn = !slow && (int32_t)col[CS * (nd32 - 1)] < 0 ? -1 : 0;
        stashed = crt_finish<ROUND, STASH>(a, i, jj, col, CS, slow, sgn);
    }
    if constexpr (STASH) store_limbs(a, sdig, stashed, i * a.ldc + jj);
}

// planes [G][R][C] (int8, row stride ldi) -> [G][Co][Ro] (row stride Ro), zero where
// the source row is out of range.  A block moves a 128 x 128 byte tile.  Thread t loads the
// 16-byte column chunk t % 8 of source rows 4 (t / 8) .. + 3 (four loads in flight), turns
// each 4 x 4 byte block into four dwords (one source column, four source rows each) and
// writes them to an LDS tile of output rows; the 16-byte chunks of an output row are stored
// XOR-swizzled by its column chunk, so that a dword write instruction touches 32 banks
// rather than 8.  Then 8 consecutive threads read one output row's eight chunks and store
// them as one 128-byte segment.  Requires ldi to be a multiple of 16 with C <= ldi (a chunk
// that starts below C stays in its row; its bytes past C, the planes' zero padding, land in
// output rows >= C) and Ro, Co multiples of 128 (the residue planes are padded to 128 and
// the GEMM tiles to 128 or 256).
__global__ __launch_bounds__(256) void k_plane_transpose(const int8_t *__restrict__ in, int64_t R,
                                                         int64_t C, int64_t ldi, int64_t ips,
                                                         int8_t *__restrict__ out, int64_t Ro,
                                                         int64_t Co, int64_t ops) {
    __shared__ __attribute__((aligned(16))) uint32_t tile[128 * 32];   // [output row][32 dwords]
    const int64_t g = blockIdx.z;
    const int64_t c0 = (int64_t)blockIdx.x * 128, r0 = (int64_t)blockIdx.y * 128;   // source tile
    const int t = threadIdx.x;
    {
        const int cc = t & 7, rg = t >> 3;   // column chunk, group of four source rows
        const int64_t c = c0 + 16 * cc;
        v4i x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t r = r0 + 4 * rg + i;
            x[i] = v4i{0, 0, 0, 0};
            if (r < R && c < C) x[i] = *(const v4i *)(in + g * ips + r * ldi + c);
        }
        // dword of output row o = 16 cc + 4 q + j: byte j of each of the four rows' word q
        const int pc = 4 * ((rg >> 2) ^ cc) + (rg & 3);   // swizzled dword position in the row
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t d = (((uint32_t)x[0][q] >> (8 * j)) & 0xFFu) |
                                   ((((uint32_t)x[1][q] >> (8 * j)) & 0xFFu) << 8) |
                                   ((((uint32_t)x[2][q] >> (8 * j)) & 0xFFu) << 16) |
                                   ((((uint32_t)x[3][q] >> (8 * j)) & 0xFFu) << 24);
                tile[(16 * cc + 4 * q + j) * 32 + pc] = d;
            }
    }
    __syncthreads();
    const int qc = t & 7;   // logical chunk: output columns r0 + 16 qc .. + 15
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = (t >> 3) + 32 * i;   // output row c0 + o
        const v4i v = *(const v4i *)&tile[o * 32 + 4 * (qc ^ ((o >> 4) & 7))];
        *(v4i *)(out + g * ops + (c0 + o) * Ro + r0 + 16 * qc) = v;
    }
}

// zero output for K = 0
__global__ void k_zero_out(int8_t *__restrict__ s, int32_t *__restrict__ e,
                           uint64_t *__restrict__ limbs, int64_t M, int64_t N, int64_t ld, int nl) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= M * N) return;
    const int64_t i = idx / N, j = idx - i * N;
    const int64_t o = i * ld + j;
    s[o] = 0;
    e[o] = 0;
    for (int l = 0; l < nl; ++l) limbs[o * nl + l] = 0;
}

// ---------------------------------------------------------------- float64 carriers
// Element (r, c) of a carrier is CW = 2 + 2 nl doubles: [0] the value truncated
// to 53 bits, [1] 4 exp + sign + 1, [2 + 2l], [3 + 2l] the 32-bit halves of limb l.
// Every slot but [0] is an exactly representable integer, so the encoding
// survives any copy, view or device move of a floating tensor.

// the CW slots of element src of X into o
__device__ __forceinline__ void carrier_encode(int p, int nl, const int8_t *__restrict__ sign,
                                               const int32_t *__restrict__ exps,
                                               const uint64_t *__restrict__ limbs, int64_t src,
                                               double *o) {
    const int s = sign[src];
    const int e = s ? exps[src] : 0;
    const int top = p - 64 * (nl - 1);   // bits of the top limb, 1..64
    uint64_t hi = 0;                     // the 64 (or p, if fewer) leading bits of mant
    for (int l = 0; l < nl; ++l) {
        uint64_t x = s ? limbs[src * nl + l] : 0;
        if (l == nl - 1 && top < 64) x &= (~0ull) >> (64 - top);
        o[2 + 2 * l] = (double)(uint32_t)x;
        o[3 + 2 * l] = (double)(uint32_t)(x >> 32);
        if (l == nl - 1) {
            if (top == 64 || nl == 1) hi = x;
            else hi = (x << (64 - top)) | (limbs[src * nl + l - 1] >> top);
        }
    }
    const int hb = p < 64 ? p : 64;      // bits held in `hi`
    double approx = 0.0;
    if (s) {
        const uint64_t m53 = hb > 53 ? hi >> (hb - 53) : hi;
        const int mb = hb > 53 ? 53 : hb;
        approx = ldexp((double)m53, e - mb);
        if (s < 0) approx = -approx;
    }
    o[0] = approx;
    o[1] = 4.0 * (double)e + (double)(s + 1);
}

// STAGED: a block's elements are consecutive, so its part of the carrier is one contiguous
// run of blockDim.x * CW doubles; each thread writes its CW slots into LDS and the block then
// copies the run out with consecutive lanes on consecutive doubles (one thread per element
// writing its own slots directly puts lanes CW * 8 bytes apart).  Dynamic LDS:
// blockDim.x * CW doubles.
template <bool STAGED>
__global__ __launch_bounds__(256) void k_carrier_pack(int64_t rows, int64_t cols, int p, int nl,
                                                      const int8_t *__restrict__ sign,
                                                      const int32_t *__restrict__ exps,
                                                      const uint64_t *__restrict__ limbs,
                                                      int64_t ld, double *__restrict__ car) {
    extern __shared__ __attribute__((aligned(16))) double cstage[];
    const int64_t n = rows * cols, e0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t idx = e0 + threadIdx.x;
    const int cw = 2 + 2 * nl;
    if (idx < n) {
        const int64_t r = idx / cols, c = idx - r * cols;
        carrier_encode(p, nl, sign, exps, limbs, r * ld + c,
                       STAGED ? cstage + (size_t)threadIdx.x * cw : car + idx * cw);
    }
    if constexpr (STAGED) {
        __syncthreads();
        const int64_t total = (n - e0 < (int64_t)blockDim.x ? n - e0 : (int64_t)blockDim.x) * cw;
        double *dst = car + e0 * cw;
        for (int64_t i = threadIdx.x; i < total; i += blockDim.x) dst[i] = cstage[i];
    }
}

// bad (nullable) gets a 1 if any element is not a valid encoding; such an
// element is written as zero
// STAGED: the block first copies its contiguous run of the carrier into LDS (consecutive
// lanes on consecutive doubles), then each thread decodes its element from there.
template <bool STAGED>
__global__ __launch_bounds__(256) void k_carrier_unpack(int64_t rows, int64_t cols, int p, int nl,
                                                        const double *__restrict__ car,
                                                        int8_t *__restrict__ sign,
                                                        int32_t *__restrict__ exps,
                                                        uint64_t *__restrict__ limbs, int64_t ld,
                                                        int32_t *bad) {
    extern __shared__ __attribute__((aligned(16))) double cstage[];
    const int64_t n = rows * cols, e0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t idx = e0 + threadIdx.x;
    const int cw = 2 + 2 * nl;
    if constexpr (STAGED) {
        const int64_t total = (n - e0 < (int64_t)blockDim.x ? n - e0 : (int64_t)blockDim.x) * cw;
        const double *src = car + e0 * cw;
        for (int64_t i = threadIdx.x; i < total; i += blockDim.x) cstage[i] = src[i];
        __syncthreads();
    }
    // STAGED with ld == cols: the block's limbs are one contiguous run too; each thread puts
    // its limbs over its own (already read) LDS slots and the block stores the run together
    const bool dense = STAGED && ld == cols;
    if (!dense && idx >= n) return;
    if (idx < n) {
        const int64_t r = idx / cols, c = idx - r * cols, dst = r * ld + c;
        double *in = STAGED ? cstage + (size_t)threadIdx.x * cw : const_cast<double *>(car) + idx * cw;
        const double code = in[1];
        bool ok = code == rint(code) && fabs(code) < 0x1p33;
        const double q = floor(code * 0.25);
        const int s = ok ? (int)(code - 4.0 * q) - 1 : 0;
        const int64_t e = (int64_t)q;
        ok = ok && s <= 1 && e >= INT_MIN && e <= INT_MAX;
        const int top = p - 64 * (nl - 1);
        for (int l = 0; l < nl; ++l) {
            const double lo = in[2 + 2 * l], hi = in[3 + 2 * l];
            ok = ok && lo == rint(lo) && hi == rint(hi) && lo >= 0.0 && hi >= 0.0 &&
                 lo < 0x1p32 && hi < 0x1p32;
        }
        uint64_t topl = 0, any = 0;
        // dense: limb l goes over LDS slot l, kept as a double bit pattern (slot l was read
        // before: limb l reads slots 2 + 2l and 3 + 2l)
        auto put = [&](int l, uint64_t v) {
            if (dense) in[l] = __builtin_bit_cast(double, v);
            else limbs[dst * nl + l] = v;
        };
        for (int l = 0; l < nl; ++l) {
            const uint64_t x = ok ? ((uint64_t)(uint32_t)in[2 + 2 * l] |
                                     ((uint64_t)(uint32_t)in[3 + 2 * l] << 32)) : 0;
            if (l == nl - 1) topl = x;
            any |= x;
            put(l, s && ok ? x : 0);
        }
        // a nonzero value must be normalised (bit p - 1 set, nothing above it), a
        // zero must have zero limbs
        if (ok) ok = s ? (topl >> (top - 1)) == 1 : any == 0;
        if (!ok) {
            for (int l = 0; l < nl; ++l) put(l, 0);
            if (bad) *bad = 1;
        }
        sign[dst] = ok ? (int8_t)s : 0;
        exps[dst] = ok && s ? (int32_t)e : 0;
    }
    if (dense) {
        __syncthreads();
        const int64_t cnt = n - e0 < (int64_t)blockDim.x ? n - e0 : (int64_t)blockDim.x;
        uint64_t *out = limbs + e0 * nl;
        const int bd = blockDim.x, dt = bd / nl, dw = bd % nl;   // flat f = t nl + l advances by bd
        int t = (int)threadIdx.x / nl, l = (int)threadIdx.x - t * nl;
        for (int64_t f = threadIdx.x; f < cnt * nl; f += bd) {
            out[f] = __builtin_bit_cast(uint64_t, cstage[(size_t)t * cw + l]);
            t += dt;
            l += dw;
            if (l >= nl) {
                l -= nl;
                ++t;
            }
        }
    }
}

}  // namespace oz2h
