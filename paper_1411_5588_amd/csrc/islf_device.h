// Device code shared by the kernel files of libislf: Philox4x32-10, lattice
// accesses, the per-replica view, and the single-column / single-word updates
// that work on any row of a replica.  Not part of the public ABI.
#pragma once

#include <type_traits>

#include "islf_internal.h"

#pragma clang fp contract(off)

namespace islf {

// a ^ b ^ c in one gfx950 three-input bitwise op (truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies
// whose halves are xored into the other counter words with the round key; the
// key advances by the Weyl constants after each round.
// ---------------------------------------------------------------------------
// The first round's product of c0 = base + OFF is formed as one multiply-add,
// M0 base + M0 OFF, which is M0 c0 whenever base + OFF < 2^32 (every counter
// of a valid site: the group index is checked against 2^32 when a replica is
// created); OFF = 0 is the plain generator.
template <uint32_t OFF = 0>
__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         uint32_t k0, uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t pa = (uint64_t)0xD2511F53u * c0 + (r == 0 ? (uint64_t)0xD2511F53u * OFF : 0ull);
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

constexpr uint64_t kOnes8 = 0x0101010101010101ull;

__device__ __forceinline__ uint32_t bytesum64(uint64_t v)
{
    return __builtin_amdgcn_sad_u8((uint32_t)v, 0u, __builtin_amdgcn_sad_u8((uint32_t)(v >> 32), 0u, 0u));
}

struct Acc {
    int dB, dM, dM1, dMn;
};

// Per-replica parameters as the update loop uses them: loaded once per
// replica change from the descriptor table, uniform across the workgroup (the
// compiler keeps them in scalar registers).
struct RepView {
    uint8_t *spins;
    long long *acc;
    int Lx, Ly, Lz, C, Wq, K;
    uint32_t Hp, RB;        // int8 sublattice row and row bytes
    int seam_reflect, seam_invert;
    uint32_t key0, key1, replica, t;
    int tj, ty, mx;          // marching tile (tj = 0: linear tiles)
    int my_ty, my_tj;        // this thread's row and column inside a box tile
    bool never;              // some move can never be accepted (thr == 0)
    bool sym;                // bulk thresholds by aligned neighbours alone (RepDesc::sym)
};

__device__ __forceinline__ RepView load_view(const RepDesc *__restrict__ descs, const RepState *__restrict__ st,
                                             int rep, uint32_t t_offset)
{
    const RepDesc &d = descs[rep];
    RepView v;
    v.spins = d.spins;
    v.acc = d.acc;
    v.Lx = d.Lx; v.Ly = d.Ly; v.Lz = d.Lz; v.C = d.C; v.Wq = d.Wq; v.K = d.K;
    v.Hp = (uint32_t)d.Hp;
    v.RB = (uint32_t)d.RB;
    v.seam_reflect = d.seam_reflect;
    v.seam_invert = d.seam_invert;
    v.key0 = d.key0; v.key1 = d.key1; v.replica = d.replica;
    v.t = st[rep].t + t_offset;
    v.tj = d.i8_tj;
    v.ty = d.i8_ty;
    v.mx = d.i8_mx;
    v.my_ty = v.tj > 0 ? (int)threadIdx.x / v.tj : 0;
    v.my_tj = (int)threadIdx.x - v.my_ty * v.tj;
    v.never = d.never_mask != 0;
    v.sym = d.sym != 0;
    return v;
}

// ---------------------------------------------------------------------------
// int8 format: update the current-phase sites of one 8-byte column.
// Byte offsets are 32-bit (a replica's spin array is below 4 GiB).
// ---------------------------------------------------------------------------
// Loads through the global address space (the spin arrays always live in
// device memory), addressed as a uniform base plus a 32-bit offset.
typedef __attribute__((address_space(1))) const uint8_t gcu8;
typedef __attribute__((address_space(1))) const uint32_t gcu32;
typedef __attribute__((address_space(1))) const uint64_t gcu64;
typedef __attribute__((address_space(1))) uint64_t gu64;
typedef __attribute__((address_space(1))) uint32_t gu32;
typedef __attribute__((address_space(1))) uint8_t gu8;

// Lattice accesses.  COH (the persistent kernel) makes them relaxed
// device-scope atomics, which the compiler marks device-coherent: stores
// write through the XCD's L2 and loads do not use a stale copy in it, so a
// block on any XCD sees another's stores once they are complete, and the
// grid barrier needs no L2 write-back or invalidate (see grid_barrier).
template <bool COH>
__device__ __forceinline__ uint64_t ld64(const uint8_t *base, uint32_t off)
{
    gu64 *p = (gu64 *)((gcu8 *)base + off);
    if (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}
template <bool COH>
__device__ __forceinline__ uint32_t ld32(const uint8_t *base, uint32_t off)
{
    gu32 *p = (gu32 *)((gcu8 *)base + off);
    if (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}
template <bool COH>
__device__ __forceinline__ uint64_t ld8(const uint8_t *base, uint32_t off)
{
    gu8 *p = (gu8 *)((gcu8 *)base + off);
    if (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}
template <bool COH>
__device__ __forceinline__ void st64(uint8_t *base, uint32_t off, uint64_t v)
{
    gu64 *p = (gu64 *)((gcu8 *)base + off);
    if (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
template <bool COH>
__device__ __forceinline__ void st32(uint8_t *base, uint32_t off, uint32_t v)
{
    gu32 *p = (gu32 *)((gcu8 *)base + off);
    if (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// Bytes [0, nv) of an 8-byte column set.
__device__ __forceinline__ uint64_t byte_mask(int nv)
{
    return nv >= 8 ? ~0ull : ((1ull << (8 * nv)) - 1ull);
}

// One 8-byte column k of the phase's sublattice of row (x, y): 8 sites
// z = 2i + q, i = 8k .. 8k+7 (the last column of a row may hold fewer).
// Philox call c (counter g + 2c) draws for sites i = 8k + 4c .. 8k + 4c + 3
// (their 8-site group is i >> 2 = 2k + c, word i & 3).  Used by the
// seam-slab stages: any row, the y seam, 64-bit thresholds of any class.
template <bool COH>
__device__ __forceinline__ void i8_update_col(const RepView &v, int x, int y, int k, int parity,
                                              const uint64_t *sthr, Acc &a)
{
    const int Lx = v.Lx, Ly = v.Ly, K = v.K;
    const int Lzh = v.Lz >> 1;
    const uint32_t RB = v.RB, Hp = v.Hp;
    uint8_t *sp = v.spins;
    const int q = (parity + x + y) & 1;
    const uint32_t row = (uint32_t)x * (uint32_t)Ly + (uint32_t)y;
    const uint32_t rowoff = row * RB;
    const uint32_t co = 8u * (uint32_t)k;
    const uint32_t qo = (uint32_t)q * Hp + co;            // column offset inside a row
    const uint32_t own = rowoff + qo;
    const uint32_t oth = rowoff + (uint32_t)(q ^ 1) * Hp + co;
    const bool last = (k == K - 1);
    const int nv = last ? Lzh - 8 * (K - 1) : 8;

    // z neighbours from the other sublattice O of the row: q = 0 (z = 2i):
    // z+1 is odd index i, z-1 odd index i-1; q = 1 (z = 2i+1): z-1 is even
    // index i, z+1 even index i+1 (wrapping at the row's ends)
    const uint64_t O = ld64<COH>(sp, oth);
    uint64_t Z;
    if (q == 0) {
        const uint32_t eo = k > 0 ? oth - 1u : rowoff + Hp + (uint32_t)(Lzh - 1);
        Z = (O << 8) | ld8<COH>(sp, eo);
    } else {
        const uint32_t eo = last ? rowoff : oth + 8u;
        Z = (O >> 8) | (ld8<COH>(sp, eo) << (8 * (nv - 1)));
    }
    // y neighbours (the seam remaps x and inverts when eps = -1; a padding
    // byte may turn to 1 there, it is never a site) and x neighbours (a free
    // surface contributes 0)
    const uint32_t xs = v.seam_reflect ? (uint32_t)(Lx - 1 - x) : (uint32_t)x;
    const uint64_t seam_mask = v.seam_invert ? kOnes8 : 0ull;
    const bool ytop = (y == Ly - 1), ybot = (y == 0);
    const uint32_t rp = ytop ? xs * (uint32_t)Ly : row + 1u;
    const uint32_t rm = ybot ? xs * (uint32_t)Ly + (uint32_t)(Ly - 1) : row - 1u;
    const uint64_t Yp = ld64<COH>(sp, rp * RB + qo) ^ (ytop ? seam_mask : 0ull);
    const uint64_t Ym = ld64<COH>(sp, rm * RB + qo) ^ (ybot ? seam_mask : 0ull);
    const uint32_t xstride = (uint32_t)Ly * RB;
    const uint64_t Xm = x > 0 ? ld64<COH>(sp, own - xstride) : 0ull;
    const uint64_t Xp = x < Lx - 1 ? ld64<COH>(sp, own + xstride) : 0ull;
    const uint64_t S = ld64<COH>(sp, own);

    const uint64_t cnt = ((O + Z) + (Yp + Ym)) + (Xm + Xp);
    const int cls = (x == 0 ? 1 : 0) + (x == Lx - 1 ? 2 : 0);
    const int kn = 6 - (x == 0) - (x == Lx - 1);
    const uint64_t idxw = cnt + (S << 3);   // per byte: 8*u + count

    const uint32_t g = ((row * (uint32_t)v.C + 2u * (uint32_t)k) << 1) | (uint32_t)q;
    uint32_t r0[4], r1[4];
    philox10<0u>(g, v.t, v.replica, 0u, v.key0, v.key1, r0);
    philox10<2u>(g, v.t, v.replica, 0u, v.key0, v.key1, r1);

    const uint64_t *tc = sthr + cls * kThrPerClass;
    uint64_t flip = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t e = (uint32_t)(idxw >> (8 * b)) & 0xFFu;
        const uint32_t u = b < 4 ? r0[b] : r1[b - 4];
        flip |= (uint64_t)((uint64_t)u < tc[e & 0xF]) << (8 * b);
    }
    flip &= byte_mask(nv);
    st64<COH>(sp, own, S ^ flip);

    // dB = -2 sum_f s n with s = 2u-1, n = 2 cnt - k;  dM = sum_f (2 - 4u)
    const uint64_t fu = flip & S;
    const int nf = __popcll(flip), nfu = __popcll(fu);
    const uint64_t fm = (flip << 8) - flip, fum = (fu << 8) - fu;
    const int Sf = (int)bytesum64(cnt & fm), Sfu = (int)bytesum64(cnt & fum);
    a.dB += -2 * (4 * Sfu - 2 * kn * nfu - 2 * Sf + kn * nf);
    const int dm = 2 * nf - 4 * nfu;
    a.dM += dm;
    if (x == 0) a.dM1 += dm;
    if (x == Lx - 1) a.dMn += dm;
}

// ---------------------------------------------------------------------------
// bit-packed format: update one 32-bit word (32 same-phase sites).
// Row layout: words [0, Wq) hold even z (z = 2i), words [Wq, 2Wq) odd z.
// ---------------------------------------------------------------------------
template <bool COH>
__device__ __forceinline__ void bp_update_word(const RepView &v, int x, int y, int w, int parity,
                                               const uint64_t *sthr, Acc &a)
{
    const int Lx = v.Lx, Ly = v.Ly, C = v.C, Wq = v.Wq;
    const int nbits = v.Lz >> 1;
    const uint32_t RW = 2u * (uint32_t)Wq;
    const uint32_t row = (uint32_t)x * (uint32_t)Ly + (uint32_t)y;
    auto word = [&](uint32_t i) { return ld32<COH>(v.spins, 4u * i); };
    const int q = (parity + x + y) & 1;
    const uint32_t own = row * RW + (uint32_t)(q * Wq);
    const uint32_t oth = row * RW + (uint32_t)((q ^ 1) * Wq);
    const int nb_here = min(32, nbits - 32 * w);
    const uint32_t vmask = nb_here >= 32 ? 0xFFFFFFFFu : ((1u << nb_here) - 1u);

    const uint32_t S = word(own + w);
    uint32_t zm, zp;
    if (q == 0) {
        // z = 2i: z+1 is odd index i, z-1 is odd index i-1
        const uint32_t O = word(oth + w);
        zp = O;
        const uint32_t carry = (w > 0) ? (word(oth + w - 1) >> 31)
                                       : (word(oth + ((nbits - 1) >> 5)) >> ((nbits - 1) & 31)) & 1u;
        zm = (O << 1) | carry;
    } else {
        // z = 2i+1: z-1 is even index i, z+1 is even index i+1
        const uint32_t E = word(oth + w);
        zm = E;
        const bool lastw = (w == Wq - 1);
        const uint32_t inb = word(oth + (lastw ? 0 : w + 1)) & 1u;
        zp = (E >> 1) | (inb << (lastw ? (nb_here - 1) : 31));
    }

    const uint32_t xs = v.seam_reflect ? (uint32_t)(Lx - 1 - x) : (uint32_t)x;
    const uint32_t seam_mask = v.seam_invert ? 0xFFFFFFFFu : 0u;
    const uint32_t qo = (uint32_t)(q * Wq + w);
    uint32_t yp, ym;
    if (y < Ly - 1) yp = word((row + 1) * RW + qo);
    else yp = word((xs * (uint32_t)Ly) * RW + qo) ^ seam_mask;
    if (y > 0) ym = word((row - 1) * RW + qo);
    else ym = word((xs * (uint32_t)Ly + (uint32_t)(Ly - 1)) * RW + qo) ^ seam_mask;
    const uint32_t xstride = (uint32_t)Ly * RW;
    const uint32_t xm = (x > 0) ? word(own + w - xstride) : 0u;
    const uint32_t xp = (x < Lx - 1) ? word(own + w + xstride) : 0u;

    // bit-sliced count of the six neighbour bits
    const uint32_t s1 = zm ^ zp ^ ym, c1 = (zm & zp) | (ym & (zm ^ zp));
    const uint32_t s2 = yp ^ xm ^ xp, c2 = (yp & xm) | (xp & (yp ^ xm));
    const uint32_t b0 = s1 ^ s2, k0 = s1 & s2;
    const uint32_t b1 = c1 ^ c2 ^ k0, b2 = (c1 & c2) | (k0 & (c1 ^ c2));

    const int cls = (x == 0 ? 1 : 0) + (x == Lx - 1 ? 2 : 0);
    const int k = 6 - (x == 0) - (x == Lx - 1);
    const uint64_t *tc = sthr + cls * kThrPerClass;
    const uint32_t gbase = row * (uint32_t)C + 8u * (uint32_t)w;
    uint32_t F = 0;
    // not unrolled: this path is a small share of the work and must not raise
    // the register count of the kernels it is inlined into
#pragma unroll 1
    for (int g4 = 0; g4 < 8; ++g4) {
        uint32_t rnd[4];
        philox10(((gbase + g4) << 1) | (uint32_t)q, v.t, v.replica, 0u, v.key0, v.key1, rnd);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int b = 4 * g4 + l;
            const uint32_t e = ((S >> b) & 1u) << 3 | ((b2 >> b) & 1u) << 2 | ((b1 >> b) & 1u) << 1 |
                               ((b0 >> b) & 1u);
            F |= (uint32_t)((uint64_t)rnd[l] < tc[e]) << b;
        }
    }
    F &= vmask;
    st32<COH>(v.spins, 4u * (own + w), S ^ F);

    const uint32_t FU = F & S;
    const int nf = __popc(F), nfu = __popc(FU);
    const int Sf = __popc(F & b0) + 2 * __popc(F & b1) + 4 * __popc(F & b2);
    const int Sfu = __popc(FU & b0) + 2 * __popc(FU & b1) + 4 * __popc(FU & b2);
    a.dB += -2 * (4 * Sfu - 2 * k * nfu - 2 * Sf + k * nf);
    const int dm = 2 * nf - 4 * nfu;
    a.dM += dm;
    if (x == 0) a.dM1 += dm;
    if (x == Lx - 1) a.dMn += dm;
}

// Shifts the reject bits (thr - 1 < r) of eight sites into two words:
// lo = 2 lo + reject(site of t[l].x, r0[l]) and hi likewise with t[l].y and
// r1[l], for l = 3, 2, 1, 0 (FIRST: lo and hi start from 0).  Each compare
// writes a carry register that an add-with-carry (x + x + carry) consumes:
// two instructions per site.  Three carry registers rotate so that each is
// read two or more instructions after the compare writes it, the wait gfx950
// needs between a VALU write of a scalar register and a VALU read of it.
// VALU instructions only.
#define ISLF_REJECT8_ASM(LO0, HI0)                                                                                     \
    "v_cmp_lt_u32_e64 %[a], %[t3x], %[r03]\n\t"                                                                         \
    "v_cmp_lt_u32_e64 %[b], %[t3y], %[r13]\n\t"                                                                         \
    "v_cmp_lt_u32_e32 vcc, %[t2x], %[r02]\n\t"                                                                          \
    "v_addc_co_u32_e64 %[lo], %[a], " LO0 ", " LO0 ", %[a]\n\t"                                                         \
    "v_addc_co_u32_e64 %[hi], %[b], " HI0 ", " HI0 ", %[b]\n\t"                                                         \
    "v_cmp_lt_u32_e64 %[a], %[t2y], %[r12]\n\t"                                                                         \
    "v_addc_co_u32_e32 %[lo], vcc, %[lo], %[lo], vcc\n\t"                                                               \
    "v_cmp_lt_u32_e64 %[b], %[t1x], %[r01]\n\t"                                                                         \
    "v_cmp_lt_u32_e32 vcc, %[t1y], %[r11]\n\t"                                                                          \
    "v_addc_co_u32_e64 %[hi], %[a], %[hi], %[hi], %[a]\n\t"                                                             \
    "v_addc_co_u32_e64 %[lo], %[b], %[lo], %[lo], %[b]\n\t"                                                             \
    "v_cmp_lt_u32_e64 %[a], %[t0x], %[r00]\n\t"                                                                         \
    "v_addc_co_u32_e32 %[hi], vcc, %[hi], %[hi], vcc\n\t"                                                               \
    "v_cmp_lt_u32_e64 %[b], %[t0y], %[r10]\n\t"                                                                         \
    "v_addc_co_u32_e64 %[lo], %[a], %[lo], %[lo], %[a]\n\t"                                                             \
    "s_nop 0\n\t"                                                                                                       \
    "v_addc_co_u32_e64 %[hi], %[b], %[hi], %[hi], %[b]"
#define ISLF_REJECT8_IN                                                                                                \
    [t3x] "v"(t[3].x), [t3y] "v"(t[3].y), [t2x] "v"(t[2].x), [t2y] "v"(t[2].y), [t1x] "v"(t[1].x),                   \
        [t1y] "v"(t[1].y), [t0x] "v"(t[0].x), [t0y] "v"(t[0].y), [r03] "v"(r0[3]), [r13] "v"(r1[3]),                  \
        [r02] "v"(r0[2]), [r12] "v"(r1[2]), [r01] "v"(r0[1]), [r11] "v"(r1[1]), [r00] "v"(r0[0]), [r10] "v"(r1[0])

template <bool FIRST>
__device__ __forceinline__ void reject_bits8(uint32_t &lo, uint32_t &hi, const uint2 t[4], const uint32_t r0[4],
                                             const uint32_t r1[4])
{
    uint64_t ca, cb;
    if (FIRST)
        asm(ISLF_REJECT8_ASM("0", "0")
            : [lo] "=&v"(lo), [hi] "=&v"(hi), [a] "=&s"(ca), [b] "=&s"(cb)
            : ISLF_REJECT8_IN
            : "vcc");
    else
        asm(ISLF_REJECT8_ASM("%[lo]", "%[hi]")
            : [lo] "+v"(lo), [hi] "+v"(hi), [a] "=&s"(ca), [b] "=&s"(cb)
            : ISLF_REJECT8_IN
            : "vcc");
}
#undef ISLF_REJECT8_ASM
#undef ISLF_REJECT8_IN

// Accept bits of the 32 sites of one word, thresholds read from a class's
// pair table (see Tables) for the neighbouring sites (2m, 2m+1).  Byte m of w[k]
// interleaves the index bits e = 8u + cnt of sites 8m + 2k and 8m + 2k + 1:
// its 2-bit fields are bits (2k, 2k+1) of byte m of the planes b0, b1, b2
// and S, placed by shifts and bitfield inserts (the four fields cover every
// bit of a byte).  Philox call c (counter gq + 2c) draws for sites
// 4c .. 4c+3.
template <class KEY>
__device__ __forceinline__ uint32_t bp_flips_pairs(uint32_t S, uint32_t b2, uint32_t b1, uint32_t b0, uint32_t gq,
                                                   const KEY &v, const uint2 *pair)
{
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t acc = b0 >> (2 * k);
        acc = __builtin_amdgcn_bitop3_b32(0x0C0C0C0Cu, k == 0 ? b1 << 2 : b1 >> (2 * k - 2), acc, 0xCA);
        acc = __builtin_amdgcn_bitop3_b32(0x30303030u, k <= 2 ? b2 << (4 - 2 * k) : b2 >> 2, acc, 0xCA);
        w[k] = __builtin_amdgcn_bitop3_b32(0xC0C0C0C0u, S << (6 - 2 * k), acc, 0xCA);
    }
    // sites are visited from the top down (g = 3 .. 0, l = 3 .. 0), so that
    // the shifted-in reject bits end at their site's position; the
    // thresholds are read before the draws so that the LDS latency overlaps
    // Philox
    uint32_t rlo, rhi;
    auto group = [&](auto gc) {
        constexpr int g = decltype(gc)::value;
        // sites 4g .. 4g+3: byte g/2 of w[2(g&1)] and w[2(g&1)+1]; sites
        // 4g+16 .. 4g+19: byte 2 + g/2 of the same words
        constexpr int k = 2 * (g & 1), lo = 8 * (g >> 1), hi = lo + 16;
        const uint2 l0 = pair[(w[k] >> lo) & 0xFFu], l1 = pair[(w[k + 1] >> lo) & 0xFFu];
        const uint2 h0 = pair[(w[k] >> hi) & 0xFFu], h1 = pair[(w[k + 1] >> hi) & 0xFFu];
        // t[l]: thresholds of site 4g+l (x) and 4g+16+l (y)
        const uint2 t[4] = {make_uint2(l0.x, h0.x), make_uint2(l0.y, h0.y), make_uint2(l1.x, h1.x),
                            make_uint2(l1.y, h1.y)};
        uint32_t r0[4], r1[4];
        philox10<2u * g>(gq, v.t, v.replica, 0u, v.key0, v.key1, r0);
        philox10<2u * (g + 4)>(gq, v.t, v.replica, 0u, v.key0, v.key1, r1);
        reject_bits8<g == 3>(rlo, rhi, t, r0, r1);
    };
    group(std::integral_constant<int, 3>{});
    group(std::integral_constant<int, 2>{});
    group(std::integral_constant<int, 1>{});
    group(std::integral_constant<int, 0>{});
    return ~(rlo | (rhi << 16));
}

// Thresholds of four neighbouring sites by the number of their aligned
// neighbours (RepDesc::thr_q): entry k, low nibble the sites' low code bits,
// high nibble their high ones, code 0 for at most three aligned neighbours
// and 1, 2, 3 for four, five, six.  Entry k of the 256-entry table.
__device__ __forceinline__ uint4 quad_entry(const RepDesc &d, int k)
{
    auto thr = [&](int i) { return d.thr_q[((k >> i) & 1) | ((k >> (i + 3)) & 2)]; };
    return make_uint4(thr(0), thr(1), thr(2), thr(3));
}

// Table indices of a word's sites: byte m of w[0] for sites 8m .. 8m+3, of
// w[1] for sites 8m+4 .. 8m+7.  A site with c up neighbours has c of them
// aligned if it is up and 6 - c if it is down: the code's low bit is set for
// 4 and 6 aligned (b2 equals the spin and b0 = 0), the high bit for 5 and 6.
__device__ __forceinline__ void quad_index(uint32_t S, uint32_t b2, uint32_t b1, uint32_t b0, uint32_t w[2])
{
    const uint32_t lo = __builtin_amdgcn_bitop3_b32(S, b2, b0, 0x41);
    const uint32_t u = __builtin_amdgcn_bitop3_b32(S, b0, b1, 0xE5);   // up: b0 | b1, down: ~b1
    const uint32_t hi = __builtin_amdgcn_bitop3_b32(S, b2, u, 0x82);
    w[0] = __builtin_amdgcn_bitop3_b32(0x0F0F0F0Fu, lo, hi << 4, 0xCA);
    w[1] = __builtin_amdgcn_bitop3_b32(0x0F0F0F0Fu, lo >> 4, hi, 0xCA);
}

// bp_flips_pairs by the four-site table: 15 instead of 44 instructions and
// half the LDS accesses for the 32 thresholds of a word.  The kernels are
// bound by VALU issue; 3 x 160x480x600 bit-packed, 100 sweeps in the batched
// form: 5.98 against 6.18 ms; 64 x 40x120x120 resident: 23.1 against 23.8 us per sweep.
template <class KEY>
__device__ __forceinline__ uint32_t bp_flips_quads(uint32_t S, uint32_t b2, uint32_t b1, uint32_t b0, uint32_t gq,
                                                   const KEY &v, const uint4 *quad)
{
    uint32_t w[2];
    quad_index(S, b2, b1, b0, w);
    uint32_t rlo, rhi;
    auto group = [&](auto gc) {
        constexpr int g = decltype(gc)::value;
        constexpr int lo = 8 * (g >> 1), hi = lo + 16;
        const uint4 a = quad[(w[g & 1] >> lo) & 0xFFu], b = quad[(w[g & 1] >> hi) & 0xFFu];
        const uint2 t[4] = {make_uint2(a.x, b.x), make_uint2(a.y, b.y), make_uint2(a.z, b.z), make_uint2(a.w, b.w)};
        uint32_t r0[4], r1[4];
        philox10<2u * g>(gq, v.t, v.replica, 0u, v.key0, v.key1, r0);
        philox10<2u * (g + 4)>(gq, v.t, v.replica, 0u, v.key0, v.key1, r1);
        reject_bits8<g == 3>(rlo, rhi, t, r0, r1);
    };
    group(std::integral_constant<int, 3>{});
    group(std::integral_constant<int, 2>{});
    group(std::integral_constant<int, 1>{});
    group(std::integral_constant<int, 0>{});
    return ~(rlo | (rhi << 16));
}

}  // namespace islf
