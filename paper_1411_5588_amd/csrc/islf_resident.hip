// Resident form of the sweeps: a launch loads its replicas' spins into LDS,
// one bit per site whatever the stored format, runs all of its sweeps there
// and writes the spins back at the end.  256 CUs x 160 KB of LDS hold 3e8
// sites; between two sweeps nothing travels but the edge rows of the shares.
//
// A replica that fits one workgroup is swept by it alone (barriers inside the
// workgroup only).  A larger one is cut along y and along x (mirrored plane
// pairs) into shares (ResJob), one workgroup each, which exchange the edges of
// their shares after phases 0 and 1 through mailboxes in device memory: every
// 64-bit mailbox word carries 32 spins and the step's epoch and is written and
// polled with relaxed device-scope atomics, so a word's arrival is its own
// flag: no fence and no counter stands between an edge word and its reader.
// Edge rows and planes are updated first in a phase; one wave takes in the
// mail while the others compute the rest.
//  - Two mailbox slots (by phase) are enough: a share writes a word of step
//    k+2 only after it has read its neighbour's step k+1, which the neighbour
//    wrote after it had read step k (row 0's words in phases 2 and 3 are other
//    words than the main rows' and follow the same rule).
//  - No word that arrives in a phase is read in it: an update reads its
//    neighbours' sublattice that the phase leaves alone.
//  - The shares of a cluster wait for each other, so they must all be
//    resident.  Each first reports to a counter and waits (bounded) until all
//    of the launch's cluster workgroups have; only then does the first sweep
//    start.  If they do not all arrive, the launch leaves every cluster
//    replica as it was, and the closing kernel sweeps them itself, one
//    workgroup per replica, from device memory (slow, but without waiting
//    for anybody).
//  - Every later wait is bounded too and raises the context's error word.
// A launch is followed by a closing kernel that sums the shares' per-sweep
// changes of the observables into records and advances the sweep counters.
//
// Same Philox words, thresholds and phase order as the launch chain
// (islf_kernels.hip), hence the same chains bit for bit.
#include "islf_device.h"

#pragma clang fp contract(off)

namespace islf {

struct DrawKey {
    uint32_t t, replica, key0, key1;
};

// A column: one word position of one local row, what an update needs of it
// worked out once per launch.  The table is an array per field (consecutive
// lanes read consecutive columns: no bank conflicts).
struct Column {
    uint32_t at, gy;         // byte offset in its plane (even z); Philox counter part y * gy + 16 w
    uint32_t flags;          // RW_*, the z edge shift (see share_gather) from bit 8, the local row from bit 16 on
    uint32_t up, dn;         // steps to the next word round the row, each way
};
constexpr int kColumnFields = 7;   // and the column's parts of its mailbox addresses: y (edge rows), x

// A share as the update loop sees it (uniform over the workgroup): its
// lattice in LDS, planes (slots) of R + 2 local rows of 2 Wq words, followed
// by the plane, column and mail tables.
struct Share {
    int Lx, Wq, rem;         // words of a sublattice row, sites of a partial last word (32: none)
    uint32_t SB, RB, PB;     // LDS bytes of a sublattice row, a local row, a plane
    int R, ls, lr0, y0, np;
    uint32_t inv;            // seam inversion mask
    bool refl, never, sym;
    uint32_t gx, gy;         // Philox counter steps of x and y
    const uint4 *pt;         // plane table: slot * PB, x * gx, mirror slot * PB, flags
    const uint2 *pm;         // mailbox addresses of the planes sent to x neighbours (a second one or ~0)
    const uint32_t *ct;      // column table: whole words by row, then the rows' partial words
    int nc;                  // columns
    const uint32_t *mt;      // mail table: where word k of a slot goes in phase 0 (see mail_target)
};

// Sums over one thread's flips of a sweep (see bp_march).
struct Sums {
    int NF, NFU, A0, A1, A2, KDM, D1, Dn;
};

// Static LDS of the kernels, ahead of the lattice: pair tables (see Tables) of
// the bulk planes, x = 0 and x = Lx-1, all 64-bit thresholds, control words.
struct ResTables {
    uint4 quad[256];         // bulk planes, four sites at once (quad_entry), where RepDesc::sym holds
    uint2 pair[3 * 256];
    uint64_t thr[kThrEntries];
};
struct ResCtl {
    int4 sums[2][kResThreads / 64];   // a sweep's changes by wave, by sweep parity
    unsigned int bad;      // 1 + the first sweep in which a wait ran out, else ~0
    unsigned int state;    // the census' answer; error word at the start
    int ticket[4];         // next chunk of a phase, by phase number mod 4
};

__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Sums of four values over the first N = 16 or 64 lanes, in lane N - 1 (all
// lanes active; lanes a step has no source for add 0).  The four chains fill
// each other's latency.
template <int N>
__device__ __forceinline__ int4 wave_sums(int4 v)
{
    auto step = [&](auto ctrl, auto rows) {
        constexpr int C = decltype(ctrl)::value, R = decltype(rows)::value;
        const int x = __builtin_amdgcn_update_dpp(0, v.x, C, R, 0xF, false);
        const int y = __builtin_amdgcn_update_dpp(0, v.y, C, R, 0xF, false);
        const int z = __builtin_amdgcn_update_dpp(0, v.z, C, R, 0xF, false);
        const int w = __builtin_amdgcn_update_dpp(0, v.w, C, R, 0xF, false);
        v = make_int4(v.x + x, v.y + y, v.z + z, v.w + w);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());   // row_shr:1, :2, :4, :8
    step(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());
    if (N == 64) {
        step(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());   // row_bcast:15 to rows 1 and 3
        step(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());   // row_bcast:31 to rows 2 and 3
    }
    return v;
}

// a where the mask is set, else b
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA);
}

// n / d for n * d < 2^32 with m = ceil(2^32 / d); d = 1 has no 32-bit m
__device__ __forceinline__ uint32_t div_m(uint32_t n, uint32_t d, uint32_t m)
{
    return d == 1 ? n : __umulhi(n, m);
}

__device__ __forceinline__ int share_row_y(const Share &g, int lr)
{
    return (g.lr0 && lr >= g.lr0) ? lr - g.lr0 : g.y0 + lr - 1;
}

__device__ __forceinline__ uint32_t lds32(const char *lat, uint32_t off)
{
    return *(const uint32_t *)(lat + off);
}

// A word of the phase's sublattice: its spins, the bit planes of the
// neighbour counts, its byte offset and the Philox counter of its first group.
struct Word {
    uint32_t S, b0, b1, b2, own, gq;
};

// SEAM: the row may be y = 0 or Ly-1.  WHOLE: all 32 sites of the word exist,
// else it is the partial last word.  All selects are arithmetic (no divergent
// branches, so that the loads are issued together).
template <bool SEAM, bool WHOLE>
__device__ __forceinline__ Word share_gather(const Share &g, const char *lat, const uint4 &pl, const Column &cl,
                                             int phase)
{
    const uint32_t q = (pl.w ^ cl.flags ^ (uint32_t)phase) & 1u, qm = 0u - q;
    const uint32_t at = pl.x + cl.at;
    Word o;
    o.own = at + (qm & g.SB);
    const uint32_t oth = at + (g.SB - (qm & g.SB));
    // the other sublattice one word on: up for odd z, down for even z, round the row's ends
    const uint32_t O = lds32(lat, oth), E = lds32(lat, oth + pick(qm, cl.up, cl.dn));
    o.S = lds32(lat, o.own);
    uint32_t ua = o.own + g.RB, da = o.own - g.RB, um = 0u, dm = 0u;
    if (SEAM) {
        // the seam joins local rows ls (y = Ly-1) and lr0 (y = 0) of planes x and, reflected, Lx-1-x
        const uint32_t sx = o.own - pl.x - (cl.flags >> 16) * g.RB + (g.refl ? pl.z : pl.x);
        const bool su = (cl.flags & RW_LAST) != 0, sd = (cl.flags & RW_ROW0) != 0;
        ua = su ? sx + (uint32_t)g.lr0 * g.RB : ua;
        da = sd ? sx + (uint32_t)g.ls * g.RB : da;
        um = su ? g.inv : 0u;
        dm = sd ? g.inv : 0u;
    }
    const uint32_t yp = lds32(lat, ua) ^ um, ym = lds32(lat, da) ^ dm;
    const uint32_t xm = lds32(lat, o.own - g.PB), xp = lds32(lat, o.own + g.PB);
    // z neighbour beyond the word: the previous word's top site (the row's
    // last site for w = 0), or the next word's first one
    const uint32_t zd = __builtin_amdgcn_alignbit(O, E << ((cl.flags >> 8) & 31u), 31);
    const uint32_t zu = WHOLE ? __builtin_amdgcn_alignbit(E, O, 1) : (O >> 1) | ((E & 1u) << (g.rem - 1));
    const uint32_t Z = pick(qm, zu, zd);
    const uint32_t s1 = xor3(O, Z, ym), c1 = maj3(O, Z, ym);
    const uint32_t s2 = xor3(yp, xm, xp), c2 = maj3(yp, xm, xp);
    const uint32_t k0 = s1 & s2;
    o.b0 = s1 ^ s2;
    o.b1 = xor3(c1, c2, k0);
    o.b2 = maj3(c1, c2, k0);
    o.gq = pl.y + cl.gy + q;
    return o;
}

// Adds the flips F of a word to the sums.
__device__ __forceinline__ void share_sums(const Word &o, uint32_t F, bool surf, bool x0, bool xl, Sums &a)
{
    const uint32_t FU = F & o.S;
    a.NF += __popc(F);
    a.NFU += __popc(FU);
    a.A0 += __popc(__builtin_amdgcn_bitop3_b32(F, o.b0, o.S, 0x90));
    a.A1 += __popc(__builtin_amdgcn_bitop3_b32(F, o.b1, o.S, 0x90));
    a.A2 += __popc(__builtin_amdgcn_bitop3_b32(F, o.b2, o.S, 0x90));
    if (surf) {
        const int dm = 2 * __popc(F) - 4 * __popc(FU);
        a.D1 += x0 ? dm : 0;
        a.Dn += xl ? dm : 0;
        a.KDM += ((x0 ? 1 : 0) + (xl ? 1 : 0)) * dm;
    }
}

// F = 16 F + the reject bits (t < r) of four sites, the last site's first:
// the four-site form of reject_bits8, with the same spacing of carry writes
// and reads.
__device__ __forceinline__ uint32_t reject_bits4(uint32_t F, const uint2 &ta, const uint2 &tb, const uint32_t r[4])
{
    uint64_t ca, cb;
    asm("v_cmp_lt_u32_e64 %[a], %[t3], %[r3]\n\t"
        "v_cmp_lt_u32_e64 %[b], %[t2], %[r2]\n\t"
        "v_cmp_lt_u32_e32 vcc, %[t1], %[r1]\n\t"
        "v_addc_co_u32_e64 %[f], %[a], %[f], %[f], %[a]\n\t"
        "v_addc_co_u32_e64 %[f], %[b], %[f], %[f], %[b]\n\t"
        "v_cmp_lt_u32_e64 %[a], %[t0], %[r0]\n\t"
        "v_addc_co_u32_e32 %[f], vcc, %[f], %[f], vcc\n\t"
        "s_nop 1\n\t"
        "v_addc_co_u32_e64 %[f], %[a], %[f], %[f], %[a]"
        : [f] "+&v"(F), [a] "=&s"(ca), [b] "=&s"(cb)
        : [t3] "v"(tb.y), [t2] "v"(tb.x), [t1] "v"(ta.y), [t0] "v"(ta.x), [r3] "v"(r[3]), [r2] "v"(r[2]),
          [r1] "v"(r[1]), [r0] "v"(r[0])
        : "vcc");
    return F;
}

// Accept bits of the word's first 4 ng sites by 64-bit thresholds, one site
// at a time: the exact form for moves that are never accepted (threshold 0),
// which thr - 1 in 32 bits cannot tell from threshold 1.
__device__ __forceinline__ uint32_t exact_flips(uint32_t S, uint32_t b2, uint32_t b1, uint32_t b0, uint32_t gq, int ng,
                                             uint32_t t, uint32_t replica, uint32_t key0, uint32_t key1,
                                             const uint64_t *thr)
{
    uint32_t F = 0;
#pragma unroll 1
    for (int g = 0; g < ng; ++g) {
        uint32_t r[4];
        philox10(gq + 2u * (uint32_t)g, t, replica, 0u, key0, key1, r);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int i = 4 * g + l;
            const uint32_t e = ((S >> i) & 1u) << 3 | ((b2 >> i) & 1u) << 2 | ((b1 >> i) & 1u) << 1 | ((b0 >> i) & 1u);
            F |= (uint32_t)((uint64_t)r[l] < thr[e]) << i;
        }
    }
    return F;
}

// Accept bits of the word's first 4 ng sites from the pair tables, two groups
// at a time from the top: partial last words and, with QUADS = false, surface
// planes and replicas that the four-site table does not cover (a bulk field,
// or never-accepted moves: those are rare misreadings of a draw of 0, found
// by the smallest draw and done over).
template <bool QUADS>
__device__ __forceinline__ uint32_t few_flips(const Word &o, int ng, const DrawKey &k, const uint4 *quad,
                                              const uint2 *pair, const uint64_t *thr, bool never)
{
    uint32_t w[4];
    if (QUADS) quad_index(o.S, o.b2, o.b1, o.b0, w);
#pragma unroll
    for (int j = 0; j < 4 && !QUADS; ++j) {
        uint32_t acc = o.b0 >> (2 * j);
        acc = pick(0x0C0C0C0Cu, j == 0 ? o.b1 << 2 : o.b1 >> (2 * j - 2), acc);
        acc = pick(0x30303030u, j <= 2 ? o.b2 << (4 - 2 * j) : o.b2 >> 2, acc);
        w[j] = pick(0xC0C0C0C0u, o.S << (6 - 2 * j), acc);
    }
    uint32_t F = 0, low = ~0u, r[4];
    if (ng & 1) {
        const uint32_t sh = 4u * (uint32_t)(ng - 1);
        philox10(o.gq + 2u * (uint32_t)(ng - 1), k.t, k.replica, 0u, k.key0, k.key1, r);
        if (QUADS) {
            const uint4 a = quad[(w[0] >> sh) & 0xFFu];
            F = reject_bits4(F, make_uint2(a.x, a.y), make_uint2(a.z, a.w), r);
        } else {
            F = reject_bits4(F, pair[(w[0] >> sh) & 0xFFu], pair[(w[1] >> sh) & 0xFFu], r);
        }
        if (!QUADS) low = min(min(r[0], r[1]), min(r[2], r[3]));
    }
#pragma unroll 1
    for (int h = (ng >> 1) - 1; h >= 0; --h) {
        const uint32_t sh = 8u * (uint32_t)h, c = o.gq + 4u * (uint32_t)h;
        uint2 l0, l1, h0, h1;
        if (QUADS) {
            const uint4 a = quad[(w[0] >> sh) & 0xFFu], b = quad[(w[1] >> sh) & 0xFFu];
            l0 = make_uint2(a.x, a.y), l1 = make_uint2(a.z, a.w);
            h0 = make_uint2(b.x, b.y), h1 = make_uint2(b.z, b.w);
        } else {
            l0 = pair[(w[0] >> sh) & 0xFFu], l1 = pair[(w[1] >> sh) & 0xFFu];
            h0 = pair[(w[2] >> sh) & 0xFFu], h1 = pair[(w[3] >> sh) & 0xFFu];
        }
        uint32_t r1[4];
        philox10(c, k.t, k.replica, 0u, k.key0, k.key1, r);
        philox10<2u>(c, k.t, k.replica, 0u, k.key0, k.key1, r1);
        F = reject_bits4(F, h0, h1, r1);
        F = reject_bits4(F, l0, l1, r);
        if (!QUADS) low = min(min(low, min(min(r[0], r[1]), min(r[2], r[3]))), min(min(r1[0], r1[1]), min(r1[2], r1[3])));
    }
    F = ~F;
    if (!QUADS && never && __any(low == 0u))
        F = exact_flips(o.S, o.b2, o.b1, o.b0, o.gq, ng, k.t, k.replica, k.key0, k.key1, thr);
    return F;
}

// (a mailbox is below 4 GiB: a uniform base and a 32-bit offset)
__device__ __forceinline__ void mail_put(unsigned long long *mbox, uint32_t at, unsigned long long v)
{
    gu64 *p = (gu64 *)((gu8 *)mbox + 8u * at);
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Updates chunk c of a row set in one phase: words run planes slowest, then
// rows, then words of a row, 64 to a chunk.  send: new words of edge rows and
// edge planes go to the neighbours' mailboxes.
//
// FINE: 16 words to a chunk, four lanes to a word with two of its groups each
// (they read and count the word's neighbours alike, and join their flips).  A
// chunk takes a third of the time, all words together half as long again: for
// stages of few words, which lie on one chunk's latency (24 x 20x64x64 11.1 ->
// 7.7 us a sweep, 16 x 40x120x120 15.8 -> 11.4, 22x142x142 11.4 -> 9.9).
template <bool SEAM, bool WHOLE, bool FINE>
__device__ __forceinline__ void share_chunk(const Share &g, const ResJob &jb, char *lat, const ResTables &tb,
                                            const DrawKey &key, const ResRows &rs, int c, int phase, bool send,
                                            bool edge_rows, unsigned long long *mbox, uint32_t epoch, Sums &a)
{
    const int lane = threadIdx.x & 63;
    const int plane = WHOLE ? rs.n * jb.Wf : rs.n;
    const uint32_t m = WHOLE ? rs.m_w : rs.m;
    const uint32_t *ct = g.ct + (WHOLE ? rs.r0 * jb.Wf : g.R * jb.Wf + rs.r0);
    const int T = g.np * plane;
    constexpr int PER = FINE ? kResFineChunk : 64;
    const int tk = c * PER + (FINE ? lane >> 2 : lane);
    const uint32_t p8 = FINE ? 8u * (uint32_t)(lane & 3) : 0u;   // the lane's first site in the word
    bool ok = tk < T;
    const uint32_t tau = (uint32_t)min(tk, T - 1);
    const uint32_t pi = div_m(tau, (uint32_t)plane, m);
    const uint32_t *cp = ct + (tau - __umul24(pi, (uint32_t)plane));
    const Column cl{cp[0], cp[g.nc], cp[2 * g.nc], cp[3 * g.nc], cp[4 * g.nc]};
    const uint4 pl = g.pt[pi];
    const Word o = share_gather<SEAM, WHOLE>(g, lat, pl, cl, phase);
    // chunks of bulk planes read the bulk table at a fixed base
    const bool surf = c * PER < jb.n_head * plane || c * PER + PER - 1 >= T - jb.n_tail * plane;
    const bool x0 = (pl.w & PL_X0) != 0, xl = (pl.w & PL_XL) != 0;
    uint32_t F;
    if (FINE) {
        const Word f = {o.S >> p8, o.b0 >> p8, o.b1 >> p8, o.b2 >> p8, o.own, o.gq + (p8 >> 1)};
        if (g.sym && !surf) F = few_flips<true>(f, 2, key, tb.quad, tb.pair, tb.thr, false);
        else
            F = few_flips<false>(f, 2, key, tb.quad, tb.pair + (x0 ? 256 : xl ? 512 : 0),
                                 tb.thr + kThrPerClass * ((x0 ? 1 : 0) + (xl ? 2 : 0)), g.never);
        F = (F & 0xFFu) << p8;
        F |= (uint32_t)__builtin_amdgcn_mov_dpp((int)F, 0xB1, 0xF, 0xF, true);   // lanes 1 0 3 2 of each four
        F |= (uint32_t)__builtin_amdgcn_mov_dpp((int)F, 0x4E, 0xF, 0xF, true);   // lanes 2 3 0 1
        ok = ok && p8 == 0u;
    } else if (g.sym && !surf) {
        if (WHOLE) F = bp_flips_quads(o.S, o.b2, o.b1, o.b0, o.gq, key, tb.quad);
        else F = few_flips<true>(o, jb.ng, key, tb.quad, tb.pair, tb.thr, false);
    } else {
        F = few_flips<false>(o, WHOLE ? 8 : jb.ng, key, tb.quad, tb.pair + (x0 ? 256 : xl ? 512 : 0),
                             tb.thr + kThrPerClass * ((x0 ? 1 : 0) + (xl ? 2 : 0)), g.never);
    }
    if (!WHOLE) F &= (1u << g.rem) - 1u;
    F = ok ? F : 0u;
    const uint32_t V = o.S ^ F;
    if (ok) *(uint32_t *)(lat + o.own) = V;
    share_sums(o, F, surf, x0, xl, a);
    if (send) {
        const unsigned long long v = ((unsigned long long)epoch << 32) | V;
        const uint32_t sl = (phase & 1) ? jb.slot : 0u;
        if (edge_rows && ok) {
            const uint32_t ay = cp[5 * g.nc] + __umul24(pi, (uint32_t)g.Wq) + sl;
            mail_put(mbox, ay, v);
            if (g.R == 1) mail_put(mbox, ay + (jb.out_y[1] - jb.out_y[0]), v);   // one row is both edges
        }
        if (c * PER < jb.n_edge * plane && ok && (int)pi < jb.n_edge) {
            const uint2 px = g.pm[pi];
            const uint32_t ax = cp[6 * g.nc] + sl;
            mail_put(mbox, px.x + ax, v);
            if (px.y != ~0u) mail_put(mbox, px.y + ax, v);
        }
    }
}

// Small films: one lane per four-site group, so that a phase spreads over all
// waves and its latency is one group's, not one word's.  A lane keeps its
// groups for the whole launch, their addresses worked out once.
struct GroupTask {
    uint32_t base;       // byte offset of the word in the even-z sublattice of its row
    uint32_t ua, da;     // what leads from there to the y+1 and y-1 words
    uint32_t um, dm;     // seam masks of them
    uint32_t up, dn;     // steps to the next word round the row, each way
    uint32_t sh;         // first site of the group in its word
    uint32_t mask;       // sites that exist
    uint32_t cls;        // table offset: 0, 256 (x = 0) or 512 (x = Lx-1)
    uint32_t gq, xy;     // Philox counter for even z; x + y
    uint32_t esh, top;   // z edge shifts (see share_gather)
    int thr;             // threshold class offset
    bool on, x0, xl;
};

__device__ __forceinline__ GroupTask group_task(const Share &g, uint32_t m_c, int lr0, const ResRows &rs, int tk)
{
    const int C = (int)(g.gy >> 1);
    GroupTask t;
    t.on = tk < g.Lx * rs.n * C;
    const uint32_t k = t.on ? (uint32_t)tk : 0u;
    const uint32_t rest = div_m(k, (uint32_t)C, m_c), gr = k - rest * (uint32_t)C;
    const int x = (int)div_m(rest, (uint32_t)rs.n, rs.m);
    const int lr = lr0 + ((int)rest - x * rs.n);
    const int w = (int)(gr >> 3), y = share_row_y(g, lr);
    const int xs = g.refl ? g.Lx - 1 - x : x;
    const bool su = lr == g.ls, sd = lr == g.lr0, lastw = w == g.Wq - 1;
    t.base = (uint32_t)(x + 1) * g.PB + (uint32_t)lr * g.RB + 4u * (uint32_t)w;
    t.ua = (su ? (uint32_t)(xs - x) * g.PB + (uint32_t)(g.lr0 - lr) * g.RB : g.RB);
    t.da = (sd ? (uint32_t)(xs - x) * g.PB + (uint32_t)(g.ls - lr) * g.RB : 0u - g.RB);
    t.um = su ? g.inv : 0u;
    t.dm = sd ? g.inv : 0u;
    t.up = lastw ? 0u - 4u * (uint32_t)w : 4u;
    t.dn = w == 0 ? 4u * (uint32_t)(g.Wq - 1) : 0u - 4u;
    t.sh = 4u * (gr & 7u);
    t.mask = !t.on ? 0u : lastw && g.rem < 32 ? (1u << g.rem) - 1u : ~0u;
    t.x0 = x == 0;
    t.xl = x == g.Lx - 1;
    t.cls = t.x0 ? 256u : t.xl ? 512u : 0u;
    t.thr = kThrPerClass * ((t.x0 ? 1 : 0) + (t.xl ? 2 : 0));
    t.gq = (uint32_t)x * g.gx + (uint32_t)y * g.gy + 2u * gr;
    t.xy = (uint32_t)(x + y);
    t.esh = w == 0 ? 32u - (uint32_t)g.rem : 0u;
    t.top = lastw ? (uint32_t)g.rem - 1u : 31u;
    return t;
}

// One phase of a group (see share_gather); the lanes of a word add their
// flips with LDS xors.
__device__ __forceinline__ void group_update(const Share &g, const GroupTask &t, char *lat, const uint2 *pair,
                                             const uint64_t *thr, const DrawKey &key, int phase, Sums &a)
{
    const uint32_t q = (t.xy + (uint32_t)phase) & 1u, qm = 0u - q;
    Word o;
    o.own = t.base + (qm & g.SB);
    const uint32_t oth = t.base + (~qm & g.SB);
    const uint32_t O = lds32(lat, oth), E = lds32(lat, oth + pick(qm, t.up, t.dn));
    const uint32_t yp = lds32(lat, o.own + t.ua) ^ t.um, ym = lds32(lat, o.own + t.da) ^ t.dm;
    const uint32_t xm = lds32(lat, o.own - g.PB), xp = lds32(lat, o.own + g.PB);
    o.S = lds32(lat, o.own);
    const uint32_t gq = t.gq + q;
    uint32_t r[4];
    philox10(gq, key.t, key.replica, 0u, key.key0, key.key1, r);
    const uint32_t zd = __builtin_amdgcn_alignbit(O, E << t.esh, 31), zu = (O >> 1) | ((E & 1u) << t.top);
    const uint32_t Z = pick(qm, zu, zd);
    const uint32_t s1 = xor3(O, Z, ym), c1 = maj3(O, Z, ym);
    const uint32_t s2 = xor3(yp, xm, xp), c2 = maj3(yp, xm, xp);
    const uint32_t k0 = s1 & s2;
    o.b0 = s1 ^ s2;
    o.b1 = xor3(c1, c2, k0);
    o.b2 = maj3(c1, c2, k0);
    const uint32_t s = o.S >> t.sh, p0 = o.b0 >> t.sh, p1 = o.b1 >> t.sh, p2 = o.b2 >> t.sh;
    const uint32_t i0 = pick(0xC0u, s << 6, pick(0x30u, p2 << 4, pick(0x0Cu, p1 << 2, p0)));
    const uint32_t i1 = pick(0xC0u, s << 4, pick(0x30u, p2 << 2, pick(0x0Cu, p1, p0 >> 2)));
    const uint2 ta = pair[t.cls + (i0 & 0xFFu)], tc = pair[t.cls + (i1 & 0xFFu)];
    uint32_t f = ~reject_bits4(0u, ta, tc, r) & 15u;
    if (g.never && __any(min(min(r[0], r[1]), min(r[2], r[3])) == 0u))
        f = exact_flips(s, p2, p1, p0, gq, 1, key.t, key.replica, key.key0, key.key1, thr + t.thr);
    const uint32_t F = (f << t.sh) & t.mask;
    if (F) __hip_atomic_fetch_xor((uint32_t *)(lat + o.own), F, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    share_sums(o, F, t.x0 || t.xl, t.x0, t.xl, a);
}

// Halo plane j of a face (0 outer, 1 inner): its slot and its x.
__device__ __forceinline__ int halo_slot(const ResJob &jb, int face, int j)
{
    if (face == 0) return j == 0 ? 0 : jb.n2 ? jb.n1 + jb.n2 + 3 : jb.n1 + 1;
    return jb.n1 + 1 + j;
}
__device__ __forceinline__ int halo_x(const Share &g, const ResJob &jb, int face, int j)
{
    if (face == 0) return j == 0 ? jb.xa - 1 : g.Lx - jb.xa;
    return j == 0 ? jb.xa + jb.n1 : g.Lx - jb.xa - jb.n2 - 1;
}

// Words of a mailbox slot: y faces, then x faces.
__device__ __forceinline__ int mail_y(const Share &g, const ResJob &jb)
{
    return (jb.has & HAS_Y) ? 2 * g.np * g.Wq : 0;
}
__device__ __forceinline__ int mail_x(const Share &g, const ResJob &jb)
{
    return (((jb.has & HAS_OUTER) ? 2 : 0) + ((jb.has & HAS_INNER) ? 2 : 0)) * g.R * g.Wq;
}

// Where word k of a slot goes: its byte offset in LDS in the even-z
// sublattice, bit 0 the parity of x + y (the sublattice that a phase updates
// is that parity + phase), bit 1 set for row 0 (sent in phases 2 and 3).
__device__ __forceinline__ uint32_t mail_target(const Share &g, const ResJob &jb, int k)
{
    const int n = g.np * g.Wq, RW = g.R * g.Wq, KY = mail_y(g, jb);
    if (k < KY) {
        const int face = k >= n ? 1 : 0;
        const uint32_t kk = (uint32_t)(k - face * n), pi = div_m(kk, (uint32_t)g.Wq, jb.m_q), w = kk - pi * g.Wq;
        const uint4 pl = g.pt[pi];
        // the neighbour's row is a main row one below local row 1 or one above local row R
        const int y = face ? share_row_y(g, g.R) + 1 : g.y0 - 1;
        return pl.x + (face ? (uint32_t)(g.R + 1) * g.RB : 0u) + 4u * w + ((pl.w ^ (uint32_t)y) & 1u);
    }
    uint32_t kk = (uint32_t)(k - KY);
    const uint32_t f = div_m(kk, (uint32_t)RW, jb.m_f);
    kk -= f * RW;
    const uint32_t row = div_m(kk, (uint32_t)g.Wq, jb.m_q);
    kk -= row * g.Wq;
    const int face = (jb.has & HAS_OUTER) ? (int)(f >> 1) : 1, j = (int)(f & 1u);
    const uint32_t par = (uint32_t)(halo_x(g, jb, face, j) + share_row_y(g, (int)row + 1)) & 1u;
    return (uint32_t)halo_slot(jb, face, j) * g.PB + (row + 1u) * g.RB + 4u * kk + par +
           ((int)row + 1 == g.lr0 ? 2u : 0u);
}

// One wave receives the words that the neighbours updated in phase 0 or 1 into
// the halo rows and planes, or in phases 2 and 3 row 0's words, while the
// other waves compute (no word that arrives in a phase is read in it).
// Returns false if a wait ran out.
__device__ __forceinline__ bool share_receive(const Share &g, const ResJob &jb, char *lat, GridSync *sync,
                                              const unsigned long long *mbox, uint32_t epoch, int phase)
{
    const unsigned long long *box = mbox + jb.in + ((phase & 1) ? jb.slot : 0u);
    const int KY = mail_y(g, jb), K = KY + mail_x(g, jb), lane = threadIdx.x & 63;
    constexpr int B = 8;   // words a lane polls together
    unsigned spins = 0;
    for (int k0 = phase < 2 ? 0 : KY; k0 < K; k0 += 64 * B) {
        uint32_t to[B];
        bool some = false;
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int k = k0 + 64 * i + lane;
            to[i] = k < K ? g.mt[k] : ~0u;
            // row 0 comes in phases 2 and 3, alone
            if (((to[i] & 2u) != 0) != (phase >= 2)) to[i] = ~0u;
            some = some || to[i] != ~0u;
        }
        if (!__any(some)) continue;
        while (true) {
            unsigned long long v[B];
            bool all = true;
#pragma unroll
            for (int i = 0; i < B; ++i)
                v[i] = __hip_atomic_load(box + min(k0 + 64 * i + lane, K - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int i = 0; i < B; ++i) {
                if (to[i] == ~0u) continue;
                if ((uint32_t)(v[i] >> 32) == epoch) {
                    *(uint32_t *)(lat + (to[i] & ~3u) + (((to[i] ^ (uint32_t)phase) & 1u) ? g.SB : 0u)) = (uint32_t)v[i];
                    to[i] = ~0u;
                } else {
                    all = false;
                }
            }
            if (__all(all)) break;
            __builtin_amdgcn_s_sleep(2);
            if ((++spins & 1023u) == 0) {
                if (__hip_atomic_load(&sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
                if (spins > (1u << 21)) {
                    if (lane == 0) atomicAdd(&sync->error.v, 1ull);
                    return false;
                }
            }
        }
    }
    return true;
}

// Moves words between the replica's spin array and LDS: local rows lo .. hi of
// planes 0 .. np-1 of the plane table (or of the one halo plane given by slot
// and x), LDS word (plane, local row, sublattice, word).
template <int FMT, bool LOAD>
__device__ __forceinline__ void share_move(const Share &g, const RepDesc &d, const ResPlane *planes, char *lat, int lo,
                                           int hi, int np, int slot = 0, int hx = 0)
{
    const int nr = hi - lo + 1, RW = 2 * g.Wq;
    const int n = np * nr * RW;
    for (int k = threadIdx.x; k < n; k += kResThreads) {
        const int r = k / RW, c = k - r * RW;
        const int pi = r / nr, lr = lo + (r - pi * nr);
        const int y = share_row_y(g, lr);
        const int x = planes ? planes[pi].x : hx, sl = planes ? planes[pi].slot : slot;
        uint32_t *l = (uint32_t *)(lat + ((uint32_t)sl * g.PB + (uint32_t)lr * g.RB)) + c;
        const size_t row = (size_t)x * d.Ly + y;
        if (FMT == ISLF_SPIN_BITPACK) {
            uint32_t *p = (uint32_t *)d.spins + row * (size_t)RW + c;
            if (LOAD) *l = *p;
            else *p = *l;
        } else {
            // 32 sites = four 8-byte columns of the sublattice (fewer in the last word)
            const int q = c >= g.Wq ? 1 : 0, w = c - q * g.Wq;
            uint64_t *p = (uint64_t *)(d.spins + row * (size_t)d.RB + (size_t)q * d.Hp) + 4 * w;
            const int nc = min(4, d.K - 4 * w);
            if (LOAD) {
                uint32_t v = 0;
                for (int i = 0; i < nc; ++i) {
                    const uint64_t b = p[i];
                    // bytes of 0/1 to bits: byte j of a half lands on bit 28 + j of the product
                    const uint32_t lo4 = ((uint32_t)b * 0x10204080u) >> 28;
                    const uint32_t hi4 = ((uint32_t)(b >> 32) * 0x10204080u) >> 28;
                    v |= (lo4 | (hi4 << 4)) << (8 * i);
                }
                *l = v;
            } else {
                const uint32_t v = *l;
                for (int i = 0; i < nc; ++i) {
                    const uint32_t lo4 = (v >> (8 * i)) & 15u, hi4 = (v >> (8 * i + 4)) & 15u;
                    const uint32_t a = (lo4 * 0x00204081u) & 0x01010101u, b = (hi4 * 0x00204081u) & 0x01010101u;
                    p[i] = ((uint64_t)b << 32) | a;
                }
            }
        }
    }
}

// Waits until every cluster workgroup of the launch has started, or gives up
// and aborts the launch for all of them (whoever moves the state first
// decides for all).  Gives up after about a tenth of a second: what holds the
// CUs is then work that the library does not see (its own contexts take turns,
// see Turns in islf_api.hip), and the closing kernel's sweeps cost more than
// waiting for most of that.  (The bound fits an instruction's 16-bit constant:
// with a 32-bit one the code behind it moved by 4 bytes, and three films of
// 46 M sites took 62.6 instead of 61.3 us a sweep.)  Called by thread 0.
__device__ __forceinline__ unsigned int res_census(ResSync *rs, unsigned int members)
{
    const unsigned int old = atomicAdd(&rs->count, 1u);
    if (old + 1 == members) atomicCAS(&rs->state, (unsigned)RES_WAIT, (unsigned)RES_GO);
    for (unsigned spins = 0;; ++spins) {
        const unsigned int s = __hip_atomic_load(&rs->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s != RES_WAIT) return s;
        if (spins > 65000u) atomicCAS(&rs->state, (unsigned)RES_WAIT, (unsigned)RES_ABORT);
        __builtin_amdgcn_s_sleep(32);
    }
}

// What bounds it: VALU issue (the Philox word and the threshold lookups, as
// in bp_march).  16 waves per workgroup and one workgroup per CU: a CU's
// whole LDS is one share, which keeps the edge rows few against the interior
// (two workgroups of 8 waves per CU measured 24.3 against 23.4 us per sweep on
// 64 x 40x120x120 and 85 against 66 on 3 x 160x480x600).  Counters, 3 x
// 160x480x600: 15.8 VALU lane-ops per update (the launch chain's march 16.2,
// padding of its 300-bit rows included), VALU issue 89% of the time; without
// the exchange the same launch takes 57.6 us per sweep instead of 62.0.
// Per sweep, before (launch chain, or persistent kernel) and now: 12x24x24 14
// and 3.4 us, 168 ladder films 37 and 2.7 us, 64 x 40x120x120 31 and 21.4 us,
// 96 uneven films int8 85 and 59 us, 184x504x504 39 and 25 us, 3 x
// 160x480x600 int8 95 and 62 us, persistent 78 and 61 us.
// FORM: RES_GROUPS = no clusters, and films of few words, updated one four-site
// group per lane (group_update); RES_FINE = chunks of 16 words.
template <int FMT, int FORM>
__global__ __launch_bounds__(kResThreads) void k_resident(const RepDesc *__restrict__ descs,
                                                          const RepState *__restrict__ st,
                                                          const ResJob *__restrict__ jobs,
                                                          const int *__restrict__ first,
                                                          const ResPlane *__restrict__ plane_tables,
                                                          const ResRow *__restrict__ row_tables, const ResLaunch L)
{
    constexpr bool SMALL = FORM == RES_GROUPS, FINE = FORM == RES_FINE;
    extern __shared__ uint32_t smem[];
    __shared__ ResTables tb;
    __shared__ ResCtl ctl_s;
    static_assert(sizeof(ResTables) + sizeof(ResCtl) <= kResStaticLds, "the host's LDS budget counts on it");
    ResCtl *ctl = &ctl_s;
    char *lat = (char *)smem;
    const int tid = threadIdx.x;
    const uint32_t n = L.n;
    if (L.check_error) {
        if (tid == 0)
            ctl->state = __hip_atomic_load(&L.sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
        __syncthreads();
        if (ctl->state) return;
        __syncthreads();
    }
    const uint32_t epoch0 = L.rs->epoch;
    for (int j = first[blockIdx.x]; j < first[blockIdx.x + 1]; ++j) {
        const ResJob &jb = jobs[j];   // uniform: scalar loads where used
        const RepDesc &d = descs[jb.rep];
        const ResPlane *planes = plane_tables + jb.planes;
        Share g;
        g.Lx = d.Lx; g.Wq = d.Wq;
        g.rem = (d.Lz >> 1) - 32 * (d.Wq - 1);
        g.SB = 4u * (uint32_t)g.Wq;
        g.RB = 2u * g.SB;
        g.PB = (uint32_t)(jb.R + 2) * g.RB;
        g.R = jb.R; g.ls = jb.ls; g.lr0 = jb.lr0; g.y0 = jb.y0;
        g.np = jb.n1 + jb.n2;
        g.inv = d.seam_invert ? ~0u : 0u;
        g.refl = d.seam_reflect != 0;
        g.never = d.never_mask != 0;
        g.sym = d.sym != 0 && !g.never;
        g.gy = 2u * (uint32_t)d.C;
        g.gx = g.gy * (uint32_t)d.Ly;
        const int slots = g.np + (jb.n2 ? 4 : 2);
        uint4 *pt = (uint4 *)(lat + ((uint32_t)slots * g.PB + 15u & ~15u));
        uint2 *pm = (uint2 *)(pt + g.np);
        uint32_t *ct = (uint32_t *)(pm + g.np);
        g.pm = pm;
        g.nc = g.R * g.Wq;
        uint32_t *mt = ct + kColumnFields * g.nc;
        g.pt = pt;
        g.ct = ct;
        g.mt = mt;
        DrawKey key{st[jb.rep].t, d.replica, d.key0, d.key1};
        // tables: three classes' pair tables (a one-layer film has one class), all thresholds, planes, rows
        for (int k = tid; k < 768; k += kResThreads) {
            const int e = k & 255, cls = g.Lx == 1 ? 3 : k >> 8;
            const int ev = (e & 1) | ((e >> 1) & 2) | ((e >> 2) & 4) | ((e >> 3) & 8);
            const int od = ((e >> 1) & 1) | ((e >> 2) & 2) | ((e >> 3) & 4) | ((e >> 4) & 8);
            tb.pair[k] = make_uint2(d.thr_m1[cls * kThrPerClass + ev], d.thr_m1[cls * kThrPerClass + od]);
        }
        for (int k = tid; k < 256 && g.sym; k += kResThreads) tb.quad[k] = quad_entry(d, k);
        if (tid < kThrEntries) tb.thr[tid] = d.thr[tid];
        if (tid == 8) ctl->bad = ~0u;
        if (tid >= 12 && tid < 16) ctl->ticket[tid - 12] = 0;
        if (!SMALL) {
            for (int k = tid; k < g.np; k += kResThreads) {
                const ResPlane e = planes[k];
                pt[k] = make_uint4((uint32_t)e.slot * g.PB, (uint32_t)e.x * g.gx, (uint32_t)e.mirror * g.PB,
                                   (uint32_t)e.flags);
                // faces it is sent to: outer j = 0, 1, inner j = 0, 1
                uint32_t to[2] = {~0u, ~0u};
                int m = 0;
                for (int f = 0; f < 4; ++f)
                    if (e.flags & (PL_SEND << f)) {
                        const uint32_t v = jb.out_x[f >> 1] + (uint32_t)((f & 1) * g.R * g.Wq);
                        if (m == 0) to[0] = v;
                        else to[1] = v;
                        ++m;
                    }
                pm[k] = make_uint2(to[0], to[1]);
            }
            for (int k = tid; k < g.R * g.Wq; k += kResThreads) {
                const int ri = k / g.Wq, w = k - ri * g.Wq;
                const ResRow e = row_tables[jb.rows + ri];
                uint32_t *c = ct + (w < jb.Wf ? ri * jb.Wf + w : g.R * jb.Wf + ri);
                c[0] = (uint32_t)e.lr * g.RB + 4u * (uint32_t)w;
                c[g.nc] = (uint32_t)e.y * g.gy + 16u * (uint32_t)w;
                c[2 * g.nc] = (uint32_t)e.flags | (w == 0 ? 32u - (uint32_t)g.rem : 0u) << 8 | (uint32_t)e.lr << 16;
                c[3 * g.nc] = w == g.Wq - 1 ? 0u - 4u * (uint32_t)w : 4u;
                c[4 * g.nc] = w == 0 ? 4u * (uint32_t)(g.Wq - 1) : 0u - 4u;
                c[5 * g.nc] = jb.out_y[e.lr == 1 ? 0 : 1] + (uint32_t)w;
                c[6 * g.nc] = (uint32_t)((e.lr - 1) * g.Wq + w);
            }
        }
        // the planes beyond the free surfaces stay 0
        if (!(jb.has & HAS_OUTER))
            for (uint32_t k = tid; k < g.PB / 4; k += kResThreads) {
                ((uint32_t *)lat)[k] = 0u;
                ((uint32_t *)(lat + (uint32_t)(slots - 1) * g.PB))[k] = 0u;
            }
        const bool cluster = !SMALL && jb.P > 1;
        const bool has_x = (jb.has & (HAS_OUTER | HAS_INNER)) != 0, has_y = (jb.has & HAS_Y) != 0;
        share_move<FMT, true>(g, d, planes, lat, has_y ? 0 : 1, has_y ? g.R + 1 : g.R, g.np);
        if (!SMALL && has_x)
            for (int f = 0; f < 4; ++f)
                if (jb.has & ((f >> 1) ? HAS_INNER : HAS_OUTER))
                    share_move<FMT, true>(g, d, nullptr, lat, 1, g.R, 1, halo_slot(jb, f >> 1, f & 1),
                                          halo_x(g, jb, f >> 1, f & 1));
        if (cluster) {
            __syncthreads();   // the plane table
            for (int k = tid; k < mail_y(g, jb) + mail_x(g, jb); k += kResThreads) mt[k] = mail_target(g, jb, k);
        }
        if (cluster && tid == 0) ctl->state = res_census(L.rs, (unsigned)L.members);
        __syncthreads();
        if (cluster && ctl->state != RES_GO) {
            __syncthreads();
            continue;
        }
        // the small form's groups: rows y > 0 (at most kSmallTasks per lane), row y = 0
        GroupTask gt[kSmallTasks], gt0;
        int main_tasks = 0, row0_tasks = 0;
        if (SMALL) {
            const ResRows &m = jb.set[RES_INNER], &z = jb.set[RES_ROW0];
            for (int k = 0; k < kSmallTasks; ++k) gt[k] = group_task(g, jb.m_c, 2, m, tid + k * kResThreads);
            gt0 = group_task(g, jb.m_c, 1, z, tid);
            // whole waves without a group skip the phase
            main_tasks = g.Lx * m.n * d.C - (tid & ~63);
            row0_tasks = g.Lx * d.C;
        }
        bool good = true;
        int turn = 0;   // phases so far
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        for (uint32_t s = 0; s < n && good; ++s, ++key.t) {
            Sums a = {0, 0, 0, 0, 0, 0, 0, 0};
            if (SMALL) {
#pragma unroll 1
                for (int phase = 0; phase < 4; ++phase) {
                    if (phase < 2) {
                        for (int k = 0; k < kSmallTasks; ++k)
                            if (k * kResThreads < main_tasks) group_update(g, gt[k], lat, tb.pair, tb.thr, key, phase, a);
                    } else if ((int)(tid & ~63) < row0_tasks) {
                        group_update(g, gt0, lat, tb.pair, tb.thr, key, phase, a);
                    }
                    if (phase < 3) __syncthreads();
                }
            } else {
#pragma unroll 1
                for (int i = 0; i < jb.stages; ++i) {
                    const ResStage &sg = jb.stage[i];
                    const uint32_t ep = epoch0 + 4u * s + 1u;   // + phase
                    // the last wave takes in the mail first (nobody's input after the last sweep: phases 1 and 3)
                    if (cluster && wave == kResThreads / 64 - 1) {
                        // Ahead of the computing waves of its SIMD: its few instructions stand between one load latency
                        // and the next, and at their priority it waited for three waves of Philox in between.
                        // Three films of 46 M sites, 1,720 words a sweep: 62.8 -> 61.7 us a sweep; one 25.8 -> 24.7.
                        __builtin_amdgcn_s_setprio(3);
                        bool ok = true;
                        if (sg.mail == 0 || (sg.mail == 1 && s + 1 < n))
                            ok = share_receive(g, jb, lat, L.sync, L.mbox, ep + (uint32_t)sg.mail, sg.mail);
                        if (sg.mail_row0 == 2 || (sg.mail_row0 == 3 && s > 0))   // (phase 3's comes a sweep later)
                            ok = share_receive(g, jb, lat, L.sync, L.mbox, ep + (sg.mail_row0 == 2 ? 2u : 3u - 4u),
                                               sg.mail_row0) && ok;
                        if (!ok) atomicMin(&ctl->bad, s + 1u);
                        __builtin_amdgcn_s_setprio(0);
                    }
                    // chunks go to the waves as they come free
                    int *ticket = &ctl->ticket[turn & 3];
                    if (tid == 0) ctl->ticket[(turn + 2) & 3] = 0;   // last used two barriers ago
                    ++turn;
                    while (true) {
                        int c = 0;
                        if ((tid & 63) == 0) c = atomicAdd(ticket, 1);
                        c = __builtin_amdgcn_readfirstlane(c);
                        int k = 0;
                        while (k < 3 && c >= sg.part[k].c1 - sg.part[k].c0) {
                            c -= sg.part[k].c1 - sg.part[k].c0;
                            ++k;
                        }
                        if (k == 3) break;
                        c += sg.part[k].c0;
                        const int set = sg.part[k].set, phase = sg.part[k].phase;
                        const ResRows &rs = jb.set[set];
                        const bool edge = set == RES_EDGE;
                        const bool send = cluster && (!(phase & 1) || s + 1 < n);
                        const uint32_t e = ep + (uint32_t)phase;
                        if (c < rs.whole) {
                            if (rs.seam) share_chunk<true, true, FINE>(g, jb, lat, tb, key, rs, c, phase, send, edge, L.mbox, e, a);
                            else share_chunk<false, true, FINE>(g, jb, lat, tb, key, rs, c, phase, send, edge, L.mbox, e, a);
                        } else {
                            c -= rs.whole;
                            if (rs.seam) share_chunk<true, false, FINE>(g, jb, lat, tb, key, rs, c, phase, send, edge, L.mbox, e, a);
                            else share_chunk<false, false, FINE>(g, jb, lat, tb, key, rs, c, phase, send, edge, L.mbox, e, a);
                        }
                    }
                    if (i + 1 < jb.stages) __syncthreads();
                }
            }
            // The sweep's changes (see bp_march): summed by each wave, then over the waves by the last one, while the
            // others begin the next sweep (the first, which issues ahead of them, cost 1 us on three 46 M-site
            // films). Against masked reductions and LDS adds, one quantity after another: 12x24x24 3.85 -> 3.39 us
            // a sweep, 22x142x142 9.9 -> 9.5, 64 x 40x120x120 21.7 -> 21.4.
            const int4 w = wave_sums<64>(make_int4(-4 * (a.A0 + 2 * a.A1 + 4 * a.A2) + 16 * a.NF - 4 * a.NFU + a.KDM,
                                                   2 * a.NF - 4 * a.NFU, a.D1, a.Dn));
            int4 *sums = ctl->sums[s & 1];
            if ((tid & 63) == 63) sums[tid >> 6] = w;
            __syncthreads();
            // (written again two sweeps on, behind the next sweep's barriers)
            if (tid >= kResThreads - 64) {
                const int4 v = wave_sums<kResThreads / 64>(sums[tid & (kResThreads / 64 - 1)]);
                if ((tid & 63) == kResThreads / 64 - 1) L.part[(size_t)s * L.njobs + jb.id] = v;
            }
            // (a faster wave may be in sweep s+1 already: its failure counts there)
            good = ctl->bad > s + 1u;
        }
        if (good) share_move<FMT, false>(g, d, planes, lat, 1, g.R, g.np);
        __syncthreads();
    }
}

__device__ __forceinline__ void tell_host(unsigned long long *word, unsigned int v)
{
    __hip_atomic_store(word, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Closes a resident launch of n sweeps: one workgroup per replica.  Sums the
// shares' changes, stores the records and advances the replica; if the launch
// was aborted, sweeps the cluster replicas here first.
template <int FMT>
__global__ __launch_bounds__(kResThreads) void k_resident_close(const ResLaunch L)
{
    __shared__ long long sum[kResMaxSweeps][4];
    __shared__ uint64_t thr[kThrEntries];
    __shared__ int run;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n = L.n;
    ResSync *rs = L.rs;
    RepState *st = L.st;
    const ResRep rr = L.reps[blockIdx.x];
    const RepDesc &d = L.descs[rr.rep];
    if (tid == 0) {
        const bool err = L.check_error && __hip_atomic_load(&L.sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        run = err ? 0 : rr.P > 1 && rs->state != RES_GO ? 2 : 1;
    }
    if (tid < kThrEntries) thr[tid] = d.thr[tid];
    __syncthreads();
    const uint32_t t0 = st[rr.rep].t;
    for (int k = tid; k < 4 * kResMaxSweeps; k += kResThreads) (&sum[0][0])[k] = 0;
    __syncthreads();
    if (run == 2) {
        RepView v{};
        v.spins = d.spins;
        v.Lx = d.Lx; v.Ly = d.Ly; v.Lz = d.Lz; v.C = d.C; v.Wq = d.Wq; v.K = d.K;
        v.Hp = (uint32_t)d.Hp;
        v.RB = (uint32_t)d.RB;
        v.seam_reflect = d.seam_reflect;
        v.seam_invert = d.seam_invert;
        v.key0 = d.key0; v.key1 = d.key1; v.replica = d.replica;
        const int J = FMT == ISLF_SPIN_INT8 ? d.K : d.Wq;
        for (uint32_t s = 0; s < n; ++s) {
            v.t = t0 + s;
            Acc a = {0, 0, 0, 0};
            for (int phase = 0; phase < 4; ++phase) {
                const int ny = phase >= 2 ? 1 : d.Ly - 1;
                const long tasks = (long)d.Lx * ny * J;
                for (long k = tid; k < tasks; k += kResThreads) {
                    const long r = k / J;
                    const int x = (int)(r / ny), y = phase >= 2 ? 0 : 1 + (int)(r - (long)x * ny);
                    if (FMT == ISLF_SPIN_INT8) i8_update_col<false>(v, x, y, (int)(k - r * J), phase & 1, thr, a);
                    else bp_update_word<false>(v, x, y, (int)(k - r * J), phase & 1, thr, a);
                }
                __threadfence_block();
                __syncthreads();
            }
            const int q[4] = {a.dB, a.dM, a.dM1, a.dMn};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                long long w = q[k];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off, 64);
                if (lane == 0) atomicAdd((unsigned long long *)&sum[s][k], (unsigned long long)w);
            }
        }
    } else if (run == 1) {
        for (uint32_t s = wave; s < n; s += kResThreads / 64) {
            long long v[4] = {0, 0, 0, 0};
            for (int p = lane; p < rr.P; p += 64) {
                const int4 w = L.part[(size_t)s * L.njobs + rr.job0 + p];
                v[0] += w.x; v[1] += w.y; v[2] += w.z; v[3] += w.w;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
                if (lane == 0) sum[s][k] = v[k];
            }
        }
    }
    __syncthreads();
    if (run) {
        // running sums over the sweeps: wave k < 4 scans quantity k, four sweeps per lane
        if (wave < 4) {
            constexpr int L = kResMaxSweeps / 64;
            long long v[L], tot = 0;
#pragma unroll
            for (int i = 0; i < L; ++i) {
                const uint32_t s = (uint32_t)(L * lane + i);
                tot += s < n ? sum[s][wave] : 0;
                v[i] = tot;
            }
            long long inc = tot;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const long long u = __shfl_up(inc, off, 64);
                if (lane >= off) inc += u;
            }
            const long long before = st[rr.rep].cur[wave] + (inc - tot);
#pragma unroll
            for (int i = 0; i < L; ++i) {
                const uint32_t s = (uint32_t)(L * lane + i);
                if (s < n) sum[s][wave] = before + v[i];
            }
        }
        __syncthreads();
        // records that the ring keeps
        for (uint32_t s = tid; s < n; s += kResThreads) {
            if (n - s > d.cap) continue;
            d.rec[(t0 + s) % d.cap] = islf_obs{sum[s][0], sum[s][1], sum[s][2], sum[s][3]};
        }
        if (tid < 4) st[rr.rep].cur[tid] = sum[n - 1][tid];
        if (tid == 0) st[rr.rep].t = t0 + n;
    }
    // the last workgroup (every one has read the state by then) readies the next launch
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        if (atomicAdd(&rs->done, 1u) + 1 == gridDim.x) {
            // (launches without clusters: nobody has to wait for them, and a word to the host costs them 1 us)
            if (L.members > 0 && rs->state == RES_ABORT) tell_host(L.host + HOST_ABORTS, ++rs->aborts);
            if (L.members > 0) tell_host(L.host + HOST_ENDED, ++rs->ended);
            rs->count = 0;
            rs->state = RES_WAIT;
            rs->done = 0;
            rs->epoch += 4u * n + 4u;
        }
    }
}

// Ends a run of the launch chain as the closing kernel ends a resident launch.
__global__ void k_mark(ResSync *rs, unsigned long long *host)
{
    if (threadIdx.x == 0) tell_host(host + HOST_ENDED, ++rs->ended);
}

// ---------------------------------------------------------------------------
// Host-callable launchers
// ---------------------------------------------------------------------------
using ResKernel = void (*)(const RepDesc *, const RepState *, const ResJob *, const int *, const ResPlane *,
                           const ResRow *, ResLaunch);

static ResKernel resident_kernel(int fmt, int form)
{
    static const ResKernel k[2][3] = {
        {k_resident<ISLF_SPIN_INT8, RES_WORDS>, k_resident<ISLF_SPIN_INT8, RES_GROUPS>, k_resident<ISLF_SPIN_INT8, RES_FINE>},
        {k_resident<ISLF_SPIN_BITPACK, RES_WORDS>, k_resident<ISLF_SPIN_BITPACK, RES_GROUPS>,
         k_resident<ISLF_SPIN_BITPACK, RES_FINE>}};
    return k[fmt == ISLF_SPIN_INT8 ? 0 : 1][form];
}

// Lets the kernels use `bytes` of dynamic LDS.
hipError_t resident_lds_limit(int fmt, size_t bytes)
{
    hipError_t e = hipSuccess;
    for (int form : {RES_WORDS, RES_GROUPS, RES_FINE})
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)resident_kernel(fmt, form), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)bytes);
    return e;
}

hipError_t launch_resident(int fmt, int form, const ResLaunch &L, size_t lds, hipStream_t s)
{
    const dim3 b(kResThreads);
    hipLaunchKernelGGL(resident_kernel(fmt, form), dim3(L.grid), b, lds, s, L.descs, L.st, L.jobs, L.first, L.planes,
                       L.rows, L);
    if (fmt == ISLF_SPIN_INT8) hipLaunchKernelGGL(k_resident_close<ISLF_SPIN_INT8>, dim3(L.nreps), b, 0, s, L);
    else hipLaunchKernelGGL(k_resident_close<ISLF_SPIN_BITPACK>, dim3(L.nreps), b, 0, s, L);
    return hipGetLastError();
}

hipError_t launch_mark(ResSync *rs, unsigned long long *host, hipStream_t s)
{
    hipLaunchKernelGGL(k_mark, dim3(1), dim3(64), 0, s, rs, host);
    return hipGetLastError();
}

}  // namespace islf
