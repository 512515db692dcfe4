// Resident form of the sweeps: a launch loads its replicas' spins into LDS,
// one bit per site whatever the stored format, runs all of its sweeps there
// and writes the spins back at the end.  256 CUs x 160 KB of LDS hold 3e8
// sites; between two sweeps nothing travels but the edge rows of the shares.
//
// A replica that fits one workgroup is swept by it alone (barriers inside the
// workgroup only).  A larger one is cut along y into shares of whole rows
// (ResJob), one workgroup each, which exchange their edge rows after phases 0
// and 1 through mailboxes in device memory: every 64-bit mailbox word carries
// 32 spins and the step's epoch and is written and polled with relaxed
// device-scope atomics, so a word's arrival is its own flag: no fence and no
// counter stands between an edge word and its reader.  The edge rows are
// updated first in a phase and the interior rows cover the transfer.
//  - Two mailbox slots (by phase) are enough: a share writes step k+2 only
//    after it has read its neighbour's step k+1, which the neighbour wrote
//    after it had read step k.
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

// A share as the update loop sees it (uniform over the workgroup).  Its
// lattice in LDS: planes x = -1 .. Lx of R + 2 local rows of 2 Wq words; the
// planes -1 and Lx stay 0 (a free surface adds nothing to a neighbour count).
struct Share {
    int Lx, Wq, rem;         // words of a sublattice row, sites of a partial last word (32: none)
    uint32_t SB, RB, PB;     // LDS bytes of a sublattice row, a local row, an x plane
    int R, ls, lr0, y0;
    uint32_t inv;            // seam inversion mask
    bool refl, never, sym;
    uint32_t gx, gy;         // Philox counter steps of x and y
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
    int acc[2][4];
    unsigned int bad;      // 1 + the first sweep in which a wait ran out, else ~0
    unsigned int state;    // the census' answer; error word at the start
};

__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
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

// SEAM: the row may be y = 0 or Ly-1.  KIND: all 32 sites of the word exist, w
// is the partial last word, or either.  All selects are arithmetic (no
// divergent branches, so that the loads are issued together).
enum { WORD_WHOLE, WORD_PART, WORD_ANY };
template <bool SEAM, int KIND>
__device__ __forceinline__ Word share_gather(const Share &g, const char *lat, int x, int lr, int w, int phase)
{
    const int y = SEAM ? share_row_y(g, lr) : lr + (lr > g.ls && g.ls ? -g.lr0 : g.y0 - 1);
    const uint32_t q = (uint32_t)(phase + x + y) & 1u, qm = 0u - q;
    const uint32_t row = __umul24((uint32_t)x, g.PB) + (__umul24((uint32_t)lr, g.RB) + g.PB);   // plane -1 comes first
    const uint32_t at = row + 4u * (uint32_t)w;
    Word o;
    o.own = at + (qm & g.SB);
    const uint32_t oth = at + (~qm & g.SB);
    // the other sublattice one word on: up for odd z, down for even z, round the row's ends
    const uint32_t last = (uint32_t)g.Wq - 1u;
    const uint32_t up = (uint32_t)w == last ? 0u - 4u * last : 4u, dn = w == 0 ? 4u * last : 0u - 4u;
    const uint32_t O = lds32(lat, oth), E = lds32(lat, oth + pick(qm, up, dn));
    o.S = lds32(lat, o.own);
    uint32_t ua = o.own + g.RB, da = o.own - g.RB, um = 0u, dm = 0u;
    if (SEAM) {
        // the seam joins local rows ls (y = Ly-1) and lr0 (y = 0) of planes x and xs
        const uint32_t xs = g.refl ? (uint32_t)(g.Lx - 1 - x) : (uint32_t)x;
        const uint32_t col = o.own - row, sx = __umul24(xs, g.PB) + (g.PB + col);
        const bool su = lr == g.ls, sd = lr == g.lr0;
        ua = su ? sx + __umul24((uint32_t)g.lr0, g.RB) : ua;
        da = sd ? sx + __umul24((uint32_t)g.ls, g.RB) : da;
        um = su ? g.inv : 0u;
        dm = sd ? g.inv : 0u;
    }
    const uint32_t yp = lds32(lat, ua) ^ um, ym = lds32(lat, da) ^ dm;
    const uint32_t xm = lds32(lat, o.own - g.PB), xp = lds32(lat, o.own + g.PB);
    // z neighbour beyond the word: the previous word's top site (the row's
    // last site for w = 0), or the next word's first one
    const uint32_t Et = E << (w == 0 ? 32 - g.rem : 0);
    const uint32_t zd = __builtin_amdgcn_alignbit(O, Et, 31);
    const int top = KIND == WORD_ANY && (uint32_t)w != last ? 31 : g.rem - 1;
    const uint32_t zu = KIND == WORD_WHOLE ? __builtin_amdgcn_alignbit(E, O, 1) : (O >> 1) | ((E & 1u) << top);
    const uint32_t Z = pick(qm, zu, zd);
    const uint32_t s1 = xor3(O, Z, ym), c1 = maj3(O, Z, ym);
    const uint32_t s2 = xor3(yp, xm, xp), c2 = maj3(yp, xm, xp);
    const uint32_t k0 = s1 & s2;
    o.b0 = s1 ^ s2;
    o.b1 = xor3(c1, c2, k0);
    o.b2 = maj3(c1, c2, k0);
    o.gq = (uint32_t)x * g.gx + (uint32_t)y * g.gy + 16u * (uint32_t)w + q;
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

// Updates a row set in one phase.  Tasks (words) run x slowest, then row,
// then word; 64 consecutive tasks are a chunk, chunks go to the waves in turn
// (`turn` carries the turn from set to set), so that the SIMDs get equal
// numbers of chunks.  send: the new words of edge rows go to the neighbours'
// mailboxes.
template <bool SEAM>
__device__ __forceinline__ void share_rows(const Share &g, const ResJob &jb, char *lat, const uint4 *quad,
                                           const uint2 *pair, const uint64_t *thr, const DrawKey &key,
                                           const ResRows &rs, int phase, bool send, unsigned long long *mbox, uint32_t epoch, int &turn, Sums &a)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int W = kResThreads / 64;
    auto each = [&](auto whole_t) {
        constexpr bool WHOLE = decltype(whole_t)::value;
        const int inner = WHOLE ? jb.Wf : 1;
        const int plane = rs.n * inner;
        const int T = g.Lx * plane;
        const int chunks = (T + 63) >> 6;
        int c = wave - turn;
        if (c < 0) c += W;
        for (; c < chunks; c += W) {
            const int tk = c * 64 + lane;
            const bool ok = tk < T;
            const uint32_t tau = (uint32_t)min(tk, T - 1);
            const uint32_t rest = WHOLE ? div_m(tau, (uint32_t)inner, jb.m_w) : tau;
            const int w = WHOLE ? (int)(tau - __umul24(rest, (uint32_t)inner)) : jb.Wf;
            const int x = (int)div_m(rest, (uint32_t)rs.n, rs.m);
            int lr = rs.base + __mul24((int)rest - __mul24(x, rs.n), rs.stride);
            if (rs.skip) lr += lr >= rs.skip ? 2 : 0;
            const Word o = share_gather<SEAM, WHOLE ? WORD_WHOLE : WORD_PART>(g, lat, x, lr, w, phase);
            // chunks of bulk planes read the bulk table at a fixed base
            const bool surf = c * 64 < plane || c * 64 + 63 >= T - plane;
            const bool x0 = x == 0, xl = x == g.Lx - 1;
            uint32_t F;
            if (g.sym && !surf) {
                if (WHOLE) F = bp_flips_quads(o.S, o.b2, o.b1, o.b0, o.gq, key, quad);
                else F = few_flips<true>(o, jb.ng, key, quad, pair, thr, false);
            } else {
                F = few_flips<false>(o, WHOLE ? 8 : jb.ng, key, quad, pair + (x0 ? 256 : xl ? 512 : 0),
                                     thr + kThrPerClass * ((x0 ? 1 : 0) + (xl ? 2 : 0)), g.never);
            }
            if (!WHOLE) F &= (1u << g.rem) - 1u;
            F = ok ? F : 0u;
            const uint32_t V = o.S ^ F;
            if (ok) *(uint32_t *)(lat + o.own) = V;
            share_sums(o, F, surf, x0, xl, a);
            if (send && ok) {
                const unsigned long long v = ((unsigned long long)epoch << 32) | V;
                const uint32_t at = (uint32_t)(phase * g.Lx + x) * (uint32_t)g.Wq + (uint32_t)w;
                if (lr == 1)
                    __hip_atomic_store(mbox + jb.out_off[0] + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lr == g.R)
                    __hip_atomic_store(mbox + jb.out_off[1] + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        turn = (turn + chunks) & (W - 1);
    };
    if (jb.Wf) each(std::true_type{});
    if (jb.ng) each(std::false_type{});
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

__device__ __forceinline__ GroupTask group_task(const Share &g, uint32_t m_c, const ResRows &rs, int tk)
{
    const int C = (int)(g.gy >> 1);
    GroupTask t;
    t.on = tk < g.Lx * rs.n * C;
    const uint32_t k = t.on ? (uint32_t)tk : 0u;
    const uint32_t rest = div_m(k, (uint32_t)C, m_c), gr = k - rest * (uint32_t)C;
    const int x = (int)div_m(rest, (uint32_t)rs.n, rs.m);
    const int lr = rs.base + ((int)rest - x * rs.n) * rs.stride;
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

// Mailbox word k of a phase: words 0 .. n-1 of the lower neighbour's edge row
// (local row 0 here), then the upper neighbour's (row R+1).
__device__ __forceinline__ unsigned long long mail(const Share &g, const ResJob &jb, const unsigned long long *mbox,
                                                   uint32_t epoch, int phase, int k)
{
    const int n = g.Lx * g.Wq;
    const int face = k >= n ? 1 : 0;
    if (k >= 2 * n) return (unsigned long long)epoch << 32;   // nothing to wait for
    return __hip_atomic_load(mbox + jb.in_off[face] + (uint32_t)(phase * n + k - face * n), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

// Receives the edge words that both neighbours updated in a phase into local
// rows 0 and R+1.  Returns false if a wait ran out.
__device__ __forceinline__ bool share_receive(const Share &g, const ResJob &jb, char *lat, GridSync *sync,
                                              const unsigned long long *mbox, uint32_t epoch, int phase)
{
    const int n = g.Lx * g.Wq;
    constexpr int B = 4;   // words polled together by a thread
    unsigned spins = 0;
    for (int k0 = threadIdx.x; k0 < 2 * n; k0 += B * kResThreads) {
        unsigned long long v[B];
        while (true) {
            bool all = true;
#pragma unroll
            for (int i = 0; i < B; ++i) v[i] = mail(g, jb, mbox, epoch, phase, k0 + i * kResThreads);
#pragma unroll
            for (int i = 0; i < B; ++i) all = all && (uint32_t)(v[i] >> 32) == epoch;
            if (all) break;
            __builtin_amdgcn_s_sleep(1);
            if ((++spins & 1023u) == 0) {
                if (__hip_atomic_load(&sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
                if (spins > (1u << 21)) {
                    atomicAdd(&sync->error.v, 1ull);
                    return false;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int k = k0 + i * kResThreads;
            if (k >= 2 * n) break;
            const int face = k >= n ? 1 : 0;
            const int kk = k - face * n;
            const int x = kk / g.Wq, w = kk - x * g.Wq;
            const int lr = face ? g.R + 1 : 0;
            // the neighbour's row is a main row one below local row 1 or one above local row R
            const int y = face ? share_row_y(g, g.R) + 1 : g.y0 - 1;
            const int q = (phase + x + y) & 1;
            *(uint32_t *)(lat + ((uint32_t)(x + 1) * g.PB + (uint32_t)lr * g.RB + (q ? g.SB : 0u) + 4u * (uint32_t)w)) =
                (uint32_t)v[i];
        }
    }
    return true;
}

// Moves a share's rows between the replica's spin array and LDS: local rows
// lo .. hi, LDS word (x, local row, sublattice, word).
template <int FMT, bool LOAD>
__device__ __forceinline__ void share_move(const Share &g, const RepDesc &d, char *lat, int lo, int hi)
{
    const int nr = hi - lo + 1, RW = 2 * g.Wq;
    const int n = g.Lx * nr * RW;
    for (int k = threadIdx.x; k < n; k += kResThreads) {
        const int r = k / RW, c = k - r * RW;
        const int x = r / nr, lr = lo + (r - x * nr);
        const int y = share_row_y(g, lr);
        uint32_t *l = (uint32_t *)(lat + ((uint32_t)(x + 1) * g.PB + (uint32_t)lr * g.RB)) + c;
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
// decides for all).  About 20 ms on a busy device; called by thread 0.
__device__ __forceinline__ unsigned int res_census(ResSync *rs, unsigned int members)
{
    const unsigned int old = atomicAdd(&rs->count, 1u);
    if (old + 1 == members) atomicCAS(&rs->state, (unsigned)RES_WAIT, (unsigned)RES_GO);
    for (unsigned spins = 0;; ++spins) {
        const unsigned int s = __hip_atomic_load(&rs->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s != RES_WAIT) return s;
        if (spins > 20000u) atomicCAS(&rs->state, (unsigned)RES_WAIT, (unsigned)RES_ABORT);
        __builtin_amdgcn_s_sleep(8);
    }
}

// What bounds it: VALU issue (the Philox word and the threshold lookups, as
// in bp_march).  16 waves per workgroup and one workgroup per CU: a CU's
// whole LDS is one share, which keeps the edge rows few against the interior
// (two workgroups of 8 waves per CU: 64 x 40x120x120 25.7 against 23.8 us per
// sweep, 3 x 160x480x600 97 against 73).  Per sweep, before (launch chain, or
// persistent kernel) and now: 12x24x24 14 and 3.7 us, 168 ladder films 37 and
// 3.0 us, 64 x 40x120x120 31 and 23.8 us, 96 uneven films int8 85 and 70 us,
// 3 x 160x480x600 int8 95 and 75 us, persistent 78 and 74 us.
// SMALL: no clusters, and films of few words, updated one four-site group per
// lane (share_groups).
template <int FMT, bool SMALL>
__global__ __launch_bounds__(kResThreads) void k_resident(const RepDesc *__restrict__ descs,
                                                          const RepState *__restrict__ st,
                                                          const ResJob *__restrict__ jobs,
                                                          const int *__restrict__ first, int njobs, int members,
                                                          uint32_t n, ResSync *rs, GridSync *sync, int4 *part,
                                                          unsigned long long *mbox, int check_error)
{
    extern __shared__ uint32_t smem[];
    __shared__ ResTables tb;
    __shared__ ResCtl ctl_s;
    static_assert(sizeof(ResTables) + sizeof(ResCtl) <= kResStaticLds, "the host's LDS budget counts on it");
    uint2 *pair = tb.pair;
    uint64_t *thr = tb.thr;
    ResCtl *ctl = &ctl_s;
    char *lat = (char *)smem;
    const int tid = threadIdx.x;
    if (check_error) {
        if (tid == 0)
            ctl->state = __hip_atomic_load(&sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
        __syncthreads();
        if (ctl->state) return;
        __syncthreads();
    }
    const uint32_t epoch0 = rs->epoch;
    for (int j = first[blockIdx.x]; j < first[blockIdx.x + 1]; ++j) {
        const ResJob &jb = jobs[j];   // uniform: scalar loads where used
        const RepDesc &d = descs[jb.rep];
        Share g;
        g.Lx = d.Lx; g.Wq = d.Wq;
        g.rem = (d.Lz >> 1) - 32 * (d.Wq - 1);
        g.SB = 4u * (uint32_t)g.Wq;
        g.RB = 2u * g.SB;
        g.PB = (uint32_t)(jb.R + 2) * g.RB;
        g.R = jb.R; g.ls = jb.ls; g.lr0 = jb.lr0; g.y0 = jb.y0;
        g.inv = d.seam_invert ? ~0u : 0u;
        g.refl = d.seam_reflect != 0;
        g.never = d.never_mask != 0;
        g.sym = d.sym != 0 && !g.never;
        g.gy = 2u * (uint32_t)d.C;
        g.gx = g.gy * (uint32_t)d.Ly;
        DrawKey key{st[jb.rep].t, d.replica, d.key0, d.key1};
        // tables: three classes' pair tables (a one-layer film has one class), all thresholds
        for (int k = tid; k < 768; k += kResThreads) {
            const int e = k & 255, cls = g.Lx == 1 ? 3 : k >> 8;
            const int ev = (e & 1) | ((e >> 1) & 2) | ((e >> 2) & 4) | ((e >> 3) & 8);
            const int od = ((e >> 1) & 1) | ((e >> 2) & 2) | ((e >> 3) & 4) | ((e >> 4) & 8);
            pair[k] = make_uint2(d.thr_m1[cls * kThrPerClass + ev], d.thr_m1[cls * kThrPerClass + od]);
        }
        for (int k = tid; k < 256 && g.sym; k += kResThreads) tb.quad[k] = quad_entry(d, k);
        if (tid < kThrEntries) thr[tid] = d.thr[tid];
        if (tid < 8) (&ctl->acc[0][0])[tid] = 0;
        if (tid == 8) ctl->bad = ~0u;
        // the planes beyond the free surfaces
        for (uint32_t k = tid; k < g.PB / 4; k += kResThreads) {
            ((uint32_t *)lat)[k] = 0u;
            ((uint32_t *)(lat + (uint32_t)(g.Lx + 1) * g.PB))[k] = 0u;
        }
        const bool cluster = !SMALL && jb.P > 1;
        share_move<FMT, true>(g, d, lat, cluster ? 0 : 1, cluster ? g.R + 1 : g.R);
        if (cluster && tid == 0) ctl->state = res_census(rs, (unsigned)members);
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
            for (int k = 0; k < kSmallTasks; ++k) gt[k] = group_task(g, jb.m_c, m, tid + k * kResThreads);
            gt0 = group_task(g, jb.m_c, z, tid);
            // whole waves without a group skip the phase
            main_tasks = g.Lx * m.n * d.C - (tid & ~63);
            row0_tasks = g.Lx * d.C;
        }
        bool good = true;
        const int phases = g.lr0 ? 4 : 2;
        for (uint32_t s = 0; s < n && good; ++s, ++key.t) {
            Sums a = {0, 0, 0, 0, 0, 0, 0, 0};
            int turn = 0;
#pragma unroll 1
            for (int phase = 0; phase < phases; ++phase) {
                const bool xch = cluster && (phase == 0 || (phase == 1 && s + 1 < n));
                const uint32_t ep = epoch0 + 2u * s + (uint32_t)phase + 1u;
                if (SMALL) {
                    if (phase < 2) {
                        for (int k = 0; k < kSmallTasks; ++k)
                            if (k * kResThreads < main_tasks) group_update(g, gt[k], lat, pair, thr, key, phase, a);
                    } else if ((int)(tid & ~63) < row0_tasks) {
                        group_update(g, gt0, lat, pair, thr, key, phase, a);
                    }
                } else {
#pragma unroll 1
                    for (int k = phase < 2 ? RES_EDGE : RES_ROW0; k <= (phase < 2 ? RES_INNER : RES_ROW0); ++k) {
                        const ResRows &rs = jb.set[k];
                        if (rs.n == 0) continue;
                        const bool send = xch && k == RES_EDGE;
                        if (rs.seam) share_rows<true>(g, jb, lat, tb.quad, pair, thr, key, rs, phase, send, mbox, ep, turn, a);
                        else share_rows<false>(g, jb, lat, tb.quad, pair, thr, key, rs, phase, send, mbox, ep, turn, a);
                    }
                    if (xch && !share_receive(g, jb, lat, sync, mbox, ep, phase)) atomicMin(&ctl->bad, s + 1u);
                }
                if (phase + 1 < phases) __syncthreads();
            }
            // the sweep's changes (see bp_march), one LDS add per wave and quantity
            const int dB = -4 * (a.A0 + 2 * a.A1 + 4 * a.A2) + 16 * a.NF - 4 * a.NFU + a.KDM;
            const int dM = 2 * a.NF - 4 * a.NFU;
            int *acc = ctl->acc[s & 1];
            const int vB = __reduce_add_sync(~0ull, dB), vM = __reduce_add_sync(~0ull, dM);
            int v1 = 0, vn = 0;
            if (__any((a.D1 | a.Dn) != 0)) {
                v1 = __reduce_add_sync(~0ull, a.D1);
                vn = __reduce_add_sync(~0ull, a.Dn);
            }
            if ((tid & 63) == 0) {
                atomicAdd(&acc[0], vB);
                atomicAdd(&acc[1], vM);
                if (v1) atomicAdd(&acc[2], v1);
                if (vn) atomicAdd(&acc[3], vn);
            }
            __syncthreads();
            // the other half serves the next sweep, whose barriers order this clear before its reuse
            if (tid == 0) {
                part[(size_t)s * njobs + jb.id] = make_int4(acc[0], acc[1], acc[2], acc[3]);
                acc[0] = acc[1] = acc[2] = acc[3] = 0;
            }
            // (a faster wave may be in sweep s+1 already: its failure counts there)
            good = ctl->bad > s + 1u;
        }
        if (good) share_move<FMT, false>(g, d, lat, 1, g.R);
        __syncthreads();
    }
}

// Closes a resident launch of n sweeps: one workgroup per replica.  Sums the
// shares' changes, stores the records and advances the replica; if the launch
// was aborted, sweeps the cluster replicas here first.
template <int FMT>
__global__ __launch_bounds__(kResThreads) void k_resident_close(const RepDesc *__restrict__ descs, RepState *st,
                                                                const ResRep *__restrict__ reps, int njobs,
                                                                uint32_t n, ResSync *rs, GridSync *sync, int4 *part,
                                                                int check_error)
{
    __shared__ long long sum[kResMaxSweeps][4];
    __shared__ uint64_t thr[kThrEntries];
    __shared__ int run;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const ResRep rr = reps[blockIdx.x];
    const RepDesc &d = descs[rr.rep];
    if (tid == 0) {
        const bool err = check_error && __hip_atomic_load(&sync->error.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
                const int4 w = part[(size_t)s * njobs + rr.job0 + p];
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
            rs->count = 0;
            rs->state = RES_WAIT;
            rs->done = 0;
            rs->epoch += 2u * n + 2u;
        }
    }
}

// ---------------------------------------------------------------------------
// Host-callable launchers
// ---------------------------------------------------------------------------
template <int FMT, bool SMALL>
static hipError_t launch_resident_as(const RepDesc *descs, RepState *st, const ResJob *jobs, const int *first,
                                     const ResRep *reps, int grid, int njobs, int members, int nreps, size_t lds,
                                     uint32_t n, ResSync *rs, GridSync *sync, int4 *part, unsigned long long *mbox,
                                     int check_error, hipStream_t s)
{
    hipLaunchKernelGGL((k_resident<FMT, SMALL>), dim3(grid), dim3(kResThreads), lds, s, descs, st, jobs, first, njobs,
                       members, n, rs, sync, part, mbox, check_error);
    hipLaunchKernelGGL(k_resident_close<FMT>, dim3(nreps), dim3(kResThreads), 0, s, descs, st, reps, njobs, n, rs,
                       sync, part, check_error);
    return hipGetLastError();
}

// Lets the kernels use `bytes` of dynamic LDS.
hipError_t resident_lds_limit(int fmt, size_t bytes)
{
    const void *f[2] = {fmt == ISLF_SPIN_INT8 ? (const void *)k_resident<ISLF_SPIN_INT8, false>
                                              : (const void *)k_resident<ISLF_SPIN_BITPACK, false>,
                        fmt == ISLF_SPIN_INT8 ? (const void *)k_resident<ISLF_SPIN_INT8, true>
                                              : (const void *)k_resident<ISLF_SPIN_BITPACK, true>};
    hipError_t e = hipSuccess;
    for (int i = 0; i < 2 && e == hipSuccess; ++i)
        e = hipFuncSetAttribute(f[i], hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    return e;
}

hipError_t launch_resident(int fmt, bool small, const RepDesc *descs, RepState *st, const ResJob *jobs,
                           const int *first, const ResRep *reps, int grid, int njobs, int members, int nreps,
                           size_t lds, uint32_t n, ResSync *rs, GridSync *sync, int4 *part, unsigned long long *mbox,
                           int check_error, hipStream_t s)
{
    auto f = fmt == ISLF_SPIN_INT8
                 ? (small ? launch_resident_as<ISLF_SPIN_INT8, true> : launch_resident_as<ISLF_SPIN_INT8, false>)
                 : (small ? launch_resident_as<ISLF_SPIN_BITPACK, true> : launch_resident_as<ISLF_SPIN_BITPACK, false>);
    return f(descs, st, jobs, first, reps, grid, njobs, members, nreps, lds, n, rs, sync, part, mbox, check_error, s);
}

}  // namespace islf
