// pass.h -- device code of one heat-bath pass: addressing, staples, random
// draws and the Cabibbo-Marinari heat bath.  Shared by the single-lattice and
// the batched kernels of pass_kernels.h.
//
// What bounds a pass.  A SIMD issues one vector instruction per 4 cycles, FP64,
// FP32 and 64-bit integer alike (moves and bit operations in half of that when
// four waves share it), and one wave alone only one per 8 cycles.  A tile of 64
// updates is about 3500 vector instructions in all (three waves of 1150 to 1170
// each, 32^4) for 864 (FP64) or 432 (FP32) bytes per update, so a
// pass needs at least two, better three or four waves per SIMD that are ready
// to issue, and every instruction counts.
#pragma once

#include "launch.h"

namespace su3hb {
namespace {

// ---------------------------------------------------------------------------
// Addresses.  A link's byte offset in its block is a 32-bit number, added to a
// scalar base by the load itself, as long as a block has less than 4 GiB
// (pass_big); larger lattices take 64-bit offsets (BIG).
// ---------------------------------------------------------------------------
template <bool BIG> struct OffsetOf {
    using type = uint32_t;
};
template <> struct OffsetOf<true> {
    using type = uint64_t;
};
template <bool BIG> using offset_t = typename OffsetOf<BIG>::type;

template <typename R, bool BIG> __device__ __forceinline__ offset_t<BIG> link_offset(int n)
{
    constexpr uint32_t E = sizeof(store_t<R>);
    const uint32_t u = (uint32_t)n, in_tile = u & (kTile - 1);
    if constexpr (BIG)
        return (uint64_t)(u >> 4) * (kEntries * kTile * E) + in_tile * E;
    else
        return u * (kEntries * E) - in_tile * ((kEntries - 1) * E);
}

// One (direction, parity) block of links.
template <typename R> struct Block {
    const char *base;
};
template <typename R, bool BIG = true>
__device__ __forceinline__ Block<R> block_of(const store_t<R> *links, const Geom &g, int dir, int par)
{
    constexpr uint32_t kLink = kEntries * sizeof(store_t<R>);
    if constexpr (BIG) return Block<R>{(const char *)links + (size_t)(dir * 2 + par) * (size_t)g.stride * kLink};
    // a block has less than 4 GiB
    return Block<R>{(const char *)links + (uint64_t)(uint32_t)(dir * 2 + par) * ((uint32_t)g.stride * kLink)};
}

// Rows 0 and 1 of the link at offset o (row 2 is left undefined).
template <typename R, typename O> __device__ __forceinline__ void load_rows(M3<R> &m, Block<R> b, O o)
{
    const store_t<R> *p = (const store_t<R> *)(b.base + o);
#pragma unroll
    for (int e = 0; e < kEntries; ++e) {
        const store_t<R> v = p[e * kTile];
        m.e[e / 3][e % 3] = Cx<R>{v.x, v.y};
    }
}
// Rows 0 and 1 of two links, entry by entry in turn: the two are the same
// link for two neighbouring sites, so the second use finds the line in cache.
template <typename R, typename O>
__device__ __forceinline__ void load_rows_pair(M3<R> &m, Block<R> bm, O om, M3<R> &n, Block<R> bn, O on)
{
    const store_t<R> *p = (const store_t<R> *)(bm.base + om), *q = (const store_t<R> *)(bn.base + on);
#pragma unroll
    for (int e = 0; e < kEntries; ++e) {
        const store_t<R> v = p[e * kTile], w = q[e * kTile];
        m.e[e / 3][e % 3] = Cx<R>{v.x, v.y};
        n.e[e / 3][e % 3] = Cx<R>{w.x, w.y};
    }
}

// Nontemporal access to the link a pass updates: no other thread of the pass
// reads it, so it should not displace reusable staple links from L2.
template <typename R> struct NtVec;
template <> struct NtVec<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct NtVec<float> { typedef float type __attribute__((ext_vector_type(2))); };

template <typename R, typename O> __device__ __forceinline__ void load_own(M3<R> &m, Block<R> b, O o)
{
    typedef typename NtVec<R>::type V;
    const V *p = (const V *)(b.base + o);
#pragma unroll
    for (int e = 0; e < kEntries; ++e) {
        const V v = __builtin_nontemporal_load(p + e * kTile);
        m.e[e / 3][e % 3] = Cx<R>{v.x, v.y};
    }
}
// FP64: nontemporal store (a plain one: -3 % at 32^4); FP32, which is not
// bound by memory: a plain store (+1 %).
template <typename R, typename O> __device__ __forceinline__ void store_own(Block<R> b, O o, const M3<R> &m)
{
    typedef typename NtVec<R>::type V;
    V *p = (V *)(b.base + o);
#pragma unroll
    for (int e = 0; e < kEntries; ++e) {
        V v;
        v.x = m.e[e / 3][e % 3].re;
        v.y = m.e[e / 3][e % 3].im;
        if constexpr (sizeof(R) == 8)
            __builtin_nontemporal_store(v, p + e * kTile);
        else
            p[e * kTile] = v;
    }
}

// The site of a link: coordinates, half-index and layer.
struct Site {
    int x[4];
    int i;      // half-index within the layer
    int layer;  // 0 on a single torus
};

// The site at pass-order position v (order_site), v < nlat * Vh.
template <bool DLT> __device__ __forceinline__ Site site_of(const Geom &g, int par, int v)
{
    Site s;
    s.layer = DLT && v >= g.Vh ? 1 : 0;
    s.i = order_site(g, par, DLT ? v - s.layer * g.Vh : v, s.x);
    return s;
}

// What one step along a direction adds to the half-index, and the layer bit it
// flips.  Along directions 1..3 a step moves lex by an even number, so the
// half-index moves by the same amount whatever the other coordinates; along
// direction 0 it depends on x0 alone.  So steps along two directions add up.
struct Step {
    int di;
    int flip;
};
template <int D, int S> __device__ __forceinline__ Step step_of(const Geom &g, const Site &s)
{
    const bool edge = S > 0 ? s.x[D] == g.L[D] - 1 : s.x[D] == 0;
    const int odd = s.x[0] & 1;
    const int by = D != 0 ? g.hs[D] : S > 0 ? odd : 1 - odd;
    Step r;
    r.di = S > 0 ? (edge ? -g.wrap[D] : by) : (edge ? g.wrap[D] : -by);
    r.flip = edge ? (int)((g.flip >> D) & 1u) : 0;
    return r;
}

// Plane element of the site after the steps a (and b).
template <bool DLT> __device__ __forceinline__ int elem(const Geom &g, const Site &s, Step a)
{
    const int i = s.i + a.di;
    return DLT ? i + ((s.layer ^ a.flip) ? g.Vh : 0) : i;
}
template <bool DLT> __device__ __forceinline__ int elem(const Geom &g, const Site &s, Step a, Step b)
{
    const int i = s.i + a.di + b.di;
    return DLT ? i + ((s.layer ^ a.flip ^ b.flip) ? g.Vh : 0) : i;
}

// The staple directions nu != MU in increasing order.
template <int MU> constexpr int kNu0 = MU == 0 ? 1 : 0;
template <int MU> constexpr int kNu1 = MU <= 1 ? 2 : 1;
template <int MU> constexpr int kNu2 = MU <= 2 ? 3 : 2;

// The two steps along the direction of wave w (2, 0, 1 of the staple
// directions for w = 0, 1, 2): step_of with the direction chosen by selects
// that are uniform over the wave, without branches.
template <int MU, bool DLT>
__device__ __forceinline__ void steps_of(const Geom &g, const Site &s, int w, Step &up, Step &dn)
{
    constexpr int A = kNu2<MU>, B = kNu0<MU>, C = kNu1<MU>;
    const auto pick = [w](int a, int b, int c) { return w == 0 ? a : w == 1 ? b : c; };
    const int x = pick(s.x[A], s.x[B], s.x[C]), L = pick(g.L[A], g.L[B], g.L[C]);
    const int hs = pick(g.hs[A], g.hs[B], g.hs[C]), wrap = pick(g.wrap[A], g.wrap[B], g.wrap[C]);
    const int odd = s.x[0] & 1;
    const bool along0 = B == 0 && w == 1;
    const bool top = x == L - 1, bottom = x == 0;
    up.di = top ? -wrap : along0 ? odd : hs;
    dn.di = bottom ? wrap : along0 ? odd - 1 : -hs;
    const int bit = DLT ? (int)((g.flip >> pick(A, B, C)) & 1u) : 0;
    up.flip = DLT && top ? bit : 0;
    dn.flip = DLT && bottom ? bit : 0;
}

// ---------------------------------------------------------------------------
// Staple of U_MU(x): A = sum over nu != MU (ascending) of D_nu,
//   D_nu = up_nu + dn_nu,
//   up_nu = U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+ = a (c b)^+,
//   dn_nu = U_nu(x+mu-nu)^+ U_mu(x-nu)^+ U_nu(x-nu) = (e d)^+ f,
// with a = U_nu(x+mu), b = U_mu(x+nu), c = U_nu(x), d = U_nu(x+mu-nu),
// e = U_mu(x-nu), f = U_nu(x-nu).  up_nu is the plaquette based at x, dn_nu
// the one based at x - nu.
//
// Rounding order, fixed for every kernel: c b, e d and a (c b)^+ are SU(3)
// products (rows 0 and 1 formed, row 2 rebuilt); dn_nu is formed entry by
// entry; D_nu = up_nu + dn_nu entry by entry; A = (D_0 + D_1) + D_2 over the
// three directions in increasing order.  With per-layer couplings A is the sum
// of the six weighted terms, one multiply-add after the other.  All kernels
// add in exactly this order, so a lattice gets the same bits from each of them.
// ---------------------------------------------------------------------------

// (ed^+ f)_rc
template <typename R> __device__ __forceinline__ Cx<R> dn_entry(const M3<R> &ed, const M3<R> &f, int r, int c)
{
    Cx<R> dn = cmul_cn(ed.e[0][r], f.e[0][c]);
    dn = cmadd_cn(dn, ed.e[1][r], f.e[1][c]);
    return cmadd_cn(dn, ed.e[2][r], f.e[2][c]);
}

// D = up + (e d)^+ f with D = up on entry.  CROSS: also cross = (e d)^+ f where
// `crosses` (the lower plaquette's base site lies in the other layer of a
// double-layered torus), else 0.
template <typename R, bool CROSS>
__device__ __forceinline__ void add_dn(M3<R> &D, const M3<R> &ed, const M3<R> &f, M3<R> &cross, bool crosses)
{
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Cx<R> dn = dn_entry(ed, f, r, c);
            D.e[r][c].re += dn.re;
            D.e[r][c].im += dn.im;
            if constexpr (CROSS) {
                cross.e[r][c].re = crosses ? dn.re : R(0);
                cross.e[r][c].im = crosses ? dn.im : R(0);
            }
        }
}

// Offsets of the six links of direction nu's two staples.
template <bool BIG> struct StapleAt {
    offset_t<BIG> here, mu, up, dn, mu_dn;  // x, x + mu, x + nu, x - nu, x + mu - nu
    bool crosses;                           // x - nu lies in the other layer
};
template <int MU, typename R, bool DLT, bool BIG>
__device__ __forceinline__ StapleAt<BIG> staple_at(const Geom &g, const Site &s, Step mu, Step up, Step dn)
{
    StapleAt<BIG> a;
    a.here = link_offset<R, BIG>(DLT ? s.i + (s.layer ? g.Vh : 0) : s.i);
    a.mu = link_offset<R, BIG>(elem<DLT>(g, s, mu));
    a.up = link_offset<R, BIG>(elem<DLT>(g, s, up));
    a.dn = link_offset<R, BIG>(elem<DLT>(g, s, dn));
    a.mu_dn = link_offset<R, BIG>(elem<DLT>(g, s, mu, dn));
    a.crosses = DLT && dn.flip;
    return a;
}

// How many of the six links of a direction are requested before the random
// draw.  More cost registers, and so waves that share a SIMD: FP64 four (152
// registers, three waves; with two 8^4 takes 460 instead of 420 us per 8
// sweeps, 16^4 708 instead of 676 us), FP32 two (six waves; with four 16^4
// takes 525 instead of 508 us, a batch of jobs 22.4 instead of 22.1 ms).
template <typename R> constexpr int kEarlyLinks = sizeof(R) == 8 ? 4 : 2;

// The two staples of direction nu.  TWOB: D = up and cross = dn, to be weighted
// where they are added.  between(): work that needs none of the links, done while
// the first kEarlyLinks are on their way (the compiler would sink the loads or
// hoist the products, hence the barriers).
template <int MU, typename R, bool CROSS, bool TWOB, bool BIG, typename Between>
__device__ __forceinline__ void staple_nu(M3<R> &D, M3<R> &cross, const store_t<R> *links, const Geom &g, int par, int nu,
                                          const StapleAt<BIG> &at, Between between)
{
    const int opp = par ^ 1;
    const Block<R> umu = block_of<R, BIG>(links, g, MU, opp), unu_par = block_of<R, BIG>(links, g, nu, par),
                   unu_opp = block_of<R, BIG>(links, g, nu, opp);
    M3<R> b, e, c, d, a, f;
    load_rows_pair(b, umu, at.up, e, umu, at.dn);
    if constexpr (kEarlyLinks<R> == 4) load_rows_pair(c, unu_par, at.here, d, unu_par, at.mu_dn);
    __builtin_amdgcn_sched_barrier(0);
    between();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kEarlyLinks<R> == 2) {
        load_rows_pair(c, unu_par, at.here, d, unu_par, at.mu_dn);
        load_rows_pair(a, unu_opp, at.mu, f, unu_opp, at.dn);
    }
    rebuild_row2(b);
    rebuild_row2(d);
    const M3<R> cb = mul_nn_su3(c, b);
    if constexpr (kEarlyLinks<R> == 4) load_rows_pair(a, unu_opp, at.mu, f, unu_opp, at.dn);
    const M3<R> ed = mul_nn_su3(e, d);
    D = mul_nd_su3(a, cb);
    rebuild_row2(f);
    if constexpr (TWOB) {
        set_zero(cross);
        acc_dn(cross, ed, f);
    } else {
        add_dn<R, CROSS>(D, ed, f, cross, at.crosses);
    }
}

// The same from b and e (rows 0 and 1) at hand, in a wave that forms all three
// directions in turn.
template <int MU, typename R, bool CROSS, bool TWOB, bool BIG>
__device__ __forceinline__ void staple_from(M3<R> &D, M3<R> &cross, M3<R> b, const M3<R> &e, const store_t<R> *links,
                                            const Geom &g, int par, int nu, const StapleAt<BIG> &at)
{
    const Block<R> unu_par = block_of<R, BIG>(links, g, nu, par), unu_opp = block_of<R, BIG>(links, g, nu, par ^ 1);
    M3<R> c, d, a, f;
    load_rows_pair(c, unu_par, at.here, d, unu_par, at.mu_dn);
    rebuild_row2(b);
    rebuild_row2(d);
    const M3<R> cb = mul_nn_su3(c, b);
    const M3<R> ed = mul_nn_su3(e, d);
    load_rows_pair(a, unu_opp, at.mu, f, unu_opp, at.dn);
    D = mul_nd_su3(a, cb);
    rebuild_row2(f);
    if constexpr (TWOB) {
        set_zero(cross);
        acc_dn(cross, ed, f);
    } else {
        add_dn<R, CROSS>(D, ed, f, cross, at.crosses);
    }
}

// ---------------------------------------------------------------------------
// Cabibbo-Marinari heat bath of one link in staple A.  W = U A; for subgroup
// (i,j): v = 1/2 (Re(w_ii + w_jj), -Im(w_ij + w_ji), Re(w_ji - w_ij),
// Im(w_jj - w_ii)), k = |v|, alpha = 2 beta k / 3.  Kennedy-Pendleton attempt t
// uses Philox block (lid, sweep, sub<<32 | t, heat-bath tag):
//   lambda^2 = -(ln u1 + cos^2(2 pi u2) ln u3) / (2 alpha), accept iff u4^2 <= 1 - lambda^2,
//   a0 = 1 - 2 lambda^2, cos(theta) = 2 u5 - 1, phi = 2 pi u6;
// then rows i, j of U and W are multiplied from the left by r = P(a) P(v/k)
// with P(p) = [[p0 + i p3, p2 + i p1], [-p2 + i p1, p0 - i p3]].
// The SU(2) step runs in the link precision R (FP64 links: FP64 throughout,
// accept decisions in FP64); the uniforms are formed exactly in FP64 first.
// The link is reunitarised in FP64 at the end.
// ---------------------------------------------------------------------------

// What an attempt needs from its random numbers, independent of the link:
// q = ln u1 + cos^2(2 pi u2) ln u3 (so lambda^2 = -q / (2 alpha)), u4^2,
// cos(theta), sin(theta) cos(phi), sin(theta) sin(phi).
template <typename R> struct KPDraw {
    R q, u4sq, cth, sc, ss;
};

template <typename R> __device__ __forceinline__ KPDraw<R> kp_draw(uint32_t lid, uint64_t sweep, uint64_t seed, int sub, int t)
{
    const U64x4 w = philox_link(lid, sweep, ((uint64_t)sub << 32) | (uint64_t)t, seed);
    const uint32_t h2 = (uint32_t)w.w[2], h4 = (uint32_t)(w.w[2] >> 32);
    const uint32_t h5 = (uint32_t)w.w[3], h6 = (uint32_t)(w.w[3] >> 32);
    const R u1 = R(unif52(w.w[0])), u3 = R(unif52(w.w[1]));
    const R u4 = R(unif32(h4)), u5 = R(unif32(h5));
    KPDraw<R> d;
    d.u4sq = u4 * u4;
    d.cth = R(2) * u5 - R(1);
    // FP64: |cth| < 1 (u5 is never 0 or 1), so the argument is positive
    const R sth = sqrt_pos_r(R(1) - d.cth * d.cth);
    R sph, cph, c2;
    if constexpr (sizeof(R) == 8) {
        c2 = cos2_2pi_u32(h2);
        d.q = log_unit(u1) + c2 * log_unit(u3);
        sincos_2pi_u32(h6, &sph, &cph);
    } else {
        c2 = cospi_sq_0to2(R(2) * R(unif32(h2)));
        d.q = logf(u1) + c2 * logf(u3);
        sincospi_0to2(R(2) * R(unif32(h6)), &sph, &cph);
    }
    d.sc = sth * cph;
    d.ss = sth * sph;
    return d;
}

// A matrix in LDS, entry-major over the 64 lanes.
template <typename R, int N> __device__ __forceinline__ void lds_put(store_t<R> (*buf)[64], int lane, const M3<R> &m)
{
#pragma unroll
    for (int e = 0; e < N; ++e) {
        store_t<R> v;
        v.x = m.e[e / 3][e % 3].re;
        v.y = m.e[e / 3][e % 3].im;
        buf[e][lane] = v;
    }
}
template <typename R, int N> __device__ __forceinline__ M3<R> lds_get(const store_t<R> (*buf)[64], int lane)
{
    M3<R> m;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const store_t<R> v = buf[e][lane];
        m.e[e / 3][e % 3] = Cx<R>{v.x, v.y};
    }
    return m;
}

// The draws of 64 lanes in LDS.
template <typename R> struct DrawLds {
    store_t<R> q_u4sq[64], cth_sc[64];
    R ss[64];
};
template <typename R> __device__ __forceinline__ void draw_put(DrawLds<R> &buf, int lane, const KPDraw<R> &d)
{
    store_t<R> a, b;
    a.x = d.q;
    a.y = d.u4sq;
    b.x = d.cth;
    b.y = d.sc;
    buf.q_u4sq[lane] = a;
    buf.cth_sc[lane] = b;
    buf.ss[lane] = d.ss;
}
template <typename R> __device__ __forceinline__ KPDraw<R> draw_get(const DrawLds<R> &buf, int lane)
{
    const store_t<R> a = buf.q_u4sq[lane], b = buf.cth_sc[lane];
    return KPDraw<R>{a.x, a.y, b.x, b.y, buf.ss[lane]};
}

// Attempts and acceptances of a wave, uniform over it.
struct Counts {
    uint32_t att, acc;
};
__device__ __forceinline__ uint32_t lanes_of(bool p) { return (uint32_t)__popcll(__ballot(p)); }

// Second attempts made ahead by three waves.  An attempt misses where u4^2 >
// 1 - lambda^2; lambda^2 is a few per cent at the usual couplings, so all but
// some misses in a thousand have u4^2 above kMayMiss: 22.5 % of the lanes, 14 of 64, of
// which two do miss.  The second draws of the first kPoolSlots of these lanes, for all
// three subgroups, are made together by one wave: a third of the work of
// drawing for every lane.  A lane that misses without one draws when it does.
constexpr int kPoolSlots = 21;
constexpr double kMayMiss = 0.6;
template <typename R> __device__ __forceinline__ int pool_slot(R u4sq, int sub, int lane)
{
    const bool may = u4sq > R(kMayMiss);
    const uint64_t m = __ballot(may);
    const int rank = __popcll(m & ((1ull << lane) - 1));
    return may && rank < kPoolSlots ? sub * kPoolSlots + rank : -1;
}

// A round of 64 further attempts for the lanes of the mask m, each lane one: the
// asking lanes get 64 / (their number) attempts each, which lanes rank, rank +
// count, rank + 2 count, ... make.  So a wave at strong coupling, where all its
// lanes may miss many times, waits for some tens of attempts, not for the
// slowest lane's, and a single asker has all its attempts at once.
struct Round {
    int rank;        // of an asking lane among them
    int asker;       // the lane whose attempt this one makes,
    int ahead;       // and which of its `each` attempts
    int each;
    uint64_t every;  // bits 0, count, 2 count, ... below each count
    uint32_t inv;
    // x / count for x < 64, exact: inv = floor(2^16 / count) + 1 is above 2^16 / count by at most 1, and 64 < 2^16 / 64
    __device__ __forceinline__ int attempts(int x) const { return (int)((uint32_t)x * inv >> 16); }
    __device__ __forceinline__ Round(uint64_t m, int lane)
    {
        const int count = __popcll(m);
        inv = 65536u / (uint32_t)count + 1;
        each = 64 / count;
        every = 1;
        for (int s = count; s < each * count; s += s) every |= every << s;
        if (each * count < 64) every &= (1ull << each * count) - 1;
        const uint64_t below = (1ull << lane) - 1;
        const bool asks = m >> lane & 1;
        rank = __popcll(m & below);
        // lane r learns which lane has rank r: the others take the ranks from count on
        const int to = asks ? rank : count + __popcll(~m & below);
        const int holder = __builtin_amdgcn_ds_permute(to << 2, lane);
        ahead = attempts(lane);
        asker = __shfl(holder, lane - ahead * count);
    }
};
// Sum over the wave of a number below 128.
__device__ __forceinline__ uint32_t sum_small(int x)
{
    uint32_t s = 0;
#pragma unroll
    for (int b = 0; b < 7; ++b) s += lanes_of(x >> b & 1) << b;
    return s;
}

// Has the matrix formed here, not later.
template <typename R> __device__ __forceinline__ void pin(M3<R> &m)
{
#pragma unroll
    for (int e = 0; e < 9; ++e) __asm__ __volatile__("" : "+v"(m.e[e / 3][e % 3].re), "+v"(m.e[e / 3][e % 3].im));
}

// The heat bath proper.  Returns Re Tr W after the last subgroup, i.e.
// Re Tr(U_new A) before the final reunitarisation.  Projections are of 2 v; the
// factor is exact and cancels.  q32 = 3/(2 beta).
// All 64 lanes take part; only the `active` ones count.  There is no branch
// per lane: a rejected attempt (3 % of them, so nearly every wave has one)
// rotates by the identity, which leaves finite rows as they are (and carries a
// NaN of one row into others: keep_nan_rows).
//
// The draw of attempt 0 is made ahead, first(sub), and that of attempt 1 for
// some lanes, second(sub, u4sq, made), u4sq being the first draw's: PARK, the
// wave then has registers for U and W but not for a draw beside them, and
// leaves them in park_u and park_w (nine entries per lane of LDS each) during
// any further one.  Without PARK all attempts of several are made here.
// MASK: lanes that want no attempt are masked off.  Drawing in all of them
// takes power and so clock rate (one wave per tile, 32^4 to 64^4 FP64: +3 to
// +5 %; three waves, FP32 32^4 +3 %); waves that wait for the chain of
// instructions and not for the clock lose up to 15 % by the branch.
template <typename R, bool HIT1, bool PARK, bool MASK, typename First, typename Second>
__device__ __forceinline__ double heatbath(M3<R> &U, const M3<R> &A, R q32, uint32_t lid, uint64_t sweep, uint64_t seed,
                                           int nhit, bool active, Counts &n, store_t<R> (*park_u)[64],
                                           store_t<R> (*park_w)[64], int lane, First first, Second second)
{
    M3<R> W = mul_nn(U, A);
    // without this, rows that the first subgroup does not read are formed after its round of attempts,
    // and everything they are made of waits in registers
    if constexpr (!HIT1) pin(W);
#pragma unroll
    for (int sub = 0; sub < 3; ++sub) {
        const int i = (sub == 1) ? 1 : 0;
        const int j = (sub == 0) ? 1 : 2;
        const R v0 = W.e[i][i].re + W.e[j][j].re;
        const R v1 = -(W.e[i][j].im + W.e[j][i].im);
        const R v2 = W.e[j][i].re - W.e[i][j].re;
        const R v3 = W.e[j][j].im - W.e[i][i].im;
        const R k2 = v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
        // a staple projection that vanishes exactly: nothing to sample, no attempt
        const bool sample = k2 != R(0);
        const R rk = rsqrt_r(k2);
        const R inv2alpha = q32 * rk;
        KPDraw<R> d;
        R lam2;
        bool ok;
        // the lanes whose turn it is take this draw's values if it hits
        const auto take = [&](const KPDraw<R> &e, bool turn) {
            const R l = -e.q * inv2alpha;
            const bool hit = turn && e.u4sq <= R(1) - l;
            lam2 = hit ? l : lam2;
            d.cth = hit ? e.cth : d.cth;
            d.sc = hit ? e.sc : d.sc;
            d.ss = hit ? e.ss : d.ss;
            ok = ok || hit;
        };
        int t = 1;  // attempts that all lanes have had which still want one
        if constexpr (HIT1 || PARK) {
            d = first(sub);
            lam2 = -d.q * inv2alpha;
            ok = sample && d.u4sq <= R(1) - lam2;
            n.att += lanes_of(sample && active);
            n.acc += lanes_of(ok && active);
        } else {
            d = KPDraw<R>{};
            lam2 = R(0);
            ok = false;
            t = 0;
        }
        if constexpr (!HIT1) {
            bool made = false;
            if constexpr (PARK) {
                if (nhit > 1) {
                    const KPDraw<R> e = second(sub, d.u4sq, made);
                    const bool turn = sample && !ok && made && active;
                    take(e, turn);
                    n.att += lanes_of(turn);
                    n.acc += lanes_of(turn && ok);
                    if (__ballot(active && sample && !ok && !made) == 0) t = 2;
                }
            }
            // Each lane its own attempt; without PARK as long as most lanes want one, there is one left or none
            // has had three.
            uint64_t m = __ballot(active && sample && !ok);
            while (t < nhit && m != 0 && (PARK || t < 3 || t + 1 == nhit || __popcll(m) > 32)) {
                const bool turn = active && sample && !ok && (t > 1 || !made);
                if constexpr (PARK) {
                    lds_put<R, 9>(park_u, lane, U);
                    lds_put<R, 9>(park_w, lane, W);
                    __asm__ __volatile__("" ::: "memory");
                }
                if constexpr (!MASK)
                    take(kp_draw<R>(lid, sweep, seed, sub, t), turn);
                else if (turn)
                    take(kp_draw<R>(lid, sweep, seed, sub, t), true);
                if constexpr (PARK) {
                    __asm__ __volatile__("" ::: "memory");
                    U = lds_get<R, 9>(park_u, lane);
                    W = lds_get<R, 9>(park_w, lane);
                }
                n.att += lanes_of(turn);
                n.acc += lanes_of(turn && ok);
                ++t;
                m = __ballot(active && sample && !ok);
            }
            // further attempts, a round of 64 at a time
            if constexpr (!PARK)
                while (t < nhit && m != 0) {
                    const Round r(m, lane);
                    const int at = t + r.ahead;
                    const KPDraw<R> e = kp_draw<R>(__shfl(lid, r.asker), sweep, seed, sub, at);
                    const R l = -e.q * __shfl(inv2alpha, r.asker);
                    const bool hit = r.ahead < r.each && at < nhit && e.u4sq <= R(1) - l;
                    // the asker takes the first of its attempts that hit, which lane `from` made
                    const bool asks = m >> lane & 1;
                    const uint64_t hits = __ballot(hit);
                    const uint64_t mine = asks ? (hits >> r.rank) & r.every : 0;
                    const bool got = mine != 0;
                    const int skip = got ? __builtin_ctzll(mine) : 0;
                    const int from = (r.rank + skip) & 63;
                    const R lam = __shfl(l, from), cth = __shfl(e.cth, from), sc = __shfl(e.sc, from),
                            ss = __shfl(e.ss, from);
                    lam2 = got ? lam : lam2;
                    d.cth = got ? cth : d.cth;
                    d.sc = got ? sc : d.sc;
                    d.ss = got ? ss : d.ss;
                    ok = ok || got;
                    n.att += sum_small(!asks ? 0 : got ? r.attempts(skip) + 1 : min(r.each, nhit - t));
                    n.acc += lanes_of(got);
                    t += r.each;
                    m = __ballot(asks && !got);
                }
        }
        const R a0 = R(1) - R(2) * lam2;
        const R rho2 = R(1) - a0 * a0;
        const R rho = rho2 > R(0) ? sqrt_pos_r(rho2) : R(0);
        const R a1 = rho * d.sc, a2 = rho * d.ss, a3 = rho * d.cth;
        const R b0 = v0 * rk, b1 = v1 * rk, b2 = v2 * rk, b3 = v3 * rk;
        // quaternion product c = a * b  <=>  P(c) = P(a) P(b)
        const R p0 = a0 * b0 - a1 * b1 - a2 * b2 - a3 * b3;
        const R p1 = a0 * b1 + b0 * a1 - (a2 * b3 - a3 * b2);
        const R p2 = a0 * b2 + b0 * a2 - (a3 * b1 - a1 * b3);
        const R p3 = a0 * b3 + b0 * a3 - (a1 * b2 - a2 * b1);
        const R c0 = ok ? p0 : R(1), c1 = ok ? p1 : R(0), c2 = ok ? p2 : R(0), c3 = ok ? p3 : R(0);
        const Cx<R> r00{c0, c3}, r01{c2, c1}, r10{-c2, c1}, r11{c0, -c3};
#pragma unroll
        for (int col = 0; col < 3; ++col) {
            const Cx<R> ui = U.e[i][col], uj = U.e[j][col];
            U.e[i][col] = cmadd(cmul(r00, ui), r01, uj);
            U.e[j][col] = cmadd(cmul(r10, ui), r11, uj);
            const Cx<R> wi = W.e[i][col], wj = W.e[j][col];
            W.e[i][col] = cmadd(cmul(r00, wi), r01, wj);
            W.e[j][col] = cmadd(cmul(r10, wi), r11, wj);
        }
    }
    M3<double> Ud = convert<double>(U);
    reunit(Ud);
    U = convert<R>(Ud);
    return double(W.e[0][0].re) + double(W.e[1][1].re) + double(W.e[2][2].re);
}

// A link that was stored with a NaN in row 0 or 1 has two rows of W NaN and so
// every projection: it accepts no attempt and keeps its rows, reunitarised.
// The heat bath's identity rotations have made its row 0 NaN throughout.
template <typename R> __device__ __forceinline__ bool has_nan(const M3<R> &m)
{
    bool r = false;
#pragma unroll
    for (int e = 0; e < kEntries; ++e) {
        const Cx<R> c = m.e[e / 3][e % 3];
        r = r || c.re != c.re || c.im != c.im;
    }
    return r;
}
template <typename R, typename O> __device__ __forceinline__ void keep_nan_rows(M3<R> &U, Block<R> own, O o)
{
    if (__ballot(U.e[0][0].re != U.e[0][0].re) == 0) return;
    M3<R> V;
    load_own(V, own, o);
    if (has_nan(V)) {
        rebuild_row2(V);
        M3<double> Vd = convert<double>(V);
        reunit(Vd);
        U = convert<R>(Vd);
    }
}

// Re Tr(u s), accumulated in FP64.
template <typename R> __device__ __forceinline__ double retr_mul(const M3<R> &u, const M3<R> &s)
{
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            t += (double)u.e[i][k].re * (double)s.e[k][i].re - (double)u.e[i][k].im * (double)s.e[k][i].im;
    return t;
}

// Sum over the wave, in a fixed order.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// A wave's counts go to counter slot `slot`, so that few concurrent
// workgroups update the same address.
__device__ __forceinline__ void add_counts(Counts n, unsigned long long *__restrict__ counters, int slot, int lane)
{
    if (lane == 0 && n.att != 0) {
        unsigned long long *c = counters + 2 * slot;
        atomicAdd(&c[0], (unsigned long long)n.att);
        atomicAdd(&c[1], (unsigned long long)n.acc);
    }
}

// The job of tile t: the last one whose tile_begin is at most t.  The lanes of
// a wave look at 64 jobs at once.
__device__ __forceinline__ int job_of_tile(const BatchJob *__restrict__ jobs, int njobs, int t)
{
    const int lane = threadIdx.x & 63;
    int lo = 0, n = njobs;
    while (n > 1) {
        const int stride = (n + 63) / 64, k = lane * stride;
        const int c = (int)lanes_of(k < n && jobs[lo + (k < n ? k : 0)].tile_begin <= t);  // job lo always counts
        lo += (c - 1) * stride;
        n = min(stride, n - (c - 1) * stride);
        if (stride == 1) break;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Tile of this workgroup in a pass of parity `par`.  Every pass reads the
// whole lattice, and the passes of a sweep alternate in parity, so the odd
// passes walk the tiles backwards: a pass begins on the links its
// predecessor read last, which are still in L2 and in the memory-side cache.
// The order does not change the result, only which links are in cache.
__device__ __forceinline__ int pass_tile(int par)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    return par ? (int)gridDim.x - 1 - t : t;
}

// The couplings as the kernels take them: 3/(2 beta), or, for per-layer
// couplings, half of each, which goes into the staple.  Its projections (of 2 v)
// then overflow no sooner than those of the full weights would.
template <typename R> struct Couplings {
    R q32, w0, w1;
};
template <typename R, bool TWOB> Couplings<R> couplings_of(const PassArgs &a)
{
    return Couplings<R>{TWOB ? R(0.75) : R(1.5) / R(a.beta0), R(0.5) * R(a.beta0), R(0.5) * R(a.beta1)};
}

}  // namespace
}  // namespace su3hb
