// pass_kernels.h -- the kernels of a heat-bath pass, for one lattice and for a
// batch of them, and their launch.  Instantiated per link precision
// (pass_f64.hip, pass_f32.hip).
#pragma once

#include <type_traits>

#include "pass.h"

namespace su3hb {
namespace {

// Waves per SIMD the kernels are compiled for.  FP64: 168 registers are allowed;
// 1-hit passes take 152 to 168 (a measured one of two layers spills 8 to 24
// bytes), several attempts 157 (measured ones and those with layer couplings
// spill 60 to 72 bytes).  Asked for four waves, the compiler schedules for
// registers and the pass is 10 % slower; held to exactly three it is 3 % slower.
// FP32 with per-layer couplings has two more terms in registers and spills at five.
template <typename R, bool TWOB = false> constexpr int kSplitWaves = sizeof(R) == 8 ? 3 : TWOB ? 4 : 5;

// Several attempts: the second draws.  Six waves make them for every link and
// subgroup; three for the lanes that pool_slot picks, whose links are listed.
template <typename R, bool HIT1, bool SIX> struct SecondDraws {};
template <typename R> struct SecondDraws<R, false, true> {
    DrawLds<R> second[3];
};
template <typename R> struct SecondDraws<R, false, false> {
    DrawLds<R> pool;
    uint32_t list[64];
};

// Per-layer couplings: the lower staple of the second direction, D being the
// weighted sum of the first one's staples and the second one's upper one.
template <typename R, bool TWOB> struct LowerTerm {};
template <typename R> struct LowerTerm<R, true> {
    store_t<R> dn[9][64];
};

// Several attempts: U and W wait in LDS during a round of further ones, over the
// two D, which wave 0 alone reads and has read by then.  A measured pass of mu = 1
// or 2 needs D of the directions below mu again (KEEP; their sum stays in D[0])
// and has a place of its own for W.
template <typename R, bool OWN> struct Parking {};
template <typename R> struct Parking<R, true> {
    store_t<R> w[9][64];
};
template <typename R, bool HIT1, bool TWOB, bool KEEP, bool SIX, bool ROOM = TWOB>
struct SplitLds : SecondDraws<R, HIT1, SIX>, LowerTerm<R, TWOB>, Parking<R, !HIT1 && KEEP> {
    store_t<R> D[2][9][64];  // D of the first two directions
    // wave 0 keeps its own draw in registers, unless these are short
    static constexpr bool kAllDraws = SIX || (!HIT1 && ROOM);
    DrawLds<R> draw[kAllDraws ? 3 : 2];
    __device__ store_t<R> (*park_u())[64] { return D[1]; }
    __device__ store_t<R> (*park_w())[64]
    {
        if constexpr (!HIT1 && KEEP)
            return this->w;
        else
            return D[0];
    }
};
// A measured pass of a double-layered torus: the new link, after the heat bath
// (several attempts: over D[1], which is free then).
template <typename R, bool OWN> struct NewLink {};
template <typename R> struct NewLink<R, true> {
    store_t<R> U[9][64];
};
template <typename R, bool HIT1, int MU, bool SIX>
struct CrossLds : SplitLds<R, HIT1, false, (MU < 3), SIX, true>, NewLink<R, HIT1> {
    store_t<R> X[MU == 3 ? 9 : 1][64];  // wave 0's cross-layer part
    double part[3][2];
    __device__ store_t<R> (*new_link())[64]
    {
        if constexpr (HIT1)
            return this->U;
        else
            return this->D[1];
    }
};
template <typename R, bool HIT1, bool DLT, bool MEAS, bool TWOB, int MU, bool SIX>
using PassLds = std::conditional_t<MEAS && DLT, CrossLds<R, HIT1, MU, SIX>, SplitLds<R, HIT1, TWOB, MEAS && (MU < 3), SIX, TWOB || MEAS>>;

// A wave's share of a measured tile per layer: tr is filed under the link's
// layer but for its part trx, which belongs to the other one.
template <typename Lds>
__device__ __forceinline__ void cross_share(Lds &lds, bool active, bool l1, double tr, double trx, int w, int lane)
{
    const double s0 = wave_sum(active ? (l1 ? trx : tr - trx) : 0.0);
    const double s1 = wave_sum(active ? (l1 ? tr - trx : trx) : 0.0);
    if (lane == 0) {
        lds.part[w][0] = s0;
        lds.part[w][1] = s1;
    }
}

// One tile of 64 links with three waves: wave w forms the two staples of one
// direction and the random draw of one subgroup for all 64 links, and wave 0
// then adds the three and runs the heat bath.  SIX: three more waves make the
// draws (pass_six_waves says when).
//
// One lane per link, all in one thread, takes 3900 instructions (FP64) and 220
// registers: two waves per SIMD, each of which spends a third of its time on
// memory while the other alone issues at half rate.  Here no wave has more
// than one direction in registers (152 in FP64, 77 in FP32), the loads of four
// links (FP32: two) are in flight while the draw is made, the chain from the
// first load to the store is 1580 instructions instead of 3900 (1100 with six
// waves), and nothing is computed twice but the addresses.  us per pass, one
// lane per link (up to 8192 links four, up to 32768 two) -> this:
//   FP64          8^4 9.6 -> 6.0, 16^4 12.9 -> 9.5, 2 x 16^4 18.1 -> 15.6, 24^4 35.6
//                 -> 31.2, 32^4 98 -> 93, 64^4 1608 -> 1600;
//   FP64, 3 hits  8^4 16.3 -> 9.3, 16^4 18.4 -> 14.1, 32^4 106 -> 103 (larger ones: one wave, pass_lane.h);
//   FP32          8^4 9.1 -> 5.7, 16^4 10.7 -> 7.4, 2 x 16^4 13.9 -> 10.2, 24^4 22.3 ->
//                 19.4, 32^4 51.8 -> 48.5, 64^4 867 -> 856;
//   FP32, 3 hits  16^4 19.2 -> 9.9, 32^4 65 -> 57, 64^4 1040 -> 974;
//   measured sweeps (three of whose eight passes measure), 2 x 16^4: FP64 19.2 -> 17.4, FP32 15.3 -> 11.6.
// What bounds it now: 32^4 FP64 moves 500 MB past L2 with the vector unit 57 %
// busy (its loads and stores alone take 76 us, its arithmetic alone 64); FP32
// keeps the vector unit 86 % busy; 8^4 has a quarter of a wave per SIMD and
// takes the chain's latency.
//
// Several attempts: three waves make the first draws while the links arrive,
// wave 1 then the pool's second ones while wave 0 multiplies U by the staple.
// Second draws for every link instead: 32^4 FP64 111, FP32 59 us.  Third draws
// for the pool as well, by wave 2: 109 us (FP64).
template <int MU, typename R, bool HIT1, bool DLT, bool MEAS, bool TWOB, bool BIG, bool SIX>
__device__ __forceinline__ void pass_split(store_t<R> *__restrict__ links, const Geom &g, int par, int tile, R q32, R w0,
                                           R w1, uint64_t sweep, uint64_t seed, int nhit,
                                           unsigned long long *__restrict__ counters, int slot,
                                           double *__restrict__ meas,
                                           PassLds<R, HIT1, DLT, MEAS, TWOB, MU, SIX> &lds)
{
    static_assert(!MEAS || (MU > 0 && !TWOB), "measured passes: MU = 1, 2, 3 with one coupling");
    constexpr bool CROSS = MEAS && DLT;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nlinks = g.nlat * g.Vh;
    int v = tile * 64 + lane;
    const bool active = v < nlinks;
    v = active ? v : nlinks - 1;  // a lane past the end works on the last link and stores nothing
    const Site s = site_of<DLT>(g, par, v);
    const uint32_t lid = 4u * (uint32_t)(s.layer * 2 * g.Vh + 2 * s.i + (s.x[0] & 1)) + MU;
    if constexpr (SIX)
        if (w >= 3) {
            draw_put<R>(lds.draw[w - 3], lane, kp_draw<R>(lid, sweep, seed, w - 3, 0));
            if constexpr (!HIT1)
                if (nhit > 1) draw_put<R>(lds.second[w - 3], lane, kp_draw<R>(lid, sweep, seed, w - 3, 1));
            __syncthreads();
            if constexpr (CROSS) {
                __syncthreads();
                __syncthreads();
            }
            return;
        }
    const int nu = w == 0 ? kNu2<MU> : w == 1 ? kNu0<MU> : kNu1<MU>;
    Step up, dn;
    steps_of<MU, DLT>(g, s, w, up, dn);
    const StapleAt<BIG> at = staple_at<MU, R, DLT, BIG>(g, s, step_of<MU, +1>(g, s), up, dn);
    // D: the direction's sum; X: its part whose base lies in the other layer
    // (CROSS), or the lower term (TWOB; D is then the upper one)
    M3<R> D, X;
    KPDraw<R> mine;  // three waves: the draw of subgroup w - 1, or 2 for wave 0, which keeps it
    staple_nu<MU, R, CROSS, TWOB, BIG>(D, X, links, g, par, nu, at, [&] {
        if constexpr (!SIX) {
            const int sub = w == 0 ? 2 : w - 1;
            mine = kp_draw<R>(lid, sweep, seed, sub, 0);
            if constexpr (!HIT1) {
                const int slot = pool_slot(mine.u4sq, sub, lane);
                if (slot >= 0) lds.list[slot] = lid;
            }
        }
    });
    // A += the two terms of a direction, each with half the coupling of its base's layer
    const R wu = s.layer ? w1 : w0, wd = (s.layer ^ dn.flip) ? w1 : w0;
    if (w != 0) {
        if constexpr (TWOB) {
            if (w == 1) {
                M3<R> A;
                set_zero(A);
                scale_acc(A, D, wu);
                scale_acc(A, X, wd);
                D = A;
            } else {
                lds_put<R, 9>(lds.dn, lane, X);
            }
        }
        lds_put<R, 9>(lds.D[w - 1], lane, D);
        if constexpr (!SIX) draw_put<R>(lds.draw[w - 1], lane, mine);
        __syncthreads();
        if constexpr (!SIX && !HIT1)
            if (nhit > 1) {
                if (w == 1) {
                    // slots past a subgroup's candidates hold no link: their draws are not read
                    const int sub = lane < kPoolSlots ? 0 : lane < 2 * kPoolSlots ? 1 : 2;
                    draw_put<R>(lds.pool, lane, kp_draw<R>(lds.list[lane], sweep, seed, sub, 1));
                }
                __syncthreads();
            }
        if constexpr (CROSS) {
            __syncthreads();
            double trx = 0.0;
            if (nu < MU) trx = retr_mul(lds_get<R, 9>(lds.new_link(), lane), X);
            cross_share(lds, active, s.layer != 0, 0.0, trx, w, lane);
            __syncthreads();
        }
        return;
    }
    const Block<R> own = block_of<R, BIG>(links, g, MU, par);
    M3<R> U;
    load_own(U, own, at.here);
    if constexpr (CROSS && MU == 3) lds_put<R, 9>(lds.X, lane, X);
    if constexpr (!SIX && std::remove_reference_t<decltype(lds)>::kAllDraws) draw_put<R>(lds.draw[2], lane, mine);
    __syncthreads();
    M3<R> A;
    if constexpr (TWOB) {
        // entry by entry, so that D and X give way to A
        const R wd1 = (s.layer ^ step_of<kNu1<MU>, -1>(g, s).flip) ? w1 : w0;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const store_t<R> a = lds.D[0][e][lane], u1 = lds.D[1][e][lane], d1 = lds.dn[e][lane];
            Cx<R> t{a.x, a.y};
            t = scale_add(t, Cx<R>{u1.x, u1.y}, wu);
            t = scale_add(t, Cx<R>{d1.x, d1.y}, wd1);
            t = scale_add(t, D.e[e / 3][e % 3], wu);
            A.e[e / 3][e % 3] = scale_add(t, X.e[e / 3][e % 3], wd);
        }
    } else {
        A = lds_get<R, 9>(lds.D[0], lane);
        add_to(A, lds_get<R, 9>(lds.D[1], lane));
        if constexpr (MEAS && MU == 2) lds_put<R, 9>(lds.D[0], lane, A);  // the sum over nu < MU
        add_to(A, D);
    }
    rebuild_row2(U);
    Counts n{0, 0};
    double tr = heatbath<R, HIT1, !HIT1, !SIX && sizeof(R) == 4>(
        U, A, q32, lid, sweep, seed, nhit, active, n, lds.park_u(), lds.park_w(), lane,
        [&](int k) { return !std::remove_reference_t<decltype(lds)>::kAllDraws && k == 2 ? mine : draw_get<R>(lds.draw[k], lane); },
        [&](int k, R u4sq, bool &made) {
            if constexpr (HIT1) {
                made = false;
                return mine;
            } else if constexpr (SIX) {
                made = true;
                return draw_get<R>(lds.second[k], lane);
            } else {
                if (k == 0) __syncthreads();  // the pool is drawn
                const int slot = pool_slot(u4sq, k, lane);
                made = slot >= 0;
                return draw_get<R>(lds.pool, made ? slot : 0);
            }
        });
    keep_nan_rows(U, own, at.here);
    if (active) store_own(own, at.here, U);
    add_counts(n, counters, slot, lane);
    if constexpr (MEAS) {
        // S = sum of D_nu over nu < MU
        if constexpr (MU < 3) tr = retr_mul(U, lds_get<R, 9>(lds.D[0], lane));
        if constexpr (!CROSS) {
            tr = wave_sum(active ? tr : 0.0);
            if (lane == 0) meas[0] = tr;
        } else {
            // the lower terms whose base lies in the other layer: each wave
            // sums its own direction's share Re Tr(U_new X)
            lds_put<R, 9>(lds.new_link(), lane, U);
            __syncthreads();
            double trx = 0.0;
            if constexpr (MU == 3) trx = retr_mul(U, lds_get<R, 9>(lds.X, lane));
            cross_share(lds, active, s.layer != 0, tr, trx, 0, lane);
            __syncthreads();
            if (lane == 0) {
                meas[0] = lds.part[0][0] + lds.part[1][0] + lds.part[2][0];
                if (g.nlat == 2) meas[1] = lds.part[0][1] + lds.part[1][1] + lds.part[2][1];
            }
        }
    }
}

template <int MU, typename R, bool HIT1, bool DLT, bool MEAS, bool TWOB, bool BIG, bool SIX>
__global__ __launch_bounds__(SIX ? 384 : 192, (kSplitWaves<R, TWOB>)) void k_pass_split(
    store_t<R> *__restrict__ links, const Geom g, const int par, const R q32, const R w0, const R w1,
    const uint64_t sweep, const uint64_t seed, const int nhit, unsigned long long *__restrict__ counters,
    double *__restrict__ meas)
{
    // three waves, several attempts: four workgroups share the 160 KiB of a CU, as many as the registers allow
    static_assert(sizeof(PassLds<R, HIT1, DLT, MEAS, TWOB, MU, SIX>) <= (SIX || HIT1 ? 160 : 40) * 1024, "LDS of a pass");
    __shared__ PassLds<R, HIT1, DLT, MEAS, TWOB, MU, SIX> lds;
    pass_split<MU, R, HIT1, DLT, MEAS, TWOB, BIG, SIX>(links, g, par, pass_tile(par), q32, w0, w1, sweep, seed, nhit,
                                                  counters, blockIdx.x % kCounterSlots,
                                                  MEAS ? meas + (size_t)g.nlat * blockIdx.x : nullptr, lds);
}

// Batched pass: one launch updates the links U_MU of parity `par` of every
// job in `jobs` (sorted by tile_begin).  The grid has one workgroup per tile
// of 64 links of the batch; logical tile t (pass_tile: each XCD works on
// contiguous stretches of each job's tiles) belongs to the job whose tile range
// holds t; job j is at sweep index sweep0 + (step - admit_step).  The record
// of the job is uniform over the workgroup.
template <int MU, typename R, bool HIT1, bool DLT, bool BIG, bool SIX>
__global__ __launch_bounds__(SIX ? 384 : 192, kSplitWaves<R>) void k_batch_split(const BatchJob *__restrict__ jobs,
                                                                             const int njobs, const long long step,
                                                                             const int par)
{
    __shared__ PassLds<R, HIT1, DLT, false, false, MU, SIX> lds;
    const int t = pass_tile(par);
    const BatchJob J = jobs[job_of_tile(jobs, njobs, t)];
    const int tile = t - J.tile_begin;
    pass_split<MU, R, HIT1, DLT, false, false, BIG, SIX>((store_t<R> *)J.links, J.g, par, tile, sizeof(R) == 8 ? (R)J.q32 : (R)J.q32f,
                                                    R(0), R(0), J.sweep0 + (uint64_t)(step - J.admit_step), J.seed,
                                                    J.nhit, J.counters, tile % kCounterSlots, nullptr, lds);
}
// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
template <int MU, typename R, bool HIT1, bool DLT, bool MEAS, bool TWOB, bool BIG> void launch_one(const PassArgs &a)
{
    const unsigned grid = (unsigned)pass_blocks(a.g, kPassBlock);
    const auto [q, w0, w1] = couplings_of<R, TWOB>(a);
    if constexpr (!BIG)
        if (a.six_waves) {
            k_pass_split<MU, R, HIT1, DLT, MEAS, TWOB, BIG, true><<<grid, 384, 0, a.stream>>>(
                (store_t<R> *)a.links, a.g, a.par, q, w0, w1, a.sweep, a.seed, a.nhit, a.counters, a.meas);
            return;
        }
    k_pass_split<MU, R, HIT1, DLT, MEAS, TWOB, BIG, false><<<grid, 192, 0, a.stream>>>(
        (store_t<R> *)a.links, a.g, a.par, q, w0, w1, a.sweep, a.seed, a.nhit, a.counters, a.meas);
}

// The kernel by hit count and torus.  Blocks of 4 GiB and more (64-bit offsets)
// have one attempt here: several take one wave per tile (launch_pass).
template <int MU, typename R, bool MEAS, bool TWOB, bool DLT> void launch_torus(const PassArgs &a)
{
    if (a.big)
        launch_one<MU, R, true, DLT, MEAS, TWOB, true>(a);
    else if (a.nhit == 1)
        launch_one<MU, R, true, DLT, MEAS, TWOB, false>(a);
    else
        launch_one<MU, R, false, DLT, MEAS, TWOB, false>(a);
}

template <int MU, typename R, bool MEAS, bool TWOB> void launch_mu(const PassArgs &a)
{
    if constexpr (!TWOB)
        if (a.g.nlat == 1) return launch_torus<MU, R, MEAS, TWOB, false>(a);
    launch_torus<MU, R, MEAS, TWOB, true>(a);
}

template <typename R, bool MEAS, bool TWOB> void launch_any(const PassArgs &a)
{
    switch (a.mu) {
    case 0:
        if constexpr (!MEAS) launch_mu<0, R, MEAS, TWOB>(a);
        break;
    case 1: launch_mu<1, R, MEAS, TWOB>(a); break;
    case 2: launch_mu<2, R, MEAS, TWOB>(a); break;
    default: launch_mu<3, R, MEAS, TWOB>(a); break;
    }
}

template <typename R> hipError_t launch_pass_r(const PassArgs &a)
{
    if (a.twob)
        launch_any<R, false, true>(a);
    else if (a.meas)
        launch_any<R, true, false>(a);
    else
        launch_any<R, false, false>(a);
    return hipGetLastError();
}

template <int MU, typename R, bool HIT1, bool DLT, bool BIG> void launch_batch_one(const BatchArgs &b)
{
    if constexpr (!BIG)
        if (b.six_waves) {
            k_batch_split<MU, R, HIT1, DLT, BIG, true><<<b.ntiles, 384, 0, b.stream>>>(b.jobs, b.njobs, b.step, b.par);
            return;
        }
    k_batch_split<MU, R, HIT1, DLT, BIG, false><<<b.ntiles, 192, 0, b.stream>>>(b.jobs, b.njobs, b.step, b.par);
}

template <int MU, typename R, bool DLT> void launch_batch_torus(const BatchArgs &b)
{
    if (b.big)
        launch_batch_one<MU, R, true, DLT, true>(b);
    else if (b.hit1)
        launch_batch_one<MU, R, true, DLT, false>(b);
    else
        launch_batch_one<MU, R, false, DLT, false>(b);
}

template <int MU, typename R> void launch_batch_mu(const BatchArgs &b)
{
    if (b.dlt)
        launch_batch_torus<MU, R, true>(b);
    else
        launch_batch_torus<MU, R, false>(b);
}

template <typename R> hipError_t launch_batch_r(const BatchArgs &b)
{
    switch (b.mu) {
    case 0: launch_batch_mu<0, R>(b); break;
    case 1: launch_batch_mu<1, R>(b); break;
    case 2: launch_batch_mu<2, R>(b); break;
    default: launch_batch_mu<3, R>(b); break;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace su3hb
