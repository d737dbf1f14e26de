// pass_lane.h -- heat-bath passes with several attempts per subgroup in which
// one wave does all the work of its 64 links, and their launch (pass_one_lane
// says when).  Instantiated per link precision (pass_lane_f64.hip,
// pass_lane_f32.hip).
#pragma once

#include "pass.h"

namespace su3hb {
namespace {

// One lane per link: all three directions and the draws in one thread, 203 to 246
// registers in FP64 (two waves per SIMD) and 98 to 117 in FP32 (four), no
// spills.  Bound by instruction issue: a draw is some 400 instructions beside the
// 2700 of an update (32^4 FP64, 64 attempts, beta 0.5: 691 us per pass with each
// lane's attempts one after the other, 218 with rounds of 64 once few lanes ask).
//
// FP64: the six links U_mu(x +- nu) are links of the other parity that the
// neighbouring sites read in all three directions; loaded direction by
// direction their lines leave L2 in between.  They are loaded first, and three of
// them wait in LDS.  FP32, which is not bound by memory, loads b and e direction
// by direction.  Measured passes keep the sums for the measurement there after that.
template <typename R, bool MEAS, bool CROSS, int MU> struct LaneLds {
    static constexpr bool kStash = sizeof(R) == 8;
    static constexpr int kSum = MEAS && MU < 3 ? 9 : 0, kCross = CROSS ? 9 : 0;
    store_t<R> room[kStash ? 18 : kSum + kCross > 0 ? kSum + kCross : 1][64];
};
template <int MU, typename R, bool DLT, bool MEAS, bool TWOB, bool BIG>
__device__ __forceinline__ void pass_lane(store_t<R> *__restrict__ links, const Geom &g, int par, int tile, R q32, R w0,
                                          R w1, uint64_t sweep, uint64_t seed, int nhit,
                                          unsigned long long *__restrict__ counters, int slot,
                                          double *__restrict__ meas,
                                          LaneLds<R, MEAS, (MEAS && DLT), MU> &lds)
{
    constexpr bool CROSS = MEAS && DLT, STASH = sizeof(R) == 8;
    constexpr int kSum = LaneLds<R, MEAS, CROSS, MU>::kSum;
    constexpr int N0 = kNu0<MU>, N1 = kNu1<MU>, N2 = kNu2<MU>;
    const int lane = threadIdx.x & 63;
    const int nlinks = g.nlat * g.Vh;
    int v = tile * 64 + lane;
    const bool active = v < nlinks;
    v = active ? v : nlinks - 1;
    const Site s = site_of<DLT>(g, par, v);
    const uint32_t lid = 4u * (uint32_t)(s.layer * 2 * g.Vh + 2 * s.i + (s.x[0] & 1)) + MU;
    const Step mu = step_of<MU, +1>(g, s);
    const Step dn0 = step_of<N0, -1>(g, s), dn1 = step_of<N1, -1>(g, s), dn2 = step_of<N2, -1>(g, s);
    const StapleAt<BIG> at0 = staple_at<MU, R, DLT, BIG>(g, s, mu, step_of<N0, +1>(g, s), dn0);
    const StapleAt<BIG> at1 = staple_at<MU, R, DLT, BIG>(g, s, mu, step_of<N1, +1>(g, s), dn1);
    const StapleAt<BIG> at2 = staple_at<MU, R, DLT, BIG>(g, s, mu, step_of<N2, +1>(g, s), dn2);
    const Block<R> umu = block_of<R, BIG>(links, g, MU, par ^ 1);
    const R wu = s.layer ? w1 : w0;
    M3<R> A, Sx, b, e;
    if constexpr (CROSS) set_zero(Sx);
    // D_nu into A; counts: its cross-layer part into Sx
    const auto add = [&](const M3<R> &D, const M3<R> &X, Step dn, bool first, bool counts) {
        if constexpr (TWOB) {
            if (first) set_zero(A);
            scale_acc(A, D, wu);
            scale_acc(A, X, (s.layer ^ dn.flip) ? w1 : w0);
        } else {
            if (first)
                A = D;
            else
                add_to(A, D);
            if constexpr (CROSS)
                if (counts) add_to(Sx, X);
        }
    };
    // FP32: gathering the staple, issue loads ahead of waves in the heat bath (-2 to -3 %; FP64 +1 to +4 %)
    if constexpr (sizeof(R) == 4) __builtin_amdgcn_s_setprio(1);
    // FP32: one direction after the other (loads of the next one early cost registers and so waves: +1 to +4 %;
    // FP64 -1 %)
    const auto phase = [] {
        if constexpr (sizeof(R) == 4) {
            __asm__ __volatile__("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    M3<R> D, X;
    if constexpr (STASH) {
        M3<R> b1, e1, b2, e2;
        load_rows_pair(b, umu, at0.up, e, umu, at0.dn);
        load_rows_pair(b1, umu, at1.up, e1, umu, at1.dn);
        load_rows_pair(b2, umu, at2.up, e2, umu, at2.dn);
        lds_put<R, 6>(lds.room, lane, b1);
        lds_put<R, 6>(lds.room + 6, lane, e1);
        lds_put<R, 6>(lds.room + 12, lane, b2);
        __asm__ __volatile__("" ::: "memory");
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e, links, g, par, N0, at0);
        add(D, X, dn0, true, N0 < MU);
        phase();
        b = lds_get<R, 6>(lds.room, lane);
        e = lds_get<R, 6>(lds.room + 6, lane);
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e, links, g, par, N1, at1);
        if constexpr (MEAS && MU == 1) {
            __asm__ __volatile__("" ::: "memory");
            lds_put<R, 9>(lds.room, lane, A);
        }
        add(D, X, dn1, false, N1 < MU);
        phase();
        b = lds_get<R, 6>(lds.room + 12, lane);
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e2, links, g, par, N2, at2);
        if constexpr (MEAS && MU == 2) {
            __asm__ __volatile__("" ::: "memory");
            lds_put<R, 9>(lds.room, lane, A);
        }
        add(D, X, dn2, false, N2 < MU);
    } else {
        load_rows_pair(b, umu, at0.up, e, umu, at0.dn);
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e, links, g, par, N0, at0);
        add(D, X, dn0, true, N0 < MU);
        phase();
        if constexpr (MEAS && MU == 1) lds_put<R, 9>(lds.room, lane, A);
        load_rows_pair(b, umu, at1.up, e, umu, at1.dn);
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e, links, g, par, N1, at1);
        add(D, X, dn1, false, N1 < MU);
        phase();
        if constexpr (MEAS && MU == 2) lds_put<R, 9>(lds.room, lane, A);
        load_rows_pair(b, umu, at2.up, e, umu, at2.dn);
        staple_from<MU, R, CROSS, TWOB, BIG>(D, X, b, e, links, g, par, N2, at2);
        add(D, X, dn2, false, N2 < MU);
    }
    if constexpr (CROSS) lds_put<R, 9>(lds.room + kSum, lane, Sx);
    __asm__ __volatile__("" ::: "memory");
    const Block<R> own = block_of<R, BIG>(links, g, MU, par);
    M3<R> U;
    load_own(U, own, at0.here);
    if constexpr (sizeof(R) == 4) __builtin_amdgcn_s_setprio(0);
    rebuild_row2(U);
    Counts n{0, 0};
    double tr = heatbath<R, false, false, true>(
        U, A, q32, lid, sweep, seed, nhit, active, n, nullptr, nullptr, lane,
        [](int) { return KPDraw<R>{}; },
        [](int, R, bool &) { return KPDraw<R>{}; });
    keep_nan_rows(U, own, at0.here);
    if (active) store_own(own, at0.here, U);
    add_counts(n, counters, slot, lane);
    if constexpr (MEAS) {
        if constexpr (MU < 3) tr = retr_mul(U, lds_get<R, 9>(lds.room, lane));
        double trx = 0.0;
        if constexpr (CROSS) trx = retr_mul(U, lds_get<R, 9>(lds.room + kSum, lane));
        const bool l1 = s.layer != 0;
        const double s0 = wave_sum(active ? (l1 ? trx : tr - trx) : 0.0);
        if (lane == 0) meas[0] = s0;
        if constexpr (CROSS) {
            const double s1 = wave_sum(active ? (l1 ? tr - trx : trx) : 0.0);
            if (lane == 0 && g.nlat == 2) meas[1] = s1;
        }
    }
}
template <int MU, typename R, bool DLT, bool MEAS, bool TWOB, bool BIG>
__global__ __launch_bounds__(64, (sizeof(R) == 8 ? 2 : 4)) void k_pass_lane(
    store_t<R> *__restrict__ links, const Geom g, const int par, const R q32, const R w0, const R w1,
    const uint64_t sweep, const uint64_t seed, const int nhit, unsigned long long *__restrict__ counters,
    double *__restrict__ meas)
{
    __shared__ LaneLds<R, MEAS, (MEAS && DLT), MU> lds;
    pass_lane<MU, R, DLT, MEAS, TWOB, BIG>(links, g, par, pass_tile(par), q32, w0, w1, sweep, seed, nhit, counters,
                                           blockIdx.x % kCounterSlots, MEAS ? meas + (size_t)g.nlat * blockIdx.x : nullptr,
                                           lds);
}

// The same for the jobs of a batch (k_batch_split).
template <int MU, typename R, bool DLT, bool BIG>
__global__ __launch_bounds__(64, (sizeof(R) == 8 ? 2 : 4)) void k_batch_lane(const BatchJob *__restrict__ jobs,
                                                                            const int njobs, const long long step,
                                                                            const int par)
{
    __shared__ LaneLds<R, false, false, MU> lds;
    const int t = pass_tile(par);
    const BatchJob J = jobs[job_of_tile(jobs, njobs, t)];
    const int tile = t - J.tile_begin;
    pass_lane<MU, R, DLT, false, false, BIG>((store_t<R> *)J.links, J.g, par, tile, sizeof(R) == 8 ? (R)J.q32 : (R)J.q32f,
                                             R(0), R(0), J.sweep0 + (uint64_t)(step - J.admit_step), J.seed, J.nhit,
                                             J.counters, tile % kCounterSlots, nullptr, lds);
}
template <int MU, typename R, bool DLT, bool MEAS, bool TWOB, bool BIG> void launch_lane_one(const PassArgs &a)
{
    const auto [q, w0, w1] = couplings_of<R, TWOB>(a);
    k_pass_lane<MU, R, DLT, MEAS, TWOB, BIG><<<(unsigned)pass_blocks(a.g, kPassBlock), 64, 0, a.stream>>>(
        (store_t<R> *)a.links, a.g, a.par, q, w0, w1, a.sweep, a.seed, a.nhit, a.counters, a.meas);
}

template <int MU, typename R, bool MEAS, bool TWOB> void launch_lane_mu(const PassArgs &a)
{
    if (a.big) return launch_lane_one<MU, R, true, MEAS, TWOB, true>(a);
    if constexpr (!TWOB)
        if (a.g.nlat == 1) return launch_lane_one<MU, R, false, MEAS, TWOB, false>(a);
    launch_lane_one<MU, R, true, MEAS, TWOB, false>(a);
}

template <int MU, typename R> void launch_lane_any(const PassArgs &a)
{
    if (a.twob) return launch_lane_mu<MU, R, false, true>(a);
    if constexpr (MU > 0)
        if (a.meas) return launch_lane_mu<MU, R, true, false>(a);
    launch_lane_mu<MU, R, false, false>(a);
}

template <typename R> hipError_t launch_lane_r(const PassArgs &a)
{
    switch (a.mu) {
    case 0: launch_lane_any<0, R>(a); break;
    case 1: launch_lane_any<1, R>(a); break;
    case 2: launch_lane_any<2, R>(a); break;
    default: launch_lane_any<3, R>(a); break;
    }
    return hipGetLastError();
}

template <int MU, typename R> void launch_lane_batch_mu(const BatchArgs &b)
{
    if (b.big)
        k_batch_lane<MU, R, true, true><<<b.ntiles, 64, 0, b.stream>>>(b.jobs, b.njobs, b.step, b.par);
    else if (b.dlt)
        k_batch_lane<MU, R, true, false><<<b.ntiles, 64, 0, b.stream>>>(b.jobs, b.njobs, b.step, b.par);
    else
        k_batch_lane<MU, R, false, false><<<b.ntiles, 64, 0, b.stream>>>(b.jobs, b.njobs, b.step, b.par);
}

template <typename R> hipError_t launch_lane_batch_r(const BatchArgs &b)
{
    switch (b.mu) {
    case 0: launch_lane_batch_mu<0, R>(b); break;
    case 1: launch_lane_batch_mu<1, R>(b); break;
    case 2: launch_lane_batch_mu<2, R>(b); break;
    default: launch_lane_batch_mu<3, R>(b); break;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace su3hb
