// launch.h -- host-side launchers of the gfx950 kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"
#include "layout.h"

namespace su3hb {

// One job of a batched pass (continuous batching of several lattices).
struct BatchJob {
    void *links;                   // this job's link buffer (tiled layout, its own precision)
    unsigned long long *counters;  // this job's heat-bath counter slots
    Geom g;
    double q32;                    // 3 / (2 beta), in both precisions
    float q32f;
    int nhit;
    uint64_t seed;
    uint64_t sweep0;               // sweep index at global step admit_step
    long long admit_step;
    int tile_begin;                // first workgroup of this job in the launch
};

// One checkerboard pass of one lattice.
struct PassArgs {
    void *links;
    Geom g;
    int mu, par;
    double beta0, beta1;           // the coupling, or one per layer (twob)
    bool twob;                     // double-layered torus: a plaquette takes its base site's layer coupling
    bool big;                      // 64-bit link offsets (pass_big)
    bool six_waves;                // six waves per 64 links instead of three (pass_six_waves)
    bool one_lane;                 // one wave per 64 links, several attempts only (pass_one_lane); always with `big`
    uint64_t sweep, seed;
    int nhit;
    unsigned long long *counters;
    // measured pass (odd pass of mu = 1, 2, 3) if not null: also store, per
    // workgroup of 64 links, the sum of its final plaquettes in the planes
    // (nu, mu), nu < mu: meas[b] on a single torus, meas[2 b + l] for layer l on
    // a double-layered torus (each plaquette under its base site's layer), b <
    // meas_blocks(g).  The three passes write consecutive slices of nlat *
    // meas_blocks(g) doubles, which launch_measure_final adds up into sums[0]
    // (total) and sums[1 + l] (layer l).
    double *meas;
    hipStream_t stream;
};
hipError_t launch_pass_f64(const PassArgs &a);
hipError_t launch_pass_f32(const PassArgs &a);
hipError_t launch_lane_f64(const PassArgs &a);
hipError_t launch_lane_f32(const PassArgs &a);
inline hipError_t launch_pass(int precision, const PassArgs &a)
{
    if (a.one_lane || (a.big && a.nhit > 1)) return precision == 64 ? launch_lane_f64(a) : launch_lane_f32(a);
    return precision == 64 ? launch_pass_f64(a) : launch_pass_f32(a);
}

// One pass (mu, par) of every job in `jobs` (device copy, sorted by
// tile_begin).  All jobs share the precision; hit1: every job has nhit = 1;
// dlt: every job is a double-layered torus (else every job is a single torus);
// big: some job needs 64-bit link offsets.  A job takes ceil(nlat Vh / 64)
// workgroups.
struct BatchArgs {
    const BatchJob *jobs;
    int njobs, ntiles;
    long long step;
    int mu, par;
    bool hit1, dlt, big, six_waves, one_lane;
    hipStream_t stream;
};
hipError_t launch_batch_f64(const BatchArgs &b);
hipError_t launch_batch_f32(const BatchArgs &b);
hipError_t launch_lane_batch_f64(const BatchArgs &b);
hipError_t launch_lane_batch_f32(const BatchArgs &b);
inline hipError_t launch_batch(int precision, const BatchArgs &b)
{
    if (b.njobs <= 0 || b.ntiles <= 0) return hipSuccess;
    if (b.one_lane || (b.big && !b.hit1)) return precision == 64 ? launch_lane_batch_f64(b) : launch_lane_batch_f32(b);
    return precision == 64 ? launch_batch_f64(b) : launch_batch_f32(b);
}

hipError_t launch_start(int precision, void *links, const Geom &g, int hot, uint64_t seed, hipStream_t s);
// Plaquette sums of the whole lattice into sums[0..3] (total, per layer,
// number of links failing the unitarity check); partials: plaq_partial_bytes(g,
// precision) bytes.  With `mean` non-null also the normalised values
// mean[0..nlat] and the failing-link count mean[1 + nlat], on the device.
hipError_t launch_plaquette(int precision, const void *links, const Geom &g, double *partials, double *sums,
                            hipStream_t s, double *mean = nullptr);
// Adds the partial sums of a measured sweep (PassArgs::meas).
hipError_t launch_measure_final(const double *meas, const Geom &g, double *sums, hipStream_t s);
// Polyakov loops along direction 3: out[2 l], out[2 l + 1] = sums of Re, Im of Tr/3 over the starts in layer l;
// partials: 2 * nlat * polyakov_blocks(g) doubles
hipError_t launch_polyakov(int precision, const void *links, const Geom &g, double *partials, double *out,
                           hipStream_t s);
hipError_t launch_reunit(int precision, void *links, const Geom &g, hipStream_t s);
hipError_t launch_gauge(int precision, void *links, const Geom &g, uint64_t gseed, hipStream_t s);
hipError_t launch_zero_u64(unsigned long long *p, int n, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s);

}  // namespace su3hb
