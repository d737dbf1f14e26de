// kernels.hip -- gfx950 kernels around the heat-bath passes (pass_kernels.h):
// start configurations, reunitarisation, gauge transformation, plaquette,
// Polyakov loops, the sums of measured sweeps and the copy probe.
//
// Link storage: the links of one (direction, parity) form a block of tiles of
// 16 consecutive links, each tile holding the 6 complex entries of rows 0 and 1
// entry-major (double2 or float2; row 2 is rebuilt by every reader); see
// link_at.  The link U_dir(x) of site
// x = (layer, parity, i) is element n = layer * Vh + i of block (dir, parity).
// Sixteen lanes with consecutive n read 16 consecutive complex numbers per
// entry: whole 128-byte lines, fully coalesced vector loads.
#include <algorithm>

#include "pass.h"

namespace su3hb {

namespace {

// Sum of v over the workgroup, in a fixed order (valid in thread 0).
template <int NB = kBlock> __device__ __forceinline__ double block_sum(double v)
{
    __shared__ double wsum[NB / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NB / 64; ++w) s += wsum[w];
    return s;
}

// Polyakov loops along direction 3: thread (layer, x0, x1, x2) walks the
// closed path x3 = 0, 1, ... (2 L3 links when crossing the direction-3
// boundary switches the layer) multiplying U_3 in FP64; partial sums of
// Re and Im of Tr/3 per workgroup and layer.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_polyakov(const store_t<R> *__restrict__ links, const Geom g,
                                                     double *__restrict__ partials)
{
    const int layer = blockIdx.y;
    const int V3 = g.L[0] * g.L[1] * g.L[2];
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double re = 0.0, im = 0.0;
    if (s < V3) {
        int y[4] = {s % g.L[0], (s / g.L[0]) % g.L[1], s / (g.L[0] * g.L[1]), 0};
        int ly = layer;
        M3<double> P;
        set_zero(P);
        P.e[0][0].re = P.e[1][1].re = P.e[2][2].re = 1.0;
        do {
            const int lex = lex_of(g, y);
            const int par = (y[0] + y[1] + y[2] + y[3]) & 1;
            const M3<double> u = convert<double>(load_link12<R>(planes<R>(links, g, 3, par), ly * g.Vh + (lex >> 1)));
            P = mul_nn(P, u);
            step<3, +1, true>(g, y, ly);
        } while (y[3] != 0 || ly != layer);
        re = (P.e[0][0].re + P.e[1][1].re + P.e[2][2].re) / 3.0;
        im = (P.e[0][0].im + P.e[1][1].im + P.e[2][2].im) / 3.0;
    }
    const double br = block_sum(re);
    __syncthreads();
    const double bi = block_sum(im);
    if (threadIdx.x == 0) {
        partials[2 * (layer * gridDim.x + blockIdx.x)] = br;
        partials[2 * (layer * gridDim.x + blockIdx.x) + 1] = bi;
    }
}

// out[2 l], out[2 l + 1] = sums of Re, Im over the partials of layer l (fixed order)
__global__ __launch_bounds__(kBlock) void k_polyakov_final(const double *__restrict__ partials, int nblk, int nlat,
                                                           double *__restrict__ out)
{
    for (int l = 0; l < nlat; ++l)
        for (int c = 0; c < 2; ++c) {
            double s = 0.0;
            for (int b = threadIdx.x; b < nblk; b += kBlock) s += partials[2 * (l * nblk + b) + c];
            const double r = block_sum(s);
            __syncthreads();
            if (threadIdx.x == 0) out[2 * l + c] = r;
        }
}

// ---------------------------------------------------------------------------
// start configurations, reunitarisation, gauge transformation: one thread per
// link; blockIdx.y = dir * 2 + parity
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool link_of_thread(const Geom &g, int &n, int &dir, int &par, int &layer, int x[4])
{
    n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.nlat * g.Vh) return false;
    dir = blockIdx.y >> 1;
    par = blockIdx.y & 1;
    layer = n >= g.Vh ? 1 : 0;
    site_coords(g, par, n - layer * g.Vh, x);
    return true;
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_start(store_t<R> *__restrict__ links, const Geom g, const int hot,
                                                  const uint64_t seed)
{
    int n, dir, par, layer, x[4];
    if (!link_of_thread(g, n, dir, par, layer, x)) return;
    M3<double> u;
    if (hot) {
        const uint64_t site = (uint64_t)layer * (uint64_t)(2 * g.Vh) + (uint64_t)lex_of(g, x);
        u = haar_element(seed, 4 * site + dir, kTagHot);
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) u.e[r][c] = Cx<double>{r == c ? 1.0 : 0.0, 0.0};
    }
    store_link<R>(planes<R>(links, g, dir, par), n, convert<R>(u));
}

template <typename R> __global__ __launch_bounds__(kBlock) void k_reunit(store_t<R> *__restrict__ links, const Geom g)
{
    int n, dir, par, layer, x[4];
    if (!link_of_thread(g, n, dir, par, layer, x)) return;
    store_t<R> *base = planes<R>(links, g, dir, par);
    M3<double> u = convert<double>(load_link12<R>(base, n));
    reunit(u);
    store_link<R>(base, n, convert<R>(u));
}

template <int D>
__device__ __forceinline__ uint64_t forward_site(const Geom &g, const int x[4], int layer)
{
    int y[4] = {x[0], x[1], x[2], x[3]};
    int ly = layer;
    step<D, +1>(g, y, ly);
    return (uint64_t)ly * (uint64_t)(2 * g.Vh) + (uint64_t)lex_of(g, y);
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_gauge(store_t<R> *__restrict__ links, const Geom g, const uint64_t gseed)
{
    int n, dir, par, layer, x[4];
    if (!link_of_thread(g, n, dir, par, layer, x)) return;
    const uint64_t site = (uint64_t)layer * (uint64_t)(2 * g.Vh) + (uint64_t)lex_of(g, x);
    uint64_t fwd;
    switch (dir) {
    case 0: fwd = forward_site<0>(g, x, layer); break;
    case 1: fwd = forward_site<1>(g, x, layer); break;
    case 2: fwd = forward_site<2>(g, x, layer); break;
    default: fwd = forward_site<3>(g, x, layer); break;
    }
    const M3<double> gx = haar_element(gseed, site, kTagGauge);
    const M3<double> gy = haar_element(gseed, fwd, kTagGauge);
    store_t<R> *base = planes<R>(links, g, dir, par);
    const M3<double> u = convert<double>(load_link12<R>(base, n));
    const M3<double> t = mul_nn(gx, u);
    M3<double> out;
    set_zero(out);
    acc_nd(out, t, gy);
    store_link<R>(base, n, convert<R>(out));
}

// ---------------------------------------------------------------------------
// plaquette: sum over sites of Re Tr U_mu(x) U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
// = Re Tr P Q^+ with P = U_mu(x) U_nu(x+mu), Q = U_nu(x) U_mu(x+nu), in FP64.
// ---------------------------------------------------------------------------

// Re Tr P Q^+ of two SU(3) matrices from their rows 0 and 1: with G_ij = p_i .
// q_j^* for i, j < 2, the third rows' product is conj(det G) (the third row is
// the conjugate cross product of the first two).
__device__ __forceinline__ double retr_pq(const M3<double> &P, const M3<double> &Q)
{
    Cx<double> G[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            G[i][j] = cmul_cn(Q.e[j][0], P.e[i][0]);
            G[i][j] = cmadd_cn(G[i][j], Q.e[j][1], P.e[i][1]);
            G[i][j] = cmadd_cn(G[i][j], Q.e[j][2], P.e[i][2]);
        }
    double s = G[0][0].re + G[1][1].re;
    s = fma(G[0][0].re, G[1][1].re, s);
    s = fma(-G[0][0].im, G[1][1].im, s);
    s = fma(-G[0][1].re, G[1][0].re, s);
    return fma(G[0][1].im, G[1][0].im, s);
}

// rows 0 and 1 of A B (B with its row 2)
__device__ __forceinline__ M3<double> rows_nn(const M3<double> &A, const M3<double> &B)
{
    M3<double> C;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            Cx<double> t = cmul(A.e[a][0], B.e[0][b]);
            t = cmadd(t, A.e[a][1], B.e[1][b]);
            C.e[a][b] = cmadd(t, A.e[a][2], B.e[2][b]);
        }
    return C;
}

// Rows 0 and 1 of a link in FP64.
template <typename R, typename O> __device__ __forceinline__ M3<double> rows_of(Block<R> b, O o)
{
    M3<R> m;
    load_rows(m, b, o);
    M3<double> d;
#pragma unroll
    for (int e = 0; e < kEntries; ++e)
        d.e[e / 3][e % 3] = Cx<double>{(double)m.e[e / 3][e % 3].re, (double)m.e[e / 3][e % 3].im};
    return d;
}

// rebuild_row2 with each real entry a sum of four products in one chain of
// fused multiply-adds: 24 instructions instead of 30, and fewer roundings
__device__ __forceinline__ void row2_chain(M3<double> &u)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const Cx<double> a = u.e[0][(k + 1) % 3], b = u.e[1][(k + 2) % 3];
        const Cx<double> c = u.e[0][(k + 2) % 3], d = u.e[1][(k + 1) % 3];
        u.e[2][k].re = fma(c.im, d.im, fma(-c.re, d.re, fma(-a.im, b.im, a.re * b.re)));
        u.e[2][k].im = fma(c.im, d.re, fma(c.re, d.im, fma(-a.im, b.re, -(a.re * b.im))));
    }
}

// Plane (mu, nu) of a site: own links Um, Un (rows 0, 1), neighbours Vn =
// U_nu(x+mu), Vm = U_mu(x+nu).
__device__ __forceinline__ double plaq_plane(const M3<double> &Um, const M3<double> &Un, M3<double> Vn, M3<double> Vm)
{
    row2_chain(Vn);
    row2_chain(Vm);
    return retr_pq(rows_nn(Um, Vn), rows_nn(Un, Vm));
}

// 1 if the stored rows 0 and 1 of u are not finite or not orthonormal within
// tol (|r0|^2 - 1, |r1|^2 - 1, <r0, r1>), else 0.  Row 2 is conj(r0 x r1), so
// orthonormal rows 0 and 1 make u an SU(3) matrix.  NaN fails every test.
__device__ __forceinline__ int link_bad(const M3<double> &u, double tol)
{
    double n0 = 0.0, n1 = 0.0;
    Cx<double> d{0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        n0 += u.e[0][k].re * u.e[0][k].re + u.e[0][k].im * u.e[0][k].im;
        n1 += u.e[1][k].re * u.e[1][k].re + u.e[1][k].im * u.e[1][k].im;
        d = cmadd_cn(d, u.e[0][k], u.e[1][k]);
    }
    const bool ok = fabs(n0 - 1.0) <= tol && fabs(n1 - 1.0) <= tol && fabs(d.re) <= tol && fabs(d.im) <= tol;
    return ok ? 0 : 1;
}

// Grid (nblk, nlat), four waves per workgroup.  Workgroup b (XCD-remapped) sums
// the contiguous run of tiles [b T, (b+1) T) of its layer in the pass order; a
// tile is 64 half-indices, and each parity's 64 sites are taken by two waves:
// one for the planes of directions 0, 1, 2, one for the three planes with
// direction 3.  Fixed order per lane, per wave and per workgroup: the sum is
// bitwise reproducible.  partials[l nblk + b]: plaquette sum of workgroup b of
// layer l; partials[(nlat + l) nblk + b]: its number of failing links.
// Half a site per lane needs 160 registers, three waves per SIMD; one lane per
// FP64 site took 256.  us per call, one lane per site (FP32: two sites) ->
// this: FP64 8^4 42 -> 30, 16^4 44 -> 34, 20^4 63 -> 50, 24^4 (walk below) 74 -> 66;
// FP32 16^4 37 -> 33, 32^4 110 -> 106, 40^4 368 -> 245.  It reads each link 4.75
// times on average and L2 hits are few, so large FP64 lattices walk instead
// (32^4 185 us here, 161 there).  Keeping the tile's own links in LDS for its
// waves spilled.
template <typename R, bool DLT, bool BIG>
__global__ __launch_bounds__(kBlock, 2) void k_plaq(const store_t<R> *__restrict__ links, const Geom g,
                                                    const int tiles_per_block, const double tol,
                                                    double *__restrict__ partials)
{
    const int layer = DLT ? (int)blockIdx.y : 0;
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int par = w & 1, opp = par ^ 1;
    const bool with3 = w >> 1;
    double s = 0.0;
    int bad = 0;
    for (int t = 0; t < tiles_per_block; ++t) {
        const int v = (b * tiles_per_block + t) * 64 + lane;
        if (v >= g.Vh) break;
        Site x;
        x.layer = layer;
        x.i = order_site(g, par, v, x.x);
        const auto at = [&](Step d) { return link_offset<R, BIG>(elem<DLT>(g, x, d)); };
        const offset_t<BIG> here = link_offset<R, BIG>(DLT && layer ? x.i + g.Vh : x.i);
        const auto own = [&](int d) { return rows_of<R>(block_of<R>(links, g, d, par), here); };
        const auto nbr = [&](int d, offset_t<BIG> o) { return rows_of<R>(block_of<R>(links, g, d, opp), o); };
        const offset_t<BIG> o0 = at(step_of<0, +1>(g, x)), o1 = at(step_of<1, +1>(g, x)), o2 = at(step_of<2, +1>(g, x));
        if (!with3) {
            const M3<double> U0 = own(0), U1 = own(1);
            s += plaq_plane(U0, U1, nbr(1, o0), nbr(0, o1));
            bad += link_bad(U0, tol) + link_bad(U1, tol);
            const M3<double> U2 = own(2);
            s += plaq_plane(U0, U2, nbr(2, o0), nbr(0, o2));
            bad += link_bad(U2, tol);
            s += plaq_plane(U1, U2, nbr(2, o1), nbr(1, o2));
        } else {
            const offset_t<BIG> o3 = at(step_of<3, +1>(g, x));
            const M3<double> U3 = own(3);
            bad += link_bad(U3, tol);
            s += plaq_plane(own(0), U3, nbr(3, o0), nbr(0, o3));
            s += plaq_plane(own(1), U3, nbr(3, o1), nbr(1, o3));
            s += plaq_plane(own(2), U3, nbr(3, o2), nbr(2, o3));
        }
    }
    const double bs = block_sum(s);
    __syncthreads();
    const double bb = block_sum((double)bad);
    if (threadIdx.x == 0) {
        partials[blockIdx.y * gridDim.x + blockIdx.x] = bs;
        partials[(gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = bb;
    }
}

// Rows 0 and 1 of a link (row 2 never formed), in FP64.
template <typename R> __device__ __forceinline__ M3<double> load_rows01(const store_t<R> *block, int n)
{
    M3<double> m;
    const store_t<R> *p = link_at<R>(block, n);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        const store_t<R> v = p[e * kTile];
        m.e[e / 3][e % 3] = Cx<double>{(double)v.x, (double)v.y};
    }
    return m;
}

// rows 0 and 1 of A^+ B (both with row 2)
__device__ __forceinline__ M3<double> rows_dn(const M3<double> &A, const M3<double> &B)
{
    M3<double> C;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            Cx<double> t = cmul_cn(A.e[0][a], B.e[0][b]);
            t = cmadd_cn(t, A.e[1][a], B.e[1][b]);
            C.e[a][b] = cmadd_cn(t, A.e[2][a], B.e[2][b]);
        }
    return C;
}

// One column of the plaquette walk: the sites (x0, x1, x2, x3) of the
// thread's chunk [x3a, x3b) of x3, in increasing x3.  At each site the four
// own links are loaded once (and checked); the planes (mu, nu), nu < 3, take
// the links of the forward neighbours x + mu in the same x3 slab.  A plane
// (mu, 3) needs U_mu(x + 3), the next site's own link:
//   Re Tr U_mu(x) U_3(x + mu) U_mu(x + 3)^+ U_3(x)^+ = Re Tr M_mu U_mu(x + 3)^+,
//   M_mu = U_3(x)^+ U_mu(x) U_3(x + mu),
// so M_mu (rows 0, 1) is formed at x and carried to the next site.  Every
// link is then read as an own link and by its three backward neighbours in
// the same step of the walk, each own link is loaded and checked once, and
// only the last site of a chunk reads links of the slab above it.
// Summation order: fixed per thread.
template <typename R, bool DLT>
__device__ __forceinline__ double plaq_column(const store_t<R> *__restrict__ links, const Geom &g, int layer,
                                              int nch, int w, double tol, int &bad)
{
    int x[4];
    const int c = walk_column(g, nch, w, x);
    const int x3a = (int)((long long)c * g.L[3] / nch), x3b = (int)((long long)(c + 1) * g.L[3] / nch);
    const int lbase = DLT ? layer * g.Vh : 0;
    M3<double> M0, M1, M2;
    double s = 0.0;
    for (int x3 = x3a; x3 < x3b; ++x3) {
        x[3] = x3;
        const int par = (x[0] + x[1] + x[2] + x3) & 1, opp = par ^ 1;
        const int n = lbase + (lex_of(g, x) >> 1);
        const M3<double> U0 = load_rows01<R>(planes<R>(links, g, 0, par), n);
        const M3<double> U1 = load_rows01<R>(planes<R>(links, g, 1, par), n);
        const M3<double> U2 = load_rows01<R>(planes<R>(links, g, 2, par), n);
        M3<double> U3 = load_rows01<R>(planes<R>(links, g, 3, par), n);
        bad += link_bad(U0, tol) + link_bad(U1, tol) + link_bad(U2, tol) + link_bad(U3, tol);
        if (x3 > x3a) {
            // planes (mu, 3) of the site below
            s += retr_pq(M0, U0);
            s += retr_pq(M1, U1);
            s += retr_pq(M2, U2);
        }
        const int e0 = nbr_elem<0, +1, 0, 0, DLT>(g, x, layer);
        const int e1 = nbr_elem<1, +1, 0, 0, DLT>(g, x, layer);
        const int e2 = nbr_elem<2, +1, 0, 0, DLT>(g, x, layer);
        rebuild_row2(U3);
        s += retr_pq(rows_nn(U0, convert<double>(load_link12<R>(planes<R>(links, g, 1, opp), e0))),
                       rows_nn(U1, convert<double>(load_link12<R>(planes<R>(links, g, 0, opp), e1))));
        s += retr_pq(rows_nn(U0, convert<double>(load_link12<R>(planes<R>(links, g, 2, opp), e0))),
                       rows_nn(U2, convert<double>(load_link12<R>(planes<R>(links, g, 0, opp), e2))));
        M0 = rows_dn(U3, mul_nn_su3(U0, convert<double>(load_link12<R>(planes<R>(links, g, 3, opp), e0))));
        s += retr_pq(rows_nn(U1, convert<double>(load_link12<R>(planes<R>(links, g, 2, opp), e1))),
                       rows_nn(U2, convert<double>(load_link12<R>(planes<R>(links, g, 1, opp), e2))));
        M1 = rows_dn(U3, mul_nn_su3(U1, convert<double>(load_link12<R>(planes<R>(links, g, 3, opp), e1))));
        M2 = rows_dn(U3, mul_nn_su3(U2, convert<double>(load_link12<R>(planes<R>(links, g, 3, opp), e2))));
    }
    if (x3b > x3a) {
        // planes (mu, 3) of the chunk's last site: the links of the slab above
        x[3] = x3b - 1;
        const int opp = ((x[0] + x[1] + x[2] + x[3]) & 1) ^ 1;
        const int e3 = nbr_elem<3, +1, 0, 0, DLT>(g, x, layer);
        s += retr_pq(M0, load_rows01<R>(planes<R>(links, g, 0, opp), e3));
        s += retr_pq(M1, load_rows01<R>(planes<R>(links, g, 1, opp), e3));
        s += retr_pq(M2, load_rows01<R>(planes<R>(links, g, 2, opp), e3));
    }
    return s;
}

// Plaquette of FP64 lattices by walking x3 (plaq_walk_chunks says which): grid
// (nblk, nlat), workgroup b (XCD-remapped) takes the threads [b T, (b+1) T) of
// the column order (walk_column), T = tiles_per_block kPlaqWalkBlock.  Output as
// k_plaq.  The reuse of a link along x3 comes from registers; its reuse by the
// three backward neighbours in the slab comes from L2 as far as that holds the
// sites in flight (32^4: 2.4 times the stored bytes past L2).  A call at 32^4
// (4 chunks of 8, two waves per SIMD) takes 161 us against 185 us by tiles, at
// 64^4 1.93 against 3.6 ms.
template <typename R, bool DLT>
__global__ __launch_bounds__(kPlaqWalkBlock, 2) void k_plaq_walk(const store_t<R> *__restrict__ links, const Geom g,
                                                                 const int nch, const int tiles_per_block,
                                                                 const double tol, double *__restrict__ partials)
{
    const int layer = DLT ? (int)blockIdx.y : 0;
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const int nthreads = g.L[0] * g.L[1] * g.L[2] * nch;
    double s = 0.0;
    int bad = 0;
    for (int t = 0; t < tiles_per_block; ++t) {
        const int w = (b * tiles_per_block + t) * kPlaqWalkBlock + threadIdx.x;
        if (w < nthreads) s += plaq_column<R, DLT>(links, g, layer, nch, w, tol, bad);
    }
    const double bs = block_sum<kPlaqWalkBlock>(s);
    __syncthreads();
    const double bb = block_sum<kPlaqWalkBlock>((double)bad);
    if (threadIdx.x == 0) {
        partials[blockIdx.y * gridDim.x + blockIdx.x] = bs;
        partials[(gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = bb;
    }
}

// sums[1 + l] = sum over the partials of layer l; sums[0] = sum over layers;
// sums[3] = number of links that failed the unitarity check.  With `mean`
// non-null also the normalised values: mean[0] = sums[0] / (norm nlat),
// mean[1 + l] = sums[1 + l] / norm, mean[1 + nlat] = sums[3] (norm = 18 V).
// One workgroup of 1024 threads with four loads in flight each: 4096 partials in
// 5 us (13 us with 256 threads and one load).
constexpr int kSumBlock = 1024;
__device__ __forceinline__ double sum_range(const double *__restrict__ a, int n)
{
    double s = 0.0;
    int b = threadIdx.x;
    for (; b + 3 * kSumBlock < n; b += 4 * kSumBlock) {
        const double v0 = a[b], v1 = a[b + kSumBlock], v2 = a[b + 2 * kSumBlock], v3 = a[b + 3 * kSumBlock];
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; b < n; b += kSumBlock) s += a[b];
    return s;
}
__global__ __launch_bounds__(kSumBlock) void k_plaq_final(const double *__restrict__ partials, int nblk, int nlat,
                                                          double *__restrict__ sums, double *__restrict__ mean,
                                                          double norm)
{
    double tot = 0.0;
    const double s0 = sum_range(partials, nblk), s1 = nlat == 2 ? sum_range(partials + nblk, nblk) : 0.0;
    const double nb = sum_range(partials + nlat * nblk, nlat * nblk);
    for (int l = 0; l < nlat; ++l) {
        const double r = block_sum<kSumBlock>(l == 0 ? s0 : s1);
        __syncthreads();
        if (threadIdx.x == 0) {
            sums[1 + l] = r;
            tot += r;
        }
    }
    const double r = block_sum<kSumBlock>(nb);
    if (threadIdx.x == 0) {
        sums[0] = tot;
        if (nlat == 1) sums[2] = 0.0;
        sums[3] = r;
        if (mean) {
            mean[0] = tot / (norm * nlat);
            for (int l = 0; l < nlat; ++l) mean[1 + l] = sums[1 + l] / norm;
            mean[1 + nlat] = r;
        }
    }
}

// Double-layered torus: per-layer plaquette sums of a measured sweep from the
// nmeas pairs (layer 0, layer 1) of the three measured passes, fixed order:
// sums[1 + l] = the sum of layer l, sums[0] = sums[1] + sums[2].
__global__ __launch_bounds__(kSumBlock) void k_measure_final_dlt(const double *__restrict__ meas, int nmeas,
                                                              double *__restrict__ sums)
{
    double t0 = 0.0, t1 = 0.0;
    for (int k = threadIdx.x; k < nmeas; k += kSumBlock) {
        t0 += meas[2 * k];
        t1 += meas[2 * k + 1];
    }
    const double T0 = block_sum<kSumBlock>(t0);
    __syncthreads();
    const double T1 = block_sum<kSumBlock>(t1);
    if (threadIdx.x == 0) {
        sums[0] = T0 + T1;
        sums[1] = T0;
        sums[2] = T1;
    }
}

// single torus: sums[0] = sums[1] = sum of the partials a[0..na), fixed order
__global__ __launch_bounds__(kSumBlock) void k_sum_partials(const double *__restrict__ a, int na,
                                                            double *__restrict__ sums)
{
    // thread t adds a[t], a[t + kSumBlock], ... in that order; the loads of
    // eight terms are issued together
    double s = 0.0;
    int k = threadIdx.x;
    for (; k + 7 * kSumBlock < na; k += 8 * kSumBlock) {
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = a[k + j * kSumBlock];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; k < na; k += kSumBlock) s += a[k];
    const double r = block_sum<kSumBlock>(s);
    if (threadIdx.x == 0) {
        sums[0] = r;
        sums[1] = r;
    }
}

__global__ void k_zero_u64(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// bandwidth probe: 16-byte loads and stores, grid-stride over a grid of
// four workgroups per CU (the shape that copied fastest on this chip)
__global__ __launch_bounds__(kBlock) void k_copy(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n)
{
    const size_t step = (size_t)gridDim.x * kBlock;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += step) dst[i] = src[i];
}

inline unsigned blocks_for(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace


hipError_t launch_start(int precision, void *links, const Geom &g, int hot, uint64_t seed, hipStream_t s)
{
    const dim3 grid(blocks_for((long long)g.nlat * g.Vh), 8);
    if (precision == 64)
        k_start<double><<<grid, kBlock, 0, s>>>((double2 *)links, g, hot, seed);
    else
        k_start<float><<<grid, kBlock, 0, s>>>((float2 *)links, g, hot, seed);
    return hipGetLastError();
}

hipError_t launch_measure_final(const double *meas, const Geom &g, double *sums, hipStream_t s)
{
    const int nmeas = 3 * meas_blocks(g);
    if (g.nlat == 1)
        k_sum_partials<<<1, kSumBlock, 0, s>>>(meas, nmeas, sums);
    else
        k_measure_final_dlt<<<1, kSumBlock, 0, s>>>(meas, nmeas, sums);
    return hipGetLastError();
}

template <typename R>
static void plaq_launch(const store_t<R> *links, const Geom &g, int nblk, int tpb, double tol, bool big,
                        double *partials, hipStream_t s)
{
    const dim3 grid(nblk, g.nlat);
    if (big)
        k_plaq<R, true, true><<<grid, kBlock, 0, s>>>(links, g, tpb, tol, partials);
    else if (g.nlat == 2)
        k_plaq<R, true, false><<<grid, kBlock, 0, s>>>(links, g, tpb, tol, partials);
    else
        k_plaq<R, false, false><<<grid, kBlock, 0, s>>>(links, g, tpb, tol, partials);
}

hipError_t launch_plaquette(int precision, const void *links, const Geom &g, double *partials, double *sums,
                            hipStream_t s, double *mean)
{
    const int nch = plaq_walk_chunks(g, precision), nblk = plaq_launch_blocks(g, precision);
    const double tol = unitarity_tol(precision);
    if (nch > 0) {
        // FP64 lattices with enough columns: the x3 walk
        const dim3 grid(nblk, g.nlat);
        const long long tiles = ((long long)g.L[0] * g.L[1] * g.L[2] * nch + kPlaqWalkBlock - 1) / kPlaqWalkBlock;
        const int tpb = (int)((tiles + nblk - 1) / nblk);
        if (g.nlat == 2)
            k_plaq_walk<double, true><<<grid, kPlaqWalkBlock, 0, s>>>((const double2 *)links, g, nch, tpb, tol,
                                                                      partials);
        else
            k_plaq_walk<double, false><<<grid, kPlaqWalkBlock, 0, s>>>((const double2 *)links, g, nch, tpb, tol,
                                                                       partials);
    } else {
        const long long tiles = ((long long)g.Vh + 63) / 64;
        const int tpb = (int)((tiles + nblk - 1) / nblk);
        if (precision == 64)
            plaq_launch<double>((const double2 *)links, g, nblk, tpb, tol, pass_big(g, 64), partials, s);
        else
            plaq_launch<float>((const float2 *)links, g, nblk, tpb, tol, pass_big(g, 32), partials, s);
    }
    k_plaq_final<<<1, kSumBlock, 0, s>>>(partials, nblk, g.nlat, sums, mean, 36.0 * (double)g.Vh);
    return hipGetLastError();
}

hipError_t launch_polyakov(int precision, const void *links, const Geom &g, double *partials, double *out,
                           hipStream_t s)
{
    const int nblk = polyakov_blocks(g);
    const dim3 grid(nblk, g.nlat);
    if (precision == 64)
        k_polyakov<double><<<grid, kBlock, 0, s>>>((const double2 *)links, g, partials);
    else
        k_polyakov<float><<<grid, kBlock, 0, s>>>((const float2 *)links, g, partials);
    k_polyakov_final<<<1, kBlock, 0, s>>>(partials, nblk, g.nlat, out);
    return hipGetLastError();
}

hipError_t launch_reunit(int precision, void *links, const Geom &g, hipStream_t s)
{
    const dim3 grid(blocks_for((long long)g.nlat * g.Vh), 8);
    if (precision == 64)
        k_reunit<double><<<grid, kBlock, 0, s>>>((double2 *)links, g);
    else
        k_reunit<float><<<grid, kBlock, 0, s>>>((float2 *)links, g);
    return hipGetLastError();
}

hipError_t launch_gauge(int precision, void *links, const Geom &g, uint64_t gseed, hipStream_t s)
{
    const dim3 grid(blocks_for((long long)g.nlat * g.Vh), 8);
    if (precision == 64)
        k_gauge<double><<<grid, kBlock, 0, s>>>((double2 *)links, g, gseed);
    else
        k_gauge<float><<<grid, kBlock, 0, s>>>((float2 *)links, g, gseed);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long *p, int n, hipStream_t s)
{
    k_zero_u64<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    long long want = (long long)((n + kBlock - 1) / kBlock);
    const unsigned grid = (unsigned)(want < 1024 ? (want > 0 ? want : 1) : 1024);
    k_copy<<<grid, kBlock, 0, s>>>((const uint4 *)src, (uint4 *)dst, n);
    return hipGetLastError();
}

}  // namespace su3hb
