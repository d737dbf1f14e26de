// layout.cpp -- host-side geometry, buffer layout and launch shapes (see
// layout.h).  No HIP calls: everything here is plain arithmetic on the
// parameters, so it is validated before any device work and can be checked
// on the CPU under the address and undefined-behaviour sanitizers.
#include "layout.h"

#include <string>

namespace su3hb {

namespace {
thread_local std::string g_last_error;
long long round_up(long long a, long long m) { return (a + m - 1) / m * m; }
long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }
}  // namespace

su3_status fail(su3_status s, const std::string &msg)
{
    g_last_error = msg;
    return s;
}

const char *last_error() { return g_last_error.c_str(); }

su3_status check_params(const su3_params *p)
{
    if (!p) return fail(SU3_EINVAL, "params is NULL");
    for (int mu = 0; mu < 4; ++mu) {
        const int L = p->L[mu];
        if (L < 2 || L > 1024 || (L & 1))
            return fail(SU3_EINVAL, "L[" + std::to_string(mu) + "] = " + std::to_string(L) +
                                        ": extents must be even and in [2, 1024]");
    }
    if (p->nlat != 1 && p->nlat != 2) return fail(SU3_EINVAL, "nlat must be 1 (torus) or 2 (double-layered torus)");
    if (p->nlat == 1 && p->flip_mask != 0) return fail(SU3_EINVAL, "flip_mask must be 0 when nlat = 1");
    if (p->flip_mask > 0xF) return fail(SU3_EINVAL, "flip_mask has bits above direction 3");
    if (p->precision != 64 && p->precision != 32) return fail(SU3_EINVAL, "precision must be 64 or 32");
    if (p->nhit < 1 || p->nhit > 64) return fail(SU3_EINVAL, "nhit must be in [1, 64]");
    const long long V = (long long)p->L[0] * p->L[1] * p->L[2] * p->L[3];
    if ((long long)p->nlat * V > (1LL << 30))
        return fail(SU3_EINVAL, "lattice too large: nlat*V must not exceed 2^30 sites");
    return SU3_OK;
}

// Domains of the pass order (the (x1, x2) cross-section cut into w1 x w2
// pieces, each swept along x3).  A link on a domain's rim is read by two
// XCDs, each from HBM, so the choice takes the fewest rim links, the sum of
// 1/w over the directions that are cut, among the widths that
//  * give every XCD whole domains: nd * nlat a multiple of 8, nd = (L1/w1)(L2/w2);
//  * keep one x3 slab of a domain within kSlabMax = 4096 updates
//    (L0/2 w1 w2 <= 4096), so that the links around it are re-read while
//    still in L2;
//  * keep the lanes of a wave on whole 16-link tiles: L0/2 w1 a multiple of 16,
//    or w1 = L1.
// Ties go to the wider w1 (longer runs of consecutive links).  Without such
// widths the rule keeps w1 = L1 and the largest w2 <= L2/8.
void pick_domains(const int32_t L[4], int nlat, int &w1, int &w2)
{
    constexpr long long kSlabMax = 4096;
    const int l0h = L[0] / 2;
    double best = 1e30;
    w1 = L[1];
    w2 = 0;
    for (int a = L[1]; a >= 1; --a) {
        if (L[1] % a || (a != L[1] && (l0h * a) % 16)) continue;
        for (int b = L[2]; b >= 1; --b) {
            if (L[2] % b) continue;
            const long long nd = (long long)(L[1] / a) * (L[2] / b) * nlat;
            if (nd % 8 || (long long)l0h * a * b > kSlabMax) continue;
            const double rim = (a < L[1] ? 1.0 / a : 0.0) + (b < L[2] ? 1.0 / b : 0.0);
            if (rim < best - 1e-12) {
                best = rim;
                w1 = a;
                w2 = b;
            }
        }
    }
    if (w2 == 0) {
        w1 = L[1];
        w2 = 1;
        for (int b = 1; b <= L[2] / 8; ++b)
            if (L[2] % b == 0) w2 = b;
    }
}

Geom make_geom(const su3_params *p)
{
    Geom g;
    for (int mu = 0; mu < 4; ++mu) g.L[mu] = p->L[mu];
    const long long V = (long long)p->L[0] * p->L[1] * p->L[2] * p->L[3];
    g.Vh = (int)(V / 2);
    g.nlat = p->nlat;
    g.flip = p->nlat == 2 ? p->flip_mask : 0u;
    // +64: the (direction, parity) blocks are offset by 64 links from a large
    // power-of-two spacing, so equal positions in different blocks do not all
    // fall in the same L2 channel and set
    g.stride = round_up((long long)p->nlat * (V / 2), 64) + 64;
    // a step along direction 0 moves the half-index by 0 or 1; the others by
    // half the lexicographic stride, which is even
    g.hs[0] = 1;
    g.wrap[0] = p->L[0] / 2 - 1;
    for (int mu = 1, h = p->L[0] / 2; mu < 4; h *= p->L[mu], ++mu) {
        g.hs[mu] = h;
        g.wrap[mu] = (p->L[mu] - 1) * h;
    }
    pick_domains(p->L, p->nlat, g.w1, g.w2);
    g.nd1 = p->L[1] / g.w1;
    g.dl0h = make_fastdiv((uint32_t)(p->L[0] / 2));
    g.dl1 = make_fastdiv((uint32_t)p->L[1]);
    g.dl2 = make_fastdiv((uint32_t)p->L[2]);
    g.dl3 = make_fastdiv((uint32_t)p->L[3]);
    g.dw1 = make_fastdiv((uint32_t)g.w1);
    g.dw2 = make_fastdiv((uint32_t)g.w2);
    g.dnd1 = make_fastdiv((uint32_t)g.nd1);
    return g;
}

size_t link_bytes_of(const su3_params *p, const Geom &g)
{
    // 8 (direction, parity) blocks of `stride` links, 6 complex entries each
    return (size_t)8 * kEntries * (size_t)g.stride * (p->precision == 64 ? 16u : 8u);
}

// The sizes at which small passes shared one link's work between 2 or 4 lanes,
// kept for what su3_get_lanes_per_link reports; pass_six_waves has its own.
constexpr long long kLanes4Max = 8192, kLanes2Max = 32768;

int lanes_per_link(const Geom &g, int nhit, int requested)
{
    if (requested > 0) return requested;
    if (nhit != 1) return 1;
    const long long n = (long long)g.nlat * g.Vh;
    return n <= kLanes4Max ? 4 : (n <= kLanes2Max ? 2 : 1);
}

bool pass_big(const Geom &g, int precision)
{
    return (unsigned long long)g.stride * kEntries * (precision == 64 ? 16u : 8u) >= (1ull << 32);
}

// Six waves per tile instead of three take the draws out of the chain that a
// pass with few tiles waits for; with more tiles than run at once only the
// number of instructions and the waves per SIMD count, and six waves hold
// their registers until the slowest ends.  us per pass, six against three waves
// (measured: of a sweep whose odd passes of mu = 1, 2, 3 measure):
//   FP64           256 tiles 6.8 / 7.5, 320 9.9 / 9.2 (a second workgroup of six
//                  waves of 152 registers does not fit a CU beside the first);
//   FP64, 3 hits   256 tiles 10.5 / 11.5, 320 13.1 / 13.0;
//   FP64 measured  256 tiles 7.7 / 8.3, 320 10.9 / 10.1; two layers 8.5 / 9.1, 12.5 / 10.8;
//   FP64 couplings 256 tiles 7.3 / 8.0, 320 10.7 / 9.6;
//   FP32           768 tiles 8.4 / 8.7, 896 9.4 / 9.3;
//   FP32, 3 hits   512 tiles 9.8 / 11.0, 576 11.6 / 11.4 (six waves make every
//                  second draw, three only the likely ones);
//   FP32 measured  768 tiles 9.5 / 9.7, 896 10.7 / 10.4; two layers 10.9 / 10.9, 12.5 / 12.0;
//   FP32 couplings 512 tiles 7.8 / 8.6, 640 10.1 / 9.1 (100 registers: four waves per SIMD).
bool pass_six_waves(int precision, bool plain, long long tiles, int requested)
{
    if (requested > 0) return requested > 1;
    return tiles <= (precision == 64 ? 256 : plain ? 768 : 512);
}

// Several attempts, one wave per tile instead of three (or six): it has all its
// attempts to itself, two such waves share a SIMD, and a few lanes that miss
// often get a round of 64 at once, where the three waves' first one draws for
// the others while these hold their registers or have ended.  So it takes
// lattices where many attempts miss (beta below 4: those made ahead do not
// cover them any more), unless few waves are there to share the work, and large
// ones, whose waves wait for memory anyway (FP64 ones first; with layer couplings
// the three waves spill).  us per pass, one wave / three
// (six where these are in brackets), from one run each:
//   FP64, 2 hits  16^4 beta 2 17.4 / 15.9, 24^4 beta 2 42.5 / 45.7, beta 3.5 42.5 / 42.3, beta 4.5
//                 42.1 / 38.4, 32^4 beta 2 110 / 125, beta 4.5 108 / 107, 40^4 beta 4.5 257 / 263;
//   FP64, 3 hits  16^4 beta 2 20.9 / 19.6, 24^4 49.4 / 55.1, 32^4 120 / 150, 64^4 beta 5.7 1684 / 1759;
//   FP64, 8 hits  8^4 beta 2 24.4 [26.1], 16^4 beta 2 25.5 / 36.3, beta 3.5 24.4 / 25.4;
//   FP64, 64 hits 8^4 beta 0.5 41 [192], beta 2 24 [41];
//   FP32, 2 hits  20^4 beta 2 19.4 / 17.0, 24^4 26.9 / 29.2, 32^4 60 / 67, beta 4.5 59.5 / 56.0;
//   FP32, 8 hits  20^4 beta 2 28.0 / 35.9, beta 3.5 25.5 / 24.5;
//   FP32, 3 hits, beta 5.7  40^4 141 / 139, 64^4 911 / 939, 48^4 measured 299 / 304;
//   measured FP64, 2 hits  24^4 beta 5 43.8 / 40.4, 32^4 beta 5 110 / 113;
//   layer couplings FP64, 2 hits, beta 5.7  2 x 12^4 16.8 / 13.7, 2 x 16^4 20.8 / 22.7, 2 x 32^4 213 / 279.
bool pass_one_lane(int precision, int nhit, double beta, bool measured, bool twob, long long tiles)
{
    if (nhit == 1) return false;
    if (tiles >= (precision == 32 ? 32768 : twob ? 1024 : measured ? 8192 : 16384)) return true;
    if (beta >= 4.0) return false;
    if (tiles >= (precision == 64 ? 1024 : 2048)) return true;
    return nhit >= (pass_six_waves(precision, false, tiles) ? 16 : 6) && beta < (precision == 64 ? 4.0 : 3.0);
}

int pass_links_per_block(const Geom &, int) { return kPassBlock; }

int pass_blocks(const Geom &g, int nb) { return (int)ceil_div((long long)g.nlat * g.Vh, nb); }

// Workgroups for n tiles, at most `most`, each with the same number of tiles
// but the last: the XCDs take contiguous runs of workgroups, so empty ones at
// the end would leave whole XCDs idle (8 x 38 x 56 x 34 in FP32, 4522 tiles: 116 us
// with 4096 workgroups of up to two tiles).
static int even_blocks(long long n, int most) { return (int)ceil_div(n, ceil_div(n, most)); }

int plaq_tile_blocks(const Geom &g) { return even_blocks(ceil_div(g.Vh, 64), kPlaqBlocksMax); }

int plaq_blocks(const Geom &g)
{
    const long long need = ceil_div(g.Vh, kBlock);
    return (int)(need < kPlaqBlocksMax ? need : kPlaqBlocksMax);
}

// The plaquette walk (one thread per column and chunk of x3, which reads
// each link as an own link and as a neighbour in the same step of the walk)
// takes FP64 lattices with enough columns for two waves per SIMD
// (kPlaqWalkThreads) in chunks of at least kPlaqWalkMinSteps sites: 32^4 161 us
// against 185 us by tiles, 64^4 1.93 against 3.6 ms.  Smaller ones, which fit
// the memory-side cache, are faster by tiles, as the last workgroups of the walk
// leave half the CUs idle, and so is FP32 (32^4 106 us, 64^4 1.49 ms).  But from
// one wave per SIMD on (kPlaqWalkMin) the walk keeps, us per call by walk / by tiles:
//   one workgroup on every CU (65536 threads): 32^3 x 8 57 / 61, 64 x 64 x 16 x 4 58 / 68,
//     2 x 32^3 x 6 71 / 90, 8^3 x 512 60 / 64 (12^3 x 160, 276 workgroups: 72 / 62);
//   whole columns: 64 x 64 x 20 x 4 72 / 74, 48^3 x 6 105 / 129 (64 x 64 x 18 x 4, 288 workgroups:
//     71 / 68; 24^4 in six chunks 73 / 66);
//   on two layers up to four chunks with 1.5 workgroups per CU: 2 x 24^3 x 16 84 / 89,
//     2 x 32 x 32 x 16 x 12 78 / 82 (2 x 20^3 x 24 in six chunks 82 / 78; one layer, 32^3 x 12 74 / 74);
//   more than kPlaqBlocksMax tiles per layer, of which a workgroup then takes two: 26^3 x 30 98 / 115,
//     6 x 10 x 14 x 626 117 / 139 (600: 109 / 97).
constexpr long long kPlaqWalkThreads = 131072, kPlaqWalkMin = 65536, kPlaqWalkMinSteps = 4;

int plaq_walk_chunks(const Geom &g, int precision)
{
    if (precision != 64) return 0;
    const long long cols = (long long)g.nlat * g.L[0] * g.L[1] * g.L[2];
    long long nch = ceil_div(kPlaqWalkThreads, cols);
    if (nch > g.L[3] / kPlaqWalkMinSteps) nch = g.L[3] / kPlaqWalkMinSteps;
    const long long threads = cols * nch;
    if (nch < 1 || threads < kPlaqWalkMin) return 0;
    const bool walks = threads >= kPlaqWalkThreads || threads == kPlaqWalkMin ||
                       (nch == 1 && 4 * threads >= 5 * kPlaqWalkMin) ||
                       (g.nlat == 2 && nch <= 4 && 2 * threads >= 3 * kPlaqWalkMin) ||
                       ceil_div(g.Vh, 64) > kPlaqBlocksMax;
    return walks ? (int)nch : 0;
}

int plaq_walk_blocks(const Geom &g, int nch)
{
    return even_blocks(ceil_div((long long)g.L[0] * g.L[1] * g.L[2] * nch, kPlaqWalkBlock), plaq_blocks(g));
}

int plaq_launch_blocks(const Geom &g, int precision)
{
    const int nch = plaq_walk_chunks(g, precision);
    return nch > 0 ? plaq_walk_blocks(g, nch) : plaq_tile_blocks(g);
}

size_t plaq_partial_bytes(const Geom &g, int precision)
{
    return 2 * sizeof(double) * (size_t)g.nlat * (size_t)plaq_launch_blocks(g, precision);
}

int meas_blocks(const Geom &g, int lanes) { return pass_blocks(g, pass_links_per_block(g, lanes)); }

int polyakov_blocks(const Geom &g) { return (int)ceil_div((long long)g.L[0] * g.L[1] * g.L[2], kBlock); }

// Plaquette partials: per layer and workgroup the plaquette sum, then the
// number of links that fail the unitarity check.  plaq_blocks(g) of them have
// room of their own; the others (plaq_tile_blocks) run on into the measured-pass
// partials, 24 nlat bytes or more per 64 half-indices: either set is written
// and summed up within one call, in stream order, and holds nothing between calls.
size_t meas_offset(const Geom &g) { return (size_t)round_up(kOffPartials + 2 * 8LL * g.nlat * plaq_blocks(g), 256); }

// measured-pass partials: 3 passes x nlat doubles per workgroup
size_t polyakov_offset(const Geom &g)
{
    return (size_t)round_up((long long)meas_offset(g) + 3 * 8LL * g.nlat * meas_blocks(g), 256);
}

size_t scratch_bytes_of(const Geom &g)
{
    return (size_t)round_up((long long)polyakov_offset(g) + 16LL * g.nlat * polyakov_blocks(g), 256);
}

size_t dev_index(const Geom &g, int dir, int par, int e, long long n)
{
    return (size_t)(dir * 2 + par) * (size_t)g.stride * kEntries + (size_t)(n >> 4) * (kEntries * kTile) +
           (size_t)e * kTile + (size_t)(n & (kTile - 1));
}

long long site_of_elem(const Geom &g, int par, long long n)
{
    const int layer = n >= g.Vh ? 1 : 0;
    const long long i = n - (long long)layer * g.Vh;
    const int l0h = g.L[0] / 2;
    long long r = i / l0h;
    const int x0h = (int)(i - r * l0h);
    const int x1 = (int)(r % g.L[1]);
    r /= g.L[1];
    const int x2 = (int)(r % g.L[2]);
    const int x3 = (int)(r / g.L[2]);
    const int x0 = 2 * x0h + ((par + x1 + x2 + x3) & 1);
    const long long lex = x0 + (long long)g.L[0] * (x1 + (long long)g.L[1] * (x2 + (long long)g.L[2] * x3));
    return (long long)layer * 2LL * g.Vh + lex;
}

bool elem_of_lid(const Geom &g, uint64_t lid, int *dir, int *par, long long *n)
{
    const uint64_t V = 2ull * (uint64_t)g.Vh;
    if (lid >= 4ull * V * (uint64_t)g.nlat) return false;
    const uint64_t site = lid / 4;
    *dir = (int)(lid % 4);
    const uint64_t layer = site / V;
    const uint64_t lex = site % V;
    uint64_t r = lex;
    int sum = 0;
    for (int mu = 0; mu < 4; ++mu) {
        sum += (int)(r % (uint64_t)g.L[mu]);
        r /= (uint64_t)g.L[mu];
    }
    *par = sum & 1;
    *n = (long long)(layer * (uint64_t)g.Vh + (lex >> 1));
    return true;
}

void rebuild_row2_host(double *m)
{
    for (int k = 0; k < 3; ++k) {
        const int a = (k + 1) % 3, b = (k + 2) % 3;
        const double p_re = m[2 * a] * m[6 + 2 * b] - m[2 * a + 1] * m[6 + 2 * b + 1];
        const double p_im = m[2 * a] * m[6 + 2 * b + 1] + m[2 * a + 1] * m[6 + 2 * b];
        const double q_re = m[2 * b] * m[6 + 2 * a] - m[2 * b + 1] * m[6 + 2 * a + 1];
        const double q_im = m[2 * b] * m[6 + 2 * a + 1] + m[2 * b + 1] * m[6 + 2 * a];
        m[12 + 2 * k] = p_re - q_re;
        m[12 + 2 * k + 1] = -(p_im - q_im);
    }
}

void unpack_links(int precision, const Geom &g, const void *image, double *host)
{
    const long long nelem = (long long)g.nlat * g.Vh;
    for (int par = 0; par < 2; ++par)
        for (long long n = 0; n < nelem; ++n) {
            const long long site = site_of_elem(g, par, n);
            for (int dir = 0; dir < 4; ++dir) {
                double *dst = host + (size_t)(4 * site + dir) * 18;
                for (int el = 0; el < kEntries; ++el) {
                    const size_t idx = dev_index(g, dir, par, el, n);
                    if (precision == 64) {
                        const double *v = (const double *)image + 2 * idx;
                        dst[2 * el] = v[0];
                        dst[2 * el + 1] = v[1];
                    } else {
                        const float *v = (const float *)image + 2 * idx;
                        dst[2 * el] = (double)v[0];
                        dst[2 * el + 1] = (double)v[1];
                    }
                }
                rebuild_row2_host(dst);
            }
        }
}

void pack_links(int precision, const Geom &g, const double *host, void *image)
{
    const long long nelem = (long long)g.nlat * g.Vh;
    for (int par = 0; par < 2; ++par)
        for (long long n = 0; n < nelem; ++n) {
            const long long site = site_of_elem(g, par, n);
            for (int dir = 0; dir < 4; ++dir) {
                const double *src = host + (size_t)(4 * site + dir) * 18;
                for (int el = 0; el < kEntries; ++el) {
                    const size_t idx = dev_index(g, dir, par, el, n);
                    if (precision == 64) {
                        double *v = (double *)image + 2 * idx;
                        v[0] = src[2 * el];
                        v[1] = src[2 * el + 1];
                    } else {
                        float *v = (float *)image + 2 * idx;
                        v[0] = (float)src[2 * el];
                        v[1] = (float)src[2 * el + 1];
                    }
                }
            }
        }
}

}  // namespace su3hb
