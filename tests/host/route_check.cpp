// Which kernel a call takes (paper_0904_1179_amd/csrc/layout.cpp), on the
// CPU: the rules at the sizes where they change, so that the GPU tests of a
// route do take it.
#include <cstdio>
#include <random>

#include "../../paper_0904_1179_amd/csrc/layout.h"

using namespace su3hb;

static int fails = 0;
#define CHECK(c, ...)                                                \
    do {                                                             \
        if (!(c)) {                                                  \
            std::fprintf(stderr, "FAIL line %d: %s: ", __LINE__, #c); \
            std::fprintf(stderr, __VA_ARGS__);                       \
            std::fprintf(stderr, "\n");                              \
            ++fails;                                                 \
        }                                                            \
    } while (0)

static su3_params params(int L0, int L1, int L2, int L3, int nlat = 1, int prec = 64, int nhit = 1)
{
    su3_params p{};
    p.L[0] = L0;
    p.L[1] = L1;
    p.L[2] = L2;
    p.L[3] = L3;
    p.nlat = nlat;
    p.flip_mask = nlat == 2 ? 7u : 0u;
    p.precision = prec;
    p.nhit = nhit;
    p.seed = 1;
    return p;
}

// chunks of the plaquette walk, 0: by tiles
static void walks()
{
    const struct {
        int L[4], nlat, nch;
    } c[] = {
        {{32, 32, 32, 32}, 1, 4},   {{24, 24, 24, 24}, 1, 0},  {{16, 16, 32, 32}, 2, 8}, {{6, 10, 14, 626}, 1, 156},
        {{6, 10, 14, 630}, 1, 157}, {{6, 10, 14, 600}, 1, 0},  {{6, 10, 14, 318}, 2, 79}, {{6, 10, 14, 314}, 2, 0},
        {{32, 32, 32, 8}, 1, 2},    {{64, 64, 16, 4}, 1, 1},   {{64, 64, 18, 4}, 1, 0},  {{64, 64, 20, 4}, 1, 1},
        {{48, 48, 48, 6}, 1, 1},    {{24, 24, 24, 16}, 2, 4},  {{24, 24, 24, 12}, 2, 0}, {{20, 20, 20, 24}, 2, 0},
        {{26, 26, 26, 30}, 1, 7},   {{26, 26, 26, 26}, 1, 0},  {{32, 32, 32, 6}, 2, 1},  {{12, 12, 12, 160}, 1, 0},
        {{16, 16, 16, 16}, 2, 0},   {{2, 2, 2, 2}, 1, 0},      {{64, 64, 64, 2}, 1, 0},  {{32, 32, 16, 16}, 2, 4},
        {{16, 16, 8, 66}, 2, 16},   {{66, 34, 30, 6}, 1, 0},
    };
    for (const auto &k : c) {
        const su3_params p = params(k.L[0], k.L[1], k.L[2], k.L[3], k.nlat);
        const Geom g = make_geom(&p);
        CHECK(plaq_walk_chunks(g, 64) == k.nch, "%d %d %d %d x %d: %d chunks, expected %d", k.L[0], k.L[1], k.L[2], k.L[3],
              k.nlat, plaq_walk_chunks(g, 64), k.nch);
        CHECK(plaq_walk_chunks(g, 32) == 0, "FP32 walks");
    }
}

// The plaquette's partials, by whichever route, lie before the Polyakov loops'
// (a context: they may run on into those of the measured passes) and within
// 131072 bytes, half of what su3_plaquette_noalloc has; measured passes have theirs.
static void scratch_case(const su3_params &p)
{
    if (check_params(&p) != SU3_OK) return;
    const Geom g = make_geom(&p);
    const size_t need = plaq_partial_bytes(g, p.precision);
    CHECK(kOffPartials + need <= polyakov_offset(g), "%d %d %d %d x %d f%d", p.L[0], p.L[1], p.L[2], p.L[3], p.nlat, p.precision);
    CHECK(need <= 131072, "%zu bytes: %d %d %d %d x %d", need, p.L[0], p.L[1], p.L[2], p.L[3], p.nlat);
    const int nblk = plaq_launch_blocks(g, p.precision), nch = plaq_walk_chunks(g, p.precision);
    const long long tiles = nch > 0 ? ((long long)g.L[0] * g.L[1] * g.L[2] * nch + kPlaqWalkBlock - 1) / kPlaqWalkBlock
                                    : ((long long)g.Vh + 63) / 64;
    const long long tpb = (tiles + nblk - 1) / nblk;
    CHECK(nblk >= 1 && tpb * nblk >= tiles && tpb * (nblk - 1) < tiles, "grid of %d workgroups for %lld tiles", nblk, tiles);
    CHECK(meas_offset(g) + 24 * (size_t)g.nlat * meas_blocks(g) <= polyakov_offset(g), "measured partials");
    CHECK(polyakov_offset(g) + 16 * (size_t)g.nlat * polyakov_blocks(g) <= scratch_bytes_of(g), "Polyakov partials");
}
static void scratch()
{
    std::mt19937_64 rng(7);
    for (int k = 0; k < 200000; ++k) {
        const auto extent = [&] { return 2 << (rng() % 9) | (int)(2 * (rng() % 40)); };
        scratch_case(params(extent(), extent(), extent(), extent(), 1 + (int)(rng() & 1), rng() & 1 ? 64 : 32));
    }
    for (int a = 2; a <= 96; a += 2)
        for (int b = 2; b <= 64; b += 2)
            for (int nlat : {1, 2}) scratch_case(params(a, a, b, a, nlat));
}

// a step of +1 or -1 along a direction, as the passes take it, against the coordinates
static void steps(const su3_params &p)
{
    const Geom g = make_geom(&p);
    const auto lex = [&](const int x[4]) { return x[0] + g.L[0] * (x[1] + g.L[1] * (x[2] + g.L[2] * x[3])); };
    int x[4];
    for (x[3] = 0; x[3] < g.L[3]; ++x[3])
        for (x[2] = 0; x[2] < g.L[2]; ++x[2])
            for (x[1] = 0; x[1] < g.L[1]; ++x[1])
                for (x[0] = 0; x[0] < g.L[0]; ++x[0])
                    for (int d = 0; d < 4; ++d)
                        for (int s : {1, -1}) {
                            int y[4] = {x[0], x[1], x[2], x[3]};
                            y[d] = (y[d] + s + g.L[d]) % g.L[d];
                            const bool edge = s > 0 ? x[d] == g.L[d] - 1 : x[d] == 0;
                            const int odd = x[0] & 1, by = d != 0 ? g.hs[d] : s > 0 ? odd : 1 - odd;
                            const int di = s > 0 ? (edge ? -g.wrap[d] : by) : (edge ? g.wrap[d] : -by);
                            CHECK((lex(x) >> 1) + di == lex(y) >> 1, "direction %d step %d", d, s);
                        }
}

int main()
{
    walks();
    scratch();
    for (const su3_params &p : {params(2, 2, 2, 2), params(4, 6, 2, 8), params(10, 2, 6, 4, 2), params(6, 8, 10, 2)}) steps(p);
    std::printf("%d failures\n", fails);
    return fails != 0;
}
