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

// waves per tile of 64 links: six, three or one
static void waves()
{
    CHECK(pass_six_waves(64, true, 256) && !pass_six_waves(64, true, 257), "FP64");
    CHECK(pass_six_waves(32, true, 768) && !pass_six_waves(32, true, 769), "FP32");
    CHECK(pass_six_waves(32, false, 512) && !pass_six_waves(32, false, 513), "FP32, several attempts or couplings");
    // asked for: three waves on the smallest lattice, six on a large one
    for (int prec : {64, 32}) {
        CHECK(!pass_six_waves(prec, true, 1, 1) && !pass_six_waves(prec, false, 1, 1), "lanes = 1");
        CHECK(pass_six_waves(prec, true, 8192, 2) && pass_six_waves(prec, true, 8192, 4), "lanes = 2, 4");
    }
    const struct {
        int prec, nhit;
        double beta;
        bool measured, twob;
        int tiles;
        bool one;
    } c[] = {
        {64, 1, 0.5, false, false, 1000000, false}, {64, 3, 0.5, false, false, 3, false},  {64, 64, 0.2, false, false, 1, true},
        {64, 17, 2.0, false, false, 32, true},      {64, 17, 5.7, false, false, 32, false}, {64, 3, 4.2, false, false, 284, false},
        {64, 7, 0.5, true, false, 284, true},       {32, 7, 0.5, true, false, 284, false},  {64, 2, 0.5, false, false, 1088, true},
        {64, 3, 2.0, true, false, 1088, true},      {64, 3, 5.5, false, true, 324, false},  {64, 2, 5.5, false, true, 1088, true},
        {32, 2, 0.5, false, false, 1088, false},    {32, 2, 0.5, false, false, 2176, true}, {32, 3, 5.7, false, false, 32767, false},
        {32, 3, 5.7, false, false, 32768, true},    {64, 3, 5.7, true, false, 8192, true},  {64, 3, 5.7, false, false, 8192, false},
        {64, 3, 5.7, false, false, 16384, true},    {64, 9, 0.4, false, false, 600, true},  {32, 9, 0.4, false, false, 600, true},
    };
    for (const auto &k : c)
        CHECK(pass_one_lane(k.prec, k.nhit, k.beta, k.measured, k.twob, k.tiles) == k.one, "FP%d, %d attempts, beta %g, %d tiles",
              k.prec, k.nhit, k.beta, k.tiles);
    // 64-bit offsets and several attempts: one wave per tile by size alone
    for (const su3_params &p : {params(96, 96, 98, 100, 1, 64, 2), params(128, 128, 112, 100, 1, 32, 2), params(96, 96, 98, 100, 2, 32, 2)}) {
        const Geom g = make_geom(&p);
        CHECK(pass_big(g, p.precision), "blocks over 4 GiB");
        CHECK(pass_one_lane(p.precision, p.nhit, 1e9, false, false, pass_blocks(g, kPassBlock)), "one wave per tile");
    }
    const su3_params below = params(96, 96, 96, 96);
    CHECK(!pass_big(make_geom(&below), 64), "96^4");
}

int main()
{
    walks();
    waves();
    scratch();
    for (const su3_params &p : {params(2, 2, 2, 2), params(4, 6, 2, 8), params(10, 2, 6, 4, 2), params(6, 8, 10, 2)}) steps(p);
    std::printf("%d failures\n", fails);
    return fails != 0;
}
