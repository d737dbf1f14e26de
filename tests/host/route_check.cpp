// Which kernel a call takes (paper_0904_1179_amd/csrc/layout.cpp), on the
// CPU: the rules at the sizes where they change, so that the GPU tests of a
// route do take it.
#include <cstdio>

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

int main()
{
    walks();
    std::printf("%d failures\n", fails);
    return fails != 0;
}
