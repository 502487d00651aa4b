// CPU test of the traversal's query mapping (paper_1901_08088_amd/csrc/
// launch_geometry.h) for systems without particles, whose tree descriptions
// nothing writes: such a system gets no workgroup, and whatever an earlier
// call left in its descriptions no lane of it has a query.  Beside it the
// mapping itself: over all workgroups of a system every particle is some
// lane's query exactly once and no other position is, each wavefront's valid
// lanes come first and are of one type.
// Built with g++ by tests/test_empty_systems.py; exits non-zero on failure.
#include <stdint.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_1901_08088_amd/csrc/launch_geometry.h"

using namespace qbi;

struct Meta {
    int32_t start, count;
};

static int empty(std::mt19937_64 &rng, int32_t ntypes, int32_t block, int32_t qpw) {
    if (trav_blocks(0, ntypes, block, qpw) != 0) {
        fprintf(stderr, "an empty system of %d types gets workgroups\n", ntypes);
        return 1;
    }
    // a system of the same place in an earlier call, before or behind the present offset
    Meta m[4];
    int32_t at = (int32_t)(rng() % 100000);
    const int32_t start = (int32_t)(rng() % 100000);
    for (auto &t : m) {
        t.start = at;
        t.count = (int32_t)(rng() % 2000);
        at += t.count;
    }
    for (int32_t nwg = 8; nwg <= 32; nwg += 8)
        for (int32_t wg = 0; wg < nwg; ++wg)
            for (int32_t wave = 0; wave < block / 64; ++wave)
                for (int32_t lane = 0; lane < 64; ++lane) {
                    const int32_t li = query_position(m, 0, ntypes, qpw, start, block / 64, wg, nwg, wave, lane);
                    if (li < 0) {
                        fprintf(stderr, "empty system, %d types: a lane takes position %d\n", ntypes, li);
                        return 1;
                    }
                }
    return 0;
}

static int cover(std::mt19937_64 &rng, int32_t ntypes, int32_t block, int32_t qpw) {
    const int32_t start = (int32_t)(rng() % 1000);
    Meta m[4] = {};
    int32_t n = 0;
    for (int32_t t = 0; t < ntypes; ++t) {
        m[t].start = start + n;
        m[t].count = (int32_t)(rng() % (rng() % 3 ? 40 : 900));
        n += m[t].count;
    }
    std::vector<int> seen((size_t)n, 0);
    const int32_t nwg = (int32_t)trav_blocks(n, ntypes, block, qpw);
    for (int32_t wg = 0; wg < nwg; ++wg)
        for (int32_t wave = 0; wave < block / 64; ++wave) {
            int32_t first = -1;
            bool idle = false;
            for (int32_t lane = 0; lane < 64; ++lane) {
                const int32_t li = query_position(m, n, ntypes, qpw, start, block / 64, wg, nwg, wave, lane);
                if (li >= n) {
                    idle = true;
                    continue;
                }
                auto type = [&](int32_t p) {
                    int32_t t = 0;
                    while (p >= m[t].start - start + m[t].count) ++t;
                    return t;
                };
                if (li < 0 || idle || (first >= 0 && li != first + lane) || (first >= 0 && type(li) != type(first))) {
                    fprintf(stderr, "n=%d types=%d block=%d qpw=%d: lane %d takes %d\n", n, ntypes, block, qpw, lane,
                            li);
                    return 1;
                }
                if (first < 0) first = li;
                ++seen[(size_t)li];
            }
        }
    for (int32_t i = 0; i < n; ++i)
        if (seen[(size_t)i] != 1) {
            fprintf(stderr, "n=%d types=%d block=%d qpw=%d: position %d taken %d times\n", n, ntypes, block, qpw, i,
                    seen[(size_t)i]);
            return 1;
        }
    return 0;
}

int main() {
    std::mt19937_64 rng(1088);
    for (int32_t ntypes = 1; ntypes <= 4; ++ntypes)
        for (int32_t block = 64; block <= 256; block += 64)
            for (int32_t qpw = 1; qpw <= 64; qpw *= 2)
                for (int rep = 0; rep < 6; ++rep)
                    if (empty(rng, ntypes, block, qpw) || cover(rng, ntypes, block, qpw)) return 1;
    printf("all checks passed\n");
    return 0;
}
