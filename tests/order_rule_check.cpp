// Host check of the default block orders by operation, an XCD's share of what
// is read again, and direction mask, on both sides of every line, compiled from
// the sources the launches use.  Prints "ok".
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#include "../include/qdpx.h"
#include "../paper_1105_2279_amd/csrc/qdpx_impl.hpp"

#include <cstdio>

using namespace qdpx;

static int fails = 0;
#define EXPECT(cond) \
    do { \
        if (!(cond)) { \
            ++fails; \
            std::printf("line %d: %s\n", __LINE__, #cond); \
        } \
    } while (0)

int main() {
    constexpr int64_t MB = 1 << 20;
    // all directions
    EXPECT(!tiles_by_default(QDPX_OP_JACOBI, 4 * MB) && tiles_by_default(QDPX_OP_JACOBI, 4 * MB + 1));
    for (int op : {QDPX_OP_APE, QDPX_OP_SHIFT, QDPX_OP_CHAIN})
        EXPECT(!tiles_by_default(op, 6 * MB) && tiles_by_default(op, 6 * MB + 1) && tiles_by_default(op, 16 * MB));
    EXPECT(!tiles_by_default(QDPX_OP_SHIFT, 16 * MB + 1) && !tiles_by_default(QDPX_OP_SHIFT, 26 * MB));
    EXPECT(tiles_by_default(QDPX_OP_SHIFT, 26 * MB + 1));
    for (int op : {QDPX_OP_APE, QDPX_OP_CHAIN, QDPX_OP_JACOBI}) EXPECT(tiles_by_default(op, 20 * MB));
    // masks: the last share in ranges, or none
    for (unsigned mask = 0; mask < 16; ++mask)
        for (int planes = 0; planes < 2; ++planes) {
            const int n = __builtin_popcount(mask & 7u);
            const bool t = mask & 8u;
            const int64_t shift = !t || n == 0 ? 26 * MB : 0, hop = t ? 0 : n == 3 ? 28 * MB : 50 * MB,
                          ape = t ? 0 : planes ? 40 * MB : 60 * MB;
            EXPECT(ranges_for_mask(QDPX_OP_SHIFT, planes, shift, mask) && !ranges_for_mask(QDPX_OP_SHIFT, planes, shift + 1, mask));
            EXPECT(ranges_for_mask(QDPX_OP_JACOBI, planes, hop, mask) && !ranges_for_mask(QDPX_OP_JACOBI, planes, hop + 1, mask));
            EXPECT(ranges_for_mask(QDPX_OP_APE, planes, ape, mask) && !ranges_for_mask(QDPX_OP_APE, planes, ape + 1, mask));
        }
    // a geometry given by the caller is told from the others; the default is not one
    EXPECT(!LaunchCfg{}.given);
    if (fails) return 1;
    std::printf("ok\n");
    return 0;
}
