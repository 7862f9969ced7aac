// Host check of the slab walk's tile plans, compiled from the headers and
// sources the launches use: for many lattices, bytes re-read per site and
// groups per block, the grid of a launch in block order 2 gives every group
// exactly once and nothing outside the lattice (-1 elsewhere); a plan leaves
// at most a sixteenth of the launched groups empty.  Prints "ok" and the
// number of plans checked.
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#include "../paper_1105_2279_amd/csrc/qdpx_impl.hpp"

#include <cstdio>
#include <vector>

using namespace qdpx;

int main() {
    long fails = 0, plans = 0;
    const int xs[] = {2, 3, 4, 8, 12, 16, 20, 24, 32, 40}, ys[] = {2, 4, 5, 8, 12, 16}, zs[] = {2, 3, 4, 9, 16},
              ts[] = {2, 3, 4, 6, 10, 16};
    std::vector<std::vector<int32_t>> Ls;
    for (int x : xs)
        for (int y : ys)
            for (int z : zs)
                for (int t : ts) Ls.push_back({x, y, z, t});
    for (auto L : {std::vector<int32_t>{32, 32, 32, 64}, {24, 24, 24, 48}, {48, 48, 48, 96}, {20, 20, 20, 40},
                   {40, 24, 18, 30}, {28, 28, 28, 28}, {64, 2, 3, 5}})
        Ls.push_back(L);
    for (auto &L : Ls)
        for (int bytes : {96, 192, 384, 576})
            for (int fwd = 0; fwd < 2; ++fwd)
                for (int m = 1; m <= 8; m *= 2) {
                    Geo g = make_geo(L.data());
                    LaunchCfg c;
                    c.xcd = 2;
                    order_blocks(g, c, m, bytes, fwd);
                    const int ng = num_groups(g);
                    std::vector<char> seen(ng, 0);
                    long n = 0;
                    if (c.xcd != 2) {  // no plan: the grid of the plain orders
                        fails += c.xcd != 0 || (long)c.grid * m < ng || (long)(c.grid - 1) * m >= ng;
                        continue;
                    }
                    ++plans;
                    for (long i = 0; i < (long)c.grid * m; ++i) {
                        const int grp = slabwalk(g, (int)i, m);
                        if (grp == -1) continue;
                        if (grp < 0 || grp >= ng || seen[grp]) {
                            if (fails++ < 10)
                                std::printf("%dx%dx%dx%d bytes %d m %d: group %d at %ld\n", L[0], L[1], L[2], L[3],
                                            bytes, m, grp, i);
                            continue;
                        }
                        seen[grp] = 1;
                        ++n;
                    }
                    if (n != ng || (double)c.grid * m > (1.0 + 1.0 / 16) * ng + 1e-9) {
                        if (fails++ < 10)
                            std::printf("%dx%dx%dx%d bytes %d m %d: %ld of %d groups, grid %d\n", L[0], L[1], L[2], L[3],
                                        bytes, m, n, ng, c.grid);
                    }
                }
    if (!fails && plans) std::printf("ok %ld plans\n", plans);
    return fails != 0 || plans == 0;
}
