// Host check that a tile plan does not depend on the plans asked for before it:
// every plan asked for on a new thread, then all of them again in other orders
// on one thread that has asked for them before, and while other threads ask.
// Prints "ok".
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#include "../paper_1105_2279_amd/csrc/qdpx_impl.hpp"

#include <atomic>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

using namespace qdpx;

struct Key {
    int32_t L[4];
    int bytes, fwd, m;
};
struct Got {
    bool ok = false;
    Geo g;
};
static Got ask(const Key &k) {
    Got r;
    memset((void *)&r.g, 0, sizeof r.g);
    r.g = make_geo(k.L);
    r.ok = tile_plan(r.g, k.bytes, k.fwd, k.m);
    return r;
}
static bool same(const Got &a, const Got &b) {
    return a.ok == b.ok && a.g.pz == b.g.pz && a.g.nz == b.g.nz && a.g.wp == b.g.wp && a.g.wz == b.g.wz &&
           a.g.wseg == b.g.wseg && a.g.dunit.d == b.g.dunit.d && a.g.dwc.d == b.g.dwc.d && a.g.dwp.d == b.g.dwp.d &&
           a.g.dnyt.d == b.g.dnyt.d && a.g.dtiles.d == b.g.dtiles.d;
}

int main() {
    std::vector<Key> keys;
    const int32_t Ls[][4] = {{32, 32, 32, 64}, {24, 24, 24, 48}, {24, 24, 48, 24}, {20, 20, 20, 40}, {16, 12, 9, 12},
                             {6, 5, 4, 7},     {2, 2, 2, 2},     {20, 8, 10, 16}};
    for (auto &L : Ls)
        for (int bytes : {96, 384})
            for (int fwd = 0; fwd < 2; ++fwd)
                for (int m : {1, 4}) keys.push_back(Key{{L[0], L[1], L[2], L[3]}, bytes, fwd, m});
    std::vector<Got> fresh(keys.size());
    for (size_t i = 0; i < keys.size(); ++i) std::thread([&] { fresh[i] = ask(keys[i]); }).join();
    std::atomic<int> fails{0};
    auto again = [&](unsigned seed) {
        for (int n = 0; n < 4000; ++n) {
            seed = seed * 1664525u + 1013904223u;
            // runs of few keys, so that kept plans are found, and jumps among all
            const size_t i = (n / 500 % 2 ? seed >> 8 : (n / 50) * 3 + (seed >> 8) % 5) % keys.size();
            if (!same(ask(keys[i]), fresh[i])) ++fails;
        }
    };
    again(1);
    std::vector<std::thread> ts;
    for (unsigned t = 0; t < 4; ++t) ts.emplace_back(again, 17 * t + 3);
    for (auto &t : ts) t.join();
    if (fails) return 1;
    std::printf("ok\n");
    return 0;
}
