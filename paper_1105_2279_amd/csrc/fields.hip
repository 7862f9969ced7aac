// Layout conversion (host canonical AoS <-> library SoA), the shift
// expression chi = sum_mu U_mu(x) psi(x+mu) + a phi(x) with its fused FP64
// norm, the chain update psi - c chi, and the deterministic finalisation of
// FP64 partial sums.
#include <type_traits>

#include "../../include/qdpx.h"
#include "qdpx_impl.hpp"
#include "reduce_device.hpp"

namespace qdpx {

Geo make_geo(const int32_t L[4]) {
    Geo g;
    for (int d = 0; d < 4; ++d) g.L[d] = L[d];
    g.st[0] = 1;
    g.st[1] = L[0];
    g.st[2] = L[0] * L[1];
    g.st[3] = L[0] * L[1] * L[2];
    g.V = g.st[3] * L[3];
    g.S = ((int64_t)g.V + 255) / 256 * 256;
    g.P = g.st[2] % 64 == 0 ? g.st[2] / 64 : 0;
    g.ncol = g.st[3] % 64 == 0 ? g.st[3] / 64 : 0;
    g.dL0 = FastDiv::make(L[0]);
    g.dL1 = FastDiv::make(L[1]);
    g.dL2 = FastDiv::make(L[2]);
    g.dP = FastDiv::make(g.P ? g.P : 1);
    g.dncol = FastDiv::make(g.ncol ? g.ncol : 1);
    // the slab walk's tiles: eight of ncol / 8 consecutive columns (tile_plan
    // chooses others)
    g.pz = g.ncol;
    g.nz = g.wz = 1;
    g.wseg = 0;
    g.wp = g.ncol >= 8 ? g.ncol >> 3 : 1;
    g.dwp = g.dwc = FastDiv::make(g.wp);
    g.dunit = FastDiv::make(g.wp * L[3]);
    g.dnyt = g.dtiles = FastDiv::make(8);
    return g;
}

// The block order where no tiles were planned: order 2 only where make_geo's own
// tiles, eight equal ranges of columns, hold every group (tile_plan finds a plan
// wherever they do, so order_blocks has the identity order from here), else the
// identity order.
int launch_order(const Geo &g, const LaunchCfg &cfg, int groups_per_block) {
    if (cfg.xcd != 2) return cfg.xcd;
    const int groups = (g.V + 63) / 64;
    if (g.ncol && g.ncol % 8 == 0 && groups % (8 * groups_per_block) == 0) return 2;
    return 0;
}

// The tiles of the slab walk for a kernel that reads `bytes` of each site
// again from its neighbours, to both sides or (fwd_only) one.  What a tile
// reads beyond itself is its halo in y and z, so a wide tile is better, as
// long as the t planes between the first and the last read of a site (about
// three, with the groups in flight) stay in the 4 MB L2: kTilePlane bytes a
// plane with its halo, beyond which the t neighbours are fetched again.  At
// 32^3x64 the FP64 smearing step's eight slabs of four z planes (2.4 MB a
// plane) read 2.97 times their links from beyond L2, 8 x 8 tiles of (y, z)
// (1.2 MB) a modelled 1.5.  A t range cut in two or more, where tiles alone
// do not fill eight XCDs, reads its end planes again.  False where the
// groups do not form (column, t) pairs or every plan leaves more than a
// sixteenth of the blocks without a group.
constexpr double kTilePlane = 1.25e6;
// Added to the cost where the XCDs do not all work on tiles to the end.
constexpr double kTilesUneven = 0.25;

// The search takes 1 to 11 us of the host, once or twice a call, so a thread
// keeps its last few plans by what they depend on (a smearing call with two
// steps and their plaquettes on 64^3x16 in FP32: 48 us on the host with a search
// for each launch, 37 before there were plans).
struct TilePlan {
    int L[4], bytes, fwd_only, groups_per_block;
    int by, bz, bseg;  // by 0: no plan
};
static TilePlan search_tiles(const Geo &g, int bytes, bool fwd_only, int groups_per_block) {
    const int Lt = g.L[3];
    const int nz = g.P ? g.L[2] : 1, pz = g.ncol / nz;  // Lz layers, or one of whole z planes
    const double sides = fwd_only ? 1.0 : 2.0;
    const double yhalo = g.P ? g.L[0] : g.st[2];  // sites a layer and side
    // Tile sides tried: the whole extent and the numbers below it of at most
    // two set bits.
    auto next = [](int n, int all) {
        do ++n;
        while (n < all && (n & (n - 1) & ((n & (n - 1)) - 1)));
        return n;
    };
    double best = 1e300;
    int by = 0, bz = 0, bseg = 0;
    for (int ty = 1; ty <= pz; ty = next(ty, pz))
        for (int tz = 1; tz <= nz; tz = next(tz, nz)) {
            const int nyt = (pz + ty - 1) / ty, nzt = (nz + tz - 1) / tz;
            const double area = 64.0 * ty * tz;
            const double all = area + (nyt > 1 ? sides * yhalo * tz : 0.0) + (nzt > 1 ? sides * 64.0 * ty : 0.0);
            const double over = all * bytes / kTilePlane - 1.0;
            const double planes = all / area * (over > 0.0 ? 1.0 + 0.9 * (over < 1.0 ? over : 1.0) : 1.0);
            if (planes >= best) continue;
            for (int seg = 0; seg <= 4 && Lt % (1 << seg) == 0 && (Lt >> seg) >= (seg ? 4 : 1); ++seg) {
                const int64_t unit = (int64_t)ty * tz * (Lt >> seg), upx = (((int64_t)nyt * nzt << seg) + 7) / 8;
                const int64_t blocks = 8 * ((upx * unit + groups_per_block - 1) / groups_per_block);
                const double waste = (double)(blocks * groups_per_block) / ((double)g.ncol * Lt) - 1.0;
                const double cost = planes * (seg ? 1.0 + 2.0 * sides / (Lt >> seg) : 1.0) + waste +
                                    ((nyt * nzt << seg) % 8 ? kTilesUneven : 0.0);
                if (waste > 1.0 / 16 || cost >= best) continue;
                best = cost;
                by = ty;
                bz = tz;
                bseg = seg;
            }
        }
    return TilePlan{{g.L[0], g.L[1], g.L[2], g.L[3]}, bytes, fwd_only, groups_per_block, by, bz, bseg};
}

bool tile_plan(Geo &g, int bytes, bool fwd_only, int groups_per_block) {
    if (!g.ncol) return false;
    constexpr int kKept = 8;
    static thread_local TilePlan kept[kKept] = {};  // L 0: none
    static thread_local int oldest = 0;
    const TilePlan *p = nullptr;
    for (const TilePlan &k : kept)
        if (k.L[0] == g.L[0] && k.L[1] == g.L[1] && k.L[2] == g.L[2] && k.L[3] == g.L[3] && k.bytes == bytes &&
            k.fwd_only == (int)fwd_only && k.groups_per_block == groups_per_block)
            p = &k;
    if (!p) {
        kept[oldest] = search_tiles(g, bytes, fwd_only, groups_per_block);
        p = &kept[oldest];
        oldest = (oldest + 1) % kKept;
    }
    if (!p->by) return false;
    const int nz = g.P ? g.L[2] : 1, pz = g.ncol / nz;
    const int nyt = (pz + p->by - 1) / p->by, nzt = (nz + p->bz - 1) / p->bz;
    g.pz = pz;
    g.nz = nz;
    g.wp = p->by;
    g.wz = p->bz;
    g.wseg = p->bseg;
    g.dwp = FastDiv::make(g.wp);
    g.dwc = FastDiv::make(g.wp * g.wz);
    g.dunit = FastDiv::make(g.wp * g.wz * (g.L[3] >> g.wseg));
    g.dnyt = FastDiv::make(nyt);
    g.dtiles = FastDiv::make(nyt * nzt);
    return true;
}

// Tiles where an XCD's share no longer fits its L2.  The Jacobi hop, to both
// sides in every direction: from 4 MB (FP64 12x24x16x28, 5.9 MB, ranges / tiles
// 27.7 / 24.2 us).  Smearing steps, shift and chain: from 6 MB on, as contiguous
// ranges lose little to 4 MB and balance better on so few groups (FP32-18 step
// 16^3x32, 4.5 MB, 32.7 / 35.4; FP64 6 MB 47.8 / 48.9; 20^3x40 11 MB 77.4 / 76.2;
// FP64 chain 16x20^2x36, 5.3 MB, 47.3 / 49.7).  The shift also keeps ranges where
// its field as a whole is within the 256 MB cache but not much smaller, so that
// the t neighbours come from there (FP32: 36^4, 19 MB, 1.07 times the time in
// tiles, 16^2x256x32 and 32^3x64, 24 MB, 1.04 to 1.08; below and above tiles win:
// 128^2x8^2, 12 MB, 118 / 92 us; FP64 28^3x56, 28 MB, 1.12 times the time in
// ranges).
bool tiles_by_default(int op, int64_t share) {
    if (op == QDPX_OP_JACOBI) return share > kXcdL2;
    if (op == QDPX_OP_SHIFT && share > 16 << 20 && share <= 26 << 20) return false;
    return share > kXcdL2 * 3 / 2;
}

// A slab walk keeps a t plane for the next; without the t direction, or for the
// shift in t alone, its tiles only have their halos to read twice.  Contiguous
// ranges then, unless the lattice is so large that eight ranges that far apart
// cost more.  Ranges over tiles, time: the shift (to one side) 0.88 to 1.0 up to
// 24 MB, 1.06 and more from 27 MB on; the hop in x, y and z 0.90 to 1.0 up to 28
// MB, 1.02 to 1.11 at 30 to 38; in one or two of them 0.80 to 0.97 up to 48 MB,
// 1.02 to 1.1 from 54 on; the smearing step 0.87 to 1.0 up to 38 MB, 1.01 to 1.08
// from 40 on, where the groups of an xy plane are not a whole number and a tile
// is a stretch of z planes 0.95 to 1.0 up to 58 MB.
bool ranges_for_mask(int op, bool planes, int64_t share, unsigned mask) {
    const int n = __builtin_popcount(mask & 7u);
    int mb = 0;
    if (op == QDPX_OP_SHIFT) mb = !(mask & 8u) || n == 0 ? 26 : 0;
    else if (mask & 8u) mb = 0;
    else if (op == QDPX_OP_JACOBI) mb = n == 3 ? 28 : 50;
    else mb = planes ? 40 : 60;
    return share <= (int64_t)mb << 20;
}

void order_blocks(Geo &g, LaunchCfg &cfg, int groups_per_block, int bytes, bool fwd_only) {
    const int groups = (g.V + 63) / 64;
    cfg.grid = (groups + groups_per_block - 1) / groups_per_block;
    if (cfg.xcd != 2) return;
    if (tile_plan(g, bytes, fwd_only, groups_per_block))
        cfg.grid = 8 * (((((int)g.dtiles.d << g.wseg) + 7) / 8 * (int)g.dunit.d + groups_per_block - 1) / groups_per_block);
    else
        cfg.xcd = launch_order(g, cfg, groups_per_block);
}

// ------------------------------------------------------------ pack / unpack
// AoS double[V][4][3][3][2] <-> the SoA link layout (LinkLayout), and the same
// for Dirac fields.  Both directions are bound by HBM: a site's components
// are adjacent on the AoS side and a whole array apart on the SoA side, so a
// block takes a run of consecutive sites, whose AoS image is one contiguous
// stretch of memory, through LDS and touches global memory only in whole
// 1 KB wave accesses on both sides.  At 32^3x64 FP32-12 the four conversions
// (links and a Dirac field, there and back) take 778 us, 5.7 TB/s of the 6.2
// a streaming kernel reaches; with a thread per component and site, whose
// AoS accesses were 16 bytes every 576 or 192, they took 3135 us.
constexpr int kLinkTileSites = 64;   // one site per lane, one direction per wave
constexpr int kFermTileSites = 128;  // twelve (component pair, half) items for four waves
// Entries of a site in the LDS tile: one more than it has, so that 16-byte
// accesses of eight neighbouring sites (one LDS cycle) fall on different banks.
constexpr int kLinkTilePitch = 36 + 1, kFermTilePitch = 12 + 1;

// ENTRIES entries of each of the block's SITES sites (n of them inside the
// lattice), contiguous in `mem`, to or from the tile.
template <int ENTRIES, int SITES, int PITCH>
__device__ __forceinline__ void aos_to_tile(const double2 *__restrict__ mem, int n, double2 *tile) {
    constexpr int kPer = ENTRIES * SITES / 256;
    static_assert(kPer * 256 == ENTRIES * SITES, "whole trips");
    nv2_t<double> v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {  // every load in flight before the first LDS write
        const int e = i * 256 + (int)threadIdx.x;
        if (n == SITES || e < n * ENTRIES) v[i] = gptr<nv2_t<double>>(mem)[e];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = i * 256 + (int)threadIdx.x, site = e / ENTRIES;
        if (n == SITES || e < n * ENTRIES) tile[site * PITCH + (e - site * ENTRIES)] = double2{v[i].x, v[i].y};
    }
}
template <int ENTRIES, int SITES, int PITCH>
__device__ __forceinline__ void tile_to_aos(const double2 *tile, int n, double2 *__restrict__ mem) {
    constexpr int kPer = ENTRIES * SITES / 256;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = i * 256 + (int)threadIdx.x, site = e / ENTRIES;
        if (n == SITES || e < n * ENTRIES) {
            const double2 t = tile[site * PITCH + (e - site * ENTRIES)];
            store_stream<double>(mem + e, t.x, t.y);
        }
    }
}

// One block per 64 sites, wave mu storing the links of direction mu.
template <typename R, int NR>
__global__ void __launch_bounds__(256) k_pack_links(Geo g, const double2 *__restrict__ aos,
                                                    vec2_t<R> *__restrict__ soa) {
    __shared__ double2 tile[kLinkTileSites * kLinkTilePitch];
    const int s0 = blockIdx.x * kLinkTileSites;
    aos_to_tile<36, kLinkTileSites, kLinkTilePitch>(aos + (int64_t)s0 * 36, min(kLinkTileSites, g.V - s0), tile);
    __syncthreads();
    const int lane = threadIdx.x & 63, mu = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (s0 + lane >= g.V) return;
    Cx<R> e[3][3];
#pragma unroll
    for (int c = 0; c < 3 * NR; ++c) {
        const double2 v = tile[lane * kLinkTilePitch + mu * 9 + c];
        e[c / 3][c % 3] = Cx<R>{(R)v.x, (R)v.y};  // FP64 -> FP32 conversion rounds to nearest even
    }
    const LinksWO<R, NR> out{soa, g.S};
    out.store(mu, s0 + lane, e);
}

// SoA -> AoS, row 2 rebuilt in FP64 for NR == 2.
template <typename R, int NR>
__global__ void __launch_bounds__(256) k_unpack_links(Geo g, const vec2_t<R> *__restrict__ soa,
                                                      double2 *__restrict__ aos) {
    __shared__ double2 tile[kLinkTileSites * kLinkTilePitch];
    const int s0 = blockIdx.x * kLinkTileSites;
    const int lane = threadIdx.x & 63, mu = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (s0 + lane < g.V) {
        const LinksRO<R, NR> U{soa, g.S};
        Cx<R> e[3][3];
        U.template load_rows<false, NR>(mu, s0 + lane, e);
        M3<double> m;
#pragma unroll
        for (int c = 0; c < 3 * NR; ++c)
            m.e[c / 3][c % 3] = Cx<double>{(double)e[c / 3][c % 3].re, (double)e[c / 3][c % 3].im};
        if constexpr (NR == 2) rebuild_row2(m);
#pragma unroll
        for (int c = 0; c < 9; ++c)
            tile[lane * kLinkTilePitch + mu * 9 + c] = double2{m.e[c / 3][c % 3].re, m.e[c / 3][c % 3].im};
    }
    __syncthreads();
    tile_to_aos<36, kLinkTileSites, kLinkTilePitch>(tile, min(kLinkTileSites, g.V - s0), aos + (int64_t)s0 * 36);
}

// Dirac fields: one block per 128 sites; item i of the SoA side is array
// i / 2 (FP64: one component; FP32: a pair) of the sites' half i % 2.
template <typename R>
__global__ void __launch_bounds__(256) k_pack_fermion(Geo g, const double2 *__restrict__ aos,
                                                      vec2_t<R> *__restrict__ soa) {
    __shared__ double2 tile[kFermTileSites * kFermTilePitch];
    const int s0 = blockIdx.x * kFermTileSites;
    aos_to_tile<12, kFermTileSites, kFermTilePitch>(aos + (int64_t)s0 * 12, min(kFermTileSites, g.V - s0), tile);
    __syncthreads();
    constexpr int kPair = FermLayout<R>::kPaired ? 2 : 1;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int j = 0; j < 6 / kPair; ++j) {
        const int i = j * 4 + w, k = i >> 1, site = (i & 1) * 64 + lane;
        if (s0 + site >= g.V) continue;
        const double2 *t = tile + site * kFermTilePitch + k * kPair;
        if constexpr (kPair == 2) {
            nv4_t<R> v;
            v.x = (R)t[0].x;
            v.y = (R)t[0].y;
            v.z = (R)t[1].x;
            v.w = (R)t[1].y;
            __builtin_nontemporal_store(v, gptr_w<nv4_t<R>>((nv4_t<R> *)soa + (int64_t)k * g.S + s0 + site));
        } else {
            store_stream<R>(soa + (int64_t)k * g.S + s0 + site, t[0].x, t[0].y);
        }
    }
}

template <typename R>
__global__ void __launch_bounds__(256) k_unpack_fermion(Geo g, const vec2_t<R> *__restrict__ soa,
                                                        double2 *__restrict__ aos) {
    __shared__ double2 tile[kFermTileSites * kFermTilePitch];
    const int s0 = blockIdx.x * kFermTileSites;
    constexpr int kPair = FermLayout<R>::kPaired ? 2 : 1;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int j = 0; j < 6 / kPair; ++j) {
        const int i = j * 4 + w, k = i >> 1, site = (i & 1) * 64 + lane;
        if (s0 + site >= g.V) continue;
        double2 *t = tile + site * kFermTilePitch + k * kPair;
        if constexpr (kPair == 2) {
            const nv4_t<R> v = gptr<nv4_t<R>>(soa)[(int64_t)k * g.S + s0 + site];
            t[0] = double2{(double)v.x, (double)v.y};
            t[1] = double2{(double)v.z, (double)v.w};
        } else {
            const nv2_t<R> v = gptr<nv2_t<R>>(soa)[(int64_t)k * g.S + s0 + site];
            t[0] = double2{(double)v.x, (double)v.y};
        }
    }
    __syncthreads();
    tile_to_aos<12, kFermTileSites, kFermTilePitch>(tile, min(kFermTileSites, g.V - s0), aos + (int64_t)s0 * 12);
}

static dim3 tile_grid(const Geo &g, int sites) { return dim3((g.V + sites - 1) / sites); }

hipError_t launch_pack_links(const Geo &g, int prec, int nrows, const double *aos, void *soa, hipStream_t st) {
    const dim3 grid = tile_grid(g, kLinkTileSites);
    const double2 *in = reinterpret_cast<const double2 *>(aos);
    if (prec == 0) {
        k_pack_links<double, 3><<<grid, 256, 0, st>>>(g, in, (double2 *)soa);
    } else if (nrows == 3) {
        k_pack_links<float, 3><<<grid, 256, 0, st>>>(g, in, (float2 *)soa);
    } else {
        k_pack_links<float, 2><<<grid, 256, 0, st>>>(g, in, (float2 *)soa);
    }
    return hipGetLastError();
}

hipError_t launch_unpack_links(const Geo &g, int prec, int nrows, const void *soa, double *aos, hipStream_t st) {
    const dim3 grid = tile_grid(g, kLinkTileSites);
    double2 *out = reinterpret_cast<double2 *>(aos);
    if (prec == 0) {
        k_unpack_links<double, 3><<<grid, 256, 0, st>>>(g, (const double2 *)soa, out);
    } else if (nrows == 3) {
        k_unpack_links<float, 3><<<grid, 256, 0, st>>>(g, (const float2 *)soa, out);
    } else {
        k_unpack_links<float, 2><<<grid, 256, 0, st>>>(g, (const float2 *)soa, out);
    }
    return hipGetLastError();
}

hipError_t launch_pack_fermion(const Geo &g, int prec, const double *aos, void *soa, hipStream_t st) {
    const dim3 grid = tile_grid(g, kFermTileSites);
    const double2 *in = reinterpret_cast<const double2 *>(aos);
    if (prec == 0) k_pack_fermion<double><<<grid, 256, 0, st>>>(g, in, (double2 *)soa);
    else k_pack_fermion<float><<<grid, 256, 0, st>>>(g, in, (float2 *)soa);
    return hipGetLastError();
}

hipError_t launch_unpack_fermion(const Geo &g, int prec, const void *soa, double *aos, hipStream_t st) {
    const dim3 grid = tile_grid(g, kFermTileSites);
    double2 *out = reinterpret_cast<double2 *>(aos);
    if (prec == 0) k_unpack_fermion<double><<<grid, 256, 0, st>>>(g, (const double2 *)soa, out);
    else k_unpack_fermion<float><<<grid, 256, 0, st>>>(g, (const float2 *)soa, out);
    return hipGetLastError();
}

// What a kernel with and without the slab walk takes of the geometry (a
// launch copies its arguments: a tenth of its cost on the host for the walk's
// 84 bytes).
template <bool SLAB> using launch_geo = std::conditional_t<SLAB, Geo, GeoBase>;

// ------------------------------------------------------- shift expression
// chi(x) = sum_{mu in mask} h_mu(x) + a phi(x), with the forward hop
// h_mu = U_mu(x) psi(x+mu) or (bwd) the backward hop
// h_mu = U_mu(x-mu)^dag psi(x-mu); MODE 1 (one chain step) stores
// psi(x) - c chi(x) instead of chi.  A block of 256 threads holds one
// 64-site group per iteration and wave w computes direction mu = w for all 12
// spinor components, so the four directions' loads are in flight together.
// Either hop reads each link once per launch, so links are streamed.
// The four partial products meet in LDS; after a barrier wave w adds them in
// direction order for the components it owns (FermLayout), adds a phi, forms
// the FP64 |chi|^2 of those components and stores them.  The four waves'
// norms are added in wave
// order and reduced by a wave butterfly into one partial per group, so
// every sum has a fixed order and nothing depends on the launch geometry.
template <typename R, int NR, int MODE, int NS, bool SLAB>
__global__ void __launch_bounds__(256) k_shift(launch_geo<SLAB> g, LinksRO<R, NR> U, FermRO<R> psi, FermRO<R> phi, R a, R c,
                                                unsigned mask, int bwd, FermWO<R> out, double *__restrict__ partials,
                                                int xcd, int tw) {
    __shared__ vec2_t<R> part[4][12][64];  // [direction][component][lane]
    __shared__ double nrm[4][64];          // [wave][lane]
    const int tile = xcd == 1 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ngroups = num_groups(g);
#pragma unroll 1
    for (int j = 0; j < NS; ++j) {
        const int i = tile * NS + j;  // the same for the four waves
        if (!SLAB && i >= ngroups) return;
        int grp;
        if constexpr (SLAB) {
            grp = slabwalk(g, i, NS);
            if (grp < 0) continue;
        } else {
            grp = traverse(g, i, tw);
        }
        Site x;
        const bool live = group_site(g, grp, lane, x);
        const int s = x.s;
        const int cmu = coord(x, mu);
        // phi and (MODE 1) psi of the components this wave stores are
        // fetched now so that their latency overlaps the products and the
        // exchange
        constexpr int NO = FermLayout<R>::kOwn;
        Cx<R> f0[NO], p0[NO];
#pragma unroll
        for (int t = 0; t < NO; ++t) f0[t] = p0[t] = Cx<R>{(R)0, (R)0};
        if (live && phi.p) phi.ld_owned(mu, s, f0);
        if constexpr (MODE == 1) {
            if (live) psi.ld_owned(mu, s, p0);
        }
        Cx<R> acc[4][3];
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) acc[sp][cc] = Cx<R>{(R)0, (R)0};
        if (live && ((mask >> mu) & 1u)) {  // wave-uniform
            const int f = bwd ? hop_bwd(g, s, cmu, mu) : hop_fwd(g, s, cmu, mu);
            M3<R> u;
            U.template su3<true>(mu, bwd ? f : s, u);  // each link is read once
            if (bwd) {  // U^dag: transpose and conjugate in registers
#pragma unroll
                for (int ca = 0; ca < 3; ++ca) {
                    u.e[ca][ca].im = -u.e[ca][ca].im;
#pragma unroll
                    for (int cb = ca + 1; cb < 3; ++cb) {
                        const Cx<R> t = u.e[ca][cb];
                        u.e[ca][cb] = Cx<R>{u.e[cb][ca].re, -u.e[cb][ca].im};
                        u.e[cb][ca] = Cx<R>{t.re, -t.im};
                    }
                }
            }
            Cx<R> pf[4][3];
            psi.ld_all(f, pf);
            __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the arithmetic
#pragma unroll
            for (int sp = 0; sp < 4; ++sp)
#pragma unroll
                for (int ca = 0; ca < 3; ++ca)
#pragma unroll
                    for (int cb = 0; cb < 3; ++cb) cmac(acc[sp][ca], u.e[ca][cb], pf[sp][cb]);
        }
        if (j > 0) __syncthreads();  // the previous group's partials have been read
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                vec2_t<R> v;
                v.x = acc[sp][cc].re;
                v.y = acc[sp][cc].im;
                part[mu][3 * sp + cc][lane] = v;
            }
        __syncthreads();
        double n2 = 0.0;
        if (live) {
            Cx<R> o[NO];
#pragma unroll
            for (int t = 0; t < NO; ++t) {
                Cx<R> v{(R)0, (R)0};
                const int q = FermLayout<R>::owned(mu, t);
                if (q >= 0) {  // wave-uniform
#pragma unroll
                    for (int w = 0; w < 4; ++w) {  // directions in order
                        const vec2_t<R> e = part[w][q][lane];
                        v.re += e.x;
                        v.im += e.y;
                    }
                    if (phi.p) {
                        v.re = fma(a, f0[t].re, v.re);
                        v.im = fma(a, f0[t].im, v.im);
                    }
                    n2 = fma((double)v.re, (double)v.re, fma((double)v.im, (double)v.im, n2));
                    if constexpr (MODE == 1) {
                        v.re = fma(-c, v.re, p0[t].re);
                        v.im = fma(-c, v.im, p0[t].im);
                    }
                }
                o[t] = v;
            }
            out.st_owned(mu, s, o);
        }
        if (partials) {
            nrm[mu][lane] = n2;
            __syncthreads();
            if (mu == 0) {
                const double t = ((nrm[0][lane] + nrm[1][lane]) + nrm[2][lane]) + nrm[3][lane];
                const double w = wave_sum(t);
                if (lane == 0) partials[grp] = w;
            }
        }
    }
}

int shift_num_partials(const Geo &g) { return (g.V + 63) / 64; }

template <typename R, int NR, int MODE>
static void shift_dispatch_ns(const Geo &g, const void *U, const void *psi, const void *phi, double a, double c,
                              unsigned mask, int bwd, void *out, double *partials, const LaunchCfg &cfg,
                              hipStream_t st) {
    using V = vec2_t<R>;
    LinksRO<R, NR> u{(const V *)U, g.S};
    FermRO<R> p{(const V *)psi, g.S}, f{(const V *)phi, g.S};
    FermWO<R> o{(V *)out, g.S};
    const int grid = cfg.grid, xcd = cfg.xcd;
#define QDPX_SHIFT_LAUNCH(NS)                                                                                       \
    if (xcd == 2)                                                                                                   \
        k_shift<R, NR, MODE, NS, true><<<grid, 256, 0, st>>>(g, u, p, f, (R)a, (R)c, mask, bwd, o, partials, 2, 1); \
    else                                                                                                            \
        k_shift<R, NR, MODE, NS, false><<<grid, 256, 0, st>>>(g, u, p, f, (R)a, (R)c, mask, bwd, o, partials, xcd, cfg.tw)
    switch (cfg.nsite) {
    case 2: QDPX_SHIFT_LAUNCH(2); break;
    case 4: QDPX_SHIFT_LAUNCH(4); break;
    case 8: QDPX_SHIFT_LAUNCH(8); break;
    default: QDPX_SHIFT_LAUNCH(1); break;
    }
#undef QDPX_SHIFT_LAUNCH
}

template <int MODE>
static void shift_dispatch(const Geo &g, int prec, int nrows, const void *U, const void *psi, const void *phi,
                           double a, double c, unsigned mask, int bwd, void *out, double *partials,
                           const LaunchCfg &cfg, hipStream_t st) {
    if (prec == 0) shift_dispatch_ns<double, 3, MODE>(g, U, psi, phi, a, c, mask, bwd, out, partials, cfg, st);
    else if (nrows == 3) shift_dispatch_ns<float, 3, MODE>(g, U, psi, phi, a, c, mask, bwd, out, partials, cfg, st);
    else shift_dispatch_ns<float, 2, MODE>(g, U, psi, phi, a, c, mask, bwd, out, partials, cfg, st);
}

hipError_t launch_shift(const Geo &g, int prec, int nrows, const void *U, const void *psi, const void *phi,
                        double a, int mode, double c, void *out, double *partials, const LaunchCfg &cfg,
                        hipStream_t st, unsigned mask, int bwd) {
    if (mode == 0) shift_dispatch<0>(g, prec, nrows, U, psi, phi, a, c, mask, bwd, out, partials, cfg, st);
    else shift_dispatch<1>(g, prec, nrows, U, psi, phi, a, c, mask, bwd, out, partials, cfg, st);
    return hipGetLastError();
}

// ------------------------------------------------------------ Jacobi hop
// out(x) = [s0(x) + kappa * (H psi)(x)] / norm, with
// (H psi)(x) = sum_{mu in mask} [U_mu(x) psi(x+mu) + U_mu(x-mu)^dag psi(x-mu)],
// the hopping term of the smearing operator K.  s0 may be absent (then
// out = kappa H psi / norm); DIV selects the division by norm.  keep, where
// given, receives a copy of s0.
//
// A block of 256 threads holds one 64-site group per iteration and wave w
// computes direction mu = w: its forward and backward hop for all 12 spinor
// components, so the four directions' loads are in flight at once rather
// than one direction after another.  The four partial sums meet in LDS:
// every wave writes its twelve components and, after a barrier, wave w adds
// the four partials of the components it owns (FermLayout) in direction
// order, applies s0, kappa and norm, and stores them.  The order of every
// sum is fixed,
// so each site's result does not depend on the launch geometry.
// SLAB: the slab walk, compiled apart: its decoding in the same kernel took
// 1.5 % off the other orders on small lattices (20^3x40 in x, y, z: 52 us).
template <typename R, int NR, int NS, bool DIV, bool SLAB>
__global__ void __launch_bounds__(256) k_hop(launch_geo<SLAB> g, LinksRO<R, NR> U, FermRO<R> psi, FermRO<R> s0, R kappa, R norm,
                                              unsigned mask, FermWO<R> out, FermWO<R> keep, int xcd, int tw) {
    __shared__ vec2_t<R> part[4][12][64];  // [direction][component][lane]
    const int tile = xcd == 1 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ngroups = num_groups(g);
#pragma unroll 1
    for (int j = 0; j < NS; ++j) {
        const int i = tile * NS + j;  // the same for the four waves
        if (!SLAB && i >= ngroups) return;
        int grp;
        if constexpr (SLAB) {
            grp = slabwalk(g, i, NS);
            if (grp < 0) continue;
        } else {
            grp = traverse(g, i, tw);
        }
        Site x;
        const bool live = group_site(g, grp, lane, x);
        const int s = x.s;
        Cx<R> acc[4][3];
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) acc[sp][cc] = Cx<R>{(R)0, (R)0};
        const int cmu = coord(x, mu);
        // s0 of the components this wave stores is fetched now so that its
        // latency overlaps the hops and the exchange
        constexpr int NO = FermLayout<R>::kOwn;
        Cx<R> z[NO];
#pragma unroll
        for (int t = 0; t < NO; ++t) z[t] = Cx<R>{(R)0, (R)0};
        if (live && s0.p) s0.ld_owned(mu, s, z);
        if (live && ((mask >> mu) & 1u)) {
            // every load of this direction first, then the arithmetic: one
            // memory round trip per group
            const int f = hop_fwd(g, s, cmu, mu), bk = hop_bwd(g, s, cmu, mu);
            M3<R> uf, ub;
            U.template su3<false>(mu, s, uf);   // U_mu(x), also the backward link of x+mu
            U.template su3<false>(mu, bk, ub);  // U_mu(x-mu)
            Cx<R> pf[4][3], pb[4][3];
            psi.ld_all(f, pf);
            psi.ld_all(bk, pb);
            __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the arithmetic
#pragma unroll
            for (int sp = 0; sp < 4; ++sp) {
#pragma unroll
                for (int ca = 0; ca < 3; ++ca)
#pragma unroll
                    for (int cb = 0; cb < 3; ++cb) cmac(acc[sp][ca], uf.e[ca][cb], pf[sp][cb]);
                // (U^dag p)_a = sum_b conj(U_ba) p_b
#pragma unroll
                for (int ca = 0; ca < 3; ++ca)
#pragma unroll
                    for (int cb = 0; cb < 3; ++cb) cmac_ca(acc[sp][ca], ub.e[cb][ca], pb[sp][cb]);
            }
        }
        if (j > 0) __syncthreads();  // the previous group's partials have been read
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                vec2_t<R> v;
                v.x = acc[sp][cc].re;
                v.y = acc[sp][cc].im;
                part[mu][3 * sp + cc][lane] = v;
            }
        __syncthreads();
        if (live) {
            Cx<R> o[NO];
#pragma unroll
            for (int t = 0; t < NO; ++t) {
                Cx<R> v{(R)0, (R)0};
                const int q = FermLayout<R>::owned(mu, t);
                if (q >= 0) {  // wave-uniform
#pragma unroll
                    for (int w = 0; w < 4; ++w) {  // directions in order
                        const vec2_t<R> e = part[w][q][lane];
                        v.re += e.x;
                        v.im += e.y;
                    }
                    if (s0.p) {
                        v.re = fma(kappa, v.re, z[t].re);
                        v.im = fma(kappa, v.im, z[t].im);
                    } else {
                        v.re *= kappa;
                        v.im *= kappa;
                    }
                    if constexpr (DIV) {
                        v.re = v.re / norm;
                        v.im = v.im / norm;
                    }
                }
                o[t] = v;
            }
            out.st_owned(mu, s, o);
            if (keep.p) keep.st_owned(mu, s, z);
        }
    }
}

template <typename R, int NR, bool DIV>
static void hop_dispatch_ns(const Geo &g, const void *U, const void *psi, const void *s0, double kappa, double norm,
                            unsigned mask, void *out, const LaunchCfg &cfg, hipStream_t st, void *keep) {
    using V = vec2_t<R>;
    LinksRO<R, NR> u{(const V *)U, g.S};
    FermRO<R> p{(const V *)psi, g.S}, z{(const V *)s0, g.S};
    FermWO<R> o{(V *)out, g.S}, c{(V *)keep, g.S};
    const int grid = cfg.grid, xcd = cfg.xcd;
#define QDPX_HOP_LAUNCH(NS)                                                                                  \
    if (xcd == 2)                                                                                            \
        k_hop<R, NR, NS, DIV, true><<<grid, 256, 0, st>>>(g, u, p, z, (R)kappa, (R)norm, mask, o, c, 2, 1);  \
    else                                                                                                     \
        k_hop<R, NR, NS, DIV, false><<<grid, 256, 0, st>>>(g, u, p, z, (R)kappa, (R)norm, mask, o, c, xcd, cfg.tw)
    switch (cfg.nsite) {
    case 2: QDPX_HOP_LAUNCH(2); break;
    case 4: QDPX_HOP_LAUNCH(4); break;
    case 8: QDPX_HOP_LAUNCH(8); break;
    default: QDPX_HOP_LAUNCH(1); break;
    }
#undef QDPX_HOP_LAUNCH
}

template <bool DIV>
static void hop_dispatch(const Geo &g, int prec, int nrows, const void *U, const void *psi, const void *s0,
                         double kappa, double norm, unsigned mask, void *out, const LaunchCfg &cfg, hipStream_t st,
                         void *keep) {
    if (prec == 0) hop_dispatch_ns<double, 3, DIV>(g, U, psi, s0, kappa, norm, mask, out, cfg, st, keep);
    else if (nrows == 3) hop_dispatch_ns<float, 3, DIV>(g, U, psi, s0, kappa, norm, mask, out, cfg, st, keep);
    else hop_dispatch_ns<float, 2, DIV>(g, U, psi, s0, kappa, norm, mask, out, cfg, st, keep);
}

hipError_t launch_hop(const Geo &g, int prec, int nrows, const void *U, const void *psi, const void *s0, double kappa,
                      double norm, bool divide, unsigned mask, void *out, const LaunchCfg &cfg, hipStream_t st,
                      void *keep) {
    if (divide) hop_dispatch<true>(g, prec, nrows, U, psi, s0, kappa, norm, mask, out, cfg, st, keep);
    else hop_dispatch<false>(g, prec, nrows, U, psi, s0, kappa, norm, mask, out, cfg, st, keep);
    return hipGetLastError();
}

template <typename V>
__global__ void __launch_bounds__(256) k_copy_fermion(Geo g, const V *__restrict__ src, V *__restrict__ dst) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V) return;
    const int64_t o = (int64_t)blockIdx.y * g.S + s;
    dst[o] = src[o];
}

static dim3 site_grid(const Geo &g, int comps) { return dim3((g.V + 255) / 256, comps, 1); }

// One 16-byte entry per (array, site): 12 arrays of double2 (FP64) or the
// six paired arrays of FP32 fields.
hipError_t launch_copy_fermion(const Geo &g, int prec, const void *src, void *dst, hipStream_t st) {
    if (prec == 0)
        k_copy_fermion<double2><<<site_grid(g, 12), 256, 0, st>>>(g, (const double2 *)src, (double2 *)dst);
    else
        k_copy_fermion<float4><<<site_grid(g, 6), 256, 0, st>>>(g, (const float4 *)src, (float4 *)dst);
    return hipGetLastError();
}

// ------------------------------------------------------------ finalisation
// Stage A: block b sums partials [b*4096, (b+1)*4096) of each component;
// stage B: one block sums the stage-A values and applies the mode.  The
// arithmetic lives in reduce_device.hpp so the batched kernel can repeat it
// bit for bit inside one block.
__global__ void __launch_bounds__(kReduceBlock) k_finalize_a(const double *__restrict__ in, int n, int ncomp,
                                                            double *__restrict__ out) {
    __shared__ double lds[kReduceBlock / 64];
    const int nb = gridDim.x;
    for (int comp = 0; comp < ncomp; ++comp) {
        const double v = fin_stage_a(in + (int64_t)comp * n, n, blockIdx.x, lds);
        if (threadIdx.x == 0) out[comp * nb + blockIdx.x] = v;
    }
}

__global__ void __launch_bounds__(kReduceBlock) k_finalize_b(const double *__restrict__ in, int n, int mode,
                                                            double volume, double *__restrict__ out) {
    __shared__ double lds[kReduceBlock / 64];
    const int ncomp = (mode == 1) ? 2 : 1;
    double r[2] = {0.0, 0.0};
    for (int comp = 0; comp < ncomp; ++comp) r[comp] = fin_stage_b(in + comp * n, n, lds);
    if (threadIdx.x == 0) fin_write(r, mode, volume, out);
}

// Both stages as one launch, every chunk taken by 256 threads of one block at
// once.  Used for at most two chunks (a plaquette of up to 1365 groups, a
// norm of up to 8192): a launch less took the plaquette of 8^3x16 from 13.6
// to 10.2 us and the shift's norm there from 5.7 to 2.9 us.  With more, one
// CU fetching them all loses to the second launch: eight chunks of a norm
// took 19 us against 7.4 us, sixteen of a plaquette 30 us against 7 us.
constexpr int kFinOneChunks = 2;
__global__ void __launch_bounds__(kReduceBlock *kFinOneChunks) k_finalize_one(const double *__restrict__ in, int n, int mode,
                                                               double volume, double *__restrict__ out) {
    __shared__ double part[4 * kFinOneChunks];
    double r[2] = {0.0, 0.0};
    fin_both(in, n, mode == 1 ? 2 : 1, part, r);
    if (threadIdx.x == 0) fin_write(r, mode, volume, out);
}

int finalize_stage_a_blocks(int n) { return (n + kFinPerBlock - 1) / kFinPerBlock; }

hipError_t launch_finalize(const double *partials, int n, int mode, double volume, double *out, hipStream_t st) {
    // The stage-A results are stored right after the partials (the workspace
    // reserves room for them: finalize_stage_a_blocks(n) per component).
    const int ncomp = (mode == 1) ? 2 : 1;
    const int nb = finalize_stage_a_blocks(n);
    if (ncomp * nb <= kFinOneChunks) {
        k_finalize_one<<<1, kReduceBlock * ncomp * nb, 0, st>>>(partials, n, mode, volume, out);
        return hipGetLastError();
    }
    double *stage = const_cast<double *>(partials) + (int64_t)ncomp * n;
    k_finalize_a<<<nb, kReduceBlock, 0, st>>>(partials, n, ncomp, stage);
    k_finalize_b<<<1, kReduceBlock, 0, st>>>(stage, nb, mode, volume, out);
    return hipGetLastError();
}

}  // namespace qdpx
