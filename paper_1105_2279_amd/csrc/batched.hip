// Persistent batched APE smearing: many independent lattices of any extents,
// n_steps APE steps each in one persistent launch, then the final plaquettes.
//
// The persistent launch walks through phases, one per APE step.  Within a
// phase the work items are runs of 64-site groups of one lattice.  A
// lattice's groups form a (column, t-row) grid, a column being one group of a
// t plane (where those are a whole number; else all groups form one row); its
// columns are split into 8 contiguous ranges, one per XCD, and XCD x's queue
// (ticket counter) walks its range t-row by t-row, so a group's x, y and z
// neighbours are queued a few items away and its t neighbours one range
// further, all on the XCD whose L2 holds them (the slab walk of the
// single-lattice step, per lattice).  A block reads its XCD from the XCC_ID
// hardware register, drains its own queue first and then takes items from the
// other queues, so the load still balances; which queue a block uses only
// affects speed.
//
// When a block finds every queue of the phase empty it publishes how many
// items it finished and waits until the count of finished items reaches the
// phase's (one acquire).  Every item it waits for was already taken by a
// running block, so the wait always ends and no co-residency assumption is
// needed.  Fencing once per phase, not per item, matters on the multi-XCD
// MI355X: an agent-scope acquire invalidates the XCD's L2 and a release
// writes it back.  What a phase costs beyond its items is therefore one
// write-back per XCD for all of its blocks that are ready (publish), one
// acquire per block, polls without one, and counters on lines of their own:
// 35 us with 512 blocks, where a release and an acquire by every wave, an
// acquire with every poll and the counters of a phase side by side took 170
// (3 lattices, 68280 sites, FP32-12, five steps: 774 to 174 us; 64 lattices of
// 14.4 million sites 15.4 to 15.0 ms).  Every wait is bounded; on timeout the block
// records the failure in the status word and leaves, so the grid drains.
//
// The plaquettes of the outputs follow as two ordinary launches (the traces
// of every group of every lattice, then one reducing block per lattice) with
// exactly the arithmetic and partial layout of the standalone plaquette
// pass, in FP64 for every link precision.  Keeping them out of the
// persistent kernel keeps its register budget that of the step alone.
#include "ape_device.hpp"
#include "qdpx_impl.hpp"
#include "reduce_device.hpp"

namespace qdpx {

// LDS tile of the FP32 steps, a level of the single-lattice step's: 3, the
// own and backward links and the plane products (levels 2 and 4 measured the
// same for 12-real links and slower for 18-real ones).
constexpr int kBatchedLds = 3;

// Largest number of stage-A values a lattice's plaquette reduction may need
// (held in LDS): 3*ngroups <= kBatchMaxStage * kFinPerBlock (bounded with 4
// partials per group).
constexpr int kBatchMaxStage = 64;

// Counters, in words of the workspace: [1] the status; [32] the count of
// finished items; [64 + 32 x] XCD x's pending items; from kTicketWord on 8
// ticket counters a phase.  Atomics of all XCDs on one 128-byte line run
// one after another, so each counter has a line of its own, as far as the
// workspace has room for the phases (batched_ticket_stride).  With the counters
// of a phase side by side a phase of 3 lattices (68280 sites, FP32-12) took 67
// us, apart 35.
constexpr int kTicketWord = 64 + 32 * kXcds;

__global__ void __launch_bounds__(256) k_batched_init(unsigned *__restrict__ counters, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) counters[i] = 0u;
}

// XCD this block runs on (XCC_ID hardware register, bits 3:0).
__device__ __forceinline__ int xcd_id() {
    return (int)(__builtin_amdgcn_s_getreg((20) | (0 << 6) | ((4 - 1) << 11)) & (kXcds - 1));
}

// Take the next ticket (thread 0) and broadcast it to the block: of queue q,
// or, when that is empty, of the first of the others, in cyclic order, that
// is not.  Returns the ticket with q the queue it came from, or -1 when every
// queue was seen empty.  One read of the counters finds the queues that are
// left, where an atomic on each, 8 in a row with two barriers each for every
// block and phase, made them wait for one another.
__device__ __forceinline__ int take_ticket(unsigned *counters, int stride, const int (&total)[kXcds], int &q,
                                           int2 *s_ticket) {
    if (threadIdx.x == 0) {
        int r = -1, from = q;
        unsigned left = (1u << kXcds) - 1;  // queues not seen empty
        while (left) {
            const unsigned n =
                __hip_atomic_fetch_add(counters + stride * from, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (n < (unsigned)total[from]) {
                r = (int)n;
                break;
            }
            left &= ~(1u << from);
            unsigned seen[kXcds];
#pragma unroll
            for (int k = 0; k < kXcds; ++k)
                seen[k] = __hip_atomic_load(counters + stride * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int k = 0; k < kXcds; ++k)
                if (seen[k] >= (unsigned)total[k]) left &= ~(1u << k);
            if (left) {  // the next one after `from`
                const unsigned after = left >> from;
                from = after ? from + __builtin_ctz(after) : __builtin_ctz(left);
            }
        }
        *s_ticket = int2{r, from};
    }
    __syncthreads();
    const int r = __builtin_amdgcn_readfirstlane(s_ticket->x);
    q = __builtin_amdgcn_readfirstlane(s_ticket->y);
    __syncthreads();  // s_ticket is rewritten by the next call
    return r;
}

// Count `items` finished items of this block as done, device-wide.  Every
// store of theirs is in the XCD's L2 (its wave has waited for it); what makes
// it visible to the other XCDs is the write-back of that L2, which covers all
// of the XCD's blocks.  That rests on the MI355X beyond what the language's
// memory model says: every workgroup with one XCC_ID stores through one L2, a
// store counted down by vmcnt has reached it, and the waves of a workgroup share
// a CU (no threadgroup split).  So the blocks of an XCD share
// write-backs: `pending` holds the XCD's items that are in L2 and not yet
// counted; the block that finds it empty writes back and counts for all,
// until nothing is left.  A write-back by every block: 60 us a phase with 512
// blocks (3 lattices, 68280 sites, FP32-12), this 35.
__device__ __forceinline__ void publish(unsigned *pending, unsigned *done, unsigned items) {
    if (__hip_atomic_fetch_add(pending, items, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
    unsigned n = __hip_atomic_load(pending, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (n) {
        asm volatile("" ::"v"(n) : "memory");  // n has arrived before the write-back begins
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        // The write-back has finished.  It counts in vmcnt, but the compiler tracks
        // none for it: with no store of its own outstanding it leaves the fence's wait out.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __hip_atomic_fetch_add(done, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        n = __hip_atomic_fetch_sub(pending, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - n;
    }
}

// Lattice whose entry base(q) is the last one <= r (bases ascending).
template <typename F> __device__ __forceinline__ int find_lattice(int n_lat, int r, F base) {
    int lo = 0, hi = n_lat - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base(mid) <= r) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The lattice table comes as its own const __restrict__ argument: the compiler
// may then read it (at wave-uniform indices) with scalar loads, as the
// single-lattice kernels read their geometry from the kernel arguments.
// GPB 64-site groups are processed at once per block (4 waves each).  FP32:
// at most 128 registers, four waves per SIMD, what the LDS tile (36 KB per
// group) leaves room for.
template <typename R, int NR, int GPB>
__global__ void __launch_bounds__(256 * GPB) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 4 : 3)))
k_ape_batched(BatchArgs a, const BatchLat *__restrict__ lats) {
    __shared__ int2 s_ticket;
    __shared__ int s_ok;
    // FP32: the LDS tile of the single-lattice step at level kBatchedLds,
    // each group's own links, backward links and plane-product slots
    __shared__ nv4_t<R> own[GPB][sizeof(R) == 4 ? 4 * 3 * 64 : 1];
    __shared__ nv4_t<R> back[GPB][sizeof(R) == 4 && ape_lds_back(kBatchedLds) ? kApeTileF4 : 1];
    __shared__ nv4_t<R> slots[GPB][sizeof(R) == 4 && ape_lds_slots(kBatchedLds) ? 4 * kApeSlotF4 : 1];
    __shared__ double2 lds64[sizeof(R) == 8 ? 4 * GPB * f64_lds_per_wave(kApe) : 1];  // FP64: own and backward links
    // mu is wave-uniform; readfirstlane lets the compiler keep it in an SGPR
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int mu = w & 3, half = w >> 2;
    const int xid = __builtin_amdgcn_readfirstlane(xcd_id());
    const int nph = a.n_steps;
    unsigned *status = a.counters + 1;
    unsigned *done = a.counters + 32;  // items finished, over all phases (modulo 2^32)
    unsigned *pending = a.counters + 64 + 32 * xid;
    unsigned *tickets = a.counters + kTicketWord;  // [nph][kXcds], a.stride words apart
    const int per_ticket = a.group_chunk;           // groups per ticket
    for (int phase = 0; phase < nph; ++phase) {
        unsigned mine = 0;
        // step p reads the output of step p-1: step k writes to U_out when
        // n_steps-1-k is even, else to the lattice's scratch links
        const int src_odd = (a.n_steps - phase) & 1, dst_odd = (a.n_steps - 1 - phase) & 1;
        int q = xid;  // own queue first, then the others
        for (;;) {
            const int r = take_ticket(tickets + phase * kXcds * a.stride, a.stride, a.xtotal, q, &s_ticket);
            if (r < 0) break;
            ++mine;
            const BatchLat &L =
                lats[find_lattice(a.n_lat, r, [&](int i) { return lats[i].xbase[q]; })];  // read in place
            const int ncols = L.xcol1[q] - L.xcol0[q];
            const int j0 = (r - L.xbase[q]) * per_ticket;
            const int j1 = min(j0 + per_ticket, ncols * L.nrow);
            const void *src = (phase == 0) ? L.in : (src_odd == 0 ? L.out : L.tmp);
            void *dst = dst_odd == 0 ? L.out : L.tmp;
            const LinksRO<R, NR> U{(const vec2_t<R> *)src, L.g.S};
            const LinksWO<R, NR> O{(vec2_t<R> *)dst, L.g.S};
            // GPB groups at a time, half h of the block taking j0 + h, ...
            // (no early exit: every wave meets every barrier)
#pragma unroll 1
            for (int jj = j0; jj < j1; jj += GPB) {
                const int j = jj + half;
                const bool valid = j < j1;
                int grp = 0;
                if (valid) {
                    const int row = L.dcols[q].div(j);
                    grp = (L.xcol0[q] + (j - row * ncols)) + L.ncol * row;
                }
                if constexpr (sizeof(R) == 4) {  // links staged in LDS, as the single-lattice step
                    nv4_t<R> *bk = ape_lds_back(kBatchedLds) ? back[half] : nullptr;
                    if (jj > j0) __syncthreads();  // take_ticket's barriers separate items
                    if (valid) {
                        stage_own_link(L.g, U, grp, mu, lane, own[half]);
                        if constexpr (ape_lds_back(kBatchedLds)) stage_back_link(L.g, U, grp, mu, lane, bk);
                    }
                    __syncthreads();
                    if constexpr (ape_lds_slots(kBatchedLds))  // block barriers inside: every wave takes part
                        ape_group_shared<R, NR>(L.g, U, O, a.c1, a.c2, 0xFu, grp, valid, mu, lane, own[half], bk,
                                                slots[half]);
                    else if (valid)
                        ape_group<R, NR, kApe>(L.g, U, O, a.c1, a.c2, 0xFu, nullptr, grp, mu, lane, own[half],
                                               nullptr, bk);
                } else {
                    if (valid)
                        ape_group<R, NR, kApe>(L.g, U, O, a.c1, a.c2, 0xFu, nullptr, grp, mu, lane, nullptr,
                                               lds64 + w * f64_lds_per_wave(kApe));
                }
            }
        }
        if (phase + 1 == nph) break;
        const unsigned nitems = (unsigned)a.items_per_phase;
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's stores have reached the XCD's L2
        __syncthreads();
        if (threadIdx.x == 0) {
            if (mine) publish(pending, done, mine);
            const unsigned target = (unsigned)(phase + 1) * nitems;
            unsigned spins = 0;
            int ok = 1;
            // relaxed: an acquire on every poll would drop the L2 of the blocks still at work
            while ((int)(__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
                __builtin_amdgcn_s_sleep(8);
                if (++spins > a.spin_limit) {
                    ok = 0;
                    break;
                }
            }
            if (!ok) atomicOr(status, 1u);
            s_ok = ok;
            // the phase's results, for the whole block: its waves share the CU's L1
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (!s_ok) return;  // block-uniform
    }
}

// Plaquette traces of every lattice's output links into its partials: one
// 64-site group per block, the single-lattice plaquette pass's arithmetic
// and partial layout (plaquette_wave), so each lattice's plaquette is the
// one qdpx_plaquette gives for its links, bit for bit.  Contiguous ranges of
// groups per XCD, as there: 64 lattices with one step FP32-12 4.26 to 4.19 ms,
// FP64 7.35 to 7.30.
template <typename R, int NR>
__global__ void __launch_bounds__(64 * kPlaqWavesPerGroup) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 4 : 1)))
k_batched_plaq(BatchArgs a, const BatchLat *__restrict__ lats) {
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const BatchLat &L = lats[find_lattice(a.n_lat, b, [&](int i) { return lats[i].pbase; })];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    plaquette_wave(L.g, LinksRO<R, NR>{(const vec2_t<R> *)L.out, L.g.S}, b - L.pbase, w, lane, L.partials);
}

// One block per lattice: its partials reduced exactly as the two
// finalisation kernels of the single-lattice path do.
__global__ void __launch_bounds__(kReduceBlock) k_batched_fin(const BatchLat *__restrict__ lats, int per_group,
                                                             double *__restrict__ plaq) {
    __shared__ double lds[kReduceBlock / 64];
    __shared__ double stage[2][kBatchMaxStage];
    const BatchLat &L = lats[blockIdx.x];
    const int n = per_group * L.ngroups;
    const int nb = (n + kFinPerBlock - 1) / kFinPerBlock;
    double res[2];
    for (int comp = 0; comp < 2; ++comp) {
        for (int b = 0; b < nb; ++b) {
            const double v = fin_stage_a(L.partials + (int64_t)comp * n, n, b, lds);
            if (threadIdx.x == 0) stage[comp][b] = v;
        }
        __syncthreads();
        res[comp] = fin_stage_b(stage[comp], nb, lds);
    }
    if (threadIdx.x == 0) fin_write(res, 1, (double)L.g.V, plaq + 3 * blockIdx.x);
}

int batched_max_stage_groups() { return kBatchMaxStage * kFinPerBlock / 4; }

int batched_plaq_blocks(int, int ngroups) { return ngroups; }

template <typename R, int NR> static hipError_t resident(int gpb, int *per_cu) {
    if (gpb == 2) return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_ape_batched<R, NR, 2>, 512, 0);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_ape_batched<R, NR, 1>, 256, 0);
}

int batched_resident_blocks(int prec, int nrows, int block) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const int gpb = block / 256;
    hipError_t e;
    if (prec == 0) e = resident<double, 3>(gpb, &per_cu);
    else if (nrows == 3) e = resident<float, 3>(gpb, &per_cu);
    else e = resident<float, 2>(gpb, &per_cu);
    // (the occupancy does not depend on the kernel's arguments)
    if (e != hipSuccess) return 0;
    return cus * std::max(per_cu, 1);
}

int batched_counter_words(int max_phases) { return 2 + (kXcds + 1) * (max_phases + 1); }

int batched_ticket_stride(int n_steps, int words) {
    int stride = 32;
    while (stride > 1 && kTicketWord + n_steps * kXcds * stride > words) stride /= 2;
    return stride;
}

template <typename R, int NR>
static void launch_all(const BatchArgs &a, int block, int grid, hipStream_t st) {
    if (block == 512) k_ape_batched<R, NR, 2><<<grid, 512, 0, st>>>(a, a.lats);
    else k_ape_batched<R, NR, 1><<<grid, 256, 0, st>>>(a, a.lats);
    if (a.plaq) {
        k_batched_plaq<R, NR><<<a.plaq_blocks, 64 * kPlaqWavesPerGroup, 0, st>>>(a, a.lats);
        k_batched_fin<<<a.n_lat, kReduceBlock, 0, st>>>(a.lats, kPlaqWavesPerGroup, a.plaq);
    }
}

hipError_t launch_ape_batched(const BatchArgs &a, int prec, int nrows, int block, int grid, hipStream_t st) {
    const int ncount = kTicketWord + a.n_steps * kXcds * a.stride;
    k_batched_init<<<std::min((ncount + 255) / 256, 1024), 256, 0, st>>>(a.counters, ncount);
    if (prec == 0) launch_all<double, 3>(a, block, grid, st);
    else if (nrows == 3) launch_all<float, 3>(a, block, grid, st);
    else launch_all<float, 2>(a, block, grid, st);
    return hipGetLastError();
}

}  // namespace qdpx
