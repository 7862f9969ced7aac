// Deterministic FP64 reduction of per-group partial sums.  The same code
// runs as two kernels (single-lattice calls) or inside one block (the
// batched kernel), so both give bit-identical results.
#pragma once

#include "qdpx_impl.hpp"
#include "su3_device.hpp"

namespace qdpx {

constexpr int kFinChunk = 16;
constexpr int kFinPerBlock = kReduceBlock * kFinChunk;

// This thread's share of chunk b of n values: thread t of kReduceBlock adds
// its 16 consecutive values in order.  The loads do not depend on the bound
// (an index past the end reads the last value, which is not added), so all 16
// are in flight together.
__device__ __forceinline__ double fin_chunk(const double *__restrict__ p, int n, int b, int t) {
    const int base = b * kFinPerBlock + t * kFinChunk;
    const auto *gp = gptr<double>(p);  // partials always live in global memory
    double x[kFinChunk];
#pragma unroll
    for (int k = 0; k < kFinChunk; ++k) x[k] = gp[min(base + k, n - 1)];
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kFinChunk; ++k) v = base + k < n ? v + x[k] : v;
    return v;
}

// Stage A for chunk b: the threads' shares in a fixed block tree.  Result
// valid in thread 0.
__device__ __forceinline__ double fin_stage_a(const double *__restrict__ p, int n, int b, double *lds) {
    return block_sum<kReduceBlock / 64>(fin_chunk(p, n, b, (int)threadIdx.x), lds);
}

// Stage B over nb stage-A values: strided per-thread sums, then the tree.
__device__ __forceinline__ double fin_stage_b(const double *p, int nb, double *lds) {
    double v = 0.0;
    for (int i = threadIdx.x; i < nb; i += kReduceBlock) v += p[i];
    return block_sum<kReduceBlock / 64>(v, lds);
}

// Both stages in one block of any multiple of kReduceBlock threads (that many
// chunks at a time), the sums formed in the order of the two stages: nb <= 64
// chunks per component (stage B then holds one value per lane of one wave).
// part: 4 * ncomp * nb doubles of LDS.  r valid in thread 0.
__device__ __forceinline__ void fin_both(const double *__restrict__ p, int n, int ncomp, double *part, double r[2]) {
    const int nb = (n + kFinPerBlock - 1) / kFinPerBlock;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = threadIdx.x & (kReduceBlock - 1);
    for (int c = w >> 2; c < ncomp * nb; c += (int)blockDim.x / kReduceBlock) {
        const int comp = c >= nb;
        const double v = wave_sum(fin_chunk(p + (int64_t)comp * n, n, c - comp * nb, t));
        if (lane == 0) part[4 * c + (w & 3)] = v;
    }
    __syncthreads();
    if (w == 0)
        for (int comp = 0; comp < ncomp; ++comp) {
            double v = 0.0;
            if (lane < nb) {
                const double *q = part + 4 * (comp * nb + lane);
                v += ((q[0] + q[1]) + q[2]) + q[3];
            }
            r[comp] = wave_sum(v);
        }
}

// mode 0: out[0] = r[0]; mode 1: plaquette triple from spatial r[0] and temporal r[1].
__device__ __forceinline__ void fin_write(const double r[2], int mode, double volume, double *out) {
    if (mode == 0) {
        out[0] = r[0];
    } else {
        out[0] = (r[0] + r[1]) / (18.0 * volume);
        out[1] = r[0] / (9.0 * volume);
        out[2] = r[1] / (9.0 * volume);
    }
}

}  // namespace qdpx
