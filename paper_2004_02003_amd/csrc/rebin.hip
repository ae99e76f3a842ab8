// Spatial re-sort of live particles ("rebin", part of particle management).
//
// Particles start in lattice order, so the 64 lanes of a wavefront read nearby
// cells and share cache lines; as the flow disperses them that locality
// decays and every lane touches its own lines.  Between advection launches the
// live particles of each XCD segment are re-ordered by the 32x2x2-cell bin
// that holds them, bins in x-fastest order (a wavefront's particles then lie
// along a few grid rows, so each of a cell's row loads covers long runs of
// contiguous memory -- the same reason the lattice is seeded x-fastest), with
// a counting sort:
//   count   - atomically add to each (segment, bin) counter, once for a
//             wavefront's particles of the bin; the old value and the place
//             among them are a particle's rank inside the bin;
//   scan    - exclusive prefix sum over all bins (segment-major; radix.hip);
//   scatter - move each particle to its segment base + bin offset + rank, and
//             zero its bin for the next rebin.
// Order inside a bin is unspecified; results do not depend on particle
// order.
#include "bto_internal.h"

namespace bto {

__device__ __forceinline__ int segment_of(const Segs& sg, int64_t i) {
    int seg = 0;
#pragma unroll
    for (int x = 1; x < NSEG; ++x) seg += (i >= sg.base[x]) ? 1 : 0;
    return seg;
}

// The counters are memory atomics whose old value is needed, and those bound
// the kernel (2 million particles of a 256^3 turbulence block, re-sorted every
// 5 steps: 98 us with one atomic each, 40 now).  Most of a wavefront's particles
// still share their bins, so the lanes of one bin, found with a ballot per bit
// of the bin number, send one atomic together.
__global__ __launch_bounds__(BLOCK) void rebin_count_kernel(const RebinArgs a) {
    const unsigned long long lt = (1ull << (threadIdx.x % WAVE)) - 1ull;
    const int64_t n = (a.P + WAVE - 1) / WAVE * WAVE;  // whole wavefronts stay together
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) {
        const int seg = segment_of(a.segs, i);
        // (slots beyond the segment's live count hold none)
        const bool live = i < a.P && i - a.segs.base[seg] < (int64_t)a.count[seg * CSTRIDE];
        const uint32_t c = live ? a.pos[i].cell : 0u;
        const uint32_t key = (c & 1023u) / REBIN_BIN[0] +
                             a.nbx * (((c >> 10) & 1023u) / REBIN_BIN[1] + a.nby * (((c >> 20) & 1023u) / REBIN_BIN[2]));
        const uint32_t bin = (uint32_t)seg * a.nbins + key;
        unsigned long long peers = __ballot(live);
        if (!peers) continue;
        for (int b = 0; b < a.bin_bits; ++b) {
            const unsigned long long m = __ballot((bin >> b) & 1u);
            peers &= (bin >> b) & 1u ? m : ~m;
        }
        const int first = live ? __ffsll((long long)peers) - 1 : 0;
        uint32_t old = 0u;
        if (live && !(peers & lt)) old = atomicAdd(&a.hist[bin], (uint32_t)__popcll(peers));
        const uint32_t base = __shfl(old, first);
        if (live) {
            a.bin[i] = bin;
            a.rank[i] = base + (uint32_t)__popcll(peers & lt);
        }
    }
}

__global__ __launch_bounds__(BLOCK) void rebin_scatter_kernel(const RebinArgs a) {
    uint32_t start[NSEG];
    uint32_t acc = 0;
#pragma unroll
    for (int x = 0; x < NSEG; ++x) {
        start[x] = acc;
        acc += a.count[x * CSTRIDE];
    }
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < a.P; i += (int64_t)gridDim.x * BLOCK) {
        const int seg = segment_of(a.segs, i);
        if (i - a.segs.base[seg] >= (int64_t)a.count[seg * CSTRIDE]) continue;
        const uint32_t bin = a.bin[i];
        const int64_t dst = a.segs.base[seg] + (int64_t)(a.offs[bin] - start[seg]) + a.rank[i];
        a.out_pos[dst] = a.pos[i];
        a.out_id[dst] = a.id[i];
        a.hist[bin] = 0u;  // every particle of the bin writes the same zero
    }
}

static int grid_of(int64_t n) {
    int64_t b = (n + BLOCK - 1) / BLOCK;
    return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

size_t rebin_temp_bytes(int64_t nbins_total) { return scan_temp_bytes((uint64_t)nbins_total); }

hipError_t launch_rebin(const RebinArgs& a, hipStream_t s) {
    if (a.P == 0) return hipSuccess;
    hipLaunchKernelGGL(rebin_count_kernel, dim3(grid_of(a.P)), dim3(BLOCK), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_exclusive_scan(a.hist, a.offs, (uint64_t)NSEG * a.nbins, a.temp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rebin_scatter_kernel, dim3(grid_of(a.P)), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

}  // namespace bto
