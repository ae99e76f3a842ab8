// Deterministic reduction of the adjoint's grid-gradient records.
//
// The reverse sweep writes one record per accumulator flush into a slot fixed
// by (flush rank, seed): the 8 corner gradients (x 3 components) of one cell
// of one grid level, keyed by parity colour | level | cell (unused slots carry
// the bit above).  A stable radix sort (radix.hip) orders the records by key;
// then, one colour at a time (a contiguous range of the sorted keys), each
// (level, cell) group is summed in slot order (the flush's rank, then the
// seed id) and added to the grid's 8 corners with plain loads and stores.
// Two different cells of one colour differ by at least two cells along some
// axis, so their corner sets are disjoint and the stores of one colour never
// collide; the colours are applied in a fixed order.  The result does not
// depend on thread timing, unlike FP32 atomics, and each corner costs one
// read and one write per group instead of one memory-side atomic per
// contribution.
#include "bto_internal.h"

namespace bto {

// Before a sweep: every slot unused.
template <class K>
__global__ __launch_bounds__(BLOCK) void grad_clear_kernel(K* key, uint64_t n, K empty) {
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (uint64_t)gridDim.x * BLOCK)
        key[i] = empty;
}

// bounds[c] = first sorted record of colour c (c = 0..8; bounds[8]: their
// number, found by the sort in bounds[9]).
template <class K>
__global__ __launch_bounds__(BLOCK) void grad_bounds_kernel(const K* key, int colour_shift, uint32_t* bounds) {
    const uint32_t n = bounds[9];
    for (uint32_t i = blockIdx.x * BLOCK + threadIdx.x; i <= n; i += gridDim.x * BLOCK) {
        const uint32_t c = i < n ? (uint32_t)(key[i] >> colour_shift) : 8u;
        const uint32_t lo = i > 0 ? (uint32_t)(key[i - 1] >> colour_shift) + 1u : 0u;
        for (uint32_t q = lo; q <= c; ++q) bounds[q] = i;
    }
}

// A corner's gradient.
struct __attribute__((packed, aligned(4))) Corner {
    float v[3];
};

// Eight lanes per record of the colour, one per corner; those of the first
// record of a group (one (colour, level, cell): a run of equal keys) sum the
// group.  The grids' lines bound it, 90 MB read and 46 MB written per colour: 46
// us.  With a lane per record (six 16-byte loads 96 bytes apart from lane to
// lane, eight 12-byte corners) 49 us, and 60 with each load where its value is
// used; so the keys around the record and its index load together, then the
// corner's gradient and the grid's.
template <class K>
__global__ __launch_bounds__(BLOCK) void grad_apply_kernel(const K* key, const uint32_t* idx, const float* val,
                                                           const uint32_t* bounds, int colour, K cell_mask,
                                                           int level_shift, K level_mask, float* const* gf, Geom g) {
    const uint32_t lo = bounds[colour], hi = bounds[colour + 1];
    const uint32_t corner = threadIdx.x % 8;
    const uint64_t step = 3 * ((uint64_t)(corner & 1) + (uint64_t)g.sy * (corner >> 1 & 1) +
                               (uint64_t)g.sz * (corner >> 2));
    const float* v0 = val + 3 * corner;
    for (uint32_t i = lo + (blockIdx.x * BLOCK + threadIdx.x) / 8; i < hi; i += gridDim.x * (BLOCK / 8)) {
        const K k = key[i], before = key[i > lo ? i - 1 : i], after = key[i + 1 < hi ? i + 1 : i];
        const uint32_t rec = idx[i];
        if (i > lo && before == k) continue;  // not the first record of its group
        Corner s = *reinterpret_cast<const Corner*>(v0 + 24 * (size_t)rec);
        Corner* p = reinterpret_cast<Corner*>(in_global(gf[(int)((k >> level_shift) & level_mask)]) +
                                              3 * (uint64_t)(k & cell_mask) + step);
        const Corner old = *p;
        if (i + 1 < hi && after == k) {
            for (uint32_t j = i + 1; j < hi && key[j] == k; ++j) {
                const Corner y = *reinterpret_cast<const Corner*>(v0 + 24 * (size_t)idx[j]);
#pragma unroll
                for (int d = 0; d < 3; ++d) s.v[d] += y.v[d];
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) s.v[d] = old.v[d] + s.v[d];
        *p = s;
    }
}

static int key_bits(const GradRec& r) { return r.level_bits + r.cell_bits + 3; }

static unsigned grid_of(uint64_t n) {
    const uint64_t b = (n + BLOCK - 1) / BLOCK;
    return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

hipError_t launch_grad_clear(const GradRec& r, uint64_t n, hipStream_t s) {
    // unused slots: the bit above the key's
    const uint64_t empty = 1ull << key_bits(r);
    if (r.key_bytes == 4)
        hipLaunchKernelGGL((grad_clear_kernel<uint32_t>), dim3(grid_of(n)), dim3(BLOCK), 0, s,
                           static_cast<uint32_t*>(r.key), n, (uint32_t)empty);
    else
        hipLaunchKernelGGL((grad_clear_kernel<uint64_t>), dim3(grid_of(n)), dim3(BLOCK), 0, s,
                           static_cast<uint64_t*>(r.key), n, empty);
    return hipGetLastError();
}

template <class K>
static hipError_t apply(const GradRec& r, const K* key, const uint32_t* idx, uint32_t* bounds, uint64_t n,
                        float* const* gf, const Geom& g, hipStream_t s) {
    hipLaunchKernelGGL((grad_bounds_kernel<K>), dim3(grid_of(n + 1)), dim3(BLOCK), 0, s, key, key_bits(r) - 3, bounds);
    hipError_t e = hipGetLastError();
    const K cell_mask = (K)((1ull << r.cell_bits) - 1ull), level_mask = (K)((1ull << r.level_bits) - 1ull);
    for (int colour = 0; colour < 8 && e == hipSuccess; ++colour) {
        hipLaunchKernelGGL((grad_apply_kernel<K>), dim3(grid_of(n)), dim3(BLOCK), 0, s, key, idx, r.val,
                           bounds, colour, cell_mask, r.cell_bits, level_mask, gf, g);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_grad_reduce(const GradRec& r, const GradSort& w, uint64_t n, float* const* gf, const Geom& g,
                              hipStream_t s) {
    if (n == 0) return hipSuccess;
    bool in_alt = false;
    hipError_t e = launch_radix_sort_slots(r.key, w.key_alt, w.idx[0], w.idx[1], r.key_bytes, n, key_bits(r),
                                           w.bounds + 9, w.temp, &in_alt, s);
    if (e != hipSuccess) return e;
    const void* key = in_alt ? w.key_alt : r.key;
    const uint32_t* idx = w.idx[in_alt ? 1 : 0];
    if (r.key_bytes == 4) return apply(r, static_cast<const uint32_t*>(key), idx, w.bounds, n, gf, g, s);
    return apply(r, static_cast<const uint64_t*>(key), idx, w.bounds, n, gf, g, s);
}

}  // namespace bto
