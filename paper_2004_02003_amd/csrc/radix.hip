// Device-wide exclusive scan of 32-bit counts and a stable LSD radix sort of
// record slots by 32- or 64-bit keys, for the two reorderings of the path: the
// grid-gradient records (sorted by colour | level | cell, equal keys kept in
// slot order) and the rebin's bin offsets.
//
// Scan: each workgroup sums a chunk of 4,096 counts; then each scans its chunk
// from the sum of the chunks before it (up to 1,024 chunks it adds their totals
// itself, four per thread: a launch less; beyond, one workgroup scans the
// totals in between).
//
// Sort, per 8-bit digit from the lowest: a histogram of the digit per tile of
// 4,096 pairs (digit-major: count[digit][tile]), its exclusive scan (the first
// output slot of every (digit, tile)), and a scatter.  In the scatter
// wavefront w of a tile takes the tile's pairs [1024 w, 1024 w + 1024) in 16
// rounds of 64 consecutive pairs; lanes with equal digits find each other with
// one ballot per digit bit, and a pair's place is its digit's first in the
// tile, plus the counts of its digit in the tile's earlier wavefronts, earlier
// rounds and lower lanes -- the input order, so equal keys keep their order.
// The pairs are put in that order in LDS and leave from there, so a wavefront
// stores a few runs of consecutive slots instead of 64 scattered pairs.  The
// first pass takes the slot number as the value (nothing to read) and leaves
// the unused slots out, and the later ones work on the used ones alone.
//
// The passes move bytes: 3.4 million slots of which 1.6 million are used, 30
// key bits (gradient of 32,768 seeds over 50 steps, 128^3): 137 us, 17 of them
// per scatter and 11 per scan.  64-bit keys, every slot in every pass, scattered
// stores and a scan of three launches took 262 (34 and 16).
#include "bto_internal.h"

namespace bto {

constexpr int SCAN_CHUNK = 4096;          // counts per scan workgroup (256 threads x 16)
constexpr int RADIX_BITS = 8;
constexpr int RADIX_BINS = 1 << RADIX_BITS;
constexpr int SORT_ROUNDS = 16;           // rounds of 64 pairs per wavefront
constexpr int SORT_TILE = BLOCK * SORT_ROUNDS;  // 4,096 pairs per workgroup
static_assert(RADIX_BINS == BLOCK, "one digit per thread");

// ---------------------------------------------------------------------------
// Scan.
// ---------------------------------------------------------------------------
// Sum of one value per thread over the workgroup; excl: the sum of the threads
// before this one.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* s_wave, uint32_t& excl) {
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    if (lane == WAVE - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / WAVE; ++w) {
        const uint32_t t = s_wave[w];
        before += w < wave ? t : 0u;
        total += t;
    }
    excl = before + incl - v;
    __syncthreads();  // s_wave may be used again
    return total;
}

constexpr int SCAN_PER = SCAN_CHUNK / BLOCK;  // 16 consecutive counts per thread

// Number of counts: n, or one per digit and tile of *pairs sorted pairs.
__device__ __forceinline__ uint64_t scan_size(uint64_t n, const uint32_t* pairs) {
    return pairs ? (uint64_t)((*pairs + SORT_TILE - 1u) / SORT_TILE) * RADIX_BINS : n;
}

__global__ __launch_bounds__(BLOCK) void scan_total_kernel(const uint32_t* in, uint64_t n, const uint32_t* pairs,
                                                           uint32_t* totals) {
    __shared__ uint32_t s_wave[BLOCK / WAVE];
    n = scan_size(n, pairs);
    const uint64_t c0 = (uint64_t)blockIdx.x * SCAN_CHUNK + threadIdx.x;
    uint32_t sum = 0, excl;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) sum += c0 + k * BLOCK < n ? in[c0 + k * BLOCK] : 0u;
    const uint32_t total = block_scan(sum, s_wave, excl);
    if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

// Exclusive scan of the chunk totals (any count) by one workgroup, in place.
__global__ __launch_bounds__(BLOCK) void scan_totals_kernel(uint32_t* t, uint32_t n) {
    __shared__ uint32_t s_wave[BLOCK / WAVE];
    uint32_t carry = 0;
    for (uint32_t b = 0; b < n; b += BLOCK) {
        const uint32_t i = b + threadIdx.x;
        const uint32_t x = i < n ? t[i] : 0u;
        uint32_t excl;
        const uint32_t total = block_scan(x, s_wave, excl);
        if (i < n) t[i] = carry + excl;
        carry += total;
    }
}

// Exclusive scan of one chunk.  totals: the chunks' totals, or (scanned) their
// exclusive scan, or null (one chunk).  The sum of all counts goes to *all.
__global__ __launch_bounds__(BLOCK) void scan_chunk_kernel(const uint32_t* in, uint32_t* out, uint64_t n,
                                                           const uint32_t* pairs, const uint32_t* totals, int scanned,
                                                           uint32_t* all) {
    __shared__ uint32_t s_wave[BLOCK / WAVE];
    n = scan_size(n, pairs);
    const uint64_t first = (uint64_t)blockIdx.x * SCAN_CHUNK, c0 = first + (uint64_t)threadIdx.x * SCAN_PER;
    if (first >= n && blockIdx.x) return;
    uint32_t v[SCAN_PER], sum = 0, excl;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) v[k] = c0 + k < n ? in[c0 + k] : 0u;
    uint32_t before = 0;
    if (totals && scanned) {
        before = totals[blockIdx.x];
    } else if (totals) {
        uint32_t t = 0;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += BLOCK) t += totals[i];
        before = block_scan(t, s_wave, excl);
    }
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) sum += v[k];
    const uint32_t total = block_scan(sum, s_wave, excl);
    uint32_t run = before + excl;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) {
        if (c0 + k < n) out[c0 + k] = run;
        run += v[k];
    }
    if (all && threadIdx.x == 0 && first + SCAN_CHUNK >= n) *all = before + total;
}

size_t scan_temp_bytes(uint64_t n) {
    const uint64_t chunks = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    return (size_t)(chunks > 0 ? chunks : 1) * sizeof(uint32_t);
}

static hipError_t scan(const uint32_t* in, uint32_t* out, uint64_t n, const uint32_t* pairs, uint32_t* all,
                       void* temp, hipStream_t s) {
    const uint64_t chunks = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    uint32_t* totals = chunks > 1 ? static_cast<uint32_t*>(temp) : nullptr;
    const int scanned = chunks > 1024;
    if (totals) {
        hipLaunchKernelGGL(scan_total_kernel, dim3((unsigned)chunks), dim3(BLOCK), 0, s, in, n, pairs, totals);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (scanned) hipLaunchKernelGGL(scan_totals_kernel, dim3(1), dim3(BLOCK), 0, s, totals, (uint32_t)chunks);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(scan_chunk_kernel, dim3((unsigned)chunks), dim3(BLOCK), 0, s, in, out, n, pairs, totals,
                       scanned, all);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const uint32_t* in, uint32_t* out, uint64_t n, void* temp, hipStream_t s) {
    return n == 0 ? hipSuccess : scan(in, out, n, nullptr, nullptr, temp, s);
}

// ---------------------------------------------------------------------------
// Radix sort.  FIRST: the n slots themselves, unused ones (bit `drop` set) left
// out; otherwise the *count pairs of the pass before.
// ---------------------------------------------------------------------------
template <class K, bool FIRST>
__global__ __launch_bounds__(BLOCK) void radix_hist_kernel(const K* key, uint64_t n, const uint32_t* count, int drop,
                                                           int shift, uint32_t* hist) {
    __shared__ uint32_t s_h[RADIX_BINS];
    if (!FIRST) n = *count;
    const uint32_t tiles = (uint32_t)((n + SORT_TILE - 1) / SORT_TILE);
    if (blockIdx.x >= tiles) return;
    const uint64_t t0 = (uint64_t)blockIdx.x * SORT_TILE + threadIdx.x;
    K k[SORT_ROUNDS];
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r) k[r] = t0 + r * BLOCK < n ? key[t0 + r * BLOCK] : (K)0;
    s_h[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r)
        if (t0 + r * BLOCK < n && !(FIRST && (k[r] >> drop)))
            atomicAdd(&s_h[(uint32_t)(k[r] >> shift) & (RADIX_BINS - 1)], 1u);
    __syncthreads();
    hist[(uint64_t)threadIdx.x * tiles + blockIdx.x] = s_h[threadIdx.x];
}

// Lanes of the wavefront whose digit equals this lane's (among the lanes in
// `active`).
__device__ __forceinline__ unsigned long long digit_peers(uint32_t d, unsigned long long active) {
    unsigned long long m = active;
#pragma unroll
    for (int b = 0; b < RADIX_BITS; ++b) {
        const unsigned long long bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

template <class K, bool FIRST>
__global__ __launch_bounds__(BLOCK) void radix_scatter_kernel(const K* key, const uint32_t* val, uint64_t n,
                                                              const uint32_t* count, int drop, int shift,
                                                              const uint32_t* offs, K* key_out, uint32_t* val_out) {
    constexpr int W = BLOCK / WAVE;
    __shared__ uint32_t s_cnt[W][RADIX_BINS];
    __shared__ uint32_t s_out[RADIX_BINS];
    __shared__ uint32_t s_wave[W];
    __shared__ K s_key[SORT_TILE];
    __shared__ uint32_t s_val[SORT_TILE];
    if (!FIRST) n = *count;
    const uint32_t tiles = (uint32_t)((n + SORT_TILE - 1) / SORT_TILE);
    if (blockIdx.x >= tiles) return;
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const uint64_t w0 = (uint64_t)blockIdx.x * SORT_TILE + (uint64_t)wave * (WAVE * SORT_ROUNDS);
    K k[SORT_ROUNDS];
    uint32_t v[SORT_ROUNDS];
    uint32_t rg[SORT_ROUNDS];  // rank among the round's equal digits | group size << 8 (0: no pair)
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r) {
        const uint64_t i = w0 + (uint64_t)r * WAVE + lane;
        k[r] = i < n ? key[i] : (K)0;
        v[r] = FIRST ? (uint32_t)i : i < n ? val[i] : 0u;
    }
    const uint32_t out0 = offs[(uint64_t)threadIdx.x * tiles + blockIdx.x];
#pragma unroll
    for (int w = 0; w < W; ++w) s_cnt[w][threadIdx.x] = 0u;
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    // counts of each digit in this wavefront's 1,024 pairs
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r) {
        const bool ok = w0 + (uint64_t)r * WAVE + lane < n && !(FIRST && (k[r] >> drop));
        const uint32_t d = (uint32_t)(k[r] >> shift) & (RADIX_BINS - 1);
        const unsigned long long peers = digit_peers(d, __ballot(ok));
        const uint32_t rank = (uint32_t)__popcll(peers & lt), size = (uint32_t)__popcll(peers);
        rg[r] = ok ? rank | (size << 8) : 0u;
        if (ok && rank == 0u) s_cnt[wave][d] += size;  // the group's lowest lane
    }
    __syncthreads();
    // first place of each digit in the tile, for each of its wavefronts
    uint32_t mine = 0, start;
#pragma unroll
    for (int w = 0; w < W; ++w) mine += s_cnt[w][threadIdx.x];
    const uint32_t used = block_scan(mine, s_wave, start);
    s_out[threadIdx.x] = out0 - start;  // modulo 2^32
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t c = s_cnt[w][threadIdx.x];
        s_cnt[w][threadIdx.x] = start;
        start += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r) {
        const uint32_t d = (uint32_t)(k[r] >> shift) & (RADIX_BINS - 1);
        const uint32_t size = rg[r] >> 8, rank = rg[r] & 0xFFu;
        const uint32_t base = s_cnt[wave][d];  // read by every lane of the group before the lowest one adds
        if (size) {
            s_key[base + rank] = k[r];
            s_val[base + rank] = v[r];
        }
        if (size && rank == 0u) s_cnt[wave][d] = base + size;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SORT_ROUNDS; ++r) {
        const uint32_t i = r * BLOCK + threadIdx.x;
        if (i < used) {
            const K x = s_key[i];
            const uint32_t o = s_out[(uint32_t)(x >> shift) & (RADIX_BINS - 1)] + i;
            key_out[o] = x;
            val_out[o] = s_val[i];
        }
    }
}

size_t radix_temp_bytes(uint64_t n) {
    const uint64_t tiles = (n + SORT_TILE - 1) / SORT_TILE;
    const uint64_t cnt = (tiles > 0 ? tiles : 1) * RADIX_BINS;
    return (size_t)(2 * cnt) * sizeof(uint32_t) + scan_temp_bytes(cnt) + 256;
}

template <class K>
static hipError_t sort_slots(K* key, K* key_alt, uint32_t* idx0, uint32_t* idx1, uint64_t n, int bits,
                             uint32_t* count, void* temp, bool* result_in_alt, hipStream_t s) {
    const uint64_t tiles = (n + SORT_TILE - 1) / SORT_TILE;
    const uint64_t cnt = tiles * RADIX_BINS;
    uint32_t* hist = static_cast<uint32_t*>(temp);
    uint32_t* offs = hist + cnt;
    void* stemp = offs + cnt;
    const dim3 grid((unsigned)tiles), block(BLOCK);
    K* ka = key;
    K* kb = key_alt;
    uint32_t* va = idx0;
    uint32_t* vb = idx1;
    *result_in_alt = false;
    for (int shift = 0; shift < bits; shift += RADIX_BITS) {
        const bool first = shift == 0;
        if (first) hipLaunchKernelGGL((radix_hist_kernel<K, true>), grid, block, 0, s, ka, n, count, bits, shift, hist);
        else hipLaunchKernelGGL((radix_hist_kernel<K, false>), grid, block, 0, s, ka, n, count, bits, shift, hist);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = scan(hist, offs, cnt, first ? nullptr : count, first ? count : nullptr, stemp, s);
        if (e != hipSuccess) return e;
        if (first)
            hipLaunchKernelGGL((radix_scatter_kernel<K, true>), grid, block, 0, s, ka, va, n, count, bits, shift, offs,
                               kb, vb);
        else
            hipLaunchKernelGGL((radix_scatter_kernel<K, false>), grid, block, 0, s, ka, va, n, count, bits, shift,
                               offs, kb, vb);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        std::swap(ka, kb);
        std::swap(va, vb);
        *result_in_alt = !*result_in_alt;
    }
    return hipSuccess;
}

hipError_t launch_radix_sort_slots(void* key, void* key_alt, uint32_t* idx0, uint32_t* idx1, int key_bytes,
                                   uint64_t n, int bits, uint32_t* count, void* temp, bool* result_in_alt,
                                   hipStream_t s) {
    if (n == 0 || n > 0xFFFFFFFFull) return hipErrorInvalidValue;
    if (key_bytes == 4)
        return sort_slots(static_cast<uint32_t*>(key), static_cast<uint32_t*>(key_alt), idx0, idx1, n, bits, count,
                          temp, result_in_alt, s);
    return sort_slots(static_cast<uint64_t*>(key), static_cast<uint64_t*>(key_alt), idx0, idx1, n, bits, count, temp,
                      result_in_alt, s);
}

}  // namespace bto
