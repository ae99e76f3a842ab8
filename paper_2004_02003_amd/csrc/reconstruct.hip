// Post hoc side of the flow map on the seed lattice: placing per-block flow
// maps into one lattice, rebuilding terminated entries by the one-dimensional
// linear interpolation of Eq. (1) (Section 3.2; Eq. (2) shows the rebuilt
// value changes no later linear interpolation), and the accuracy metric of
// Eq. (5) and Eq. (6) (Section 4).
//
// Layout: lattice entries in x-fastest order, end positions as 3 doubles per
// entry, states as bytes (0 missing, 1 known, 2 rebuilt).  The rebuild runs
// one pass per axis (x, then y, then z), which fills every run of unknown
// entries that has known entries on both sides.  Lines of one pass are
// disjoint, so a pass needs no synchronisation beyond the kernel boundary.
// The passes read the states (a byte per entry) and move the positions of the
// entries they fill, so their time is that of reading the states in whole
// lines: the x pass, whose lines are contiguous, gives each to one wavefront
// and makes the states from the flags on the way; the y and z passes give each
// line to one lane, the lanes side by side along x.  128^3 entries of eight
// blocks with a smooth flow: x 12.6 us, y and z 7.7 each.  With the states made
// by a pass of their own (6.4 us) and one wavefront per line on every axis, 64
// scattered bytes per read, 13.3 us per pass.
#include <mutex>

#include "bto_internal.h"

namespace bto {

constexpr uint8_t ST_MISSING = 0, ST_KNOWN = 1, ST_REBUILT = 2;

__global__ __launch_bounds__(BLOCK) void recon_init_kernel(int64_t P, double* end, const uint8_t* flag,
                                                           uint8_t* state) {
    for (int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x; t < P; t += (int64_t)gridDim.x * BLOCK) {
        const bool known = flag[t] == (uint8_t)S_VALID;
        state[t] = known ? ST_KNOWN : ST_MISSING;
        if (!known) {
            const double nan = __builtin_nan("");
            end[3 * t] = nan;
            end[3 * t + 1] = nan;
            end[3 * t + 2] = nan;
        }
    }
}

constexpr int MAX_LINE = 1024;  // a lattice line never exceeds the grid's points per axis

// The x pass, and the y and z passes of lattices with few lines (see below): one
// wavefront per line, read in chunks of 64 entries.  A ballot
// per chunk marks the known ones, and every unknown entry finds its nearest
// known neighbours from the ballot masks (below: highest set bit under its
// lane, carried across chunks left to right; above: lowest set bit over its
// lane, carried right to left).  All states are read before any entry is
// written, so only entries known at the start of the pass bracket.  INIT: the
// states come from the flags and are all written, with NaN for the entries
// that stay missing.
// NC: chunks there is room for (2 for lines of up to 128 entries, 16 for all).
// X: lines along x, contiguous; otherwise point stride st, lines indexed by x
// (n_a of them) and the other axis, whose stride is s_b.
template <bool INIT, bool X, int NC>
__global__ __launch_bounds__(BLOCK) void recon_line_kernel(int64_t n_lines, int32_t n_a, int64_t s_b, int32_t len,
                                                           int64_t st, double* end, const uint8_t* flag,
                                                           uint8_t* state) {
#pragma clang fp contract(off)  // Eq. (1) rounded as written: two products, one sum
    const int64_t line = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) / WAVE;
    const int lane = threadIdx.x % WAVE;
    if (line >= n_lines) return;  // whole wavefronts leave together
    const int64_t base = X ? line * len : line % n_a + line / n_a * s_b;
    const auto at = [&](int i) { return base + (X ? (int64_t)i : (int64_t)i * st); };
    const int nchunk = (len + WAVE - 1) / WAVE;
    unsigned long long mask[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        mask[c] = 0ull;
        if (c < nchunk) {
            const int i = c * WAVE + lane;
            const bool known = i < len && (INIT ? flag[at(i)] == (uint8_t)S_VALID : state[at(i)] != ST_MISSING);
            mask[c] = __ballot(known);
        }
    }
    // nearest known index below each of this lane's entries (-1: none)
    int lo[NC];
    int carry = -1;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        lo[c] = -1;
        if (c < nchunk) {
            const unsigned long long m = mask[c] & below;
            lo[c] = m ? c * WAVE + 63 - __clzll((long long)m) : carry;
            if (mask[c]) carry = c * WAVE + 63 - __clzll((long long)mask[c]);
        }
    }
    // nearest known index above, then Eq. (1) for the unknown entries between
    carry = -1;
    const unsigned long long above = lane == 63 ? 0ull : ~((2ull << lane) - 1ull);
#pragma unroll
    for (int c = NC - 1; c >= 0; --c) {
        if (c >= nchunk) continue;
        const unsigned long long m = mask[c] & above;
        const int hi = m ? c * WAVE + __ffsll((long long)m) - 1 : carry;
        if (mask[c]) carry = c * WAVE + __ffsll((long long)mask[c]) - 1;
        const int i = c * WAVE + lane;
        if (i >= len) continue;
        const bool known = (mask[c] >> lane) & 1ull;
        const bool fill = !known && lo[c] >= 0 && hi >= 0;
        if (fill) {
            // Eq. (1): L(x1) = (x1 - x0)/(x2 - x0) f(x2) + (x2 - x1)/(x2 - x0) f(x0)
            const double span = (double)(hi - lo[c]);
            const double w2 = (double)(i - lo[c]) / span, w0 = (double)(hi - i) / span;
            const int64_t q0 = at(lo[c]), q2 = at(hi), r = at(i);
#pragma unroll
            for (int d = 0; d < 3; ++d) end[3 * r + d] = w2 * end[3 * q2 + d] + w0 * end[3 * q0 + d];
        }
        if (INIT) {
            state[at(i)] = known ? ST_KNOWN : fill ? ST_REBUILT : ST_MISSING;
            if (!known && !fill) {
                const double nan = __builtin_nan("");
#pragma unroll
                for (int d = 0; d < 3; ++d) end[3 * at(i) + d] = nan;
            }
        } else if (fill) {
            state[at(i)] = ST_REBUILT;
        }
    }
}

// The y and z passes (point stride st, lines indexed by x and the other axis,
// whose stride is s_b): 64 lines per workgroup, one per lane, so a state read
// or a row of rebuilt positions is contiguous over the wavefront.  The
// wavefronts take the line in pieces of 8 entries (16 of them, so that a line
// of 128 is one piece each: a piece's entries are filled one after the other)
// and leave each piece's known entries as a bit mask in LDS; then each finds,
// for its pieces, the nearest known entries outside them from the other
// masks, and fills.
constexpr int PIECE = 8, YZ_BLOCK = 16 * WAVE;
// Fewer lines leave three quarters of the CUs without a workgroup of 64, and each
// wavefront with pieces to fill one after the other.  A rebuild with random
// missing entries (30% / 90%), all passes by a wavefront per line against this:
// 4 x 1000 x 4 28 / 29 us and 60 / 61, 3 x 300 x 300 37 / 35 and 62 / 76,
// 16 x 128 x 128 21 / 22 and 27 / 32, 64^3 15 / 15 and 15 / 19.
constexpr int64_t FEW_LINES = 4096;

__global__ __launch_bounds__(YZ_BLOCK) void recon_yz_kernel(int64_t n_lines, int32_t n_a, int64_t s_b, int32_t len,
                                                            int64_t st, double* end, uint8_t* state) {
#pragma clang fp contract(off)  // Eq. (1) rounded as written: two products, one sum
    __shared__ uint8_t s_mask[MAX_LINE / PIECE][WAVE];
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int64_t line = (int64_t)blockIdx.x * WAVE + lane;
    const bool on = line < n_lines;
    const int64_t l = on ? line : n_lines - 1, base = l % n_a + l / n_a * s_b;
    const int np = (len + PIECE - 1) / PIECE;
    for (int p = wave; p < np; p += YZ_BLOCK / WAVE) {
        uint32_t m = 0u;
#pragma unroll
        for (int b = 0; b < PIECE; ++b) {
            const int i = p * PIECE + b, c = i < len ? i : len - 1;
            const bool known = state[base + (int64_t)c * st] != ST_MISSING;
            m |= i < len && known ? 1u << b : 0u;
        }
        s_mask[p][lane] = (uint8_t)m;
    }
    __syncthreads();
    for (int p = wave; p < np; p += YZ_BLOCK / WAVE) {
        const int n = len - p * PIECE < PIECE ? len - p * PIECE : PIECE;
        const uint32_t m = s_mask[p][lane], miss = on ? ~m & ((1u << n) - 1u) : 0u;
        if (!__any(miss != 0u)) continue;
        int lo = -1, hi_in = -1;
        for (int q = p - 1; q >= 0 && lo < 0; --q)
            if (const uint32_t w = s_mask[q][lane]) lo = q * PIECE + 31 - __clz((int)w);
        for (int q = p + 1; q < np && hi_in < 0; ++q)
            if (const uint32_t w = s_mask[q][lane]) hi_in = q * PIECE + __ffs((int)w) - 1;
        int at = -1;  // the run's upper end in e2 (its lower one in e0)
        double e0[3], e2[3];
#pragma unroll 1
        for (int b = 0; b < n; ++b) {
            const int i = p * PIECE + b;
            if (m >> b & 1u) {
                lo = i;
                continue;
            }
            const uint32_t above = m >> b;
            const int hi = above ? i + __ffs((int)above) - 1 : hi_in;
            if (!on || lo < 0 || hi < 0) continue;
            if (hi != at) {
                at = hi;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    e0[d] = end[3 * (base + (int64_t)lo * st) + d];
                    e2[d] = end[3 * (base + (int64_t)hi * st) + d];
                }
            }
            const double span = (double)(hi - lo);
            const double w2 = (double)(i - lo) / span, w0 = (double)(hi - i) / span;
            const int64_t r = base + (int64_t)i * st;
#pragma unroll
            for (int d = 0; d < 3; ++d) end[3 * r + d] = w2 * e2[d] + w0 * e0[d];
            state[r] = ST_REBUILT;
        }
    }
}

// Eq. (5) partial sums: per workgroup the sum and maximum of |b - m| over the
// entries m keeps (flag valid) and b covers, and the counts of covered and
// uncovered such entries.
struct ErrPart {
    double sum, max;
    unsigned long long n, uncovered;
};

__global__ __launch_bounds__(BLOCK) void err_partial_kernel(int64_t P, const double* b, const uint8_t* bstate,
                                                            const double* m, const uint8_t* mflag, ErrPart* part) {
    double sum = 0.0, mx = 0.0;
    unsigned long long n = 0, unc = 0;
    for (int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x; t < P; t += (int64_t)gridDim.x * BLOCK) {
        if (mflag[t] != (uint8_t)S_VALID) continue;
        if (bstate[t] == ST_MISSING) {
            ++unc;
            continue;
        }
        const double dx = b[3 * t] - m[3 * t], dy = b[3 * t + 1] - m[3 * t + 1], dz = b[3 * t + 2] - m[3 * t + 2];
        const double d = sqrt(dx * dx + dy * dy + dz * dz);
        sum += d;
        mx = fmax(mx, d);
        ++n;
    }
    __shared__ double s_sum[BLOCK], s_max[BLOCK];
    __shared__ unsigned long long s_n[BLOCK], s_u[BLOCK];
    s_sum[threadIdx.x] = sum;
    s_max[threadIdx.x] = mx;
    s_n[threadIdx.x] = n;
    s_u[threadIdx.x] = unc;
    __syncthreads();
    for (int o = BLOCK / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            s_sum[threadIdx.x] += s_sum[threadIdx.x + o];
            s_max[threadIdx.x] = fmax(s_max[threadIdx.x], s_max[threadIdx.x + o]);
            s_n[threadIdx.x] += s_n[threadIdx.x + o];
            s_u[threadIdx.x] += s_u[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = ErrPart{s_sum[0], s_max[0], s_n[0], s_u[0]};
}

// Fixed-order sum of the partials (deterministic for a given grid): each of
// BLOCK threads sums a strided subset in order, then a fixed tree in LDS.
__global__ __launch_bounds__(BLOCK) void err_final_kernel(int nparts, const ErrPart* part, ErrPart* out) {
    double sum = 0.0, mx = 0.0;
    unsigned long long n = 0, unc = 0;
    for (int i = threadIdx.x; i < nparts; i += BLOCK) {
        sum += part[i].sum;
        mx = fmax(mx, part[i].max);
        n += part[i].n;
        unc += part[i].uncovered;
    }
    __shared__ double s_sum[BLOCK], s_max[BLOCK];
    __shared__ unsigned long long s_n[BLOCK], s_u[BLOCK];
    s_sum[threadIdx.x] = sum;
    s_max[threadIdx.x] = mx;
    s_n[threadIdx.x] = n;
    s_u[threadIdx.x] = unc;
    __syncthreads();
    for (int o = BLOCK / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            s_sum[threadIdx.x] += s_sum[threadIdx.x + o];
            s_max[threadIdx.x] = fmax(s_max[threadIdx.x], s_max[threadIdx.x + o]);
            s_n[threadIdx.x] += s_n[threadIdx.x + o];
            s_u[threadIdx.x] += s_u[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = ErrPart{s_sum[0], s_max[0], s_n[0], s_u[0]};
}

// Copy a block's seed-ordered flow map (lattice mb, x fastest) into a larger
// lattice M at lattice offset off, adding `shift` to the positions (block
// coordinates -> domain coordinates).
template <class I>  // uint32_t where the block's entries fit it: a 64-bit division is a subroutine
__global__ __launch_bounds__(BLOCK) void place_kernel(int32_t mb0, int32_t mb1, int64_t Pb, int32_t M0, int32_t M1,
                                                      int32_t o0, int32_t o1, int32_t o2, double sh0, double sh1,
                                                      double sh2, const double* src_xyz, const uint8_t* src_flag,
                                                      double* dst_xyz, uint8_t* dst_flag) {
    for (int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x; t < Pb; t += (int64_t)gridDim.x * BLOCK) {
        const I jk = (I)t / (I)mb0, kk = jk / (I)mb1;
        const int64_t i = (int64_t)((I)t - jk * (I)mb0), j = (int64_t)(jk - kk * (I)mb1), k = (int64_t)kk;
        const int64_t q = (i + o0) + (int64_t)M0 * ((j + o1) + (int64_t)M1 * (k + o2));
        dst_xyz[3 * q] = src_xyz[3 * t] + sh0;
        dst_xyz[3 * q + 1] = src_xyz[3 * t + 1] + sh1;
        dst_xyz[3 * q + 2] = src_xyz[3 * t + 2] + sh2;
        dst_flag[q] = src_flag[t];
    }
}

static int grid_for(int64_t n) {
    const int64_t nb = (n + BLOCK - 1) / BLOCK;
    return (int)(nb < 4096 ? (nb > 0 ? nb : 1) : 4096);
}

hipError_t launch_reconstruct(const int32_t m[3], double* end, const uint8_t* flag, uint8_t* state, hipStream_t s) {
    const int64_t P = (int64_t)m[0] * m[1] * m[2];
    if (m[0] > MAX_LINE || m[1] > MAX_LINE || m[2] > MAX_LINE) return hipErrorInvalidValue;
    // x pass: lines over (y, z).  Lines shorter than half a wavefront leave too
    // many lanes idle to make the states on the way.
    const int64_t xl = (int64_t)m[1] * m[2], xb = (xl * WAVE + BLOCK - 1) / BLOCK;  // one wavefront per line
    if (m[0] >= WAVE / 2) {
        const auto kernel = m[0] <= 2 * WAVE ? recon_line_kernel<true, true, 2>
                                             : recon_line_kernel<true, true, MAX_LINE / WAVE>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)xb), dim3(BLOCK), 0, s, xl, 1, 0, m[0], 1, end, flag, state);
    } else {
        hipLaunchKernelGGL(recon_init_kernel, dim3(grid_for(P)), dim3(BLOCK), 0, s, P, end, flag, state);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (m[0] >= 3)
            hipLaunchKernelGGL((recon_line_kernel<false, true, 2>), dim3((unsigned)xb), dim3(BLOCK), 0, s, xl, 1, 0, m[0],
                               1, end, flag, state);
    }
    hipError_t e = hipGetLastError();
    // y pass: lines over (x, z); z pass: lines over (x, y)
    const int64_t sy = m[0], sz = (int64_t)m[0] * m[1];
    for (int axis = 1; axis < 3 && e == hipSuccess; ++axis) {
        const int64_t lines = axis == 1 ? (int64_t)m[0] * m[2] : (int64_t)m[0] * m[1];
        const int64_t s_b = axis == 1 ? sz : sy, st = axis == 1 ? sy : sz;
        if (m[axis] < 3) continue;
        if (lines < FEW_LINES) {
            const auto kernel = m[axis] <= 2 * WAVE ? recon_line_kernel<false, false, 2>
                                                    : recon_line_kernel<false, false, MAX_LINE / WAVE>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)((lines * WAVE + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, lines,
                               m[0], s_b, m[axis], st, end, flag, state);
        } else {
            hipLaunchKernelGGL(recon_yz_kernel, dim3((unsigned)((lines + WAVE - 1) / WAVE)), dim3(YZ_BLOCK), 0, s, lines,
                               m[0], s_b, m[axis], st, end, state);
        }
        e = hipGetLastError();
    }
    return e;
}

int err_parts_for(int64_t P) { return grid_for(P) < 1024 ? grid_for(P) : 1024; }

constexpr size_t ERR_SET_BYTES = 1024 * sizeof(ErrPart);  // the largest partial-sum grid

size_t err_scratch_bytes(int64_t P) { return sizeof(ErrPart) * (size_t)(err_parts_for(P) + 1); }

static hipError_t sum_error(int64_t P, const double* b, const uint8_t* bstate, const double* m, const uint8_t* mflag,
                            ErrPart* part, ErrPart* out, hipStream_t s) {
    const int parts = err_parts_for(P);
    hipLaunchKernelGGL(err_partial_kernel, dim3(parts), dim3(BLOCK), 0, s, P, b, bstate, m, mflag, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(err_final_kernel, dim3(1), dim3(BLOCK), 0, s, parts, part, out);
    return hipGetLastError();
}

static void error_values(const ErrPart& r, double out4[4]) {
    out4[0] = r.sum;
    out4[1] = r.max;
    out4[2] = (double)r.n;
    out4[3] = (double)r.uncovered;
}

hipError_t launch_flowmap_error(int64_t P, const double* b, const uint8_t* bstate, const double* m, const uint8_t* mflag,
                                void* scratch, double out4[4], hipStream_t s) {
    ErrPart* part = static_cast<ErrPart*>(scratch);
    ErrPart* out = part + err_parts_for(P);
    hipError_t e = sum_error(P, b, bstate, m, mflag, part, out, s);
    if (e != hipSuccess) return e;
    ErrPart r;
    e = hipMemcpyAsync(&r, out, sizeof r, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) error_values(r, out4);
    return e;
}

// Scratch of the accuracy metric kept between calls: a few sets per process,
// each with its partial sums on the GPU that made it and a pinned host record
// that the final kernel writes (no copy back).  A call borrows a set until its
// stream has been waited for, so calls on other threads and streams never
// share one; a call that finds none free allocates its own, as every call did:
// allocating and freeing 33 KB and copying the record back took 30 us beside
// the sums' 22.
constexpr int ERR_SETS = 8;
struct ErrSet {
    int dev;
    bool busy;
    void* part;
    ErrPart* out;
};

struct ErrSets {
    std::mutex mu;
    ErrSet set[ERR_SETS] = {};
    ErrSet* take(int dev) {
        std::lock_guard<std::mutex> lock(mu);
        for (ErrSet& q : set)
            if (q.part && !q.busy && q.dev == dev) {
                q.busy = true;
                return &q;
            }
        for (ErrSet& q : set) {
            if (q.part || q.busy) continue;
            if (hipMalloc(&q.part, ERR_SET_BYTES) != hipSuccess) {
                (void)hipGetLastError();
                q.part = nullptr;
                return nullptr;
            }
            void* host = nullptr;
            if (hipHostMalloc(&host, sizeof(ErrPart), hipHostMallocDefault) != hipSuccess) {
                (void)hipGetLastError();
                (void)hipFree(q.part);
                q.part = nullptr;
                return nullptr;
            }
            q.out = static_cast<ErrPart*>(host);
            q.dev = dev;
            q.busy = true;
            return &q;
        }
        return nullptr;
    }
    void give(ErrSet* q) {
        std::lock_guard<std::mutex> lock(mu);
        q->busy = false;
    }
};

hipError_t flowmap_error(int64_t P, const double* b, const uint8_t* bstate, const double* m, const uint8_t* mflag,
                         double out4[4], hipStream_t s) {
    static ErrSets* sets = new ErrSets;  // lives as long as the process: no call may find it destroyed
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    ErrSet* q = sets->take(dev);
    if (!q) {
        void* scratch = nullptr;
        if (hipMalloc(&scratch, err_scratch_bytes(P)) != hipSuccess) {
            (void)hipGetLastError();
            return hipErrorOutOfMemory;
        }
        e = launch_flowmap_error(P, b, bstate, m, mflag, scratch, out4, s);
        (void)hipFree(scratch);
        return e;
    }
    e = sum_error(P, b, bstate, m, mflag, static_cast<ErrPart*>(q->part), q->out, s);
    const hipError_t w = hipStreamSynchronize(s);  // also after a failed launch: the first may be running
    if (e == hipSuccess) e = w;
    if (e == hipSuccess) error_values(*q->out, out4);
    if (w == hipSuccess) sets->give(q);  // a stream in error may still write: the set stays out
    return e;
}

// Fixed device scratch of the allocation-free accuracy metric: room for the
// largest partial-sum grid (1,024 workgroups) plus the final record, which
// covers every entry count.  Each GPU holds its own copy at its own address,
// found once per device with hipGetSymbolAddress; host code uses only that
// address (the array's name on the host is a stand-in, not device memory).
// Every call on one GPU shares the array: calls that overlap on one GPU race.
constexpr size_t ERR_STATIC_BYTES = 1025 * sizeof(ErrPart);
static __device__ __align__(256) char scratch[ERR_STATIC_BYTES];
constexpr int ERR_STATIC_MAX_DEVICES = 64;

hipError_t err_static_scratch(void** ptr, size_t* bytes) {
    static std::mutex mu;
    static void* addr[ERR_STATIC_MAX_DEVICES] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= ERR_STATIC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = ERR_STATIC_BYTES;
    return hipSuccess;
}

hipError_t launch_place(const int32_t mb[3], const int32_t M[3], const int32_t off[3], const double shift[3],
                        const double* src_xyz, const uint8_t* src_flag, double* dst_xyz, uint8_t* dst_flag,
                        hipStream_t s) {
    const int64_t Pb = (int64_t)mb[0] * mb[1] * mb[2];
    const auto kernel = Pb <= (int64_t)0xFFFFFFFF ? place_kernel<uint32_t> : place_kernel<uint64_t>;
    hipLaunchKernelGGL(kernel, dim3(grid_for(Pb)), dim3(BLOCK), 0, s, mb[0], mb[1], Pb, M[0], M[1], off[0], off[1],
                       off[2], shift[0], shift[1], shift[2], src_xyz, src_flag, dst_xyz, dst_flag);
    return hipGetLastError();
}

}  // namespace bto
