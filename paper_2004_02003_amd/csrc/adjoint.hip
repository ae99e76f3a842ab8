// Discrete adjoint of the per-block RK4 advection (gradients of end positions
// with respect to seed positions and velocity grids), with checkpointing, and
// the FTLE of flow-map Jacobians.
//
// A reverse step needs the cell and the offsets of each of the step's four
// stages, which only the step itself tells.  They are put on a tape (64 bytes
// per step and seed), in one of two ways:
//   * forward   one lane per seed steps through the whole interval from its
//               position, as the advection does, and writes the tape of every
//               step; where the tape would pass its budget, FP64 checkpoints
//               every `k` steps instead;
//   * recompute one lane per seed and checkpoint segment steps through the
//               segment from its checkpoint (the forward's, or recorded by the
//               advection; then the per-seed records say which seeds stayed
//               inside for the whole interval).  Segments do not depend on
//               each other, so as many as the tape holds run at once.
// The reverse sweep then walks the tape backwards, one lane per seed: with
// every stage's cell known beforehand, all the step's corner values load
// together and a step ahead, the sampler gradients G_s follow (on the cell
// chosen by the floor/clamp rule), and the transposed stage recurrences are
// applied to every cotangent vector.
// Grid gradients leave as records for the sorted, deterministic reduction
// (grad_reduce.hip), or as FP32 atomics when no record buffer is given (their
// summation order is then not fixed).  Terminated and invalid seeds contribute
// nothing (the loss covers only the basis flows that stay inside the block).
//
// What bounds the sweeps at a few tens of thousands of seeds (three wavefronts
// per CU) is the CU's L1: it keeps about 64 lines in flight, whatever the
// wavefronts ask for.  So the reverse sweep asks for each line once: a lane
// loads a stage's cell only where it differs from the neighbouring stage's, and
// level n + 1 is kept from the step before; loading all six cells of a step
// took 316 us instead of 231 (gradient of 32,768 seeds over 50 steps, 128^3 ABC,
// f32; 372 without the loads a step ahead) and 330 instead of 220 (three
// cotangents of 48,960 seeds over 49 steps, 160 x 144 x 136 f16 turbulence).
// The recompute of five segments takes 174 us in the first, the forward 264 in
// the second.  One sweep that recomputed and reversed one segment after the
// other, each step in dependent loads, took 541 and 935 us in all.
//
// The Jacobian of a recomputed interval, and the seed gradients of many seeds
// over a few steps at a time, need no reverse sweep at all: see
// adj_tangent_kernel and adj_segments_kernel.
#include "bto_internal.h"

namespace bto {

__device__ __forceinline__ void gT(const float G[3][3], const float v[3], float out[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) out[d] = G[0][d] * v[0] + G[1][d] * v[1] + G[2][d] * v[2];
}


// Grid-gradient accumulator: the 8 corner gradients of one cell of one grid
// level, summed in registers while consecutive stage contributions hit the
// same cell and level, and flushed only when the cell or level changes (and at
// the end of each call; between the launches of a call it is kept in memory, so
// that the sums do not depend on how many the tape needs).  In the reverse sweep a level receives
// its contributions from two consecutive steps (level n from step n's first
// three stages and from step n-1's last three), so a particle that stays in
// its cell flushes once per level.  A flush appends a record for the sorted,
// deterministic reduction (or, without records or when they are full, adds the
// values to the grid with FP32 atomics).
struct GradAcc {
    uint32_t val;   // cell (first value's index; NO_CELL: none)
    int level;
    uint32_t nrec;  // records written by this seed (per_seed + 1: and then flushes added with atomics)
    float v[8][3];
};

// The accumulator of seed p between two launches: words 1 .. 26 of its ACC_WORDS
// (word 0: nrec), a word of all P seeds side by side.
__device__ __forceinline__ void acc_load(const uint32_t* w, int64_t P, int64_t p, GradAcc& A) {
    A.val = w[P + p];
    A.level = (int)w[2 * P + p];
#pragma unroll
    for (int j = 0; j < 24; ++j) A.v[j / 3][j % 3] = __uint_as_float(w[(3 + j) * P + p]);
}

__device__ __forceinline__ void acc_store(uint32_t* w, int64_t P, int64_t p, const GradAcc& A) {
    w[P + p] = A.val;
    w[2 * P + p] = (uint32_t)A.level;
#pragma unroll
    for (int j = 0; j < 24; ++j) w[(3 + j) * P + p] = __float_as_uint(A.v[j / 3][j % 3]);
}

__device__ __forceinline__ void put_key(const GradRec& R, uint64_t slot, uint64_t key) {
    if (R.key_bytes == 4) static_cast<uint32_t*>(R.key)[slot] = (uint32_t)key;
    else static_cast<uint64_t*>(R.key)[slot] = key;
}

__device__ __forceinline__ void acc_flush(const Geom& g, float* const* gf, const GradRec& R, uint32_t pid,
                                          GradAcc& A) {
    if (A.val == NO_CELL) return;
    if (R.key && A.nrec < R.per_seed) {
        // the seed's next record slot: no counter, and the lanes of a wavefront
        // that flush together write neighbouring slots
        const uint64_t slot = (uint64_t)(A.nrec++) * R.P + pid;
        const uint32_t base = A.val / 3u;
        const uint32_t i = base % g.sy, j = (base / g.sy) % (uint32_t)g.n[1], k = base / g.sz;
        const uint64_t colour = (uint64_t)((i & 1u) | ((j & 1u) << 1) | ((k & 1u) << 2));
        const uint64_t key = (colour << (R.level_bits + R.cell_bits)) | ((uint64_t)A.level << R.cell_bits) |
                             (uint64_t)base;
        put_key(R, slot, key);
        float4* out = reinterpret_cast<float4*>(R.val + 24 * (size_t)slot);
#pragma unroll
        for (int q = 0; q < 6; ++q)
            out[q] = make_float4(A.v[(4 * q) / 3][(4 * q) % 3], A.v[(4 * q + 1) / 3][(4 * q + 1) % 3],
                                 A.v[(4 * q + 2) / 3][(4 * q + 2) % 3], A.v[(4 * q + 3) / 3][(4 * q + 3) % 3]);
        A.val = NO_CELL;
        return;
    }
    if (R.key) A.nrec = R.per_seed + 1u;
    float* grid = in_global(gf[A.level]) + A.val;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float* p = grid + (size_t)(3u * q + g.sy3 * b + g.sz3 * c);
                const int k = q + 2 * b + 4 * c;
                unsafeAtomicAdd(p + 0, A.v[k][0]);
                unsafeAtomicAdd(p + 1, A.v[k][1]);
                unsafeAtomicAdd(p + 2, A.v[k][2]);
            }
    A.val = NO_CELL;
}

__device__ __forceinline__ void acc_add(const Geom& g, float* const* gf, const GradRec& R, uint32_t pid, GradAcc& A,
                                        int level, const TapeEntry& t, float coef, const float lam[3]) {
    if (A.val != t.val || A.level != level) {
        acc_flush(g, gf, R, pid, A);
        A.val = t.val;
        A.level = level;
#pragma unroll
        for (int k = 0; k < 8; ++k) A.v[k][0] = A.v[k][1] = A.v[k][2] = 0.f;
    }
    const float wx[2] = {1.f - t.f[0], t.f[0]}, wy[2] = {1.f - t.f[1], t.f[1]}, wz[2] = {1.f - t.f[2], t.f[2]};
    const float l[3] = {(float)g.inv_sp[0] * lam[0] * coef, (float)g.inv_sp[1] * lam[1] * coef,
                        (float)g.inv_sp[2] * lam[2] * coef};
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float w = wx[q] * wy[b] * wz[c];
                const int k = q + 2 * b + 4 * c;
                A.v[k][0] = fmaf(w, l[0], A.v[k][0]);
                A.v[k][1] = fmaf(w, l[1], A.v[k][1]);
                A.v[k][2] = fmaf(w, l[2], A.v[k][2]);
            }
}

// One wavefront per workgroup: a seed set of a few tens of thousands fills
// only a fraction of the SIMDs; single-wavefront workgroups spread those
// wavefronts over every CU (and its L1 and texture pipeline) instead of
// packing four of them onto each of the first P/256 CUs.
constexpr int ADJ_BLOCK = WAVE;

// Steps n0 .. n1 - 1 from x, the advection's own step.  hook.begin(n, h, x)
// before step n; hook.stage(n, s, c) with the cell and the offsets stage s
// samples; hook.sample(s, c, A, B) with its corner values; hook.end() after a
// step that stayed inside.  Returns the status of the step that ended it, or
// S_VALID.
template <int DT, int MODE, class Hook>
__device__ __forceinline__ int adj_steps(const AdjointArgs& a, double* x, int n0, int n1, Hook& hook) {
    GatherCache<DT> A, B;
    forget(A);
    forget(B);
    int status = S_VALID;
    const auto step = [&](int n, GatherCache<DT>& LA, GatherCache<DT>& LB) {
        const double h = scalar_load(a.h + (n - a.f_base));
        hook.begin(n, h, x);
        StepSizes hs = step_sizes(a.g, h);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            hs.full[d] = uniform(hs.full[d]);
            hs.half[d] = uniform(hs.half[d]);
            hs.sixth[d] = uniform(hs.sixth[d]);
        }
        status = rk4_step_gather<DT, MODE>(a.g, in_global(scalar_load(a.f + (n - a.f_base))),
                                           in_global(scalar_load(a.f + (n + 1 - a.f_base))), hs, x, LA, LB, false,
                                           [](const double*) {},
                                           [&](int s, const GatherCell<float>& c) { hook.stage(n, s, c); },
                                           [&](int s, const GatherCell<float>& c) { hook.sample(s, c, LA, LB); });
        if (status == S_VALID) hook.end();
        forget(LA);  // receives level n + 2
        if (is_frozen<MODE>) forget(LB);
    };
    for (int n = n0; n < n1; ++n) {
        step(n, A, B);
        if (status != S_VALID || ++n >= n1) break;
        step(n, B, A);
        if (status != S_VALID) break;
    }
    return status;
}

// The tape of steps n0 on at t (null: none), checkpoints every a.k steps at ck
// (null: none).
struct TapeHook {
    const AdjointArgs& a;
    TapeEntry* t;
    double* ck;
    int n0;
    __device__ __forceinline__ void begin(int n, double, const double* x) const {
        if (!ck || n % a.k != 0) return;
        double* c = ck + a.ck_stride * (int64_t)(n / a.k);
#pragma unroll
        for (int d = 0; d < 3; ++d) c[d] = x[d];
    }
    __device__ __forceinline__ void stage(int n, int s, const GatherCell<float>& c) const {
        if (!t) return;
        const U4 e = {c.val, __float_as_uint(c.f[0]), __float_as_uint(c.f[1]), __float_as_uint(c.f[2])};
        *reinterpret_cast<U4*>(t + a.np * (int64_t)(4 * (n - n0) + s)) = e;
    }
    template <class C>
    __device__ __forceinline__ void sample(int, const GatherCell<float>&, const C&, const C&) const {}
    __device__ __forceinline__ void end() const {}
};

// The tangent T = d x_n / d x_0 (cell units) carried along the steps: dk_s =
// G_s dy_s with the stage points' derivatives dy_s, as the step combines the
// stage velocities.  DEV: T and the stage points' derivatives without their unit
// matrix, whose ones would round what a few steps add to them.
template <int MODE, bool DEV = false>
struct TangentHook {
    const Geom& g;
    float T[3][3], Y[3][3], S[3][3], h;
    __device__ __forceinline__ void begin(int, double hd, const double*) {
        h = (float)hd;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) Y[r][c] = T[r][c];
    }
    __device__ __forceinline__ void stage(int, int, const GatherCell<float>&) const {}
    template <class C>
    __device__ __forceinline__ void sample(int s, const GatherCell<float>& c, const C& A, const C& B) {
        constexpr bool lin = !is_frozen<MODE>;
        float unused[3], D[3][3];
        if (lin && (s == 1 || s == 2)) trilerp_grad<lin>(A.rows(g), B.rows(g), c.f, unused, D);
        else if (lin && s == 3) trilerp_grad<false>(B.rows(g), B.rows(g), c.f, unused, D);
        else trilerp_grad<false>(A.rows(g), A.rows(g), c.f, unused, D);
        const float w = s == 0 || s == 3 ? 1.f : 2.f, next = s < 2 ? 0.5f * h : h;
        float K[3][3];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float v = D[r][0] * Y[0][k] + D[r][1] * Y[1][k] + D[r][2] * Y[2][k];
                if constexpr (DEV) v += D[r][k];
                K[r][k] = (float)g.inv_sp[r] * v;
            }
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                S[r][k] = s == 0 ? K[r][k] : S[r][k] + w * K[r][k];
                Y[r][k] = T[r][k] + next * K[r][k];
            }
    }
    __device__ __forceinline__ void end() {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) T[r][c] = T[r][c] + (h / 6.f) * S[r][c];
    }
};

// Three cotangents of the adjoint's own forward, without grid gradients (the
// flow-map Jacobian): the tangent along the forward sweep instead of a tape and
// a reverse sweep, whose loads it does without: 300 us where the two sweeps take
// 264 and 220 (48,960 seeds, 49 steps, 160 x 144 x 136 f16 turbulence); the
// derivatives alone cost the forward sweep 36.  With grid gradients, or from
// checkpoints whose segments recompute in parallel, the reverse sweep stays.
template <int DT, int MODE>
__global__ __launch_bounds__(ADJ_BLOCK) void adj_tangent_kernel(const AdjointArgs a) {
    const int64_t p = (int64_t)blockIdx.x * ADJ_BLOCK + threadIdx.x;
    if (p >= a.P) return;
    double x[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = (a.seed_xyz[3 * p + d] - a.origin[d]) * a.g.inv_sp[d];
    TangentHook<MODE> hook{a.g, {{1.f, 0.f, 0.f}, {0.f, 1.f, 0.f}, {0.f, 0.f, 1.f}}, {}, {}, 0.f};
    int status = S_TERMINATED;
    if (inside(a.g, x)) status = adj_steps<DT, MODE>(a, x, 0, a.N, hook);
    if (a.status_out) a.status_out[p] = (uint8_t)status;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        float l[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) l[r] = status == S_VALID ? a.cot[9 * p + 3 * m + r] * (float)a.sp[r] : 0.f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float v = hook.T[0][d] * l[0] + hook.T[1][d] * l[1] + hook.T[2][d] * l[2];
            a.grad_seed[9 * p + 3 * m + d] = status == S_VALID ? v * (float)a.g.inv_sp[d] : 0.f;
        }
    }
}

template <int DT, int MODE>
__global__ __launch_bounds__(ADJ_BLOCK) void adj_forward_kernel(const AdjointArgs a) {
    const int64_t q = (int64_t)blockIdx.x * ADJ_BLOCK + threadIdx.x, p = a.p0 + q;
    if (q >= a.np) return;
    double x[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = (a.seed_xyz[3 * p + d] - a.origin[d]) * a.g.inv_sp[d];
    int status = S_TERMINATED;
    const TapeHook hook{a, a.tape ? a.tape + q : nullptr, a.ckpt ? a.ckpt + 3 * p : nullptr, 0};
    if (inside(a.g, x)) status = adj_steps<DT, MODE>(a, x, 0, a.N, hook);
    a.status[p] = (uint8_t)status;
    a.bad[p] = 0;
}

__device__ __forceinline__ int forward_status(const AdjointArgs& a, int64_t p) {
    if (!a.rec_meta) return (int)a.status[p];
    const int32_t meta = a.rec_meta[p];
    return meta == META_LIVE ? S_VALID : (int)((uint32_t)meta >> META_SHIFT);
}

// Few steps at a time, no grid gradients, many seeds (see SHORT_SEEDS): segment
// by segment from the last one of the call, the tangent along the segment's
// steps from its recorded checkpoint and the cotangents through its transpose; a
// recomputed step that does not stay inside drops the seed, as in
// adj_recompute_kernel.  Without a record (rec_meta null): one segment, the whole
// interval from the seeds, whose status is the one found here.
template <int DT, int MODE>
__global__ __launch_bounds__(ADJ_BLOCK) void adj_segments_kernel(const AdjointArgs a) {
    const int64_t p = (int64_t)blockIdx.x * ADJ_BLOCK + threadIdx.x;
    if (p >= a.P) return;
    const int nseg = (a.N + a.k - 1) / a.k;
    const bool own = !a.rec_meta, first = a.sg_first == nseg - 1, last = a.sg_last == 0;
    int status = own ? S_VALID : forward_status(a, p);
    const int prior = !first ? (int)a.drop[p] : 0;
    const bool on = status == S_VALID && !prior;
    float lam[3][3];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float* src = first ? a.cot : a.lam;
            lam[m][d] = on && m < a.ncot ? src[(p * a.ncot + m) * 3 + d] * (first ? (float)a.sp[d] : 1.f) : 0.f;
        }
    bool left = false;
    if (on) {
        for (int sg = a.sg_first; sg >= a.sg_last; --sg) {
            const int n0 = sg * a.k, n1 = n0 + a.k < a.N ? n0 + a.k : a.N;
            double x[3];
#pragma unroll
            for (int d = 0; d < 3; ++d)
                x[d] = own ? (a.seed_xyz[3 * p + d] - a.origin[d]) * a.g.inv_sp[d]
                           : a.ckpt[a.ck_stride * (int64_t)sg + 3 * p + d];
            TangentHook<MODE, true> hook{a.g, {}, {}, {}, 0.f};
            int st = S_TERMINATED;
            if (inside(a.g, x)) st = adj_steps<DT, MODE>(a, x, n0, n1, hook);
            if (st != S_VALID) {
                if (own) status = st;
                left = true;
                break;
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                float l[3];
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    l[d] = lam[m][d] + (hook.T[0][d] * lam[m][0] + hook.T[1][d] * lam[m][1] + hook.T[2][d] * lam[m][2]);
#pragma unroll
                for (int d = 0; d < 3; ++d) lam[m][d] = l[d];
            }
        }
    }
    const int drop = left && !own ? ADJ_DROPPED : prior;
    if (first || drop != prior) a.drop[p] = (uint8_t)drop;
    if (last && a.status_out) a.status_out[p] = (uint8_t)(drop ? drop : status);
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int d = 0; d < 3; ++d)
            if (m < a.ncot)
                (last ? a.grad_seed : a.lam)[(p * a.ncot + m) * 3 + d] =
                    left ? 0.f : lam[m][d] * (last ? (float)a.g.inv_sp[d] : 1.f);
}

// Workgroup row y: segment sg_last + y.  A recomputed step that does not stay
// inside contradicts the forward that called the seed valid: possible only
// when the forward was taken by the advection with other rounding (recorded
// checkpoints; launches cut inside a checkpoint segment, two lanes per
// particle, the tile layout).  Such a seed is marked bad.
template <int DT, int MODE>
__global__ __launch_bounds__(ADJ_BLOCK) void adj_recompute_kernel(const AdjointArgs a) {
    const int64_t q = (int64_t)blockIdx.x * ADJ_BLOCK + threadIdx.x, p = a.p0 + q;
    if (q >= a.np || forward_status(a, p) != S_VALID) return;
    const int sg = a.sg_last + (int)blockIdx.y, n0 = sg * a.k, n1 = n0 + a.k < a.N ? n0 + a.k : a.N;
    double x[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = a.ckpt[a.ck_stride * (int64_t)sg + 3 * p + d];
    const TapeHook hook{a, a.tape + 4 * a.np * (int64_t)(n0 - a.sg_last * a.k) + q, nullptr, n0};
    if (adj_steps<DT, MODE>(a, x, n0, n1, hook) != S_VALID) a.bad[p] = 1;
}

template <int DT, int MODE, int NCOT>
__global__ __launch_bounds__(ADJ_BLOCK) void adj_reverse_kernel(const AdjointArgs a) {
    constexpr bool W = is_wide<MODE>;
    const int64_t q = (int64_t)blockIdx.x * ADJ_BLOCK + threadIdx.x, p = a.p0 + q;
    if (q >= a.np) return;
    const int nseg = (a.N + a.k - 1) / a.k;
    const int n_lo = a.sg_last * a.k, n_hi = (a.sg_first + 1) * a.k < a.N ? (a.sg_first + 1) * a.k : a.N;
    const bool first = a.sg_first == nseg - 1, last = a.sg_last == 0;
    const int status = forward_status(a, p);
    // a seed dropped by an earlier launch of the interval stays dropped
    const int prior = a.drop && !first ? (int)a.drop[p] : 0;
    const bool bad = status == S_VALID && !prior && a.bad[p];
    const bool on = status == S_VALID && !prior && !bad;

    float lam[NCOT][3];
#pragma unroll
    for (int c = 0; c < NCOT; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float* src = first ? a.cot : a.lam;
            lam[c][d] = on ? src[(p * NCOT + c) * 3 + d] * (first ? (float)a.sp[d] : 1.f) : 0.f;
        }

    GradAcc acc;
    acc.val = NO_CELL;
    acc.level = -1;
    acc.nrec = 0u;
    // what the call's launch before this one left, and what this one leaves
    const bool resumes = a.carry && a.sg_first != a.call_first, leaves = a.carry && a.sg_last != a.call_last;
    if (resumes) acc.nrec = a.carry[p];
    if (on) {
        if (resumes && a.carry_acc) acc_load(a.carry, a.P, p, acc);
        const TapeEntry* t = a.tape + q;
        const auto read = [&](int n, TapeEntry* e) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const U4 w = *reinterpret_cast<const U4*>(t + a.np * (int64_t)(4 * (n - n_lo) + s));
                e[s] = TapeEntry{w.x, {__uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)}};
            }
        };
        // A step's corner values: stage 1's cell on level n (S0); stages 2 and 3
        // on levels n and n + 1, stage 4 on level n + 1, each only by the lanes
        // whose cell there differs from the one it is taken from otherwise (the
        // stage before it; on level n + 1 the stage after it, and for stage 4
        // stage 1 of the step n + 1, still held in P).
        GatherCache<DT> S0, A1, A2, B1, B2, B3, P;
        const auto corners = [&](const char* V0, const char* V1, const TapeEntry* c) {
            S0.template load<W>(a.g, V0, c[0].val);
            if (c[1].val != c[0].val) A1.template load<W>(a.g, V0, c[1].val);
            if (c[2].val != c[1].val) A2.template load<W>(a.g, V0, c[2].val);
            if constexpr (is_frozen<MODE>) {
                if (c[3].val != c[2].val) B3.template load<W>(a.g, V0, c[3].val);
            } else {
                if (c[3].val != P.val) B3.template load<W>(a.g, V1, c[3].val);
                if (c[2].val != c[3].val) B2.template load<W>(a.g, V1, c[2].val);
                if (c[1].val != c[2].val) B1.template load<W>(a.g, V1, c[1].val);
            }
        };
        P.val = NO_CELL;
        const auto grid = [&](int n) { return in_global(scalar_load(a.f + (n - a.f_base))); };
        TapeEntry c[4], e[4];
        read(n_hi - 1, c);
        const char* V0 = grid(n_hi - 1);
        double hd = scalar_load(a.h + (n_hi - 1 - a.f_base));
        corners(V0, grid(n_hi), c);
        read(n_hi - 1 > n_lo ? n_hi - 2 : n_lo, e);
        for (int n = n_hi - 1; n >= n_lo; --n) {
            const float h = (float)hd;
            float G[4][3][3];
            const auto grad = [&](int s, const GatherCache<DT>& A, const GatherCache<DT>& B, auto mid) {
                float unused[3], D[3][3];
                trilerp_grad<decltype(mid)::value>(A.rows(a.g), B.rows(a.g), c[s].f, unused, D);
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int d = 0; d < 3; ++d) G[s][r][d] = (float)a.g.inv_sp[r] * D[r][d];
            };
            constexpr std::integral_constant<bool, !is_frozen<MODE>> mid{};
            A1.take(S0, c[1].val);
            A2.take(A1, c[2].val);
            if constexpr (is_frozen<MODE>) {
                B3.take(A2, c[3].val);
            } else {
                B3.take(P, c[3].val);
                B2.take(B3, c[2].val);
                B1.take(B2, c[1].val);
            }
            grad(3, B3, B3, std::false_type{});
            grad(2, A2, is_frozen<MODE> ? A2 : B2, mid);
            grad(1, A1, is_frozen<MODE> ? A1 : B1, mid);
            grad(0, S0, S0, std::false_type{});
            P = S0;
            // the step below: its corner values and the entries of the one after it
            // load while this step's recurrences and sums run
            const int m1 = n - 1 > n_lo ? n - 1 : n_lo, m2 = n - 2 > n_lo ? n - 2 : n_lo;
            const char* Vm = grid(m1);
            hd = scalar_load(a.h + (m1 - a.f_base));
            corners(Vm, V0, e);
            V0 = Vm;
            TapeEntry e2[4];
            read(m2, e2);
            const int lv = n - a.f_base;  // grid level of cycle n in the gradient grids
#pragma unroll
            for (int m = 0; m < NCOT; ++m) {
                float lk[4][3], ly[4][3];
#pragma unroll
                for (int d = 0; d < 3; ++d) lk[3][d] = (h / 6.f) * lam[m][d];
                gT(G[3], lk[3], ly[3]);
#pragma unroll
                for (int d = 0; d < 3; ++d) lk[2][d] = (h / 3.f) * lam[m][d] + h * ly[3][d];
                gT(G[2], lk[2], ly[2]);
#pragma unroll
                for (int d = 0; d < 3; ++d) lk[1][d] = (h / 3.f) * lam[m][d] + (0.5f * h) * ly[2][d];
                gT(G[1], lk[1], ly[1]);
#pragma unroll
                for (int d = 0; d < 3; ++d) lk[0][d] = (h / 6.f) * lam[m][d] + (0.5f * h) * ly[1][d];
                gT(G[0], lk[0], ly[0]);
                if (m == 0 && a.grad_f) {
                    const auto add = [&](int level, int s, float coef) {
                        acc_add(a.g, a.grad_f, a.grec, (uint32_t)p, acc, level, c[s], coef, lk[s]);
                    };
                    if (is_frozen<MODE>) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) add(lv, s, 1.f);
                    } else {
                        // level n+1 first (it already holds step n+1's share), then level n
                        add(lv + 1, 1, 0.5f);
                        add(lv + 1, 2, 0.5f);
                        add(lv + 1, 3, 1.f);
                        add(lv, 0, 1.f);
                        add(lv, 1, 0.5f);
                        add(lv, 2, 0.5f);
                    }
                }
#pragma unroll
                for (int d = 0; d < 3; ++d) lam[m][d] += ly[0][d] + ly[1][d] + ly[2][d] + ly[3][d];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                c[s] = e[s];
                e[s] = e2[s];
            }
        }
        if (leaves && a.carry_acc) acc_store(a.carry, a.P, p, acc);
        else if (a.grad_f) acc_flush(a.g, a.grad_f, a.grec, (uint32_t)p, acc);
    }
    int drop = prior;
    if (bad) {
        // no gradient from this seed: this call's grid records are withdrawn;
        // contributions already in the grids (added with atomics after its
        // record slots ran out, or by the call of a later segment) cannot be,
        // and the status says so
        bool withdrawn = true;
        if (a.grad_f) {
            if (a.grec.key) {
                const uint32_t kept = acc.nrec < a.grec.per_seed ? acc.nrec : a.grec.per_seed;
                const uint64_t unused = 1ull << (a.grec.level_bits + a.grec.cell_bits + 3);
                for (uint32_t j = 0; j < kept; ++j) put_key(a.grec, (uint64_t)j * a.grec.P + (uint64_t)p, unused);
                withdrawn = acc.nrec <= a.grec.per_seed;
            } else {
                withdrawn = a.sg_first == a.call_first;
            }
            withdrawn = withdrawn && a.call_first == nseg - 1;
        }
        drop = withdrawn ? ADJ_DROPPED : ADJ_DROPPED_PARTIAL;
    }
    if (a.drop && (first || drop != prior)) a.drop[p] = (uint8_t)drop;
    if (leaves) a.carry[p] = acc.nrec;
    if (last) {
        if (a.status_out) a.status_out[p] = (uint8_t)(drop ? drop : status);
#pragma unroll
        for (int c = 0; c < NCOT; ++c)
#pragma unroll
            for (int d = 0; d < 3; ++d) a.grad_seed[(p * NCOT + c) * 3 + d] = lam[c][d] * (float)a.g.inv_sp[d];
    } else {
#pragma unroll
        for (int c = 0; c < NCOT; ++c)
#pragma unroll
            for (int d = 0; d < 3; ++d) a.lam[(p * NCOT + c) * 3 + d] = lam[c][d];
    }
}

struct Words {
    uint64_t v[240];
};

__global__ void put_words_kernel(uint64_t* dst, const Words w, int n) {
    if ((int)threadIdx.x < n) dst[threadIdx.x] = w.v[threadIdx.x];
}

// ---------------------------------------------------------------------------
// FTLE: sigma = ln sqrt(lambda_max(J^T J)) / |T| per seed, from row-major
// Jacobians (3x3 FP32).  The largest eigenvalue of the symmetric 3x3 matrix
// C = J^T J comes from the closed-form trigonometric solution of its
// characteristic cubic, evaluated in FP64.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void ftle_kernel(const float* jac, int64_t P, double inv_T, float* out) {
    const int64_t p = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (p >= P) return;
    double J[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) J[r][c] = (double)jac[9 * p + 3 * r + c];
    double C[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) C[i][j] = J[0][i] * J[0][j] + J[1][i] * J[1][j] + J[2][i] * J[2][j];
    const double p1 = C[0][1] * C[0][1] + C[0][2] * C[0][2] + C[1][2] * C[1][2];
    const double q = (C[0][0] + C[1][1] + C[2][2]) / 3.0;
    const double p2 = (C[0][0] - q) * (C[0][0] - q) + (C[1][1] - q) * (C[1][1] - q) + (C[2][2] - q) * (C[2][2] - q) +
                      2.0 * p1;
    double lmax;
    if (p2 <= 0.0) {
        lmax = q;
    } else {
        const double pp = sqrt(p2 / 6.0);
        double B[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) B[i][j] = (C[i][j] - (i == j ? q : 0.0)) / pp;
        double detB = B[0][0] * (B[1][1] * B[2][2] - B[1][2] * B[2][1]) -
                      B[0][1] * (B[1][0] * B[2][2] - B[1][2] * B[2][0]) +
                      B[0][2] * (B[1][0] * B[2][1] - B[1][1] * B[2][0]);
        double r = detB / 2.0;
        r = r < -1.0 ? -1.0 : (r > 1.0 ? 1.0 : r);
        const double phi = acos(r) / 3.0;
        lmax = q + 2.0 * pp * cos(phi);
    }
    out[p] = (float)(0.5 * log(lmax) * inv_T);
}

// ---------------------------------------------------------------------------
template <class F>
static hipError_t adj_dispatch(int dtype, int mode, F&& f) {
    auto by_mode = [&](auto dt) {
        switch (mode) {
        case MODE_LINEAR: return f(dt, std::integral_constant<int, MODE_LINEAR>{});
        case MODE_FROZEN: return f(dt, std::integral_constant<int, MODE_FROZEN>{});
        case MODE_LINEAR | MODE_WIDE: return f(dt, std::integral_constant<int, MODE_LINEAR | MODE_WIDE>{});
        default: return f(dt, std::integral_constant<int, MODE_FROZEN | MODE_WIDE>{});
        }
    };
    switch (dtype) {
    case DT_F32: return by_mode(std::integral_constant<int, DT_F32>{});
    case DT_F16: return by_mode(std::integral_constant<int, DT_F16>{});
    default: return by_mode(std::integral_constant<int, DT_BF16>{});
    }
}

static unsigned adj_blocks(const AdjointArgs& a) { return (unsigned)((a.np + ADJ_BLOCK - 1) / ADJ_BLOCK); }

hipError_t launch_adj_forward(const AdjointArgs& a, int dtype, int mode, hipStream_t s) {
    return adj_dispatch(dtype, mode, [&](auto dt, auto md) {
        hipLaunchKernelGGL((adj_forward_kernel<decltype(dt)::value, decltype(md)::value>), dim3(adj_blocks(a)),
                           dim3(ADJ_BLOCK), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_adj_tangent(const AdjointArgs& a, int dtype, int mode, hipStream_t s) {
    return adj_dispatch(dtype, mode, [&](auto dt, auto md) {
        hipLaunchKernelGGL((adj_tangent_kernel<decltype(dt)::value, decltype(md)::value>), dim3(adj_blocks(a)),
                           dim3(ADJ_BLOCK), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_adj_segments(const AdjointArgs& a, int dtype, int mode, hipStream_t s) {
    return adj_dispatch(dtype, mode, [&](auto dt, auto md) {
        hipLaunchKernelGGL((adj_segments_kernel<decltype(dt)::value, decltype(md)::value>), dim3(adj_blocks(a)),
                           dim3(ADJ_BLOCK), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_adj_recompute(const AdjointArgs& a, int dtype, int mode, hipStream_t s) {
    return adj_dispatch(dtype, mode, [&](auto dt, auto md) {
        hipLaunchKernelGGL((adj_recompute_kernel<decltype(dt)::value, decltype(md)::value>),
                           dim3(adj_blocks(a), (unsigned)(a.sg_first - a.sg_last + 1)), dim3(ADJ_BLOCK), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_adj_reverse(const AdjointArgs& a, int dtype, int mode, hipStream_t s) {
    return adj_dispatch(dtype, mode, [&](auto dt, auto md) {
        if (a.ncot == 1)
            hipLaunchKernelGGL((adj_reverse_kernel<decltype(dt)::value, decltype(md)::value, 1>), dim3(adj_blocks(a)),
                               dim3(ADJ_BLOCK), 0, s, a);
        else
            hipLaunchKernelGGL((adj_reverse_kernel<decltype(dt)::value, decltype(md)::value, 3>), dim3(adj_blocks(a)),
                               dim3(ADJ_BLOCK), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_put_words(uint64_t* dst, const uint64_t* src, size_t n, hipStream_t s) {
    constexpr size_t M = sizeof(Words) / sizeof(uint64_t);
    for (size_t k = 0; k < n; k += M) {
        Words w;
        const int m = (int)(n - k < M ? n - k : M);
        for (int i = 0; i < m; ++i) w.v[i] = src[k + i];
        hipLaunchKernelGGL(put_words_kernel, dim3(1), dim3(256), 0, s, dst + k, w, m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_ftle(const float* jac, int64_t P, double inv_T, float* out, hipStream_t s) {
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(ftle_kernel, dim3((unsigned)((P + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, jac, P, inv_T, out);
    return hipGetLastError();
}

}  // namespace bto
