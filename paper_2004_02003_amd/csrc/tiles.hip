// Tile layout of the live particles: the in situ step in tile order.
//
// Live particles are kept in buckets, one per tile of cells (a particle
// belongs to the tile of its sampling cell); tiles run along a Hilbert curve
// in cell space, one eighth of the curve per XCD, so neighbouring tiles run
// close in time on one XCD and share the grid lines of their common faces in
// its L2.  A step is
//   tile_gather_kernel  one workgroup per tile: advance every particle of the
//   (tiles = 2)         tile one RK4 step, gathering the grid values, and
//                       write each survivor into the bucket of the tile it
//                       ends in (next step's buffers); the workgroups behind
//                       the tiles' do the same for the list of particles that
//                       did not fit their bucket in the previous step;
// or two launches:
//   tile_stage_kernel   the same for the tiles, with the tile's cells plus a
//   (tiles = 1)         halo of H cells of level n (and n+1) first staged in
//                       LDS with coalesced row loads and sampled from there; a
//                       particle whose stage point needs a cell outside the
//                       staged box is deferred: appended unchanged to this
//                       step's list;
//   tile_list_kernel    advance the list (deferred particles and the previous
//                       step's overflow) with global gathers, into the same
//                       next-step buckets.
// All sample with the same arithmetic on the same FP32 corner values, so a
// particle's step does not depend on which kernel took it.
//
// Buffers (context-owned): two bucket arrays (ping-pong) of nbuckets x cap
// slots of state + seed id, bucket b holding the tile that workgroup b runs
// (so a workgroup loads its tile id, particle count and particles at once); a
// ring of three bucket-count arrays (a step reads ring slot s, appends to s+1
// and clears s+2); the list in the context's ping-pong particle buffers with a
// ring of three counts; per-XCD counters of the live particles and of the
// steps attempted by particles that ended, touched only where one ended.
#include <type_traits>

#include "bto_internal.h"

namespace bto {

// Tile of an inside point's sampling cell (the cell locate() picks); GATHER:
// tiles of the gathering step, whose sides are powers of two known here.
template <bool GATHER>
__device__ __forceinline__ void tile_coords(const Geom& g, const TileGeom& tg, const double x[3], int t[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        int v = (int)x[d];
        v = v > g.n[d] - 2 ? g.n[d] - 2 : v;
        t[d] = GATHER ? v / TILE_GATHER[d] : v / tg.T[d];
    }
}

__device__ __forceinline__ uint32_t tile_index(const TileGeom& tg, const int t[3]) {
    return (uint32_t)(t[0] + tg.nt[0] * (t[1] + tg.nt[1] * t[2]));
}

// Write survivors to the bucket of their tile (key: tile id): one returning
// atomic per (wavefront, destination tile) on the bucket's count, lane slots
// from the ballot.  The lookups and atomics of all the wavefront's tiles are in
// flight together (one after the other, the first step's binning of 16.8
// million seeds took 390 us instead of 203).  Slots beyond the bucket's capacity go to the next list instead
// (one atomic per wavefront).  Wave-uniform control flow.
__device__ __forceinline__ void scatter_survivors(uint32_t tid, bool surv, uint32_t key, const PState& st,
                                                  uint32_t id, const TileOut& o) {
    const int lane = (int)(tid % WAVE);
    const unsigned long long below = (1ull << lane) - 1ull;
    // the lanes of each tile first, then every tile's bucket and atomic at once
    unsigned long long pending = __ballot(surv), peers = 0ull;
    int first = 0;
    while (pending) {
        const int leader = __ffsll((long long)pending) - 1;
        const bool mine = surv && key == (uint32_t)__builtin_amdgcn_readlane((int)key, leader);
        const unsigned long long same = __ballot(mine);
        if (mine) {
            peers = same;
            first = leader;
        }
        pending &= ~same;
    }
    uint32_t slot = 0, bkt = 0;
    if (surv && lane == first) {
        bkt = (uint32_t)o.slot_of[key];
        slot = atomicAdd(&o.tc[bkt], (uint32_t)__popcll(peers));
    }
    bkt = __shfl(bkt, first);
    slot = __shfl(slot, first) + (uint32_t)__popcll(peers & below);
    const bool over = surv && slot >= o.cap;
    if (surv && !over) {
        const size_t q = (size_t)bkt * o.cap + slot;
        o.bpos[q] = st;
        o.bid[q] = id;
    }
    const unsigned long long om = __ballot(over);
    if (om) {
        const int leader = __ffsll((long long)om) - 1;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(o.list_count, (uint32_t)__popcll(om));
        base = __shfl(base, leader);
        if (over) {
            const uint32_t k = base + (uint32_t)__popcll(om & below);
            o.list_pos[k] = st;
            o.list_id[k] = id;
        }
    }
}

// Append particles to a list, one atomic per wavefront (wave-uniform).
__device__ __forceinline__ void append_list(uint32_t tid, bool on, const PState& st, uint32_t id, PState* pos,
                                            uint32_t* ids, uint32_t* count) {
    const int lane = (int)(tid % WAVE);
    const unsigned long long m = __ballot(on);
    if (!m) return;
    const int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(count, (uint32_t)__popcll(m));
    base = __shfl(base, leader);
    if (on) {
        const uint32_t k = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        pos[k] = st;
        ids[k] = id;
    }
}

// Particles that ended in this step: off the live count, and the steps that
// each attempted since the seeding onto the step total (the
// live ones' attempts are known from the steps done).  Only workgroups in
// which a particle ended touch the shared counters.
__device__ __forceinline__ void add_ended(const TileStepArgs& a, uint32_t ended) {
    const int xcd = blockIdx.x % NSEG;
    atomicAdd(&a.psteps[xcd * PSTRIDE], (unsigned long long)ended * a.attempts);
    atomicSub(&a.live[xcd * CSTRIDE], ended);
}

// The same for a wavefront of the list (wave-uniform).
__device__ __forceinline__ void list_ended(const TileStepArgs& a, bool ended) {
    const unsigned long long m = __ballot(ended);
    if (m && threadIdx.x % WAVE == 0) add_ended(a, (uint32_t)__popcll(m));
}

__device__ __forceinline__ void end_record(const TileStepArgs& a, int status, uint32_t id, const double x[3], int rec) {
    a.rec_pos[id] = pack(x);
    a.rec_meta[id] = (status << META_SHIFT) | a.step0 | (rec && status == S_TERMINATED ? META_EXITPT : 0);
}

// Bucket of each neighbour of tile ts (direction (dx, dy, dz) in -1..1 at
// index (dz + 1) * 9 + (dy + 1) * 3 + dx + 1; -1 outside the block), loaded
// by the first 27 threads at the start of a workgroup and kept in a register
// until the scatter (so the load overlaps the step instead of stalling the
// first barrier).
__device__ __forceinline__ int32_t neighbour_bucket(const TileGeom& tg, const TileOut& o, const int ts[3]) {
    int32_t b = -1;
    if (threadIdx.x < 27) {
        const int d = (int)threadIdx.x;
        const int q[3] = {ts[0] + d % 3 - 1, ts[1] + (d / 3) % 3 - 1, ts[2] + d / 9 - 1};
        if (q[0] >= 0 && q[0] < tg.nt[0] && q[1] >= 0 && q[1] < tg.nt[1] && q[2] >= 0 && q[2] < tg.nt[2])
            b = o.slot_of[q[0] + tg.nt[0] * (q[1] + tg.nt[1] * q[2])];
    }
    return b;
}

// Direction (0..26, as in neighbour_bucket) of tile td from tile ts; 27: not a
// neighbour.
__device__ __forceinline__ int tile_dir(const int ts[3], const int td[3]) {
    const unsigned dx = (unsigned)(td[0] - ts[0] + 1), dy = (unsigned)(td[1] - ts[1] + 1),
                   dz = (unsigned)(td[2] - ts[2] + 1);
    return ((dx <= 2u) & (dy <= 2u) & (dz <= 2u)) ? (int)(dz * 9u + dy * 3u + dx) : 27;
}

struct ScatterLds {
    uint32_t hist[32];  // survivors per direction (zeroed by the caller, before a barrier)
    uint32_t base[32];
    int32_t nb[32];     // neighbour buckets (written by the caller, before a barrier)
    uint32_t ended;     // particles that ended in this batch (zeroed with hist)
};

// Survivors of one workgroup batch into the buckets of the next step.  A
// survivor ends in its own tile or a neighbour unless it jumped further: ranks
// per direction from LDS atomics, then one global atomic per (batch,
// destination tile) reserves the slots.  Survivors that jumped further take
// one global atomic each; slots beyond the bucket's capacity go to the next
// list.  Block-uniform (barriers inside).
__device__ __forceinline__ void scatter_block(const TileStepArgs& a, uint32_t tid, bool surv, bool ended,
                                              const int ts[3], const int td[3], const PState& st, uint32_t id,
                                              ScatterLds& s) {
    const TileOut& o = a.out;
    const int dir = surv ? tile_dir(ts, td) : 27;
    uint32_t rank = 0;
    if (surv && dir < 27) rank = atomicAdd(&s.hist[dir], 1u);
    const unsigned long long em = __ballot(ended);
    if (em && tid % WAVE == 0) atomicAdd(&s.ended, (uint32_t)__popcll(em));
    __syncthreads();
    if (tid < 27) {
        const uint32_t c = s.hist[tid];
        s.base[tid] = c ? atomicAdd(&o.tc[s.nb[tid]], c) : 0u;
    } else if (tid == 27) {
        if (s.ended) add_ended(a, s.ended);
    }
    __syncthreads();
    bool over = false;
    if (surv) {
        uint32_t bkt, slot;
        if (dir < 27) {
            bkt = (uint32_t)s.nb[dir];
            slot = s.base[dir] + rank;
        } else {
            bkt = (uint32_t)o.slot_of[td[0] + a.tg.nt[0] * (td[1] + a.tg.nt[1] * td[2])];
            slot = atomicAdd(&o.tc[bkt], 1u);
        }
        over = slot >= o.cap;
        if (!over) {
            const size_t q = (size_t)bkt * o.cap + slot;
            o.bpos[q] = st;
            o.bid[q] = id;
        }
    }
    append_list(tid, over, st, id, o.list_pos, o.list_id, o.list_count);
}

// ---------------------------------------------------------------------------
// The staging box of tile t: the tile's cells plus a halo of H cells, clipped
// to the block (lo: first point per axis, ext: points per axis, <= S).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tile_box(const Geom& g, const TileGeom& tg, const int tc[3], int lo[3], int ext[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int l = tc[d] * tg.T[d] - tg.H;
        const int h = tc[d] * tg.T[d] + tg.T[d] + tg.H;
        lo[d] = l < 0 ? 0 : l;
        const int hi = h > g.n[d] - 1 ? g.n[d] - 1 : h;
        ext[d] = hi - lo[d] + 1;
    }
}

// Grid values of one staging box held in registers between their loads and
// their stores to LDS: every load of the box is issued at once (one round
// trip), one point per thread per pass, rows of the box contiguous in x.
template <int DT, int MODE, int S>
struct StageRegs {
    static constexpr int NPT = S * S * S;
    static constexpr int KP = (NPT + BLOCK - 1) / BLOCK;
    static constexpr int NL = is_frozen<MODE> ? 1 : 2;
    static constexpr int EB = DT == DT_F32 ? 16 : 8;  // LDS bytes per staged point
    static constexpr uint32_t PLANE = (uint32_t)NPT * EB;
    using Pt = typename std::conditional<DT == DT_F32, Pt32, Pt16>::type;
    Pt v[NL][KP];
    uint32_t ok;

    __device__ __forceinline__ void load(const Geom& g, const char* V0, const char* V1, const int lo[3],
                                         const int ext[3]) {
        ok = 0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int p = threadIdx.x + k * BLOCK;
            const int lx = p % S, ly = (p / S) % S, lz = p / (S * S);
            if (p < NPT && lx < ext[0] && ly < ext[1] && lz < ext[2]) {
                ok |= 1u << k;
                const uint64_t gp = (uint64_t)(lo[0] + lx) + (uint64_t)g.sy * (uint32_t)(lo[1] + ly) +
                                    (uint64_t)g.sz * (uint32_t)(lo[2] + lz);
                v[0][k] = *reinterpret_cast<const Pt*>(V0 + gp * sizeof(Pt));
                if constexpr (NL == 2) v[NL - 1][k] = *reinterpret_cast<const Pt*>(V1 + gp * sizeof(Pt));
            }
        }
    }

    __device__ __forceinline__ void store(char* lds) const {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (ok & (1u << k)) {
                const int p = threadIdx.x + k * BLOCK;
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    if constexpr (DT == DT_F32) {
                        *reinterpret_cast<float4*>(lds + l * PLANE + (size_t)p * EB) =
                            make_float4(v[l][k].v[0], v[l][k].v[1], v[l][k].v[2], 0.f);
                    } else {
                        *reinterpret_cast<uint2*>(lds + l * PLANE + (size_t)p * EB) =
                            make_uint2(v[l][k].xy, (uint32_t)v[l][k].z);
                    }
                }
            }
        }
    }
};

__device__ __forceinline__ void unpack_tile(int32_t t, int tc[3]) {
    tc[0] = t & 1023;
    tc[1] = (t >> 10) & 1023;
    tc[2] = t >> 20;
}

// Inclusive sum over the wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    const auto dpp = [](uint32_t x, auto ctrl, auto rows) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
    };
    using std::integral_constant;
    constexpr integral_constant<int, 0xF> all{};
    v += dpp(v, integral_constant<int, 0x111>{}, all);                             // row_shr:1
    v += dpp(v, integral_constant<int, 0x112>{}, all);                             // row_shr:2
    v += dpp(v, integral_constant<int, 0x114>{}, all);                             // row_shr:4
    v += dpp(v, integral_constant<int, 0x118>{}, all);                             // row_shr:8
    v += dpp(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});   // row_bcast:15 into rows 1, 3
    v += dpp(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});   // row_bcast:31 into rows 2, 3
    return v;
}

// ---------------------------------------------------------------------------
// Gathering tile step: one workgroup of NT threads per tile, the particles
// gather from the grids (through L2, which the tile order keeps warm).
//
// The particles of a batch are first reordered by the (z, y) row of their
// cell inside the tile (counting sort in LDS), so that the lanes of a
// wavefront share grid rows: each row load of the sampler then touches a few
// cache lines per wavefront instead of one per lane (without it 6 to 10%
// slower; a finer order along x changes nothing).  A tile has one row per
// lane, so every wavefront scans the row counts by itself.
//
// What bounds it: the L1 returns in order, so a load behind one that missed to
// HBM waits; accesses (0.38 per cycle and CU on the 512^3 f16 block) and
// stalls on pending lines (0.63) fill every cycle.  The kernel therefore gains
// from less work per wavefront and more wavefronts to hide it: 91 registers
// leave 5 wavefronts per SIMD (f16; FP32 94; 127 and 121 before).  What is
// computed from the thread index is computed anew behind the step for that
// reason.  Nothing else is shared between workgroups than the buckets: the
// live and step totals are touched only where a particle ended.
// Intervals with two launches a step and the 127 registers of the step before, and
// now: 512^3 f16, 20 steps, 20.5 and 16.8 ms; 256^3, 25 steps: f32 4.86 and 4.24,
// bf16 3.88 and 2.74; FP64 sampling at 201 x 150 x 177 1.93 and 1.68.
// Prefetching a later tile's lines into L2 (every line of it by one dword
// load, 16 to 128 tiles ahead) made it 8 to 14% slower: the loads wait in the
// same in-order L1, and a third of the lines were evicted before their use.
// ---------------------------------------------------------------------------
template <int DT, int MODE, int REC, int NT>
__global__ __launch_bounds__(NT) void tile_gather_kernel(const TileStepArgs a) {
    constexpr int Ty = TILE_GATHER[1], Tz = TILE_GATHER[2];
    static_assert(Ty * Tz == WAVE, "one row of the tile per lane");
    __shared__ ScatterLds s_sc;
    __shared__ uint32_t s_row[WAVE];
    __shared__ U4 s_pos[NT];
    __shared__ uint32_t s_id[NT];
    const uint32_t tid = threadIdx.x;
    const uint32_t ntile = (uint32_t)a.order_len;
    const bool list = blockIdx.x >= ntile;  // the workgroups behind the tiles' take the list
    if (blockIdx.x == 0 && tid == 0) *a.list_clear = 0u;
    // batches of NT particles [i, i + NT) of src_pos, src_id, every `stride`, up to n
    const U4* src_pos = reinterpret_cast<const U4*>(a.list_pos);
    const uint32_t* src_id = a.list_id;
    uint32_t i = (blockIdx.x - ntile) * NT, n, stride = (gridDim.x - ntile) * NT;
    // one state and id per thread, held as plain registers (an index past the
    // last particle reads the last one's); a tile's first ones load before its
    // count is known
    U4 st;
    uint32_t id;
    const auto load = [&](uint32_t last) {
        const uint32_t k = i + threadIdx.x < last ? i + threadIdx.x : last;
        st = src_pos[k];
        id = src_id[k];
    };
    int tc[3] = {0, 0, 0};
    int32_t nb = -1;
    if (list) {
        n = scalar_load(a.list_count);
        if (i >= n) return;
        load(n - 1u);
    } else {
        // the bucket of this workgroup: its tile, count and first particles load at
        // once.  Every other step runs each XCD's tiles backwards: what the last
        // step touched last -- level n + 1, which is this step's level n, and the
        // buckets it filled -- is then read first, while the memory-side cache
        // still holds it (the intervals above all in one direction: 17.0 ms instead
        // of 16.9, 4.41 instead of 4.25, 2.83 instead of 2.78, 1.70 instead of 1.67).
        const uint32_t b = a.backwards ? (ntile / NSEG - 1u - blockIdx.x / NSEG) * NSEG + blockIdx.x % NSEG : blockIdx.x;
        int32_t t = scalar_load(a.order + b);
        n = scalar_load(a.tc_in + b);
        src_pos = reinterpret_cast<const U4*>(a.in_pos) + (size_t)b * a.out.cap;
        src_id = a.in_id + (size_t)b * a.out.cap;
        i = 0;
        stride = NT;
        load(a.out.cap - 1u);
        asm("" : "+s"(t), "+s"(n));  // both tables' entries in flight before the first is looked at
        if (t < 0) return;
        if (tid == 0) a.tc_clear[b] = 0u;
        n = n < a.out.cap ? n : a.out.cap;
        if (n == 0) return;
        // A tile with fewer particles than threads: the wavefronts past its count
        // end here, so they hold no wave slot while the tile runs (s_barrier then
        // waits for the surviving wavefronts only).  The wave index is taken from
        // the first lane so that the branch is scalar: the whole wavefront ends.
        if (n < (uint32_t)NT && __builtin_amdgcn_readfirstlane((int)(tid / WAVE)) >= (int)((n + WAVE - 1) / WAVE)) return;
        unpack_tile(t, tc);
        nb = neighbour_bucket(a.tg, a.out, tc);
    }
    const char* V0 = in_global(a.f0);
    const char* V1 = in_global(a.f1);
    bool first = true;
    for (;;) {
        // the thread index anew before and after the step: what is computed from
        // it is then not held in registers across the step
        uint32_t tid = opaque(threadIdx.x);
        const bool alive = i + tid < n;
        if (!list) {
            if (tid < WAVE) s_row[tid] = 0u;
            if (tid < 32) s_sc.hist[tid] = 0u;
            if (tid == 0) s_sc.ended = 0u;
            __syncthreads();
            uint32_t row = 0, rank = 0;
            if (alive) {
                int ly = (int)((st.x >> 10) & 1023u) - tc[1] * Ty;
                int lz = (int)(st.x >> 20) - tc[2] * Tz;
                ly = ly > Ty - 1 ? Ty - 1 : ly;  // a point on the high face has the cell index n - 1
                lz = lz > Tz - 1 ? Tz - 1 : lz;
                row = (uint32_t)(lz * Ty + ly);
                rank = atomicAdd(&s_row[row], 1u);
            }
            __syncthreads();
            const uint32_t c = s_row[tid % WAVE];
            const uint32_t dst = __shfl(wave_scan(c) - c, (int)row) + rank;
            if (alive) {
                s_pos[dst] = st;
                s_id[dst] = id;
            }
            if (first && tid < 27) s_sc.nb[tid] = nb;
            first = false;
            nb = 0;
        } else {
            s_pos[tid] = st;
            s_id[tid] = id;
        }
        __syncthreads();
        double x[3] = {0.0, 0.0, 0.0};
        int status = S_INVALID;
        if (alive) {
            const U4 p = s_pos[tid];
            unpack(PState{p.x, {p.y, p.z, p.w}}, x);
            const auto on_exit = [&](const double* y) {
                if constexpr (REC)
                    a.rec_out[s_id[tid]] =
                        make_float4((float)(y[0] - x[0]), (float)(y[1] - x[1]), (float)(y[2] - x[2]), 0.f);
            };
            GatherCache<DT> A, B;
            forget(A);
            forget(B);
            status = rk4_step_gather<DT, MODE>(a.g, V0, V1, a.hs, x, A, B, false, on_exit);
        }
        tid = opaque(threadIdx.x);
        id = s_id[tid];
        const bool was = i + tid < n, surv = was & (status == S_VALID), ended = was & !surv;
        if (ended) end_record(a, status, id, x, REC);
        int td[3];
        tile_coords<true>(a.g, a.tg, x, td);
        if (!list) {
            scatter_block(a, tid, surv, ended, tc, td, pack(x), id, s_sc);
        } else {
            list_ended(a, ended);
            scatter_survivors(tid, surv, tile_index(a.tg, td), pack(x), id, a.out);
        }
        i += stride;
        if (i >= n) break;
        load(n - 1u);
    }
}

// ---------------------------------------------------------------------------
// Staged tile step: one workgroup per tile stages the tile's cells plus a halo
// of H cells of both levels in LDS (every load of the box issued at once),
// then advances the tile's particles sampling from LDS.  Particles whose stage
// points need cells beyond the staged box are deferred to the list.
// ---------------------------------------------------------------------------
template <int DT, int MODE, int REC, int S>
__global__ __launch_bounds__(BLOCK) void tile_stage_kernel(const TileStepArgs a) {
    extern __shared__ __align__(16) char lds[];
    __shared__ ScatterLds s_sc;
    using SR = StageRegs<DT, MODE, S>;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.list_clear = 0u;
    const uint32_t b = blockIdx.x;
    const int32_t t = scalar_load(a.order + b);
    uint32_t cnt = scalar_load(a.tc_in + b);
    const size_t bin = (size_t)b * a.out.cap;
    PState st0{};
    uint32_t id0 = 0;
    if (threadIdx.x < a.out.cap) {  // in the bucket even when beyond its count
        st0 = a.in_pos[bin + threadIdx.x];
        id0 = a.in_id[bin + threadIdx.x];
    }
    if (t < 0) return;
    if (threadIdx.x == 0) a.tc_clear[b] = 0u;
    cnt = cnt < a.out.cap ? cnt : a.out.cap;
    if (cnt == 0) return;
    int tc[3], lo[3], ext[3];
    unpack_tile(t, tc);
    tile_box(a.g, a.tg, tc, lo, ext);
    const int32_t nb = neighbour_bucket(a.tg, a.out, tc);
    {
        SR sr;
        sr.load(a.g, in_global(a.f0), in_global(a.f1), lo, ext);
        sr.store(lds);
    }
    if (threadIdx.x < 27) s_sc.nb[threadIdx.x] = nb;
    LdsCache<DT> A, B;
    A.plane = lds;
    B.plane = lds + (is_frozen<MODE> ? 0u : SR::PLANE);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        A.lo[d] = B.lo[d] = lo[d];
        A.lim[d] = B.lim[d] = ext[d] - 2;
    }
    A.S = B.S = S;
    for (uint32_t bb = 0; bb < cnt; bb += BLOCK) {
        if (threadIdx.x < 32) s_sc.hist[threadIdx.x] = 0u;
        if (threadIdx.x == 0) s_sc.ended = 0u;
        __syncthreads();
        const uint32_t i = bb + threadIdx.x;
        const bool alive = i < cnt;
        PState st = st0;
        uint32_t id = id0;
        if (bb && alive) {
            st = a.in_pos[bin + i];
            id = a.in_id[bin + i];
        }
        double x[3] = {0.0, 0.0, 0.0};
        int status = S_DEFER;
        if (alive) {
            unpack(st, x);
            const auto on_exit = [&](const double* y) {
                if constexpr (REC)
                    a.rec_out[id] = make_float4((float)(y[0] - x[0]), (float)(y[1] - x[1]), (float)(y[2] - x[2]), 0.f);
            };
            forget(A);
            forget(B);
            status = rk4_step<DT, MODE>(a.g, nullptr, nullptr, a.h, x, A, B, on_exit);
        }
        const bool surv = alive && status == S_VALID;
        const bool ended = status == S_TERMINATED || status == S_INVALID;
        if (ended) end_record(a, status, id, x, REC);
        int td[3];
        tile_coords<false>(a.g, a.tg, x, td);
        scatter_block(a, threadIdx.x, surv, ended, tc, td, surv ? pack(x) : st, id, s_sc);
        append_list(threadIdx.x, alive && status == S_DEFER, st, id, a.list_pos, a.list_id, a.list_count);
    }
}

// ---------------------------------------------------------------------------
// The list: deferred particles of this step and bucket overflows of the last
// one, advanced with global gathers into the next step's buckets.
// ---------------------------------------------------------------------------
template <int DT, int MODE, int REC>
__global__ __launch_bounds__(BLOCK) void tile_list_kernel(const TileListArgs a) {
    const uint32_t n = *a.in_count;
    const char* V0 = in_global(a.s.f0);
    const char* V1 = in_global(a.s.f1);
    // wave-uniform loop over the list
    const uint32_t wave_g = (blockIdx.x * BLOCK + threadIdx.x) / WAVE;
    const uint32_t nwaves = gridDim.x * (BLOCK / WAVE);
    for (uint32_t w0 = wave_g * WAVE; w0 < n; w0 += nwaves * WAVE) {
        const uint32_t i = w0 + threadIdx.x % WAVE;
        const bool alive = i < n;
        double x[3] = {0.0, 0.0, 0.0};
        uint32_t id = 0;
        int status = S_INVALID;
        if (alive) {
            const PState st = a.in_pos[i];
            id = a.in_id[i];
            unpack(st, x);
            GatherCache<DT> A, B;
            forget(A);
            forget(B);
            const auto on_exit = [&](const double* y) {
                if constexpr (REC)
                    a.s.rec_out[id] = make_float4((float)(y[0] - x[0]), (float)(y[1] - x[1]), (float)(y[2] - x[2]), 0.f);
            };
            status = rk4_step_gather<DT, MODE>(a.s.g, V0, V1, a.s.hs, x, A, B, false, on_exit);
            if (status != S_VALID) end_record(a.s, status, id, x, REC);
        }
        const bool surv = alive && status == S_VALID;
        list_ended(a.s, alive && !surv);
        int td[3];
        tile_coords<false>(a.s.g, a.s.tg, x, td);
        scatter_survivors(threadIdx.x, surv, tile_index(a.s.tg, td), pack(x), id, a.s.out);
    }
}

// ---------------------------------------------------------------------------
// Segment layout -> buckets (once per interval, before the first tile step):
// every live particle of the segments into the bucket of its tile, overflow
// into the list of the coming step.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void tile_bin_kernel(const TileBinArgs a) {
    const int seg = blockIdx.x % NSEG;
    const int r = blockIdx.x / NSEG;
    const int R = gridDim.x / NSEG;
    const uint32_t cnt = a.count[seg * CSTRIDE];
    const int64_t sbase = a.segs.base[seg];
    for (uint32_t b0 = (uint32_t)r * BLOCK; b0 < cnt; b0 += (uint32_t)R * BLOCK) {
        const uint32_t i = b0 + threadIdx.x;
        const bool alive = i < cnt;
        PState st{};
        uint32_t id = 0, key = 0;
        if (alive) {
            st = a.pos[sbase + i];
            id = a.id[sbase + i];
            double x[3];
            unpack(st, x);
            int td[3];
            tile_coords<false>(a.g, a.tg, x, td);
            key = tile_index(a.tg, td);
        }
        scatter_survivors(threadIdx.x, alive, key, st, id, a.out);
    }
}

// Zero n words (tile and list counts before the first tile step).
__global__ void tile_fill_kernel(uint32_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Live particles of the tile layout (buckets and the pending list), by seed
// id: end position for the flow map (out_end) or FP64 position for a
// checkpoint (ckpt non-null).  One wavefront per bucket; the last list_blocks
// workgroups share the list.
__global__ __launch_bounds__(BLOCK) void tile_live_kernel(const TileLiveArgs a) {
    const auto put = [&](const PState& st, uint32_t id) {
        double x[3];
        unpack(st, x);
        double* out = (a.ckpt ? a.ckpt : a.out_end) + 3 * (size_t)id;
#pragma unroll
        for (int d = 0; d < 3; ++d) out[d] = a.ckpt ? x[d] : a.origin[d] + a.spacing[d] * x[d];
    };
    const uint32_t tile_blocks = gridDim.x - a.list_blocks;
    if (blockIdx.x >= tile_blocks) {
        const uint32_t n = *a.list_count;
        for (uint64_t k = (uint64_t)(blockIdx.x - tile_blocks) * BLOCK + threadIdx.x; k < n;
             k += (uint64_t)a.list_blocks * BLOCK)
            put(a.list_pos[k], a.list_id[k]);
        return;
    }
    const uint32_t t = blockIdx.x * (BLOCK / WAVE) + threadIdx.x / WAVE;
    if (t >= a.ntiles) return;
    const uint32_t c = a.tc[t], n = c < a.cap ? c : a.cap;
    const uint64_t base = (uint64_t)t * a.cap;
    for (uint32_t k = threadIdx.x % WAVE; k < n; k += WAVE) put(a.bpos[base + k], a.bid[base + k]);
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
// Unused LDS of which four workgroups, but not five, find room on a CU (160 KB)
// beside their own.  FP32 cells take twice the lines of 16-bit ones, and the
// lines of four workgroups stay longer in the L1: 167 -> 165 us per step of a
// 256^3 turbulence block with 2 million particles; f16 loses (107 -> 108).
constexpr unsigned FOUR_LDS = 30 * 1024;

template <int DT, int MODE, int REC>
static hipError_t launch_tile_step_t(const TileStepArgs& a, int list_blocks, hipStream_t s) {
    hipLaunchKernelGGL((tile_gather_kernel<DT, MODE, REC, GATHER_NT>), dim3(a.order_len + list_blocks), dim3(GATHER_NT),
                       DT == DT_F32 ? FOUR_LDS : 0u, s, a);
    return hipGetLastError();
}

template <int DT, int MODE, int REC>
static hipError_t launch_tile_stage_t(const TileStepArgs& a, hipStream_t s) {
    constexpr int S = DT == DT_F32 ? TILE_S_F32 : TILE_S_16;
    using SR = StageRegs<DT, MODE, S>;
    constexpr size_t lds = (size_t)SR::NL * SR::PLANE;
    // LDS beyond the default limit: raise the kernel's dynamic-LDS limit (on
    // the current device) before the launch
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_stage_kernel<DT, MODE, REC, S>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        (void)hipGetLastError();
    hipLaunchKernelGGL((tile_stage_kernel<DT, MODE, REC, S>), dim3(a.order_len), dim3(BLOCK), lds, s, a);
    return hipGetLastError();
}

template <int DT, int MODE, int REC>
static hipError_t launch_tile_list_t(const TileListArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((tile_list_kernel<DT, MODE, REC>), dim3(grid), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

template <class F>
static hipError_t tile_dispatch(int dtype, int mode, int rec, F&& f) {
    auto by_rec = [&](auto dt, auto md) {
        return rec ? f(dt, md, std::integral_constant<int, 1>{}) : f(dt, md, std::integral_constant<int, 0>{});
    };
    auto by_mode = [&](auto dt) {
        switch (mode) {
        case MODE_LINEAR: return by_rec(dt, std::integral_constant<int, MODE_LINEAR>{});
        case MODE_FROZEN: return by_rec(dt, std::integral_constant<int, MODE_FROZEN>{});
        case MODE_LINEAR | MODE_FP64: return by_rec(dt, std::integral_constant<int, MODE_LINEAR | MODE_FP64>{});
        case MODE_FROZEN | MODE_FP64: return by_rec(dt, std::integral_constant<int, MODE_FROZEN | MODE_FP64>{});
        case MODE_LINEAR | MODE_WIDE: return by_rec(dt, std::integral_constant<int, MODE_LINEAR | MODE_WIDE>{});
        case MODE_FROZEN | MODE_WIDE: return by_rec(dt, std::integral_constant<int, MODE_FROZEN | MODE_WIDE>{});
        case MODE_LINEAR | MODE_FP64 | MODE_WIDE:
            return by_rec(dt, std::integral_constant<int, MODE_LINEAR | MODE_FP64 | MODE_WIDE>{});
        default: return by_rec(dt, std::integral_constant<int, MODE_FROZEN | MODE_FP64 | MODE_WIDE>{});
        }
    };
    switch (dtype) {
    case DT_F32: return by_mode(std::integral_constant<int, DT_F32>{});
    case DT_F16: return by_mode(std::integral_constant<int, DT_F16>{});
    default: return by_mode(std::integral_constant<int, DT_BF16>{});
    }
}

hipError_t launch_tile_step(const TileStepArgs& a, int dtype, int mode, int rec, int list_blocks, hipStream_t s) {
    return tile_dispatch(dtype, mode, rec, [&](auto dt, auto md, auto rc) {
        return launch_tile_step_t<decltype(dt)::value, decltype(md)::value, decltype(rc)::value>(a, list_blocks, s);
    });
}

hipError_t launch_tile_stage(const TileStepArgs& a, int dtype, int mode, int rec, hipStream_t s) {
    // the staging loads address 64-bit as they are
    return tile_dispatch(dtype, mode & ~MODE_WIDE, rec, [&](auto dt, auto md, auto rc) {
        return launch_tile_stage_t<decltype(dt)::value, decltype(md)::value & ~MODE_WIDE, decltype(rc)::value>(a, s);
    });
}

hipError_t launch_tile_list(const TileListArgs& a, int dtype, int mode, int rec, int grid, hipStream_t s) {
    return tile_dispatch(dtype, mode, rec, [&](auto dt, auto md, auto rc) {
        return launch_tile_list_t<decltype(dt)::value, decltype(md)::value, decltype(rc)::value>(a, grid, s);
    });
}

hipError_t launch_tile_bin(const TileBinArgs& a, int R, hipStream_t s) {
    hipLaunchKernelGGL(tile_bin_kernel, dim3(R * NSEG), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tile_fill(uint32_t* p, size_t n, hipStream_t s) {
    size_t g = (n + BLOCK - 1) / BLOCK;
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(tile_fill_kernel, dim3((unsigned)g), dim3(BLOCK), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_tile_live(const TileLiveArgs& a, hipStream_t s) {
    const uint32_t tile_blocks = (a.ntiles + BLOCK / WAVE - 1) / (BLOCK / WAVE);
    hipLaunchKernelGGL(tile_live_kernel, dim3(tile_blocks + a.list_blocks), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

}  // namespace bto
