// Host <-> kernel interface of the BTO library (not part of the public C-ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bto_device.h"

namespace bto {

// Per-segment counters (live counts, particle-step totals) lie one 128-byte
// line apart, counter x of a slot at index x * CSTRIDE (32-bit) or x * PSTRIDE
// (64-bit).  Every workgroup of a launch adds into them; device-scope atomics
// are carried out at the memory side, and spreading the counters over lines
// lets the segments' atomics proceed in parallel there.
constexpr int CSTRIDE = 32;
constexpr int PSTRIDE = 16;

// Live particles are split into NSEG contiguous segments of the ping-pong
// buffers.  Workgroup b of a launch works on segment b % NSEG: consecutive
// workgroups are dispatched round-robin over the 8 XCDs, so each XCD keeps
// one spatially compact slab of particles (and of the field) in its own L2.
// Pointers read from a device array (the grid tables) are generic to the
// compiler, which then emits flat memory instructions for every gather and
// atomic through them; flat instructions also count against the scalar-load
// counter, so their waits and those of scalar loads merge.  Every grid lives in
// global memory: rebuilding the pointer in the global address space (through
// its integer value, which no pass folds back into the generic pointer) lets
// the compiler emit the global forms.
template <class T>
__device__ __forceinline__ T* in_global(T* p) {
    using G = __attribute__((address_space(1))) T*;
    return (T*)(G)(uintptr_t)p;
}

// A value that is the same in every lane, moved to scalar registers.  Its words
// are made opaque first: the compiler drops its own builtin where it knows the
// value to be uniform, and keeps it in vector registers all the same.  The move
// itself is the builtin and not assembly, because gfx950 wants wait states
// between the vector write of a register and v_readfirstlane's read of it, and
// behind it, which the compiler puts in only for instructions that it sees.
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)opaque((uint32_t)b));
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)opaque((uint32_t)(b >> 32)));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sixteen bytes as four registers (a struct's array is kept in memory where it
// crosses a branch).
typedef uint32_t U4 __attribute__((ext_vector_type(4)));

// A table entry read through the scalar cache (constant during the launch, the
// same for the whole wavefront).
template <class T>
__device__ __forceinline__ T scalar_load(const T* p) {
    using C = const __attribute__((address_space(4))) T*;
    return *(C)(uintptr_t)p;
}

struct Segs {
    int64_t base[NSEG];  // first slot of each segment
};

struct AdvectArgs {
    const char* f[KMAX + 1];  // grids of cycles c0 .. c0 + K
    double h[KMAX];           // step sizes
    Geom g;
    int32_t K;                // steps in this launch
    int32_t step0;            // steps already done in the interval
    Segs segs;
    const PState* in_pos;
    const uint32_t* in_id;
    PState* out_pos;
    uint32_t* out_id;
    const uint32_t* in_count;   // NSEG live counts entering the launch
    uint32_t* out_count;        // NSEG counts of survivors (zero on entry)
    uint32_t* clear_count;      // NSEG counts cleared for the launch after next
    PState* rec_pos;            // per seed id: final state of ended particles
    int32_t* rec_meta;          // per seed id: flag << 28 | exit step
    float4* rec_out;            // per seed id: outside point - last inside position (terminated only)
    unsigned long long* psteps; // NSEG counters: steps attempted by the particles that ended
};

struct SeedLatticeArgs {
    int32_t m[3];        // lattice points per axis
    double off[3];       // lattice offset (cells)
    int32_t stride;
    int32_t morton;      // bricks in Morton order (power-of-two cube of bricks)
    int32_t octant;      // octant-major order: segment x = lattice octant x, x-fastest inside
    int32_t half[3];     // octant split per axis: indices < half[d] are the low half
    int64_t oct_base[NSEG];  // first slot of each octant
    int32_t brick[3];    // lattice points per brick and axis (product 64)
    int64_t P;
    Segs segs;
    double origin[3], spacing[3];
    PState* pos;
    uint32_t* id;
    double* seed_xyz;    // per seed id, world coordinates
    int32_t* rec_meta;
};

struct SeedExplicitArgs {
    const double* xyz;   // world
    int64_t P;
    Geom g;
    Segs segs;
    double origin[3], inv_sp[3];
    PState* pos;
    uint32_t* id;
    uint32_t* count;     // NSEG, zero on entry
    double* seed_xyz;
    PState* rec_pos;
    int32_t* rec_meta;
};

struct FlowmapArgs {
    int64_t P;
    int32_t steps_done;
    Segs segs;
    const uint32_t* count;
    const PState* pos;
    const uint32_t* id;
    const PState* rec_pos;
    const int32_t* rec_meta;
    const float4* rec_out;
    Geom g;
    const double* seed_xyz;
    double origin[3], spacing[3];
    double* out_seed;    // may be null
    double* out_end;
    uint8_t* out_flag;
    int32_t* out_exit;
    double* out_face;    // exit points (bto_exit_points)
};

// Grid-gradient records for the deterministic reduction: each accumulator
// flush writes (key, 8 x 3 corner gradients) instead of adding them to the
// grid with atomics; key = parity colour | level | cell (bit widths below,
// colour on top; colour field 8 marks an unused slot).  The j-th flush of seed
// p goes to slot j * P + p, a position fixed by (j, p) alone, so the stable
// sort leaves each group's records in an order that does not depend on thread
// timing.  A seed's flushes beyond per_seed fall back to atomics.  key == null:
// atomics.
struct GradRec {
    void* key;                  // uint32_t (key_bytes 4) or uint64_t per slot; null: atomics
    int32_t key_bytes;
    float* val;                 // per_seed * P x 24 floats
    uint32_t per_seed;
    uint32_t P;
    int32_t cell_bits, level_bits;
};

// The adjoint's tape: what the reverse sweep needs of a step, one 16-byte entry
// per stage -- the value index of the cell sampled and the three FP32 offsets
// in it -- at [step][stage][seed], so a wavefront's 64 entries are one
// contiguous kilobyte.
struct TapeEntry {
    uint32_t val;
    float f[3];
};

// Words per seed of what a launch leaves to the call's next: see AdjointArgs::carry.
constexpr int ACC_WORDS = 27;

struct AdjointArgs {
    const char* const* f;       // device array: grids of the call's cycles
    const double* h;            // device array: its step sizes
    Geom g;
    int32_t N;                  // steps
    int32_t k;                  // checkpoint every k steps
    int32_t ncot;               // cotangent vectors per seed (1 or 3)
    int64_t P;                  // seeds
    int64_t p0, np;             // the seeds of this launch: p0 .. p0 + np - 1
    const double* seed_xyz;     // P x 3 world
    double origin[3], sp[3];
    const float* cot;           // P x ncot x 3, d L / d x_end (world)
    float* grad_seed;           // P x ncot x 3, d L / d x_0 (world)
    float* const* grad_f;       // device array of FP32 grids (accumulated) or null
    double* ckpt;               // ceil(N/k) slots of ck_stride doubles ([slot][seed][xyz], cell units), or null
    int64_t ck_stride;          // doubles per checkpoint slot (>= 3 P)
    TapeEntry* tape;            // steps of segments sg_last .. sg_first, np seeds each (null: forward without a tape)
    uint8_t* status;            // P: status of the adjoint's own forward (rec_meta null)
    uint8_t* bad;               // P: a recomputed step contradicted the forward
    uint8_t* status_out;        // P (may be null): reported status
    const int32_t* rec_meta;    // non-null: take the forward from recorded checkpoints and these records
    GradRec grec;               // grid-gradient records (grec.key null: atomics)
    // Grid gradients between the launches of a call (null: one launch does all):
    // P words, the records that each seed has written so far; with carry_acc 26 P
    // more, its accumulator, which otherwise is flushed by each launch.
    uint32_t* carry;
    int32_t carry_acc;
    // Segments of this launch, sg_first down to sg_last (the whole interval:
    // nseg - 1 .. 0).  f, h and grad_f hold the grids, steps and gradient grids
    // from step f_base on.  lam (P x ncot x 3, cell units) carries the
    // cotangents from one launch to the next (read unless sg_first is the last
    // segment, written unless sg_last is 0); drop (P bytes, may be null where
    // one launch does all) marks seeds dropped by an earlier launch.
    int32_t sg_first, sg_last;
    int32_t f_base;
    int32_t call_first, call_last;  // first and last segment of this call
    float* lam;
    uint8_t* drop;
};

// Checkpoint of the live particles for the adjoint: FP64 positions (cell
// units) by seed id into one slot.
struct CkptArgs {
    Segs segs;
    const uint32_t* count;     // NSEG live counts
    const PState* pos;
    const uint32_t* id;
    double* out;               // slot base: [seed id][xyz]
};

// Rebin bins: REBIN_BIN[0] x REBIN_BIN[1] x REBIN_BIN[2] cells, x fastest.
constexpr int REBIN_BIN[3] = {32, 2, 2};

struct RebinArgs {
    int64_t P;                 // slots covered by the segments
    Segs segs;
    const uint32_t* count;     // NSEG live counts
    const PState* pos;         // current buffers
    const uint32_t* id;
    PState* out_pos;           // the other ping-pong buffers
    uint32_t* out_id;
    uint32_t* bin;             // per slot: (segment, brick) bin
    uint32_t* rank;            // per slot: rank inside the bin
    uint32_t* hist;            // NSEG * nbins counts (all zero between rebins)
    uint32_t* offs;            // NSEG * nbins exclusive prefix sums
    uint32_t nbins;            // bins per segment
    int32_t bin_bits;          // bits of a bin's number (segment and bin)
    uint32_t nbx, nby;         // bins along x and y
    void* temp;
    size_t temp_bytes;
};

// ---------------------------------------------------------------------------
// Tile layout of the live particles (tile-staged advection, tiles.hip).
// ---------------------------------------------------------------------------
constexpr int TILE_H = 2;       // halo cells staged around a tile
constexpr int TILE_S_16 = 17;   // staging box side in points, 16-bit grids (tile of 12 cells)
constexpr int TILE_S_F32 = 13;  // FP32 grids (tile of 8 cells)

// Tile sides in cells.  Staged tiles are cubes sized so that two workgroups'
// boxes fit a CU's LDS.  Gathering tiles are 32 x 8 x 8 cells for every
// storage type: 256 seeds at stride 2, one per thread of the workgroup, on
// rows long in x (the grid's contiguous axis), whose lines the particles of
// a row share (8% faster than 12^3 cubes on the 512^3 f16 step).
constexpr int TILE_GATHER[3] = {32, 8, 8};
constexpr int GATHER_NT = 256;  // threads per workgroup of the gathering tile step

__host__ __device__ constexpr int tile_side(int dtype, int staged, int axis) {
    return staged ? (dtype == DT_F32 ? TILE_S_F32 : TILE_S_16) - 1 - 2 * TILE_H : TILE_GATHER[axis];
}

struct __attribute__((packed, aligned(2))) Pt16 {
    uint32_t xy;
    uint16_t z;
};

struct TileGeom {
    int32_t T[3];       // tile sides (cells)
    int32_t H;          // halo of a staged tile (cells)
    int32_t nt[3];      // tiles per axis
};

struct TileOut {
    uint32_t* tc;       // bucket counts of the next step (appended)
    const int32_t* slot_of;  // bucket of each tile id
    PState* bpos;       // next step's buckets: nbuckets x cap
    uint32_t* bid;
    uint32_t cap;
    PState* list_pos;   // next step's list (bucket overflow)
    uint32_t* list_id;
    uint32_t* list_count;
};

struct TileStepArgs {
    const char* f0;           // grid of cycle n
    const char* f1;           // grid of cycle n + 1
    double h;
    StepSizes hs;             // of h, for the gathering kernels
    Geom g;
    TileGeom tg;
    int32_t step0;            // index of this step in the interval
    const int32_t* order;     // tile coordinates (10 bits each) of bucket b = workgroup b (-1: none);
                              // b = k * NSEG + x is the k-th tile of XCD x's run
    int32_t order_len;        // buckets (a multiple of NSEG)
    const uint32_t* tc_in;    // this step's bucket counts
    uint32_t* tc_clear;       // bucket counts cleared for the step after next
    const PState* in_pos;     // this step's buckets
    const uint32_t* in_id;
    TileOut out;
    PState* list_pos;         // this step's list (the staged step appends deferred particles)
    uint32_t* list_id;
    uint32_t* list_count;
    uint32_t* list_clear;     // list count cleared for the step after next
    PState* rec_pos;
    int32_t* rec_meta;
    float4* rec_out;
    unsigned long long* psteps;  // NSEG counters: steps attempted by the particles that ended
    uint32_t* live;           // NSEG counters, modulo 2^32: their sum is the live particles
    int32_t backwards;        // run each XCD's tiles in reverse order
    uint32_t attempts;        // steps attempted since the seeding by a particle ending in this step
};

struct TileListArgs {
    TileStepArgs s;
    const PState* in_pos;     // this step's list
    const uint32_t* in_id;
    const uint32_t* in_count;
};

struct TileBinArgs {
    Geom g;
    TileGeom tg;
    Segs segs;
    const uint32_t* count;    // NSEG live counts of the segments
    const PState* pos;
    const uint32_t* id;
    TileOut out;              // buckets and list of the coming step
};

struct TileLiveArgs {
    uint32_t ntiles, cap;     // buckets, slots per bucket
    const uint32_t* tc;
    const PState* bpos;
    const uint32_t* bid;
    const PState* list_pos;
    const uint32_t* list_id;
    const uint32_t* list_count;
    uint32_t list_blocks;     // workgroups for the list
    double origin[3], spacing[3];
    double* out_end;          // flow map (ckpt == null)
    double* ckpt;             // checkpoint slot base: [seed id][xyz] (cell units)
};

// One workgroup per order entry, gathering from the grids, and list_blocks for
// the list; or one per order entry sampling LDS-staged tiles, the list then by
// launch_tile_list.  mode: MODE_WIDE set for grids beyond 4 GiB.
hipError_t launch_tile_step(const TileStepArgs& a, int dtype, int mode, int rec, int list_blocks, hipStream_t s);
hipError_t launch_tile_stage(const TileStepArgs& a, int dtype, int mode, int rec, hipStream_t s);
hipError_t launch_tile_list(const TileListArgs& a, int dtype, int mode, int rec, int grid, hipStream_t s);
hipError_t launch_tile_bin(const TileBinArgs& a, int blocks_per_seg, hipStream_t s);
hipError_t launch_tile_fill(uint32_t* p, size_t n, hipStream_t s);
hipError_t launch_tile_live(const TileLiveArgs& a, hipStream_t s);

hipError_t launch_seed_lattice(const SeedLatticeArgs& a, hipStream_t s);
hipError_t launch_seed_explicit(const SeedExplicitArgs& a, hipStream_t s);
hipError_t launch_set_counts(uint32_t* counts, const uint32_t* values, int n, unsigned long long* psteps,
                             hipStream_t s);
// pair: at most two workgroups on a CU at a time.
hipError_t launch_advect(const AdvectArgs& a, int dtype, int mode, int lanes_per_particle, int record_exit,
                         int blocks_per_seg, bool pair, hipStream_t s);
hipError_t launch_exit_points(const FlowmapArgs& a, hipStream_t s);
hipError_t launch_reconstruct(const int32_t m[3], double* end, const uint8_t* flag, uint8_t* state, hipStream_t s);
size_t err_scratch_bytes(int64_t P);
// The accuracy metric with scratch of its own kept between calls (see there);
// launch_flowmap_error: with the caller's.  Both wait for the stream.
hipError_t flowmap_error(int64_t P, const double* b, const uint8_t* bstate, const double* m, const uint8_t* mflag,
                         double out4[4], hipStream_t s);
hipError_t launch_flowmap_error(int64_t P, const double* b, const uint8_t* bstate, const double* m, const uint8_t* mflag,
                                void* scratch, double out4[4], hipStream_t s);
// This GPU's copy of the fixed scratch of the allocation-free metric (looked
// up on the first call on each device) and its size in bytes.
hipError_t err_static_scratch(void** ptr, size_t* bytes);
hipError_t launch_place(const int32_t mb[3], const int32_t M[3], const int32_t off[3], const double shift[3],
                        const double* src_xyz, const uint8_t* src_flag, double* dst_xyz, uint8_t* dst_flag,
                        hipStream_t s);
hipError_t launch_flowmap(const FlowmapArgs& a, int blocks_per_seg, hipStream_t s);
hipError_t launch_ckpt_store(const CkptArgs& a, int blocks_per_seg, hipStream_t s);

// Touched grid points per step (diagnostic walk of the seeds, one step per
// launch).
struct TouchArgs {
    Geom g;
    const char* f0;                 // grids of the step's two cycles
    const char* f1;
    double h;                       // step size
    int64_t P;                      // seeds
    const double* seed_xyz;         // P x 3 world
    double origin[3];
    double* x;                      // P x 3 positions, cell units
    uint8_t* alive;                 // P
    uint32_t* bits0;                // bitmaps of the block's points: level n,
    uint32_t* bits1;                //   level n + 1
    unsigned long long* out;        // the step's counters: points of level n, n + 1, particles entering
};
hipError_t launch_touch_init(const TouchArgs& a, hipStream_t s);
hipError_t launch_touch_step(const TouchArgs& a, int dtype, int mode, hipStream_t s);
hipError_t launch_touch_count(uint32_t* bits, size_t words, unsigned long long* out, hipStream_t s);
hipError_t launch_touch_zero(unsigned long long* p, size_t n, hipStream_t s);
int advect_max_blocks_per_cu(int dtype, int mode, int lanes_per_particle, int record_exit);
// The adjoint's launches, for the seeds p0 .. p0 + np - 1: its own forward from
// the seeds (tape and checkpoints where given); the tape of segments sg_last ..
// sg_first from their checkpoints, all segments at once; the reverse sweep
// over them.  mode: MODE_WIDE set for grids beyond 4 GiB.
hipError_t launch_adj_forward(const AdjointArgs& a, int dtype, int mode, hipStream_t s);
hipError_t launch_adj_tangent(const AdjointArgs& a, int dtype, int mode, hipStream_t s);  // see the kernel
hipError_t launch_adj_segments(const AdjointArgs& a, int dtype, int mode, hipStream_t s);  // see the kernel
hipError_t launch_adj_recompute(const AdjointArgs& a, int dtype, int mode, hipStream_t s);
hipError_t launch_adj_reverse(const AdjointArgs& a, int dtype, int mode, hipStream_t s);
// n 64-bit words from the host into device memory, as kernel arguments (no
// copy whose source would have to outlive the call).
hipError_t launch_put_words(uint64_t* dst, const uint64_t* src, size_t n, hipStream_t s);
// Mark all n record slots unused (before the adjoint sweep writes them).
hipError_t launch_grad_clear(const GradRec& r, uint64_t n, hipStream_t s);
// Scratch of the reduction: the sort's second key array, its two index arrays,
// nine colour bounds and a pair count, and radix_temp_bytes(n) of temp.
struct GradSort {
    void* key_alt;
    uint32_t* idx[2];
    uint32_t* bounds;
    void* temp;
};
// Sort the n record slots by key and add each (level, cell) group's sum to the
// grids, one parity colour at a time (no two cells of one colour share a corner).
hipError_t launch_grad_reduce(const GradRec& r, const GradSort& w, uint64_t n, float* const* gf, const Geom& g,
                              hipStream_t s);
hipError_t launch_ftle(const float* jac, int64_t P, double inv_T, float* out, hipStream_t s);
size_t rebin_temp_bytes(int64_t nbins_total);

// Device-wide exclusive scan of n counts (in != out; temp: scan_temp_bytes).
size_t scan_temp_bytes(uint64_t n);
hipError_t launch_exclusive_scan(const uint32_t* in, uint32_t* out, uint64_t n, void* temp, hipStream_t s);
// Stable LSD radix sort of the slots 0 .. n - 1 by the low `bits` bits of their
// keys; slots whose bit `bits` is set are left out.  The sorted keys and slot
// numbers end in (key, idx0) or (key_alt, idx1), as *result_in_alt says, their
// number in *count (device); temp: radix_temp_bytes.  key_bytes: 4 or 8.
size_t radix_temp_bytes(uint64_t n);
hipError_t launch_radix_sort_slots(void* key, void* key_alt, uint32_t* idx0, uint32_t* idx1, int key_bytes,
                                   uint64_t n, int bits, uint32_t* count, void* temp, bool* result_in_alt,
                                   hipStream_t s);
hipError_t launch_rebin(const RebinArgs& a, hipStream_t s);

}  // namespace bto
