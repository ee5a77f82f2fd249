// Device data layout and kernel launchers of libfw2.
//
// Every per-point array (fields, memory variables, medium, labels) uses one
// padded layout: a 4-cell zero halo on each side of every axis, rows of
// `pitch` elements (a multiple of 64, so rows start on 256-byte boundaries),
// planes of `plane` = pitch * (ny + 8) elements (3D).  Element (x, y, z) is at
// origin + z * plane + y * pitch + x, and the arrays are placed so that x = 0
// of every row is 256-byte aligned.  The halo of p and v is never written, so
// stencil taps read zero outside the grid without bounds checks.  A slab of a
// grid split along z is the exception: its z halo planes hold the
// neighbouring slabs' planes, written by the halo exchange.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace fw2 {

constexpr int kHalo = 4;

// Memory variables are read and written once per step, by one kernel.  Where
// the arrays of a step exceed the last-level cache, non-temporal accesses keep
// them from displacing the stencil fields that the other kernel of the step
// reads back; where they fit, plain ones leave them there for the next step
// (2D tiles, StepArgs::stream).
__device__ __forceinline__ float ntld(const float *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void ntst(float *p, float v) { __builtin_nontemporal_store(v, p); }

struct Geometry {
    int32_t ndim;
    int32_t n[3];            // nx, ny, nz (nz = 1 in 2D)
    int64_t pitch, plane;    // element strides of y and z
    int64_t origin;          // element offset of (0, 0, 0)
    int64_t stride;          // elements between consecutive arrays
};

struct SparseArgs {
    Geometry geo;
    float *p;
    long long *step;         // device step counter
    const int64_t *idx;      // flat unpadded indices
    const int32_t *sig;      // sources: signal of each point
    const float *w;          // sources: weight of each point
    const float *signals;    // sources: [n_sig][n_t]
    float *trace;            // receivers: [cap][n]
    int32_t n;               // points
    int32_t n_t;             // sources: samples per signal
    int32_t off;             // this launch's step past the device counter
    long long cap;           // receivers: trace rows
};

struct StepArgs {
    Geometry geo;
    float *p;
    float *v;                // v_a = v + a * stride
    float *psi1;             // psi1[a][nu] = psi1 + (a * L + nu) * stride
    float *psi2;
    // Element offset from the fields a phase reads to those it writes: 0 steps
    // in place; an out-of-place step reads one state block and writes the next.
    int64_t out;
    const float *kap;        // kappa0 = 1 / (rho c^2)
    const float *nlq;        // kappa0 B, B = 1 - 2 beta as printed
    const float *rho;        // rho0
    const uint8_t *label;    // nullptr: a single relaxation tuple
    int32_t n_labels;
    int32_t stream;          // 2D tiles: memory variables by non-temporal accesses
    int32_t nb[3];           // boundary cells per axis
    const float *w2[3];      // pressure-point tables per axis: [slot][label]
    const float2 *bc2[3];    //   [slot][label][nu] (b, c)
    const float *w1[3];      // velocity-point tables per axis
    const float2 *bc1[3];
    float g[4];              // g_m0 / h
    float g11;               // g_11 / h
    float dt;
    // Momentum multiplier rho_a (1 + nlA kappa0_a pbar); nlA = 1 as printed.
    // (The mass multiplier's coefficient is folded into nlq.)
    float nlA;
    // Slab of a grid split along z: local plane k is global plane k + z_off
    // of nz_glob planes (the boundary layer and the last v_z sample follow
    // the global index).  A whole grid has z_off = 0, nz_glob = n[2].
    int32_t z_off, nz_glob;
    // Per-point stencil weights (local_stencil != 0): with s = r^2 of the
    // point, g_m0(s) / h = sum_k pw[m-1][k] s^k and g_11(s) / h = g11s * s;
    // a cell's s = q2 / (rho kappa0), q2 = (dt / h)^2.
    int32_t local_stencil;
    float pw[4][4];
    float g11s;
    float q2;
    // Receivers recorded (and the step counter advanced) by one extra block
    // of the velocity sweep launch, which reads p without writing it and runs
    // after the sources; rcv.step == nullptr: a separate launch does it.
    SparseArgs rcv;
    // Sources, for the kernels that add them in the pressure phase themselves.
    SparseArgs src;
};

// Kernel variant and tile shape.  variant 0: one thread per point over a
// (64 x 8) tile, every stencil tap a cached global load (any ndim).
// 3D: variant 1, plane sweeps of a column tile (32x16, 64x8 or 16x16 for bx =
// 32, 64, 16) over `rows` planes with a register window along z and LDS plane
// rings (each of the three adds the sources in a.src in its pressure phase);
// variant 2, the same with every load of the next plane issued during
// the current one; variant 3, only the staged planes and the z window one
// plane ahead, the point's own values at the top of their plane.
// 2D: variant 4 (at most four mechanisms), a whole step out of place in one
// launch of 64 x `rows` tiles (step_f2.hip), passed to launch_pressure;
// variant 5, the phases from LDS tiles of 64 x 8, 64 x 16 or (rows = 4, only
// with more than four mechanisms) 128 x 4 (step_t2.hip), the pressure phase
// adding the sources in a.src.
struct KernelConfig {
    int variant;
    int bx;
    int rows;
    int by = 0;              // 3D: tile rows in y (0: the default of bx)
};

// Tile of block `bid` where XCD x (blocks dealt round-robin) takes one
// contiguous band of the nblocks tiles and starts x * shift tiles into it, going
// on at the band's start past its end.  A bijection of [0, nblocks).
__host__ __device__ inline int shifted_tile(int bid, int nblocks, int shift)
{
    const int x = bid % 8, rem = nblocks % 8, count = nblocks / 8 + (x < rem ? 1 : 0);
    return x * (nblocks / 8) + (x < rem ? x : rem) + (bid / 8 + x * shift) % count;
}

// Tile of block `bid` in plain order over rows of nbx tiles, each row starting
// five tiles further on than the one before, so that a column of tiles does not
// stay on one XCD.  A bijection of whole rows.
__host__ __device__ inline int skewed_tile(int bid, int nbx)
{
    const int row = bid / nbx;
    return row * nbx + (bid - row * nbx + 5 * row) % nbx;
}

// Many 2D domains advanced by one launch per phase (batched serving).  The
// table lives in device memory; the blocks of a grid sized for the tiles of
// all entries walk them, so a captured step loop does not depend on which
// domains are active.  A domain whose step counter has reached n_steps is
// skipped (its counter keeps counting while it stays in the table).
constexpr int kMaxBatch = 64;
// Sources: added by the tiles of a kernel, each of which reads the list, or by
// a launch of their own.  The tiles take them up to kTileSources (2D) or
// kTileSources3 (3D sweeps, which list a tile's sources in LDS) and up to
// kScanPairs pairs of a tile and a source (over all entries of a batch), where
// the reading costs what the launch does.  us a step by the tiles / a launch
// (the one-launch step / two phases): reverse step 1536^2, L = 2, 2.4 M pairs
// 103.6 / 105.0, 4.7 M 104.2, 9.4 M 108.0, 19 M 112.0; one-launch step 1500^2,
// L = 2, 2.3 M 47.8 / 52.3, 4.6 M 50.0 / 52.4, 9.2 M 54.1 / 52.5; 1900^2, L = 1,
// 3.7 M 58.0 / 60.0, 7.3 M 61.0 / 59.8, 15 M 66.4 / 60.2; batch of one 2048^2,
// L = 4, 4.2 M 137.7 / 138.9, 17 M 145.6 / 140.0, of eight 384^2, L = 3, 4.7 M
// 45.0 / 43.4; two phases 4096 x 2048, L = 4, 21 M pairs 12 us a step more than
// without sources, the launch 4.5.
constexpr int32_t kTileSources = 4096;
constexpr int32_t kTileSources3 = 1024;
constexpr int64_t kScanPairs = (int64_t)4 << 20;

// a.src holds the sources that the tiles add (n = 0: none), src those that a
// launch of their own adds; a.rcv the receivers.
struct BatchEntry {
    StepArgs a;
    SparseArgs src;
};

struct BatchTable {
    int32_t n;
    // Entries are ordered by launch class; the tiles of class c are
    // [class_begin[c], class_end[c]) of the tile list.
    int32_t class_begin[4], class_end[4];
    // What a block needs to find its tile's entry and whether it is active,
    // one lane per entry: the first tile, tiles per row, mechanisms and memory
    // scheme (batch_key), the step to stop at, the next step (the domain's
    // device counter, taken anew at the start of every call) and the step
    // under way.
    int32_t tile_base[kMaxBatch], nbx[kMaxBatch], key[kMaxBatch];
    long long n_steps[kMaxBatch], next[kMaxBatch], now[kMaxBatch];
    BatchEntry e[kMaxBatch];
};

// Launch class of a batch entry: bit 0 for 5..8 mechanisms, bit 1 for
// per-point stencil weights.
__host__ __device__ inline int batch_class(int L, int local_stencil)
{
    return (L > 4 ? 1 : 0) | (local_stencil ? 2 : 0);
}

// Mechanisms 1..4 or 5..8 (by class) and scheme of an entry.
inline int batch_key(int L, int scheme) { return ((L - 1) % 4) * 2 + scheme; }

// Blocks of each class launch, a byte per class: 0 for none, else a count
// (8 + m) << e as e * 8 + m + 1, at least the class's tiles (and at most 1/8
// over; every count is a multiple of 8).
inline unsigned batch_blocks(unsigned code, int c)
{
    const unsigned v = (code >> (8 * c)) & 255u;
    return v == 0 ? 0u : (8u + (v - 1u) % 8u) << ((v - 1u) / 8u);
}
inline unsigned batch_code(int tiles, int c)
{
    if (tiles <= 0) return 0;
    for (unsigned v = 3 * 8 + 1;; ++v)               // from 64 blocks up
        if (batch_blocks(v, 0) >= (unsigned)tiles) return v << (8 * c);
}

// One step of every entry.  tile: the tile rows (8 or 16), with kBatchSources
// where the sources are added by a launch of their own; blocks: batch_code of
// every class, or-ed.  tile = kBatchTakeSteps instead moves no entry and takes
// their steps from the domains' counters.
constexpr int kBatchSources = 256, kBatchTakeSteps = 512;
hipError_t launch_batch_step(const BatchTable *dev_table, int n_entries_max, int tile, unsigned blocks,
                             hipStream_t stream);
// The library's own batch table on `device` (the current device), for a
// batch that allocates nothing: *busy is set (and *table left NULL) while
// another such batch holds it.  Released by release_static_batch_table.
hipError_t claim_static_batch_table(int device, BatchTable **table, bool *busy);
void release_static_batch_table(int device);

// Discrete adjoint of one step (adjoint.hip): device arrays of the adjoint
// state (same layout as the forward state block) and the per-step temporaries.
struct AdjointBuffers {
    float *lp, *pp, *pq, *sS, *lDv, *lqr, *lDp, *gk, *out;
};
// One reverse step.  state: forward state block at the step's input;
// state_prev: that of the step before, or nullptr.  have_pp: b.pp / b.sS
// already hold this step's p'' and S (from the previous call); *pp_next is
// set when b.pq / b.sS now hold those of step - 1 (the caller then swaps
// b.pp and b.pq).
hipError_t launch_adjoint_step(const StepArgs &f, const SparseArgs &src, const SparseArgs &rcv, int L,
                               const float *state, const float *state_prev, const AdjointBuffers &b,
                               long long step, bool have_pp, const float *residual, hipStream_t stream,
                               bool *pp_next);
hipError_t launch_adjoint_gradient(const StepArgs &f, const AdjointBuffers &b, hipStream_t stream);

// Per-dimension, per-phase launchers (step_p2/v2/p3/v3.hip), called by
// launch_pressure / launch_velocity.
hipError_t launch_pressure_2d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);
hipError_t launch_velocity_2d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);
hipError_t launch_pressure_3d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);
hipError_t launch_velocity_3d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);

hipError_t launch_tiles_2d(const StepArgs &a, int L, int scheme, bool pressure, int rows, hipStream_t stream);
hipError_t launch_fused_2d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);

// Launchers (kernels.hip).  All enqueue on `stream` and return the launch error.
hipError_t launch_pressure(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);
hipError_t launch_velocity(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t stream);
hipError_t launch_sources(const SparseArgs &s, hipStream_t stream);
hipError_t launch_receivers(const SparseArgs &s, hipStream_t stream);   // also advances the counter
hipError_t launch_fill(float *dst, int64_t n, float value, hipStream_t stream);
hipError_t launch_check(const float *p, const Geometry &g, float limit, int *flag, hipStream_t stream);
hipError_t launch_set_counter(long long *counter, long long value, hipStream_t stream);

// Planes packed or unpacked in one launch (halo.hip): the halo planes of a
// slab, or whole fields (fw2_read_fields / fw2_write_fields with device
// memory).  A set lists `n` ranges, each of `reps` consecutive arrays (one
// stride apart) from arr with planes [z0, z0 + nz); pack gathers their
// unpadded [ny][nx] planes in order into dst, unpack scatters src back into
// the same planes.  per_axis > 0 marks velocity points: array r of the range
// belongs to axis r / per_axis, and an unpack leaves out its last sample
// along that axis (outside the grid, held at zero).
struct PlaneSet {
    const float *arr[4];
    int32_t z0[4];
    int32_t nz[4];
    int32_t reps[4];
    int32_t per_axis[4];
    int32_t n;
    int32_t total;           // planes: sum of nz * reps

    void add(const float *a, int first, int count, int arrays = 1, int arrays_per_axis = 0)
    {
        arr[n] = a;
        z0[n] = first;
        nz[n] = count;
        reps[n] = arrays;
        per_axis[n] = arrays_per_axis;
        total += count * arrays;
        n++;
    }
};
hipError_t launch_pack(const PlaneSet &s, const Geometry &g, float *dst, hipStream_t stream);
hipError_t launch_unpack(const PlaneSet &s, const Geometry &g, const float *src, hipStream_t stream);

// Medium from device maps (halo.hip): kappa0 = 1/(rho c^2), kappa0 (B0 + B1
// beta) and rho into the padded arrays (FP64 arithmetic, FP32 results, the
// host conversion's operation order), labels copied; stats[0] / [1] receive
// the bits of the largest / smallest c (atomics on the bit patterns of
// positive floats) and stats[2] a nonzero flag for an invalid sample.
struct MediumArgs {
    Geometry geo;
    const float *c, *rho, *beta;
    const uint8_t *label;    // nullptr: none
    float *kap, *nlq, *rhop;
    uint8_t *labp;           // nullptr: not stored
    double B0, B1;
    int32_t n_labels;
    unsigned int *stats;     // [3], zeroed by the caller
};
hipError_t launch_medium(const MediumArgs &m, hipStream_t stream);

}  // namespace fw2
