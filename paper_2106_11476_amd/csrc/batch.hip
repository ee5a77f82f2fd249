// Batched 2D step of many domains (continuous batching): two launches a step
// over the LDS tiles (tile2d.hpp) of every active entry of a device table.
//
// 32 domains of 128..384 points a side (2.3 M points, L = 2..4): 71.2 us a step
// where 256-column row sweeps with a launch for the sources took 113.  What
// that took: tiles of 64 columns (few idle lanes on narrow grids), the entry
// found by a ballot, the entry's arguments in scalar registers and its tables
// by global (not flat) loads, registers for four blocks a CU (85 -> 60), no
// launch between the phases, and memory variables that stay in the cache (the
// last: 78.7 -> 71.2).  8 domains (0.36 M points): 16.7 against 26.6.
#include "tile2d.hpp"

#include <mutex>

// Batch table of fw2_batch_create_noalloc: file-scope device memory, one copy
// per GPU, held until the process ends.  In host code its name is only a
// stand-in: the device address of each GPU's copy comes from
// hipGetSymbolAddress with that GPU current (static_batch_table below).
static __device__ __align__(256) unsigned char scratch[sizeof(fw2::BatchTable)];

namespace fw2 {

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
void *g_static_ptr[kMaxDevices];       // device address of `scratch`, per device
bool g_static_busy[kMaxDevices];       // a no-allocation batch holds the table

}  // namespace

hipError_t claim_static_batch_table(int device, BatchTable **table, bool *busy)
{
    std::lock_guard<std::mutex> lock(g_static_mu);
    *table = nullptr;
    *busy = false;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_static_ptr[device]) {                  // once per device, with it current
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_static_ptr[device] = p;
    }
    if (g_static_busy[device]) {
        *busy = true;
        return hipSuccess;
    }
    g_static_busy[device] = true;
    *table = (BatchTable *)g_static_ptr[device];
    return hipSuccess;
}

void release_static_batch_table(int device)
{
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (device >= 0 && device < kMaxDevices) g_static_busy[device] = false;
}

namespace {

// The entry of tile t (the last whose first tile is not past t), with what
// decides the tile's work.  One lane per entry (a table holds at most 64) and
// a ballot: one memory latency, where walking the entries was a chain of up
// to 64 loads and every field another.
static_assert(kMaxBatch <= 64, "one lane per entry");
struct TileEntry {
    int d, tile, nbx, key;           // entry, tile within it
    long long step;
    bool active;
};
template <bool PRESSURE>
__device__ __forceinline__ TileEntry batch_entry_of_tile(const BatchTable *__restrict__ T, int t)
{
    const int lane = threadIdx.x % 64;
    const int base = T->tile_base[lane], nbx = T->nbx[lane], key = T->key[lane];
    const long long step = PRESSURE ? T->next[lane] : T->now[lane];
    const bool active = step < T->n_steps[lane];
    TileEntry r;
    r.d = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < T->n && base <= t)) - 1);
    r.tile = t - __builtin_amdgcn_readlane(base, r.d);
    r.nbx = __builtin_amdgcn_readlane(nbx, r.d);
    r.key = __builtin_amdgcn_readlane(key, r.d);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)step, r.d);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(step >> 32), r.d);
    r.step = (long long)(((uint64_t)hi << 32) | lo);
    r.active = (__ballot(active) >> r.d) & 1;
    return r;
}

template <int TY>
union BatchLds {
    PressureLds<TY> p;
    VelocityLds<TY> v;
};

template <bool PRESSURE, int L, bool C, bool PP, int TY>
__device__ __forceinline__ void batch_tile(const BatchEntry &e, int x0, int y0, long long step, BatchLds<TY> &lds)
{
    const StepArgs &a = e.a;
    if constexpr (PRESSURE) {
        const int n_src = step < a.src.n_t ? a.src.n : 0;
        pressure_tile<L, C, PP, TY>(a, x0, y0, a.src, n_src, step, lds.p);
    } else {
        velocity_tile<L, C, PP, TY>(a, x0, y0, lds.v);
    }
}

// Mechanism counts L0 .. L0 + 3 and both memory-variable schemes:
// key = (L - L0) * 2 + scheme (batch_key).
template <bool PRESSURE, int L0, bool PP, int TY>
__device__ __forceinline__ void batch_dispatch(int key, const BatchEntry &e, int x0, int y0, long long step,
                                               BatchLds<TY> &lds)
{
    switch (key) {
#define FW2_BCASE(K, DL, C) \
    case K: batch_tile<PRESSURE, L0 + DL, C, PP, TY>(e, x0, y0, step, lds); break;
    FW2_BCASE(0, 0, false) FW2_BCASE(1, 0, true) FW2_BCASE(2, 1, false) FW2_BCASE(3, 1, true)
    FW2_BCASE(4, 2, false) FW2_BCASE(5, 2, true) FW2_BCASE(6, 3, false) FW2_BCASE(7, 3, true)
#undef FW2_BCASE
    default: break;
    }
}

// One phase of the entries of one class of the table: CLASS bit 0 set for
// 5..8 mechanisms (else 1..4), bit 1 set for per-point stencil weights.
// Each class present gets a launch of its own, so that the larger register
// demand of many mechanisms or per-point weights does not lower the
// occupancy of the common class; entries are grouped by class, and each
// launch walks only its class's range of the tile list.  The first `extra`
// blocks (one per entry, in one of the phase's launches) keep the steps: in
// the pressure phase they copy next to now, which the velocity phase's tiles
// read; in the velocity phase they record the entry's receivers and move next
// and the domain's counter past the step, which no tile of that phase reads.
// T and W are the same table: the tiles read it through T, const, so that an
// entry's arguments load into scalar registers; only the extra blocks of the
// pressure phase write to it, a field that its tiles do not read.
template <bool PRESSURE, int TY, int CLASS>
__global__ void __launch_bounds__(kTX *TY, CLASS == 0 ? 8 : 4) batch_phase(const BatchTable *__restrict__ T, BatchTable *W, int extra)
{
    constexpr bool MANY = (CLASS & 1) != 0, PP = (CLASS & 2) != 0;
    if ((int)blockIdx.x < extra) {
        if ((int)blockIdx.x >= T->n) return;
        const int d = blockIdx.x;
        if (PRESSURE) {
            if (threadIdx.x == 0) W->now[d] = W->next[d];
            return;
        }
        const SparseArgs &r = T->e[d].a.rcv;
        const long long step = T->now[d];
        if (step < T->n_steps[d] && step < r.cap)
            for (int k = threadIdx.x; k < r.n; k += kTX * TY)
                r.trace[step * r.n + k] = r.p[padded_index(r.geo, r.idx[k])];
        if (threadIdx.x == 0) {
            r.step[0] = step + 1;
            W->next[d] = step + 1;
        }
        return;
    }
    __shared__ BatchLds<TY> lds;
    // the class's own tiles: entries are grouped by class, so they are one
    // contiguous range of the tile list
    const int begin = T->class_begin[CLASS], total = T->class_end[CLASS] - begin;
    // Blocks are dealt to the 8 XCDs round-robin; the blocks of XCD x take one
    // contiguous eighth of the range (the grid is a multiple of 8), so
    // neighbouring tiles (which share halo rows) meet in the same L2.
    const int b = (int)blockIdx.x - extra, grid = (int)gridDim.x - extra;
    const int x = b % 8, q = total / 8, rem = total % 8;
    const int start = x * q + min(x, rem), end = start + q + (x < rem ? 1 : 0);
    for (int t = start + b / 8; t < end; t += grid / 8) {
        const TileEntry e = batch_entry_of_tile<PRESSURE>(T, begin + t);
        if (!e.active) continue;                    // finished (uniform over the block)
        // the entry's arguments are read in place: the address is uniform
        // over the block, so they load into scalar registers as a kernel's
        // own arguments do
        batch_dispatch<PRESSURE, MANY ? 5 : 1, PP, TY>(e.key, T->e[e.d], (e.tile % e.nbx) * kTX, (e.tile / e.nbx) * TY,
                                                       e.step, lds);
        __syncthreads();                            // the LDS is reused by the next tile
    }
}

// Sources that the tiles do not add: kSourceBlocks blocks an entry (one block
// an entry was bound by its trips through a long list, 20 us for 4097 sources).
constexpr int kSourceBlocks = 16;
__global__ void __launch_bounds__(256) batch_sources(const BatchTable *__restrict__ T)
{
    const int d = blockIdx.y;
    if (d >= T->n) return;
    const SparseArgs &s = T->e[d].src;
    const long long step = T->now[d];
    if (step >= T->n_steps[d] || step >= s.n_t) return;
    for (int q = blockIdx.x * 256 + threadIdx.x; q < s.n; q += kSourceBlocks * 256) {
        const int64_t pi = padded_index(s.geo, s.idx[q]);
        s.p[pi] = s.p[pi] + s.w[q] * s.signals[(int64_t)s.sig[q] * s.n_t + step];
    }
}

// The entries' steps from the domains' own counters, once per call: the caller
// may have loaded a state, set a counter, stepped a member alone or replayed a
// graph of its own since.  One launch of one wavefront a call, so that the
// tiles of every step need not follow 64 pointers to find their entry's step
// (that chain is a second memory latency a tile).
__global__ void __launch_bounds__(64) batch_take_steps(BatchTable *W)
{
    const int d = threadIdx.x;
    if (d < W->n) W->next[d] = *W->e[d].a.rcv.step;
}

template <bool PRESSURE, int TY>
void launch_batch_phase(BatchTable *T, int n_entries, unsigned blocks, hipStream_t st)
{
    int extra = n_entries;                          // with the phase's first launch
#define FW2_CLASS(C)                                                                                          \
    if (const unsigned n = batch_blocks(blocks, C)) {                                                         \
        hipLaunchKernelGGL((batch_phase<PRESSURE, TY, C>), dim3(n + extra), dim3(kTX * TY), 0, st, T, T, extra); \
        extra = 0;                                                                                            \
    }
    FW2_CLASS(0) FW2_CLASS(1) FW2_CLASS(2) FW2_CLASS(3)
#undef FW2_CLASS
}

template <int TY>
void launch_batch_rows(BatchTable *T, int n_entries, bool sources, unsigned blocks, hipStream_t st)
{
    launch_batch_phase<true, TY>(T, n_entries, blocks, st);
    if (sources) hipLaunchKernelGGL(batch_sources, dim3(kSourceBlocks, n_entries), dim3(256), 0, st, T);
    launch_batch_phase<false, TY>(T, n_entries, blocks, st);
}

}  // namespace

hipError_t launch_batch_step(const BatchTable *T, int n_entries_max, int tile, unsigned blocks, hipStream_t st)
{
    BatchTable *t = const_cast<BatchTable *>(T);
    if (tile == kBatchTakeSteps)
        hipLaunchKernelGGL(batch_take_steps, dim3(1), dim3(kMaxBatch), 0, st, t);
    else if ((tile & ~kBatchSources) == 8)
        launch_batch_rows<8>(t, n_entries_max, (tile & kBatchSources) != 0, blocks, st);
    else
        launch_batch_rows<16>(t, n_entries_max, (tile & kBatchSources) != 0, blocks, st);
    return hipGetLastError();
}

}  // namespace fw2
