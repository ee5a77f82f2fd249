// 2D two-phase kernels from LDS tiles (tile2d.hpp), instantiated for every
// mechanism count, memory scheme and stencil mode.
#include "tile2d.hpp"

namespace fw2 {

namespace {

// The tile of a block by the launch's order of tiles: 0, each of the eight XCDs
// takes a contiguous band of them; > 0, the same, XCD x starting x * order tiles
// into its band (4 rows, band_shift); kSkewed, plain order, skewed by row.
constexpr int kSkewed = -1;
template <int TY>
__device__ __forceinline__ int tile_of(int bid, int nbx, int nblocks, int order)
{
    if (order == kSkewed) return skewed_tile(bid, nbx);
    return TY == 4 && order > 0 ? shifted_tile(bid, nblocks, order) : tile_of_block(bid, nblocks);
}

template <int L, bool C, bool PP, int TY, int TX>
__global__ void __launch_bounds__(TX *TY) pressure_tiles(const StepArgs a, int nbx, int nblocks, int order)
{
    __shared__ PressureLds<TY, TX> lds;
    const int tile = tile_of<TY>(blockIdx.x, nbx, nblocks, order);
    long long step = 0;
    int n_src = 0;
    if (a.src.n > 0) {
        step = *a.src.step;
        n_src = step < a.src.n_t ? a.src.n : 0;
    }
    pressure_tile<L, C, PP, TY, TX>(a, (tile % nbx) * TX, (tile / nbx) * TY, a.src, n_src, step, lds);
}

template <int L, bool C, bool PP, int TY, int TX>
__global__ void __launch_bounds__(TX *TY) velocity_tiles(const StepArgs a, int nbx, int nblocks, int order)
{
    const int rcv = a.rcv.step ? 1 : 0;              // with receivers, block 0 records them
    if ((int)blockIdx.x < rcv) {
        record_receivers(a.rcv);
        return;
    }
    __shared__ VelocityLds<TY, TX> lds;
    const int tile = tile_of<TY>((int)blockIdx.x - rcv, nbx, nblocks, order);
    velocity_tile<L, C, PP, TY, TX>(a, (tile % nbx) * TX, (tile / nbx) * TY, lds);
}

// The tiles of more than four mechanisms whose arrays pass the cache: 128
// columns by 4 rows, with LDS set aside so that a CU holds three blocks.
// Streaming 2 L + 5 arrays is bound by HBM, which serves fewer tiles in flight
// and longer rows better.  us per step, row sweeps of 256 columns by 4 rows /
// 64 x 8 / 64 x 4 with five blocks a CU / 128 x 4 with three, L = 6 and 8:
// 2000^2 170 / 174 / 168 / 165 and 212 / 225 / 216 / 210; 1000 x 4224 185 / - /
// 189 / 179 and 232 / - / 240 / 228; 4096 x 2048 338 / 344 / 335 / 333 and 438 /
// 452 / 432 / 427; 6000 x 3000 841 / 853 / 838 / 834 and 1073 / - / 1081 / 1060;
// over 37 sizes of 1.6 to 18 M points 3.6% faster than the sweeps (64 x 4: 2.3%),
// at most 1.2% slower where the rule below does not apply.
constexpr int kTX4 = 128;
constexpr unsigned kReserve4 = 40000;

// Where the bands of neighbouring XCDs start just under or at 33 x 64 KiB apart
// in each array, the eight streams meet in the same HBM channels; there each
// XCD starts its band three tile rows further in than the one before (two to
// eight rows do as well).  us per step, sweeps / 128 x 4 / shifted, L = 6 and 8:
// 2048^2 (33.0) 179 / 181 / 174 and 231 / 239 / 223; 2100 x 2048 (33.0) 188 / 192 /
// 180 and 243 / 246 / 230; 1900 x 2252 (32.8) 192 / 190 / 178 and 244 / 248 / 226;
// 1400 x 3072 (33.0) 192 / 186 / 178 and 246 / 240 / 227; 1000 x 4224 (33.0) 185 /
// 179 / 180 and 232 / 228 / 228.  On either side the shift loses: 2000 x 2048
// (32.0) 172 / 165 / 181, 3000 x 1440 (33.05) 185 / 179 / 185, 1900 x 2284 (33.3)
// 187 / 177 / 181, 2048 x 2112 (34.0) 184 / 174 / 178.
int band_shift(const Geometry &g, int nbx, int nblocks)
{
    const int64_t apart = (int64_t)(nblocks / 8) * 4 * g.pitch * 4 / nbx;
    return apart * 100 >= (int64_t)3275 * 65536 && apart * 100 <= (int64_t)3303 * 65536 ? 3 * nbx : 0;
}

// Arrays of a step past kPlainBytes (two mechanisms or more): tiles in plain
// order, skewed.  Bands keep the rows that neighbouring tiles share in one XCD's L2, but
// then eight bands stream from eight far places of every array, and the further
// past the last-level cache the arrays are, and the more of them are memory
// variables, which nothing shares, the more that costs.  us per step, bands /
// skewed (64 x 8 tiles; L = 6, 8: 128 x 4): L = 2 9000 x 2000 (968 MiB) 389 / 381,
// 12000 x 2000 623 / 518, 10000 x 4000 900 / 839, but 8100 x 4000 665 / 713; L = 3
// 3600^2 (904 MiB) 332 / 338, 6000 x 3000 508 / 480; L = 4 4096 x 2048 (718 MiB) 243 /
// 260, 3000 x 4000 (1012) 356 / 364, 2500 x 5000 (1076) 399 / 388, 12000 x 2000 992 /
// 757 (row sweeps, in plain order there, 792), 11900 x 2500 1129 / 943; L = 6 4096 x
// 2048 (978) 335 / 350, 3072^2 (1105) 488 / 388; L = 8 3000^2 472 / 466.  L = 1 gains
// and loses by as much (20000 x 2000 699 / 727, 30000 x 1200 635 / 608) and keeps
// its bands.
template <int L>
int tile_order(const Geometry &g, int nbx, int nblocks, int rows)
{
    if (L >= 2 && (6 + 4 * L) * g.stride * 4 > kPlainBytes) return kSkewed;
    return rows == 4 ? band_shift(g, nbx, nblocks) : 0;
}

template <int L, bool C, bool PP, int TY>
hipError_t launch(const StepArgs &a, bool pressure, hipStream_t st)
{
    constexpr int TX = TY == 4 ? kTX4 : kTX;
    constexpr unsigned reserve = TY == 4 ? kReserve4 : 0;
    const int nbx = (a.geo.n[0] + TX - 1) / TX, nblocks = nbx * ((a.geo.n[1] + TY - 1) / TY);
    const int order = tile_order<L>(a.geo, nbx, nblocks, TY);
    if (pressure)
        hipLaunchKernelGGL((pressure_tiles<L, C, PP, TY, TX>), dim3(nblocks), dim3(TX * TY), reserve, st, a, nbx, nblocks,
                           order);
    else
        hipLaunchKernelGGL((velocity_tiles<L, C, PP, TY, TX>), dim3(nblocks + (a.rcv.step ? 1 : 0)), dim3(TX * TY), reserve,
                           st, a, nbx, nblocks, order);
    return hipGetLastError();
}

template <int L>
hipError_t scheme_of(const StepArgs &a, int scheme, bool pressure, int rows, hipStream_t st)
{
    const bool pp = a.local_stencil != 0;
#define FW2_T(C, PP)                                                                                   \
    do {                                                                                               \
        if constexpr (L > 4)                                                                           \
            if (rows == 4) return launch<L, C, PP, 4>(a, pressure, st);                                \
        return rows == 8 ? launch<L, C, PP, 8>(a, pressure, st) : launch<L, C, PP, 16>(a, pressure, st); \
    } while (0)
    if (scheme == 0) {
        if (pp) FW2_T(false, true);
        FW2_T(false, false);
    }
    if (pp) FW2_T(true, true);
    FW2_T(true, false);
#undef FW2_T
}

}  // namespace

hipError_t launch_tiles_2d(const StepArgs &a, int L, int scheme, bool pressure, int rows, hipStream_t st)
{
    switch (L) {
    case 1: return scheme_of<1>(a, scheme, pressure, rows, st);
    case 2: return scheme_of<2>(a, scheme, pressure, rows, st);
    case 3: return scheme_of<3>(a, scheme, pressure, rows, st);
    case 4: return scheme_of<4>(a, scheme, pressure, rows, st);
    case 5: return scheme_of<5>(a, scheme, pressure, rows, st);
    case 6: return scheme_of<6>(a, scheme, pressure, rows, st);
    case 7: return scheme_of<7>(a, scheme, pressure, rows, st);
    case 8: return scheme_of<8>(a, scheme, pressure, rows, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fw2
