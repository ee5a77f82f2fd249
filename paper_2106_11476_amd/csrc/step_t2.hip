// 2D two-phase kernels from LDS tiles (tile2d.hpp), instantiated for every
// mechanism count, memory scheme and stencil mode.
#include "tile2d.hpp"

namespace fw2 {

namespace {

template <int L, bool C, bool PP, int TY>
__global__ void __launch_bounds__(kTX *TY) pressure_tiles(const StepArgs a, int nbx, int nblocks)
{
    __shared__ PressureLds<TY> lds;
    const int tile = tile_of_block(blockIdx.x, nblocks);
    long long step = 0;
    int n_src = 0;
    if (a.src.n > 0) {
        step = *a.src.step;
        n_src = step < a.src.n_t ? a.src.n : 0;
    }
    pressure_tile<L, C, PP, TY>(a, (tile % nbx) * kTX, (tile / nbx) * TY, a.src, n_src, step, lds);
}

template <int L, bool C, bool PP, int TY>
__global__ void __launch_bounds__(kTX *TY) velocity_tiles(const StepArgs a, int nbx, int nblocks)
{
    const int shift = a.rcv.step ? 1 : 0;            // with receivers, block 0 records them
    if ((int)blockIdx.x < shift) {
        record_receivers(a.rcv);
        return;
    }
    __shared__ VelocityLds<TY> lds;
    const int tile = tile_of_block((int)blockIdx.x - shift, nblocks);
    velocity_tile<L, C, PP, TY>(a, (tile % nbx) * kTX, (tile / nbx) * TY, lds);
}

// LDS set aside for each block of the 4-row tiles, so that a CU holds five of
// them.  Streaming 2 L + 5 arrays is bound by HBM, which serves fewer tiles in
// flight better: us per step, 8 rows / 4 rows, eight blocks a CU / 4 rows, five
// blocks: 4096 x 2048, L = 8 452 / 438 / 434; 6000 x 3000, L = 6 853 / 858 /
// 845; 2048^2, L = 6 185 / 190 / 183; 3000 x 1500, L = 5 166 / 164 / 164.
constexpr unsigned kReserve4 = 24000;

template <int L, bool C, bool PP, int TY>
hipError_t launch(const StepArgs &a, bool pressure, hipStream_t st)
{
    const int nbx = (a.geo.n[0] + kTX - 1) / kTX, nblocks = nbx * ((a.geo.n[1] + TY - 1) / TY);
    constexpr unsigned reserve = TY == 4 ? kReserve4 : 0;
    if (pressure)
        hipLaunchKernelGGL((pressure_tiles<L, C, PP, TY>), dim3(nblocks), dim3(kTX * TY), reserve, st, a, nbx, nblocks);
    else
        hipLaunchKernelGGL((velocity_tiles<L, C, PP, TY>), dim3(nblocks + (a.rcv.step ? 1 : 0)), dim3(kTX * TY), reserve,
                           st, a, nbx, nblocks);
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
