// 2D step of a small grid in one launch (both phases, sources and receivers).
//
// A grid of some 10^5 points is bound by latency: a step of three dependent
// launches costs three launch hand-overs, and a block that walks rows waits
// for memory once a row.  Here a block owns a 64 x TY tile: it loads
// everything the tile needs at once, advances the pressure on the tile and
// the few cells around it that its velocity points read (recomputing the
// neighbours' cells instead of waiting for them), and then the velocity, so a
// step is one launch with one exposed load latency.  The recomputed cells
// need the neighbours' old state, so the step runs out of place: from the
// block the arguments point at to the one a.out elements further.
// Per-point arithmetic is that of the two-phase sweeps (bitwise equal results).
//
// Bound by the load latency and the hand-over while every tile has a CU of its
// own (128^2, L = 2: 5.0 us a step; 480^2: 8.0), by the cache's bandwidth above
// (1536^2, L = 2: 45.7 us; a tile of 64 x 16 reads 1.6 times its cells, so the
// memory variables go through the caches plainly: with the non-temporal hint
// 1536^2 takes 63.4).
#include "step_kernels.hpp"

namespace fw2 {

namespace {

constexpr int kFX = 64;             // tile columns

// Cells of a tile (x0, y0) whose pressure its velocity points read: rows
// y0 - 1 .. y0 + TY over columns x0 - 3 .. x0 + 67, then the five rows above
// and below (y0 - 3, y0 - 2, y0 + TY + 1 .. y0 + TY + 3) over columns
// x0 - 1 .. x0 + 64: no corners, the cross terms reach one cell only.
template <int TY>
struct FusedTile {
    static constexpr int PW = kFX + 7, PH = TY + 7;                  // p rectangle from (x0 - 3, y0 - 3)
    static constexpr int N1 = PW * (TY + 2), NP = N1 + 5 * (kFX + 2);
    static constexpr int XW = kFX + 14, XH = TY + 9;                 // v_x from (x0 - 7, y0 - 4)
    static constexpr int YW = kFX + 9, YH = TY + 14;                 // v_y from (x0 - 4, y0 - 7)

    // (x - x0, y - y0) of cell e
    static __device__ __forceinline__ void cell(int e, int &x, int &y)
    {
        if (e < N1) {
            y = e / PW;
            x = e - y * PW - 3;
            y -= 1;
        } else {
            e -= N1;
            y = e / (kFX + 2);
            x = e - y * (kFX + 2) - 1;
            y = y < 2 ? y - 3 : TY - 1 + y;
        }
    }
    // cell index of (x - x0, y - y0), or -1
    static __device__ __forceinline__ int index(int x, int y)
    {
        if (y >= -1 && y <= TY) return x >= -3 && x <= kFX + 3 ? (y + 1) * PW + x + 3 : -1;
        if (x < -1 || x > kFX || y < -3 || y > TY + 3) return -1;
        return N1 + (y < 0 ? y + 3 : y + 1 - TY) * (kFX + 2) + x + 1;
    }
};

template <int L, bool CENTRED, bool PP, int TY, int NT, int WV>
__global__ void __launch_bounds__(NT, WV) fused_step2d(const StepArgs a, int nbx, int nblocks, int shift)
{
    // the receivers of the step before, from this step's input (the tiles
    // only read it); the counter stays at the first step of the chunk
    if ((int)blockIdx.x < shift) {
        const SparseArgs &s = a.rcv;
        const long long step = *s.step + s.off;
        if (step < s.cap)
            for (int r = threadIdx.x; r < s.n; r += NT) s.trace[step * s.n + r] = s.p[padded_index(s.geo, s.idx[r])];
        return;
    }
    using T = FusedTile<TY>;
    constexpr int kP = (T::NP + NT - 1) / NT;                        // pressure cells per thread
    constexpr int kX = (T::XW * T::XH + NT - 1) / NT, kY = (T::YW * T::YH + NT - 1) / NT;
    constexpr int kV = (kFX * TY + NT - 1) / NT;                     // velocity points per thread
    __shared__ float svx[T::XH * T::XW], svy[T::YH * T::YW], sp[T::PH * T::PW], sk[T::PH * T::PW];
    __shared__ int ssrc[T::NP];
    const Geometry &g = a.geo;
    const int tile = tile_of_block((int)blockIdx.x - shift, nblocks);
    const int x0 = (tile % nbx) * kFX, y0 = (tile / nbx) * TY;
    const int tid = threadIdx.x;
    const int nx = g.n[0], ny = g.n[1];

    // every load of the tile, in the order of use
    const long long step = *a.src.step + a.src.off;
    const bool active = a.src.n > 0 && step < a.src.n_t;
    float lx[kX], ly[kY];
    {
        const gbase bx = plane_base(a.v, g, 0), by = plane_base(a.v + g.stride, g, 0);
#pragma unroll
        for (int q = 0; q < kX; ++q) {
            const int e = tid + q * NT, r = e / T::XW, c = e - r * T::XW;
            lx[q] = e < T::XW * T::XH ? *at_plane(bx, plane_point(g, x0 - 7 + c, y0 - 4 + r)) : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kY; ++q) {
            const int e = tid + q * NT, r = e / T::YW, c = e - r * T::YW;
            ly[q] = e < T::YW * T::YH ? *at_plane(by, plane_point(g, x0 - 4 + c, y0 - 7 + r)) : 0.0f;
        }
    }
    struct PCell {
        int x, y, l;
        bool in;
        float p0, k0, q0, r0, m[2][L];
    } pc[kP];
#pragma unroll
    for (int q = 0; q < kP; ++q) {
        PCell &c = pc[q];
        const int e = tid + q * NT;
        T::cell(e, c.x, c.y);
        const int x = x0 + c.x, y = y0 + c.y;
        c.in = e < T::NP && (unsigned)x < (unsigned)nx && (unsigned)y < (unsigned)ny;
        if (c.in) {
            const uint32_t pt = plane_point(g, x, y);
            c.l = a.label ? label_at(plane_base(a.label, g, 0), pt) : 0;
            c.p0 = *at_plane(plane_base(a.p, g, 0), pt);
            c.k0 = *at_plane(plane_base(a.kap, g, 0), pt);
            c.q0 = *at_plane(plane_base(a.nlq, g, 0), pt);
            c.r0 = PP ? *at_plane(plane_base(a.rho, g, 0), pt) : 1.0f;
#pragma unroll
            for (int ax = 0; ax < 2; ++ax)
#pragma unroll
                for (int nu = 0; nu < L; ++nu)
                    c.m[ax][nu] = *at_plane(plane_base(a.psi2 + (int64_t)(ax * L + nu) * g.stride, g, 0), pt);
        }
    }
    struct VPoint {
        int l;
        float r0, rx, ry, m[2][L];
    } vp[kV];
#pragma unroll
    for (int q = 0; q < kV; ++q) {
        VPoint &v = vp[q];
        const int t = tid + q * NT, i = x0 + t % kFX, j = y0 + t / kFX;
        if (t < kFX * TY && i < nx && j < ny) {
            const uint32_t pt = plane_point(g, i, j);
            const gbase br = plane_base(a.rho, g, 0);
            v.l = a.label ? label_at(plane_base(a.label, g, 0), pt) : 0;
            v.r0 = *at_plane(br, pt);
            v.rx = *at_plane(br, plane_point(g, i + 1, j));
            v.ry = *at_plane(br, plane_point(g, i, j + 1));
#pragma unroll
            for (int ax = 0; ax < 2; ++ax)
#pragma unroll
                for (int nu = 0; nu < L; ++nu)
                    v.m[ax][nu] = *at_plane(plane_base(a.psi1 + (int64_t)(ax * L + nu) * g.stride, g, 0), pt);
        }
    }

    if (active) {                                    // the sources of this tile's cells
        for (int e = tid; e < T::NP; e += NT) ssrc[e] = 0;
        __syncthreads();
        for (int q = tid; q < a.src.n; q += NT) {
            const uint32_t f = (uint32_t)a.src.idx[q];
            const int y = (int)(f / (uint32_t)nx), x = (int)(f - (uint32_t)y * (uint32_t)nx);
            const int e = T::index(x - x0, y - y0);
            if (e >= 0) ssrc[e] = q + 1;
        }
    }
#pragma unroll
    for (int q = 0; q < kX; ++q)
        if (tid + q * NT < T::XW * T::XH) svx[tid + q * NT] = lx[q];
#pragma unroll
    for (int q = 0; q < kY; ++q)
        if (tid + q * NT < T::YW * T::YH) svy[tid + q * NT] = ly[q];
    __syncthreads();

    // pressure phase
#pragma unroll
    for (int q = 0; q < kP; ++q) {
        PCell &c = pc[q];
        const int e = tid + q * NT;
        if (e >= T::NP) break;
        const int at = (c.y + 3) * T::PW + c.x + 3;
        float pn = 0.0f;
        if (c.in) {
            const int x = x0 + c.x, y = y0 + c.y;
            const Wts W = weights<PP>(a, PP ? cell_r2(a, c.r0, c.k0) : 0.0f);
            const float *X = &svx[(c.y + 4) * T::XW + c.x + 7];
            float Dx = W.g0 * (X[0] - X[-1]);
            Dx = fmaf(W.g1, X[1] - X[-2], Dx);
            Dx = fmaf(W.g2, X[2] - X[-3], Dx);
            Dx = fmaf(W.g3, X[3] - X[-4], Dx);
            Dx = fmaf(W.g11, (X[T::XW] - X[T::XW - 1]) + (X[-T::XW] - X[-T::XW - 1]), Dx);
            const float *Y = &svy[(c.y + 7) * T::YW + c.x + 4];
            float Dy = W.g0 * (Y[0] - Y[-T::YW]);
            Dy = fmaf(W.g1, Y[T::YW] - Y[-2 * T::YW], Dy);
            Dy = fmaf(W.g2, Y[2 * T::YW] - Y[-3 * T::YW], Dy);
            Dy = fmaf(W.g3, Y[3 * T::YW] - Y[-4 * T::YW], Dy);
            Dy = fmaf(W.g11, (Y[1] - Y[1 - T::YW]) + (Y[-1] - Y[-1 - T::YW]), Dy);
            const int sx = max(max(a.nb[0] - x, x - (nx - 1 - a.nb[0])), 0);
            const int sy = max(max(a.nb[1] - y, y - (ny - 1 - a.nb[1])), 0);
            float S = 0.0f;
#pragma unroll
            for (int ax = 0; ax < 2; ++ax) {
                const float D = ax == 0 ? Dx : Dy;
                const int tt = (ax == 0 ? sx : sy) * a.n_labels + c.l;
                const float2 *__restrict__ bc = a.bc2[ax] + (int64_t)tt * L;
                float Sa = a.w2[ax][tt] * D;
#pragma unroll
                for (int nu = 0; nu < L; ++nu) {
                    const float2 b = bc[nu];
                    const float mn = fmaf(b.x, c.m[ax][nu], b.y * D);
                    Sa += CENTRED ? c.m[ax][nu] : mn;
                    c.m[ax][nu] = mn;
                }
                S += Sa;
            }
            const float kappa = c.k0 * (1.0f + c.q0 * c.p0);
            pn = c.p0 - a.dt * S / kappa;
            if (active && ssrc[e]) {
                const int s = ssrc[e] - 1;
                pn = fmaf(a.src.w[s], a.src.signals[(int64_t)a.src.sig[s] * a.src.n_t + step], pn);
            }
            if (c.x >= 0 && c.x < kFX && c.y >= 0 && c.y < TY) {     // the tile's own cells
                const uint32_t pt = plane_point(g, x, y);
                *at_plane_w(plane_base(a.p + a.out, g, 0), pt) = pn;
#pragma unroll
                for (int ax = 0; ax < 2; ++ax)
#pragma unroll
                    for (int nu = 0; nu < L; ++nu)
                        *at_plane_w(plane_base(a.psi2 + a.out + (int64_t)(ax * L + nu) * g.stride, g, 0), pt) =
                            c.m[ax][nu];
            }
        }
        sp[at] = pn;
        sk[at] = c.in ? c.k0 : 0.0f;
    }
    __syncthreads();

    // velocity phase
#pragma unroll
    for (int q = 0; q < kV; ++q) {
        VPoint &v = vp[q];
        const int t = tid + q * NT, tx = t % kFX, ty = t / kFX, i = x0 + tx, j = y0 + ty;
        if (t >= kFX * TY || i >= nx || j >= ny) break;
        const uint32_t pt = plane_point(g, i, j);
        const float *P = &sp[(ty + 3) * T::PW + tx + 3], *K = &sk[(ty + 3) * T::PW + tx + 3];
        const float s0 = PP ? cell_r2(a, v.r0, K[0]) : 0.0f;
#pragma unroll
        for (int ax = 0; ax < 2; ++ax) {
            if (ax == 0 ? i == nx - 1 : j == ny - 1) continue;       // outside the grid, held at zero
            constexpr int PW = T::PW;
            const int o = ax == 0 ? 1 : PW;
            const float rn = ax == 0 ? v.rx : v.ry;
            const Wts W = weights<PP>(a, PP ? 0.5f * (s0 + cell_r2(a, rn, K[o])) : 0.0f);
            float D = W.g0 * (P[o] - P[0]);
            D = fmaf(W.g1, P[2 * o] - P[-o], D);
            D = fmaf(W.g2, P[3 * o] - P[-2 * o], D);
            D = fmaf(W.g3, P[4 * o] - P[-3 * o], D);
            if (ax == 0)
                D = fmaf(W.g11, (P[PW + 1] - P[PW]) + (P[1 - PW] - P[-PW]), D);
            else
                D = fmaf(W.g11, (P[PW + 1] - P[1]) + (P[PW - 1] - P[-1]), D);
            const int s = ax == 0 ? max(max(a.nb[0] - i, i - (nx - 2 - a.nb[0])), 0)
                                  : max(max(a.nb[1] - j, j - (ny - 2 - a.nb[1])), 0);
            const int tt = s * a.n_labels + v.l;
            const float2 *__restrict__ bc = a.bc1[ax] + (int64_t)tt * L;
            float S = a.w1[ax][tt] * D;
#pragma unroll
            for (int nu = 0; nu < L; ++nu) {
                const float2 b = bc[nu];
                const float mn = fmaf(b.x, v.m[ax][nu], b.y * D);
                S += CENTRED ? v.m[ax][nu] : mn;
                v.m[ax][nu] = mn;
            }
            const float pbar = 0.5f * (P[0] + P[o]);
            const float rho_a = 0.5f * (v.r0 + rn);
            const float kap_a = 0.5f * (K[0] + K[o]);
            const float u = ax == 0 ? svx[(ty + 4) * T::XW + tx + 7] : svy[(ty + 7) * T::YW + tx + 4];
            *at_plane_w(plane_base(a.v + a.out + (int64_t)ax * g.stride, g, 0), pt) =
                u - a.dt * S / (rho_a * (1.0f + (a.nlA * kap_a) * pbar));
#pragma unroll
            for (int nu = 0; nu < L; ++nu)
                *at_plane_w(plane_base(a.psi1 + a.out + (int64_t)(ax * L + nu) * g.stride, g, 0), pt) = v.m[ax][nu];
        }
    }
}

template <int L, bool C, bool PP, int TY, int NT, int WV>
hipError_t launch_tiles(const StepArgs &a, hipStream_t st)
{
    const int shift = a.rcv.n > 0 && a.rcv.off >= 0 ? 1 : 0;         // receivers of the step before
    const int nbx = (a.geo.n[0] + kFX - 1) / kFX, nblocks = nbx * ((a.geo.n[1] + TY - 1) / TY);
    hipLaunchKernelGGL((fused_step2d<L, C, PP, TY, NT, WV>), dim3(nblocks + shift), dim3(NT), 0, st, a, nbx, nblocks,
                       shift);
    return hipGetLastError();
}

// Tile rows 8 or 16 (one_launch_rows in fw2.cpp picks them).  NT covers a
// tile's pressure cells in two passes and its velocity points in one; WV asks
// for the registers that let two blocks of 1024 threads share a CU where that
// does not spill (62 registers at L <= 2; above, such grids take two phases).
template <int L, bool C, bool PP>
hipError_t launch_fused(const StepArgs &a, const KernelConfig &kc, hipStream_t st)
{
    if (kc.rows == 8) return launch_tiles<L, C, PP, 8, 576, 1>(a, st);
    if (kc.rows == 16) return launch_tiles<L, C, PP, 16, 1024, L <= 2 ? 8 : 1>(a, st);
    return hipErrorInvalidValue;
}

template <int L>
hipError_t fused_scheme(const StepArgs &a, int scheme, const KernelConfig &kc, hipStream_t st)
{
    const bool pp = a.local_stencil != 0;
    if (scheme == 0) return pp ? launch_fused<L, false, true>(a, kc, st) : launch_fused<L, false, false>(a, kc, st);
    return pp ? launch_fused<L, true, true>(a, kc, st) : launch_fused<L, true, false>(a, kc, st);
}

}  // namespace

hipError_t launch_fused_2d(const StepArgs &a, int L, int scheme, const KernelConfig &kc, hipStream_t st)
{
    switch (L) {
    case 1: return fused_scheme<1>(a, scheme, kc, st);
    case 2: return fused_scheme<2>(a, scheme, kc, st);
    case 3: return fused_scheme<3>(a, scheme, kc, st);
    case 4: return fused_scheme<4>(a, scheme, kc, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fw2
