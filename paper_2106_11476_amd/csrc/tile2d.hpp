// 2D phases from LDS tiles of TX = 64 (or 128) columns x TY rows, one thread a
// point.
//
// A block issues every load of its tile at once (the stencil field's window
// with its halo, the point's own values), so a tile costs one exposed load
// latency, and stencil taps come from LDS.  Bound by HBM streaming on large
// grids, by the cache's bandwidth where the arrays stay there, by that latency
// on small ones.  They replace row sweeps (256 columns, a register window along
// y, one exposed latency and one barrier a row); us per step, sweeps against
// tiles of 8 rows: 128^2, L = 2 13.8 / 6.4; 1536^2, L = 4 83.8 / 67.9; 2400 x
// 2300, L = 1 99.8 / 84.0; 1237 x 893, L = 8, per-point weights 76.1 / 59.1;
// 4096 x 2048, L = 4 247 / 235-243 (6.3 TB/s of its 182 B a point); 8192 x
// 4096, L = 2 886 / 749.  Tiles of 16 rows: 254 at 4096 x 2048, L = 4, 762 at
// 8192 x 4096, 287 against 290-300 at 3072^2, L = 3; of 4 rows 241, 787, 291.
// (step_t2.hip has the tile of more than four mechanisms past the cache.)
#pragma once

#include "step_kernels.hpp"

namespace fw2 {

namespace {

// the overloads for generic pointers beside those for global ones
using fw2::ntld;
using fw2::ntst;

constexpr int kTX = 64;             // tile columns, where not said

// (W x H) window of a 2D array with corner (xs, ys), loaded into registers and
// stored to LDS; cells outside the grid are zero (the array's halo corner).
template <int W, int H, int NT>
struct Window {
    static constexpr int N = (W * H + NT - 1) / NT;
    float r[N];
    __device__ __forceinline__ void load(const float *f, const Geometry &g, int xs, int ys, int tid)
    {
        const gbase base = plane_base(f, g, 0);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int e = tid + q * NT, row = e / W;
            if (e < W * H) r[q] = *at_plane(base, plane_point(g, xs + e - row * W, ys + row));
        }
    }
    __device__ __forceinline__ void store(float *dst, int tid) const
    {
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (tid + q * NT < W * H) dst[tid + q * NT] = r[q];
    }
};

// The values at point pt of N consecutive arrays from f.  The empty
// asm statements keep the compiler from merging the two branches, which would
// drop the hint.
#define FW2_BRANCH(name) asm volatile("; " name ::: "memory")
template <int N>
__device__ __forceinline__ void load_memory(float *m, const float *f, const Geometry &g, uint32_t pt, bool stream)
{
    if (stream) {
        FW2_BRANCH("stream");
#pragma unroll
        for (int q = 0; q < N; ++q) m[q] = ntld(at_plane(plane_base(f + q * g.stride, g, 0), pt));
        FW2_BRANCH("stream end");
    } else {
        FW2_BRANCH("cached");
#pragma unroll
        for (int q = 0; q < N; ++q) m[q] = *at_plane(plane_base(f + q * g.stride, g, 0), pt);
        FW2_BRANCH("cached end");
    }
}
template <int N>
__device__ __forceinline__ void store_memory(const float *m, float *f, const Geometry &g, uint32_t pt, bool stream)
{
    if (stream) {
        FW2_BRANCH("stream");
#pragma unroll
        for (int q = 0; q < N; ++q) ntst(at_plane_w(plane_base(f + q * g.stride, g, 0), pt), m[q]);
        FW2_BRANCH("stream end");
    } else {
        FW2_BRANCH("cached");
#pragma unroll
        for (int q = 0; q < N; ++q) *at_plane_w(plane_base(f + q * g.stride, g, 0), pt) = m[q];
        FW2_BRANCH("cached end");
    }
}
#undef FW2_BRANCH

// LDS of a pressure tile: v_x and v_y with the reach of D^- (4 cells before,
// 3 after, 1 across) and the tile's sources; of a velocity tile: p with the
// reach of D^+ (3 before, 4 after, 1 across).
template <int TY, int TX = kTX>
struct PressureLds {
    static constexpr int XW = TX + 7, XH = TY + 2, YW = TX + 2, YH = TY + 7;
    float x[XW * XH], y[YW * YH];
    int src[TX * TY];
};
template <int TY, int TX = kTX>
struct VelocityLds {
    static constexpr int PW = TX + 7, PH = TY + 7;
    float p[PW * PH];
};

// Pressure phase of the tile at (x0, y0).  s: sources to add, of step `step`
// (s.n = 0: none).  All threads of the block call it.
template <int L, bool CENTRED, bool PP, int TY, int TX>
__device__ __forceinline__ void pressure_tile(const StepArgs &a, int x0, int y0, const SparseArgs &s, int n_src,
                                              long long step, PressureLds<TY, TX> &lds)
{
    using T = PressureLds<TY, TX>;
    constexpr int NT = TX * TY;
    const Geometry &g = a.geo;
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX, i = x0 + tx, j = y0 + ty;
    const int nx = g.n[0], ny = g.n[1];
    const bool live = i < nx && j < ny;
    const uint32_t pt = plane_point(g, i, j);
    Window<T::XW, T::XH, NT> wx;
    Window<T::YW, T::YH, NT> wy;
    wx.load(a.v, g, x0 - 4, y0 - 1, tid);
    wy.load(a.v + g.stride, g, x0 - 1, y0 - 4, tid);
    int l = 0;
    float p0 = 0.0f, k0 = 1.0f, q0 = 0.0f, r0 = 1.0f, m[2][L];
    if (live) {
        l = a.label ? label_at(plane_base(a.label, g, 0), pt) : 0;
        p0 = *at_plane(plane_base(a.p, g, 0), pt);
        k0 = *at_plane(plane_base(a.kap, g, 0), pt);
        q0 = *at_plane(plane_base(a.nlq, g, 0), pt);
        if (PP) r0 = *at_plane(plane_base(a.rho, g, 0), pt);
        load_memory<2 * L>(&m[0][0], a.psi2, g, pt, a.stream);
    }
    if (n_src > 0) {                                 // the sources of the tile's cells
        lds.src[tid] = 0;
        __syncthreads();
        for (int k = tid; k < n_src; k += NT) {
            const uint32_t f = (uint32_t)((const __attribute__((address_space(1))) int64_t *)s.idx)[k], y = f / (uint32_t)nx, x = f - y * (uint32_t)nx;
            if (x - (uint32_t)x0 < (uint32_t)TX && y - (uint32_t)y0 < (uint32_t)TY)
                lds.src[(y - (uint32_t)y0) * TX + (x - (uint32_t)x0)] = k + 1;
        }
    }
    wx.store(lds.x, tid);
    wy.store(lds.y, tid);
    __syncthreads();
    if (!live) return;
    const Wts W = weights<PP>(a, PP ? cell_r2(a, r0, k0) : 0.0f);
    const float *X = &lds.x[(ty + 1) * T::XW + tx + 4], *Y = &lds.y[(ty + 4) * T::YW + tx + 1];
    float Dx = W.g0 * (X[0] - X[-1]);
    Dx = fmaf(W.g1, X[1] - X[-2], Dx);
    Dx = fmaf(W.g2, X[2] - X[-3], Dx);
    Dx = fmaf(W.g3, X[3] - X[-4], Dx);
    Dx = fmaf(W.g11, (X[T::XW] - X[T::XW - 1]) + (X[-T::XW] - X[-T::XW - 1]), Dx);
    float Dy = W.g0 * (Y[0] - Y[-T::YW]);
    Dy = fmaf(W.g1, Y[T::YW] - Y[-2 * T::YW], Dy);
    Dy = fmaf(W.g2, Y[2 * T::YW] - Y[-3 * T::YW], Dy);
    Dy = fmaf(W.g3, Y[3 * T::YW] - Y[-4 * T::YW], Dy);
    Dy = fmaf(W.g11, (Y[1] - Y[1 - T::YW]) + (Y[-1] - Y[-1 - T::YW]), Dy);
    const int sx = max(max(a.nb[0] - i, i - (nx - 1 - a.nb[0])), 0);
    const int sy = max(max(a.nb[1] - j, j - (ny - 1 - a.nb[1])), 0);
    float S = 0.0f;
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) {
        const float D = ax == 0 ? Dx : Dy;
        const int tt = (ax == 0 ? sx : sy) * a.n_labels + l;
        const gcfloat bc = (gcfloat)a.bc2[ax] + tt * (2 * L);
        float Sa = ((gcfloat)a.w2[ax])[tt] * D;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 q = make_float2(bc[2 * nu], bc[2 * nu + 1]);
            const float mn = fmaf(q.x, m[ax][nu], q.y * D);
            Sa += CENTRED ? m[ax][nu] : mn;
            m[ax][nu] = mn;
        }
        S += Sa;
    }
    const float kappa = k0 * (1.0f + q0 * p0);
    float pn = p0 - a.dt * S / kappa;
    if (n_src > 0 && lds.src[tid]) {
        const int k = lds.src[tid] - 1;
        pn = fmaf(s.w[k], s.signals[(int64_t)s.sig[k] * s.n_t + step], pn);
    }
    *at_plane_w(plane_base(a.p + a.out, g, 0), pt) = pn;
    store_memory<2 * L>(&m[0][0], a.psi2 + a.out, g, pt, a.stream);
}

// Velocity phase of the tile at (x0, y0).
template <int L, bool CENTRED, bool PP, int TY, int TX>
__device__ __forceinline__ void velocity_tile(const StepArgs &a, int x0, int y0, VelocityLds<TY, TX> &lds)
{
    using T = VelocityLds<TY, TX>;
    constexpr int NT = TX * TY;
    const Geometry &g = a.geo;
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX, i = x0 + tx, j = y0 + ty;
    const int nx = g.n[0], ny = g.n[1];
    const bool live = i < nx && j < ny;
    const uint32_t pt = plane_point(g, i, j);
    Window<T::PW, T::PH, NT> wp;
    wp.load(a.p, g, x0 - 3, y0 - 3, tid);
    int l = 0;
    float r0 = 1.0f, k0 = 1.0f, rn[2] = {1.0f, 1.0f}, kn[2] = {1.0f, 1.0f}, u[2] = {0.0f, 0.0f}, m[2][L];
    if (live) {
        l = a.label ? label_at(plane_base(a.label, g, 0), pt) : 0;
        const gbase br = plane_base(a.rho, g, 0), bk = plane_base(a.kap, g, 0);
        r0 = *at_plane(br, pt);
        k0 = *at_plane(bk, pt);
#pragma unroll
        for (int ax = 0; ax < 2; ++ax) {
            const uint32_t nb = plane_point(g, i + (ax == 0), j + (ax == 1));
            rn[ax] = *at_plane(br, nb);
            kn[ax] = *at_plane(bk, nb);
            u[ax] = *at_plane(plane_base(a.v + (int64_t)ax * g.stride, g, 0), pt);
        }
        load_memory<2 * L>(&m[0][0], a.psi1, g, pt, a.stream);
    }
    wp.store(lds.p, tid);
    __syncthreads();
    if (!live) return;
    const float *P = &lds.p[(ty + 3) * T::PW + tx + 3];
    const float s0 = PP ? cell_r2(a, r0, k0) : 0.0f;
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) {
        if (ax == 0 ? i == nx - 1 : j == ny - 1) continue;           // outside the grid, held at zero
        constexpr int PW = T::PW;
        const int o = ax == 0 ? 1 : PW;
        const Wts W = weights<PP>(a, PP ? 0.5f * (s0 + cell_r2(a, rn[ax], kn[ax])) : 0.0f);
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
        const int tt = s * a.n_labels + l;
        const gcfloat bc = (gcfloat)a.bc1[ax] + tt * (2 * L);
        float S = ((gcfloat)a.w1[ax])[tt] * D;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 q = make_float2(bc[2 * nu], bc[2 * nu + 1]);
            const float mn = fmaf(q.x, m[ax][nu], q.y * D);
            S += CENTRED ? m[ax][nu] : mn;
            m[ax][nu] = mn;
        }
        const float pbar = 0.5f * (P[0] + P[o]);
        const float rho_a = 0.5f * (r0 + rn[ax]);
        const float kap_a = 0.5f * (k0 + kn[ax]);
        *at_plane_w(plane_base(a.v + a.out + (int64_t)ax * g.stride, g, 0), pt) =
            u[ax] - a.dt * S / (rho_a * (1.0f + (a.nlA * kap_a) * pbar));
        store_memory<L>(&m[ax][0], a.psi1 + a.out + (int64_t)(ax * L) * g.stride, g, pt, a.stream);
    }
}

}  // namespace

}  // namespace fw2
