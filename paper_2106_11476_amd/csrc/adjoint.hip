// gfx950 kernels of the discrete adjoint of one time step (time-centred
// memory scheme), for the gradient of J = 1/2 sum (trace - obs)^2 with
// respect to kappa0 (and through it the sound speed).
//
// The memory-variable recursion is dissipative, so running the forward
// scheme backwards in time does not give its adjoint (Sec. 5, full waveform
// inversion): the reverse step here is the transpose of the forward step's
// linearisation, taken phase by phase in
// reverse order, about the forward state at the step's input:
//   A0  pressure points: recompute S = sum_a (w2 D^-v_a + sum psi2) and
//       p'' = p - dt S / K (+ sources, A_src), K = kappa0 (1 + kappa0 B p),
//       kappa0 B = nlq (B = 1 - 2 beta as printed; B does not depend on kappa0)
//   A1  v points inside the grid: velocity phase reversed, pointwise:
//       Q = rho_a (1 + A kappa0_a pbar) (A = 1 as printed),
//       lam_S' = -dt lam_v / Q, lam_Q = dt S' lam_v / Q^2, lam_psi1 <- lam_S' + b1 lam_psi1,
//       and per axis the adjoint of D^+ p'' and lam_Q rho_a A, from which the
//       adjoints of pbar (lam_Q rho_a A kappa0_a) and kappa0_a
//       (lam_Q rho_a A pbar) follow where they are gathered
//   A_rcv  lam_p[R] += trace_n - obs_n
//   A2  pressure points: lam_p'' = lam_p - sum_a D^-(lam_D'_a) + means of lam_pbar,
//       gradient from the velocity multipliers, then the pressure phase
//       reversed: lam_S = -dt lam_p''/K, lam_K = dt S lam_p''/K^2,
//       lam_p = lam_p'' + lam_K kappa0 nlq,
//       grad += lam_K (1 + 2 nlq p), lam_psi2 <- lam_S + b2 lam_psi2,
//       lam_D_a = w2 lam_S + sum c2 lam_psi2 (new)
//   A3  v points inside the grid: lam_v_a -= D^+(lam_D_a)
// using (D^-)^T = -(D^+) and (D^+)^T = -(D^-).
// The phases run as two kernels per step (from LDS tiles in 2D, one thread per
// point in 3D): A3 of a step is deferred into the velocity kernel (A1) of the
// next call, A_rcv runs in extra blocks of that kernel, and A0 of the step
// before is fused into the pressure kernel (A2) when its state is at hand,
// writing that step's p'' into the second p'' buffer (this step's is still
// read by neighbours).
#include "tile2d.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace fw2 {

namespace {

constexpr int kABX = 256, kABY = 1;       // default block of the per-point kernels (measured best)

// Block shape of the per-point kernels: FW2_ADJ_BLOCK="bx,by" with bx * by =
// 256 (a tuning knob), else kABX x kABY.
dim3 adj_block()
{
    static dim3 b = [] {
        int bx = kABX, by = kABY;
        if (const char *e = std::getenv("FW2_ADJ_BLOCK")) {
            int x = 0, y = 0;
            if (std::sscanf(e, "%d,%d", &x, &y) == 2 && x > 0 && y > 0 && x * y == kABX * kABY) {
                bx = x;
                by = y;
            }
        }
        return dim3(bx, by);
    }();
    return b;
}

struct AdjArgs {
    StepArgs f;              // medium, tables, stencil of the domain (f.p etc. unused)
    const float *sp;         // forward state at the step input: p, v, psi1, psi2 blocks
    const float *sq;         // forward state of the step before (A0 fused into A2), or unused
    float *lp;               // adjoint state: same layout
    float *pp;               // p'' of this step (forward recompute)
    float *pq;               // p'' of the step before (written by the fused A0)
    float *sS;               // S of the pressure phase (forward recompute)
    float *lDv;              // [ndim] adjoint of D^+ p'' at v points
    float *lqr;              // [ndim] lam_Q rho_a at v points
    float *lDp;              // [ndim] adjoint of D^- v_a at p points
    float *gk;               // dJ/dkappa0
    int nbx, nby, nblocks;   // blocks along x and y; point blocks in the 1D launch
    const int64_t *rcv_idx;  // receivers (flat indices), added into lam_p by the
    const float *residual;   // velocity kernel's extra blocks: trace - obs of this step
    int n_rcv;               // 0: no receiver blocks
    SparseArgs src;          // sources of the step before, added to pq by the tile
    long long src_step;      // kernel (n = 0: none, or a launch of their own)
};

// Point block of a 1D launch.  Blocks are dealt to the 8 XCDs round-robin
// (block b runs on XCD b mod 8); renumbering them so that XCD x takes one
// contiguous run of point blocks keeps the stencil rows that neighbouring
// blocks share in that XCD's L2 instead of fetching them once per XCD.
// A bijection of [0, nblocks) for any nblocks.
__device__ __forceinline__ int xcd_block(int bid, int nblocks)
{
    const int x = bid % 8, q = nblocks / 8, rem = nblocks % 8;
    return x * q + min(x, rem) + bid / 8;
}

__device__ __forceinline__ int64_t aoff(const Geometry &g, int a)
{
    return a == 0 ? (int64_t)1 : (a == 1 ? g.pitch : g.plane);
}

__device__ __forceinline__ float dminus(const float *__restrict__ f, const Geometry &g, const float *gw, float g11,
                                        int a, int nd, int64_t idx)
{
    const int64_t o = aoff(g, a);
    float D = gw[0] * (f[idx] - f[idx - o]);
    D = fmaf(gw[1], f[idx + o] - f[idx - 2 * o], D);
    D = fmaf(gw[2], f[idx + 2 * o] - f[idx - 3 * o], D);
    D = fmaf(gw[3], f[idx + 3 * o] - f[idx - 4 * o], D);
    float cr = 0.0f;
    for (int b = 0; b < nd; ++b) {
        if (b == a) continue;
        const int64_t o2 = aoff(g, b);
        cr += (f[idx + o2] - f[idx - o + o2]) + (f[idx - o2] - f[idx - o - o2]);
    }
    return fmaf(g11, cr, D);
}

__device__ __forceinline__ float dplus(const float *__restrict__ f, const Geometry &g, const float *gw, float g11,
                                       int a, int nd, int64_t idx)
{
    const int64_t o = aoff(g, a);
    float D = gw[0] * (f[idx + o] - f[idx]);
    D = fmaf(gw[1], f[idx + 2 * o] - f[idx - o], D);
    D = fmaf(gw[2], f[idx + 3 * o] - f[idx - 2 * o], D);
    D = fmaf(gw[3], f[idx + 4 * o] - f[idx - 3 * o], D);
    float cr = 0.0f;
    for (int b = 0; b < nd; ++b) {
        if (b == a) continue;
        const int64_t o2 = aoff(g, b);
        cr += (f[idx + o + o2] - f[idx + o2]) + (f[idx + o - o2] - f[idx - o2]);
    }
    return fmaf(g11, cr, D);
}

__device__ __forceinline__ int slot_p(int x, int n, int nb) { return max(max(nb - x, x - (n - 1 - nb)), 0); }
__device__ __forceinline__ int slot_v(int x, int n, int nb) { return max(max(nb - x, x - (n - 2 - nb)), 0); }

#define ADJ_POINT                                                                  \
    const Geometry &g = A.f.geo;                                                   \
    const int blk = xcd_block(blockIdx.x, A.nblocks);                              \
    const int bxy = blk % (A.nbx * A.nby);                                         \
    const int i = (bxy % A.nbx) * blockDim.x + threadIdx.x;                        \
    const int j = (bxy / A.nbx) * blockDim.y + threadIdx.y;                        \
    const int k = blk / (A.nbx * A.nby);                                           \
    if (i >= g.n[0] || j >= g.n[1]) return;                                        \
    const int c3[3] = {i, j, k};                                                   \
    const int64_t idx = g.origin + (int64_t)k * g.plane + (int64_t)j * g.pitch + i; \
    const int lab = A.f.label ? (int)A.f.label[idx] : 0;                           \
    (void)c3;                                                                      \
    (void)lab;

// A0: forward recompute of the pressure phase (without sources).
template <int ND, int L>
__global__ void __launch_bounds__(kABX *kABY) adj_forward_p(const AdjArgs A)
{
    constexpr int nd = ND;
    ADJ_POINT
    const int64_t st = g.stride;
    const float *v = A.sp + st;
    const float *m2 = A.sp + (int64_t)(1 + nd + nd * L) * st;
    float S = 0.0f;
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        const float D = dminus(v + a * st, g, A.f.g, A.f.g11, a, nd, idx);
        const int t = slot_p(c3[a], g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
        float Sa = A.f.w2[a][t] * D;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) Sa += ntld(&m2[(int64_t)(a * L + nu) * st + idx]);
        S += Sa;
    }
    const float p0 = A.sp[idx];
    const float K = A.f.kap[idx] * (1.0f + A.f.nlq[idx] * p0);
    A.pp[idx] = p0 - A.f.dt * S / K;
    A.sS[idx] = S;
}

__device__ __forceinline__ int64_t pidx(const Geometry &g, int64_t f)
{
    const int64_t x = f % g.n[0];
    const int64_t t = f / g.n[0];
    return g.origin + (t / g.n[1]) * g.plane + (t % g.n[1]) * g.pitch + x;
}

__global__ void adj_sources(float *pp, const SparseArgs s, long long step)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= s.n || step >= s.n_t) return;
    const int64_t pi = pidx(s.geo, s.idx[q]);
    pp[pi] = pp[pi] + s.w[q] * s.signals[(int64_t)s.sig[q] * s.n_t + step];
}

// A1: velocity phase reversed at v points.  DEFER_A3: first apply the A3 of
// the step after (lam_v -= D^+ lam_Dp, lam_Dp left by the previous call).
// Blocks past the point blocks add the receiver residual into lam_p (A_rcv),
// which this kernel neither reads nor writes otherwise.
template <int ND, int L, bool DEFER_A3>
__global__ void __launch_bounds__(kABX *kABY) adj_velocity(const AdjArgs A)
{
    constexpr int nd = ND;
    if ((int)blockIdx.x >= A.nblocks) {
        const int q = ((int)blockIdx.x - A.nblocks) * (int)(blockDim.x * blockDim.y) +
                      (int)(threadIdx.y * blockDim.x + threadIdx.x);
        if (q < A.n_rcv) atomicAdd(&A.lp[pidx(A.f.geo, A.rcv_idx[q])], A.residual[q]);
        return;
    }
    ADJ_POINT
    const int64_t st = g.stride;
    const float *m1 = A.sp + (int64_t)(1 + nd) * st;
    float *lv = A.lp + st;
    float *lm1 = A.lp + (int64_t)(1 + nd) * st;
    float nv[nd], nDv[nd], nqr[nd], nm[nd][L];               // results, stored last
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        nDv[a] = nqr[a] = 0.0f;
        if (c3[a] == g.n[a] - 1) continue;                   // outside the grid: no adjoint flow
        const int64_t o = aoff(g, a);
        const float D = dplus(A.pp, g, A.f.g, A.f.g11, a, nd, idx);
        const int t = slot_v(c3[a], g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
        const float2 *bc = A.f.bc1[a] + (int64_t)t * L;
        const float w = A.f.w1[a][t];
        float Sv = w * D;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) Sv += ntld(&m1[(int64_t)(a * L + nu) * st + idx]);
        const float pbar = 0.5f * (A.pp[idx] + A.pp[idx + o]);
        const float rho_a = 0.5f * (A.f.rho[idx] + A.f.rho[idx + o]);
        const float kap_a = 0.5f * (A.f.kap[idx] + A.f.kap[idx + o]);
        const float Q = rho_a * (1.0f + (A.f.nlA * kap_a) * pbar);
        float lva = lv[a * st + idx];
        if (DEFER_A3) lva -= dplus(A.lDp + a * st, g, A.f.g, A.f.g11, a, nd, idx);
        nv[a] = lva;
        const float lS = -A.f.dt * lva / Q;
        const float lQ = A.f.dt * Sv * lva / (Q * Q);
        float lD = w * lS;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 q = bc[nu];
            const float lmn = ntld(&lm1[(int64_t)(a * L + nu) * st + idx]);
            lD = fmaf(q.y, lmn, lD);
            nm[a][nu] = fmaf(q.x, lmn, lS);
        }
        nDv[a] = lD;
        nqr[a] = (lQ * rho_a) * A.f.nlA;        // the multiplier's coefficient A folded in
    }
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        A.lDv[a * st + idx] = nDv[a];
        A.lqr[a * st + idx] = nqr[a];
        if (c3[a] == g.n[a] - 1) continue;
        if (DEFER_A3) lv[a * st + idx] = nv[a];
#pragma unroll
        for (int nu = 0; nu < L; ++nu) ntst(&lm1[(int64_t)(a * L + nu) * st + idx], nm[a][nu]);
    }
}

// A2: gather of the velocity-phase adjoints, then the pressure phase reversed.
// The adjoints of pbar and kappa0_a at the two v points of each axis are
// lam_Q rho_a times kappa0_a and pbar, recomputed here from kappa0 and this
// step's p'' as the velocity phase formed them.  WITH_A0: then A0 of the step
// before at the same point, from the state sq, into the second p'' buffer
// (S of this step is read before that of the step before overwrites it).
template <int ND, int L, bool WITH_A0>
__global__ void __launch_bounds__(kABX *kABY) adj_pressure(const AdjArgs A)
{
    constexpr int nd = ND;
    ADJ_POINT
    const int64_t st = g.stride;
    float lpp = A.lp[idx];
    float gk = A.gk[idx];
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        const int64_t o = aoff(g, a);
        lpp -= dminus(A.lDv + a * st, g, A.f.g, A.f.g11, a, nd, idx);
        // v points idx (between idx and idx + o) and idx - o
        const float q1 = A.lqr[a * st + idx], q0 = A.lqr[a * st + idx - o];
        const float k1 = 0.5f * (A.f.kap[idx] + A.f.kap[idx + o]);
        const float k0 = 0.5f * (A.f.kap[idx - o] + A.f.kap[idx]);
        const float b1 = 0.5f * (A.pp[idx] + A.pp[idx + o]);
        const float b0 = 0.5f * (A.pp[idx - o] + A.pp[idx]);
        lpp += 0.5f * (q1 * k1 + q0 * k0);
        gk += 0.5f * (q1 * b1 + q0 * b0);
    }
    const float p0 = A.sp[idx];
    const float x = A.f.kap[idx], q = A.f.nlq[idx];
    const float K = x * (1.0f + q * p0);
    const float S = A.sS[idx];
    const float lS = -A.f.dt * lpp / K;
    const float lK = A.f.dt * S * lpp / (K * K);
    const float nlp = lpp + lK * x * q, ngk = gk + lK * (1.0f + 2.0f * q * p0);
    float *lm2 = A.lp + (int64_t)(1 + nd + nd * L) * st;
    float nD[nd], nm[nd][L];                                 // results, stored last
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        const int t = slot_p(c3[a], g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
        const float2 *bc = A.f.bc2[a] + (int64_t)t * L;
        float lD = A.f.w2[a][t] * lS;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 qq = bc[nu];
            const float lmn = ntld(&lm2[(int64_t)(a * L + nu) * st + idx]);
            lD = fmaf(qq.y, lmn, lD);
            nm[a][nu] = fmaf(qq.x, lmn, lS);
        }
        nD[a] = lD;
    }
    float npq = 0.0f, nS = 0.0f;
    if (WITH_A0) {
        const float *vq = A.sq + st;
        const float *m2q = A.sq + (int64_t)(1 + nd + nd * L) * st;
        float S0 = 0.0f;
#pragma unroll
        for (int a = 0; a < nd; ++a) {
            const float D = dminus(vq + a * st, g, A.f.g, A.f.g11, a, nd, idx);
            const int t = slot_p(c3[a], g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
            float Sa = A.f.w2[a][t] * D;
#pragma unroll
            for (int nu = 0; nu < L; ++nu) Sa += ntld(&m2q[(int64_t)(a * L + nu) * st + idx]);
            S0 += Sa;
        }
        const float q0 = A.sq[idx];
        const float K0 = x * (1.0f + q * q0);
        npq = q0 - A.f.dt * S0 / K0;
        nS = S0;
    }
    A.lp[idx] = nlp;
    A.gk[idx] = ngk;
#pragma unroll
    for (int a = 0; a < nd; ++a) {
        A.lDp[a * st + idx] = nD[a];
#pragma unroll
        for (int nu = 0; nu < L; ++nu) ntst(&lm2[(int64_t)(a * L + nu) * st + idx], nm[a][nu]);
    }
    if (WITH_A0) {
        A.pq[idx] = npq;
        A.sS[idx] = nS;
    }
}

// ---------------------------------------------------------------------------
// 2D reverse step from LDS tiles of 64 columns x TY rows, one thread a point.
// One thread a point with every stencil tap a load of its own (45 and 53
// vector loads, half of them off a 64-byte boundary and so two accesses per
// 16 lanes) keeps the L1 pipeline busy three quarters of the time while HBM
// is not: 66 and 72 us for 107 and 135 B a point at 1536^2, L = 2.  Here a
// block loads the fields whose neighbours it reads once, halo included, with
// its own values, and takes the taps from LDS; the arithmetic is the same,
// point for point.  us per reverse step, per-point against tiles (with the
// sources added by the tile): 384^2, L = 2 19.5 / 14.6; 1024^2 65.9 / 48.9;
// 1536^2 141 / 105.5 (5.5 TB/s of its 246 B a point, the streaming rate);
// 1536^2, L = 4 198 / 164, L = 8 304 / 292.  Tiles of 8 rows at L <= 2, of 16
// above: 1536^2, L = 2 105.5 / 107.3, L = 8 303 / 292.
// ---------------------------------------------------------------------------

// D^- and D^+ from LDS: o and o2 are the strides along the axis and across it.
__device__ __forceinline__ float tile_dminus(const float *f, const float *gw, float g11, int o, int o2)
{
    float D = gw[0] * (f[0] - f[-o]);
    D = fmaf(gw[1], f[o] - f[-2 * o], D);
    D = fmaf(gw[2], f[2 * o] - f[-3 * o], D);
    D = fmaf(gw[3], f[3 * o] - f[-4 * o], D);
    float cr = 0.0f;
    cr += (f[o2] - f[o2 - o]) + (f[-o2] - f[-o - o2]);
    return fmaf(g11, cr, D);
}

__device__ __forceinline__ float tile_dplus(const float *f, const float *gw, float g11, int o, int o2)
{
    float D = gw[0] * (f[o] - f[0]);
    D = fmaf(gw[1], f[2 * o] - f[-o], D);
    D = fmaf(gw[2], f[3 * o] - f[-2 * o], D);
    D = fmaf(gw[3], f[4 * o] - f[-3 * o], D);
    float cr = 0.0f;
    cr += (f[o + o2] - f[o2]) + (f[o - o2] - f[-o2]);
    return fmaf(g11, cr, D);
}

#define ADJ_TILE                                                                    \
    constexpr int NT = kTX * TY;                                                    \
    const Geometry &g = A.f.geo;                                                    \
    const int blk = xcd_block(blockIdx.x, A.nblocks);                               \
    const int x0 = (blk % A.nbx) * kTX, y0 = (blk / A.nbx) * TY;                    \
    const int tid = threadIdx.x, tx = tid % kTX, ty = tid / kTX;                    \
    const int i = x0 + tx, j = y0 + ty;                                             \
    const bool live = i < g.n[0] && j < g.n[1];                                     \
    const int64_t st = g.stride;                                                    \
    const int64_t idx = g.origin + (int64_t)j * g.pitch + i;

// A1 with the deferred A3 (adj_velocity) from tiles.
template <int L, int TY>
__global__ void __launch_bounds__(kTX *TY) adj_velocity_tile(const AdjArgs A)
{
    if ((int)blockIdx.x >= A.nblocks) {
        const int q = ((int)blockIdx.x - A.nblocks) * (kTX * TY) + (int)threadIdx.x;
        if (q < A.n_rcv) atomicAdd(&A.lp[pidx(A.f.geo, A.rcv_idx[q])], A.residual[q]);
        return;
    }
    ADJ_TILE
    // p'' and lam_D with the reach of D^+: 3 cells before, 4 after, 1 across
    constexpr int PW = kTX + 7, PH = TY + 7, XH = TY + 2, YW = kTX + 2;
    __shared__ float sp[PW * PH], sx[PW * XH], sy[YW * PH];
    Window<PW, PH, NT> wp;
    Window<PW, XH, NT> wx;
    Window<YW, PH, NT> wy;
    wp.load(A.pp, g, x0 - 3, y0 - 3, tid);
    wx.load(A.lDp, g, x0 - 3, y0 - 1, tid);
    wy.load(A.lDp + st, g, x0 - 1, y0 - 3, tid);
    const float *m1 = A.sp + (int64_t)3 * st;
    float *lv = A.lp + st;
    float *lm1 = A.lp + (int64_t)3 * st;
    int lab = 0;
    float r0 = 1.0f, k0 = 1.0f, rn[2] = {1.0f, 1.0f}, kn[2] = {1.0f, 1.0f}, lva[2] = {0.0f, 0.0f}, m[2][L], lm[2][L];
    if (live) {
        lab = A.f.label ? (int)A.f.label[idx] : 0;
        r0 = A.f.rho[idx];
        k0 = A.f.kap[idx];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            rn[a] = A.f.rho[idx + aoff(g, a)];
            kn[a] = A.f.kap[idx + aoff(g, a)];
            lva[a] = lv[a * st + idx];
#pragma unroll
            for (int nu = 0; nu < L; ++nu) {
                m[a][nu] = ntld(&m1[(int64_t)(a * L + nu) * st + idx]);
                lm[a][nu] = ntld(&lm1[(int64_t)(a * L + nu) * st + idx]);
            }
        }
    }
    wp.store(sp, tid);
    wx.store(sx, tid);
    wy.store(sy, tid);
    __syncthreads();
    if (!live) return;
    const float *P = &sp[(ty + 3) * PW + tx + 3];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        float *oDv = A.lDv + a * st, *oqr = A.lqr + a * st;
        if ((a == 0 ? i : j) == g.n[a] - 1) {                // outside the grid: no adjoint flow
            oDv[idx] = 0.0f;
            oqr[idx] = 0.0f;
            continue;
        }
        const float D = tile_dplus(P, A.f.g, A.f.g11, a == 0 ? 1 : PW, a == 0 ? PW : 1);
        const int t = slot_v(a == 0 ? i : j, g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
        const float2 *__restrict__ bc = A.f.bc1[a] + (int64_t)t * L;
        const float w = A.f.w1[a][t];
        float Sv = w * D;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) Sv += m[a][nu];
        const float pbar = 0.5f * (P[0] + P[a == 0 ? 1 : PW]);
        const float rho_a = 0.5f * (r0 + rn[a]);
        const float kap_a = 0.5f * (k0 + kn[a]);
        const float Q = rho_a * (1.0f + (A.f.nlA * kap_a) * pbar);
        float l = lva[a];
        l -= a == 0 ? tile_dplus(&sx[(ty + 1) * PW + tx + 3], A.f.g, A.f.g11, 1, PW)
                    : tile_dplus(&sy[(ty + 3) * YW + tx + 1], A.f.g, A.f.g11, YW, 1);
        const float lS = -A.f.dt * l / Q;
        const float lQ = A.f.dt * Sv * l / (Q * Q);
        float lD = w * lS;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 q = bc[nu];
            lD = fmaf(q.y, lm[a][nu], lD);
            lm[a][nu] = fmaf(q.x, lm[a][nu], lS);
        }
        lv[a * st + idx] = l;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) ntst(&lm1[(int64_t)(a * L + nu) * st + idx], lm[a][nu]);
        oDv[idx] = lD;
        oqr[idx] = (lQ * rho_a) * A.f.nlA;      // the multiplier's coefficient A folded in
    }
}

// A2 and, WITH_A0, A0 of the step before (adj_pressure) from tiles.
template <int L, bool WITH_A0, int TY>
__global__ void __launch_bounds__(kTX *TY) adj_pressure_tile(const AdjArgs A)
{
    ADJ_TILE
    // lam_D^+ and v with the reach of D^-: 4 cells before, 3 after, 1 across;
    // p'' and kappa0 with one cell around
    constexpr int XW = kTX + 7, XH = TY + 2, YW = kTX + 2, YH = TY + 7;
    __shared__ float sx[XW * XH], sy[YW * YH], sp[YW * XH], sk[YW * XH];
    __shared__ float qx[WITH_A0 ? XW * XH : 1], qy[WITH_A0 ? YW * YH : 1];
    const float *vq = A.sq + st;
    Window<XW, XH, NT> wx, ux;
    Window<YW, YH, NT> wy, uy;
    Window<YW, XH, NT> wp, wk;
    wx.load(A.lDv, g, x0 - 4, y0 - 1, tid);
    wy.load(A.lDv + st, g, x0 - 1, y0 - 4, tid);
    wp.load(A.pp, g, x0 - 1, y0 - 1, tid);
    wk.load(A.f.kap, g, x0 - 1, y0 - 1, tid);
    if (WITH_A0) {
        ux.load(vq, g, x0 - 4, y0 - 1, tid);
        uy.load(vq + st, g, x0 - 1, y0 - 4, tid);
    }
    float *lm2 = A.lp + (int64_t)(3 + 2 * L) * st;
    const float *m2q = A.sq + (int64_t)(3 + 2 * L) * st;
    int lab = 0;
    float lpp = 0.0f, gk = 0.0f, p0 = 0.0f, q = 0.0f, S = 0.0f, q1[2], q0[2], lm[2][L], mq[2][L], pq0 = 0.0f;
    if (live) {
        lab = A.f.label ? (int)A.f.label[idx] : 0;
        lpp = A.lp[idx];
        gk = A.gk[idx];
        p0 = A.sp[idx];
        q = A.f.nlq[idx];
        S = A.sS[idx];
        if (WITH_A0) pq0 = A.sq[idx];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            q1[a] = A.lqr[a * st + idx];
            q0[a] = A.lqr[a * st + idx - aoff(g, a)];
#pragma unroll
            for (int nu = 0; nu < L; ++nu) {
                lm[a][nu] = ntld(&lm2[(int64_t)(a * L + nu) * st + idx]);
                if (WITH_A0) mq[a][nu] = ntld(&m2q[(int64_t)(a * L + nu) * st + idx]);
            }
        }
    }
    __shared__ int ssrc[WITH_A0 ? NT : 1];
    if (WITH_A0 && A.src.n > 0) {                    // the sources of the tile's cells
        ssrc[tid] = 0;
        __syncthreads();
        for (int k = tid; k < A.src.n; k += NT) {
            const uint32_t f = (uint32_t)A.src.idx[k], y = f / (uint32_t)g.n[0], x = f - y * (uint32_t)g.n[0];
            if (x - (uint32_t)x0 < (uint32_t)kTX && y - (uint32_t)y0 < (uint32_t)TY)
                ssrc[(y - (uint32_t)y0) * kTX + (x - (uint32_t)x0)] = k + 1;
        }
    }
    wx.store(sx, tid);
    wy.store(sy, tid);
    wp.store(sp, tid);
    wk.store(sk, tid);
    if (WITH_A0) {
        ux.store(qx, tid);
        uy.store(qy, tid);
    }
    __syncthreads();
    if (!live) return;
    const float *P = &sp[(ty + 1) * YW + tx + 1], *K1 = &sk[(ty + 1) * YW + tx + 1];
    const float *X = &sx[(ty + 1) * XW + tx + 4], *Y = &sy[(ty + 4) * YW + tx + 1];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int o = a == 0 ? 1 : YW;
        lpp -= a == 0 ? tile_dminus(X, A.f.g, A.f.g11, 1, XW) : tile_dminus(Y, A.f.g, A.f.g11, YW, 1);
        const float k1 = 0.5f * (K1[0] + K1[o]);
        const float k0 = 0.5f * (K1[-o] + K1[0]);
        const float b1 = 0.5f * (P[0] + P[o]);
        const float b0 = 0.5f * (P[-o] + P[0]);
        lpp += 0.5f * (q1[a] * k1 + q0[a] * k0);
        gk += 0.5f * (q1[a] * b1 + q0[a] * b0);
    }
    const float x = K1[0];
    const float K = x * (1.0f + q * p0);
    const float lS = -A.f.dt * lpp / K;
    const float lK = A.f.dt * S * lpp / (K * K);
    A.lp[idx] = lpp + lK * x * q;
    A.gk[idx] = gk + lK * (1.0f + 2.0f * q * p0);
    float S0 = 0.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int t = slot_p(a == 0 ? i : j, g.n[a], A.f.nb[a]) * A.f.n_labels + lab;
        const float2 *__restrict__ bc = A.f.bc2[a] + (int64_t)t * L;
        const float w = A.f.w2[a][t];
        float lD = w * lS;
#pragma unroll
        for (int nu = 0; nu < L; ++nu) {
            const float2 qq = bc[nu];
            lD = fmaf(qq.y, lm[a][nu], lD);
            ntst(&lm2[(int64_t)(a * L + nu) * st + idx], fmaf(qq.x, lm[a][nu], lS));
        }
        A.lDp[a * st + idx] = lD;
        if (WITH_A0) {
            const float D = a == 0 ? tile_dminus(&qx[(ty + 1) * XW + tx + 4], A.f.g, A.f.g11, 1, XW)
                                   : tile_dminus(&qy[(ty + 4) * YW + tx + 1], A.f.g, A.f.g11, YW, 1);
            float Sa = w * D;
#pragma unroll
            for (int nu = 0; nu < L; ++nu) Sa += mq[a][nu];
            S0 += Sa;
        }
    }
    if (WITH_A0) {
        const float K0 = x * (1.0f + q * pq0);
        float pn = pq0 - A.f.dt * S0 / K0;
        if (A.src.n > 0 && ssrc[tid]) {
            const int k = ssrc[tid] - 1;
            pn = fmaf(A.src.w[k], A.src.signals[(int64_t)A.src.sig[k] * A.src.n_t + A.src_step], pn);
        }
        A.pq[idx] = pn;
        A.sS[idx] = S0;
    }
}

// dJ/dc = dJ/dkappa0 * (-2 kappa0 / c), with c = 1/sqrt(rho kappa0).
__global__ void __launch_bounds__(kABX *kABY) adj_grad_c(const AdjArgs A, float *out)
{
    ADJ_POINT
    const float x = A.f.kap[idx];
    out[idx] = A.gk[idx] * (-2.0f * x * sqrtf(A.f.rho[idx] * x));
}

// Sets the block counts of a 1D launch of point blocks of the given shape
// over the grid (z planes of one block each) and returns the block count.
unsigned point_grid(AdjArgs &A, dim3 block)
{
    const Geometry &g = A.f.geo;
    A.nbx = (g.n[0] + (int)block.x - 1) / (int)block.x;
    A.nby = (g.n[1] + (int)block.y - 1) / (int)block.y;
    A.nblocks = A.nbx * A.nby * g.n[2];
    return (unsigned)A.nblocks;
}

// A3 of each step is deferred into the velocity kernel of the next call; A0 of
// the step before is fused into the pressure kernel when its state is given,
// else run at the start of the next call.
template <int ND, int L>
hipError_t adjoint_step(const StepArgs &f, const SparseArgs &src, const SparseArgs &rcv, const float *state,
                               const float *state_prev, const AdjointBuffers &b, long long step, bool have_pp,
                               const float *residual, hipStream_t st, bool *pp_next)
{
    AdjArgs A;
    A.f = f;
    A.sp = state;
    A.sq = state_prev;
    A.lp = b.lp;
    A.pp = b.pp;
    A.pq = b.pq;
    A.sS = b.sS;
    A.lDv = b.lDv;
    A.lqr = b.lqr;
    A.lDp = b.lDp;
    A.gk = b.gk;
    const dim3 block = adj_block();
    const dim3 grid(point_grid(A, block));
    A.rcv_idx = rcv.idx;
    A.residual = residual;
    A.n_rcv = residual ? rcv.n : 0;
    const unsigned nt = block.x * block.y;
    const dim3 vgrid(grid.x + (unsigned)((A.n_rcv + (int)nt - 1) / (int)nt));
    if (!have_pp) {
        hipLaunchKernelGGL((adj_forward_p<ND, L>), grid, block, 0, st, A);
        if (src.n > 0 && step < src.n_t)
            hipLaunchKernelGGL(adj_sources, dim3((src.n + 255) / 256), dim3(256), 0, st, b.pp, src, step);
    }
    const bool with_a0 = state_prev && step >= 1;
    const bool sources = with_a0 && src.n > 0 && step - 1 < src.n_t;
    if constexpr (ND == 2) {
        constexpr int TY = L <= 2 ? 8 : 16;
        A.nbx = (f.geo.n[0] + kTX - 1) / kTX;
        A.nby = (f.geo.n[1] + TY - 1) / TY;
        A.nblocks = A.nbx * A.nby;
        const dim3 tile(kTX * TY);
        const int rcv_blocks = (A.n_rcv + kTX * TY - 1) / (kTX * TY);
        const bool in_tiles = sources && src.n <= kTileSources && (int64_t)A.nblocks * src.n <= kScanPairs;
        A.src = src;
        if (!in_tiles) A.src.n = 0;
        A.src_step = step - 1;
        hipLaunchKernelGGL((adj_velocity_tile<L, TY>), dim3(A.nblocks + rcv_blocks), tile, 0, st, A);
        if (with_a0)
            hipLaunchKernelGGL((adj_pressure_tile<L, true, TY>), dim3(A.nblocks), tile, 0, st, A);
        else
            hipLaunchKernelGGL((adj_pressure_tile<L, false, TY>), dim3(A.nblocks), tile, 0, st, A);
        if (sources && !in_tiles)
            hipLaunchKernelGGL(adj_sources, dim3((src.n + 255) / 256), dim3(256), 0, st, b.pq, src, step - 1);
    } else {
        hipLaunchKernelGGL((adj_velocity<ND, L, true>), vgrid, block, 0, st, A);
        if (with_a0)
            hipLaunchKernelGGL((adj_pressure<ND, L, true>), grid, block, 0, st, A);
        else
            hipLaunchKernelGGL((adj_pressure<ND, L, false>), grid, block, 0, st, A);
        if (sources)
            hipLaunchKernelGGL(adj_sources, dim3((src.n + 255) / 256), dim3(256), 0, st, b.pq, src, step - 1);
    }
    *pp_next = with_a0;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint_step(const StepArgs &f, const SparseArgs &src, const SparseArgs &rcv, int L,
                               const float *state, const float *state_prev, const AdjointBuffers &b,
                               long long step, bool have_pp, const float *residual, hipStream_t st,
                               bool *pp_next)
{
    switch (f.geo.ndim * 8 + L) {            // L = 1..8
    case 2 * 8 + 1: return adjoint_step<2, 1>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 2: return adjoint_step<2, 2>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 3: return adjoint_step<2, 3>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 4: return adjoint_step<2, 4>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 1: return adjoint_step<3, 1>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 2: return adjoint_step<3, 2>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 3: return adjoint_step<3, 3>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 4: return adjoint_step<3, 4>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 5: return adjoint_step<2, 5>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 6: return adjoint_step<2, 6>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 7: return adjoint_step<2, 7>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 2 * 8 + 8: return adjoint_step<2, 8>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 5: return adjoint_step<3, 5>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 6: return adjoint_step<3, 6>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 7: return adjoint_step<3, 7>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    case 3 * 8 + 8: return adjoint_step<3, 8>(f, src, rcv, state, state_prev, b, step, have_pp, residual, st, pp_next);
    default: return hipErrorInvalidValue;
    }
}


hipError_t launch_adjoint_gradient(const StepArgs &f, const AdjointBuffers &b, hipStream_t st)
{
    AdjArgs A;
    std::memset(&A, 0, sizeof(A));
    A.f = f;
    A.gk = b.gk;
    const dim3 block = adj_block();
    const dim3 grid(point_grid(A, block));
    hipLaunchKernelGGL(adj_grad_c, grid, block, 0, st, A, b.out);
    return hipGetLastError();
}

}  // namespace fw2
