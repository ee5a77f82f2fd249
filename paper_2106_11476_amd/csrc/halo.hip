// gfx950 kernels of libfw2 around the time step: the halo planes of a slab
// of a grid split along z (pack / unpack), the medium of a domain built
// from device maps, and the streaming probes of the measurement.
//
// All are plain streaming kernels (bandwidth bound, no reuse): one thread
// per element, consecutive threads on consecutive x, so every wavefront
// reads and writes 256 contiguous bytes.
#include "kernels.hpp"
#include "probe.hpp"

#include <algorithm>

namespace fw2 {

namespace {

constexpr int kPackBX = 256;

// Grid dimensions y and z are limited to 65535 blocks: larger extents are
// covered by striding.
constexpr int kMaxGridYZ = 65535;

// Packed planes from (PACK) or to the padded arrays, V consecutive x per
// thread; packed layout [range][array][plane][ny][nx].
// grid: (elements of a plane / 256, arrays of the set, planes of an array).
// Bound by HBM streaming, each value read once and written once; one launch
// moves the whole set (a copy per plane is bound by its launches: all 16
// fields of a 160^3 grid written, one step and all read again take 0.40 ms,
// 12.5 ms with a strided copy per plane and field).
template <int V, bool PACK>
__global__ void __launch_bounds__(kPackBX) plane_copy(const PlaneSet s, const Geometry g, float *packed)
{
    const uint32_t nxv = (uint32_t)g.n[0] / V;
    const uint32_t e = blockIdx.x * kPackBX + threadIdx.x;
    if (e >= nxv * (uint32_t)g.n[1]) return;
    const int y = (int)(e / nxv), x = (int)(e - (uint32_t)y * nxv) * V;
    int q = 0, rep = blockIdx.y;
    int64_t base = 0;                               // packed planes before this array
    while (q < s.n - 1 && rep >= s.reps[q]) {
        rep -= s.reps[q];
        base += (int64_t)s.reps[q] * s.nz[q];
        ++q;
    }
    base += (int64_t)rep * s.nz[q];
    float *arr = const_cast<float *>(s.arr[q]) + (int64_t)rep * g.stride + g.origin + (int64_t)y * g.pitch + x;
    const int axis = !PACK && s.per_axis[q] > 0 ? rep / s.per_axis[q] : -1;
    if (axis == 1 && y == g.n[1] - 1) return;
    for (int k = blockIdx.z; k < s.nz[q]; k += gridDim.z) {
        if (axis == 2 && k == s.nz[q] - 1) break;
        float *f = arr + (int64_t)(s.z0[q] + k) * g.plane;
        float *b = packed + ((base + k) * g.n[1] + y) * g.n[0] + x;
        if constexpr (V == 4) {
            if (PACK) {
                *(float4 *)b = *(const float4 *)f;
            } else if (axis == 0 && x + 4 == g.n[0]) {
                const float4 v = *(const float4 *)b;
                f[0] = v.x;
                f[1] = v.y;
                f[2] = v.z;
            } else {
                *(float4 *)f = *(const float4 *)b;
            }
        } else {
            if (PACK)
                *b = *f;
            else if (!(axis == 0 && x == g.n[0] - 1))
                *f = *b;
        }
    }
}

// Medium values of one point from device maps, in FP64 with the host
// conversion's operation order and no contraction, so both give the same
// FP32 values.  hi / lo accumulate the thread's largest and smallest c.
__device__ __forceinline__ void medium_point(const MediumArgs &m, int x, int y, int z, unsigned int &hi,
                                             unsigned int &lo)
{
#pragma clang fp contract(off)
    const Geometry &g = m.geo;
    const int64_t q = ((int64_t)z * g.n[1] + y) * g.n[0] + x;
    const int64_t o = g.origin + (int64_t)z * g.plane + (int64_t)y * g.pitch + x;
    const float cf = m.c[q], rf = m.rho[q], bf = m.beta[q];
    const bool ok_c = cf > 0.0f && cf <= __FLT_MAX__;       // positive and finite (NaN fails)
    const bool ok_r = rf > 0.0f && rf <= __FLT_MAX__;
    const bool ok_b = bf >= -__FLT_MAX__ && bf <= __FLT_MAX__;
    const int lab = m.label ? (int)m.label[q] : 0;
    if (!(ok_c && ok_r && ok_b) || lab >= m.n_labels) {
        atomicOr(&m.stats[2], 1u);
        return;
    }
    // largest c: max of the bit patterns of positive floats; smallest c: max
    // of (bits of +inf - bits)
    const unsigned int bits = __float_as_uint(cf);
    hi = max(hi, bits);
    lo = max(lo, 0x7f800000u - bits);
    const double c = cf, rr = rf, b = bf;
    const double k0 = 1.0 / (rr * c * c);
    m.kap[o] = (float)k0;
    m.nlq[o] = (float)(k0 * (m.B0 + m.B1 * b));
    m.rhop[o] = (float)rr;
    if (m.labp) m.labp[o] = (uint8_t)lab;
}

// The extremes are reduced over each wavefront before the atomics: with two
// atomics per point on the same words the kernel was bound by them (47.6 ms
// for 512^3 points).
__global__ void __launch_bounds__(256) medium_kernel(const MediumArgs m)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    unsigned int hi = 0u, lo = 0u;
    if (x < m.geo.n[0])
        for (int z = blockIdx.z; z < m.geo.n[2]; z += gridDim.z)
            for (int y = blockIdx.y; y < m.geo.n[1]; y += gridDim.y) medium_point(m, x, y, z, hi, lo);
    for (int o = 32; o > 0; o >>= 1) {
        hi = max(hi, __shfl_xor(hi, o));
        lo = max(lo, __shfl_xor(lo, o));
    }
    if (threadIdx.x % 64 == 0 && hi != 0u) {        // hi == 0: no valid sample in this wavefront
        atomicMax(&m.stats[0], hi);
        atomicMax(&m.stats[1], lo);
    }
}

}  // namespace

// Four values a thread where nx is a multiple of 4 and the packed buffer
// 16-byte aligned: every packed row then starts on 16 bytes (the padded rows
// always do).  Other sizes move one value a thread.
template <bool PACK>
hipError_t launch_planes(const PlaneSet &s, const Geometry &g, float *packed, hipStream_t st)
{
    if (s.total <= 0) return hipSuccess;
    int arrays = 0, planes = 0;
    for (int q = 0; q < s.n; ++q) {
        arrays += s.reps[q];
        planes = std::max(planes, s.nz[q]);
    }
    const bool wide = g.n[0] % 4 == 0 && (uintptr_t)packed % 16 == 0;
    const unsigned per_plane = (unsigned)g.n[0] / (wide ? 4u : 1u) * (unsigned)g.n[1];
    const dim3 grid((per_plane + kPackBX - 1) / kPackBX, (unsigned)arrays, std::min(planes, kMaxGridYZ));
    if (wide)
        hipLaunchKernelGGL((plane_copy<4, PACK>), grid, dim3(kPackBX), 0, st, s, g, packed);
    else
        hipLaunchKernelGGL((plane_copy<1, PACK>), grid, dim3(kPackBX), 0, st, s, g, packed);
    return hipGetLastError();
}

hipError_t launch_pack(const PlaneSet &s, const Geometry &g, float *dst, hipStream_t st)
{
    return launch_planes<true>(s, g, dst, st);
}

hipError_t launch_unpack(const PlaneSet &s, const Geometry &g, const float *src, hipStream_t st)
{
    return launch_planes<false>(s, g, const_cast<float *>(src), st);
}

hipError_t launch_medium(const MediumArgs &m, hipStream_t st)
{
    const dim3 grid((m.geo.n[0] + 255) / 256, std::min(m.geo.n[1], kMaxGridYZ), std::min(m.geo.n[2], kMaxGridYZ));
    hipLaunchKernelGGL(medium_kernel, grid, dim3(256), 0, st, m);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Streaming probes (measurement).  They give the HBM rate that a plain
// kernel of a given access pattern reaches on the device, the reference
// against which the step kernels' measured traffic is read.  One thread per
// element, no loop, so the resident waves always cover one compact address
// window.
// ---------------------------------------------------------------------------

namespace {

constexpr int kProbeBX = 256;

__global__ void __launch_bounds__(kProbeBX) probe_copy16(const float4 *__restrict__ src, float4 *__restrict__ dst,
                                                         uint64_t n)
{
    const uint64_t i = blockIdx.x * (uint64_t)kProbeBX + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// The velocity phase's per-point byte mix at L = 2 in 3D without its
// stencil: 12 FP32 arrays read (p, three v, rho, kappa0, six memory
// variables), 9 written (three v, six memory variables).
struct MixArgs {
    const float *r[12];
    float *w[9];
};

__global__ void __launch_bounds__(kProbeBX) probe_mix(const MixArgs m, uint64_t n)
{
    const uint64_t i = blockIdx.x * (uint64_t)kProbeBX + threadIdx.x;
    if (i >= n) return;
    float x[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) x[q] = m.r[q][i];
    const float t = (x[0] + x[4]) + x[5];
#pragma unroll
    for (int q = 0; q < 3; ++q) m.w[q][i] = x[1 + q] + t;
#pragma unroll
    for (int q = 0; q < 6; ++q) m.w[3 + q][i] = fmaf(0.5f, x[6 + q], t);
}

}  // namespace

uint64_t stream_probe_elements(int kind, uint64_t bytes)
{
    if (kind == 0) return bytes / 32;                         // float4 pairs: half read, half written
    return bytes / (21 * 4) / 64 * 64;                         // points per array, arrays 256-byte aligned
}

hipError_t launch_stream_probe(int kind, void *buf, uint64_t bytes, hipStream_t stream)
{
    const uint64_t n = stream_probe_elements(kind, bytes);
    const unsigned blocks = (unsigned)((n + kProbeBX - 1) / kProbeBX);
    if (kind == 0) {
        const float4 *src = (const float4 *)buf;
        hipLaunchKernelGGL(probe_copy16, dim3(blocks), dim3(kProbeBX), 0, stream, src, (float4 *)buf + n, n);
    } else {
        MixArgs m;
        float *f = (float *)buf;
        for (int q = 0; q < 12; ++q) m.r[q] = f + (uint64_t)q * n;
        for (int q = 0; q < 9; ++q) m.w[q] = f + (uint64_t)(12 + q) * n;
        hipLaunchKernelGGL(probe_mix, dim3(blocks), dim3(kProbeBX), 0, stream, m, n);
    }
    return hipGetLastError();
}

}  // namespace fw2
