// Test double of the HIP runtime and of the device launchers, for driving the
// library's host code (fw2.cpp, setup.cpp) without a GPU: "device" memory is
// host memory registered with a device number, copies are memcpy, launches
// only count themselves.  Linked into the drivers of tests/host; the library
// itself never uses it.
#pragma once

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>

#include "kernels.hpp"
#include "probe.hpp"

namespace fake {

struct Allocation {
    uint64_t bytes;
    int device;
};
inline std::map<uintptr_t, Allocation> memory;      // start -> allocation
inline int current_device = 0;
inline int copies = 0, packs = 0, unpacks = 0;       // row or block copies; plane kernels
inline int pressure_variant = -1;                    // of the last pressure launch
inline int pressure_launches = 0, source_launches = 0;
inline fw2::StepArgs pressure_args;
inline int batch_tile = -1;                          // of the last batched step

inline void *alloc(uint64_t bytes, int device)
{
    bytes = (bytes + 255) / 256 * 256;
    void *p = std::aligned_alloc(256, bytes);
    std::memset(p, 0, bytes);
    memory[(uintptr_t)p] = Allocation{bytes, device};
    return p;
}

inline bool find(const void *p, uintptr_t *base, Allocation *a)
{
    auto it = memory.upper_bound((uintptr_t)p);
    if (it == memory.begin()) return false;
    --it;
    if ((uintptr_t)p >= it->first + it->second.bytes) return false;
    *base = it->first;
    *a = it->second;
    return true;
}

}  // namespace fake

extern "C" {
hipError_t hipGetDevice(int *d)
{
    *d = fake::current_device;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p)
{
    uintptr_t base;
    fake::Allocation a;
    if (!fake::find(p, &base, &a)) return hipErrorInvalidValue;
    std::memset(at, 0, sizeof(*at));
    at->type = hipMemoryTypeDevice;
    at->device = a.device;
    at->devicePointer = const_cast<void *>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p)
{
    uintptr_t b;
    fake::Allocation a;
    if (!fake::find(p, &b, &a)) return hipErrorInvalidValue;
    *base = (hipDeviceptr_t)b;
    *size = a.bytes;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t)
{
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memmove(d, s, n);
    ++fake::copies;
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind, hipStream_t)
{
    for (size_t r = 0; r < h; ++r) std::memcpy((char *)d + r * dp, (const char *)s + r * sp, w);
    ++fake::copies;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
}

namespace fw2 {

hipError_t launch_pressure(const StepArgs &a, int, int, const KernelConfig &kc, hipStream_t)
{
    fake::pressure_variant = kc.variant;
    fake::pressure_args = a;
    ++fake::pressure_launches;
    return hipSuccess;
}
hipError_t launch_velocity(const StepArgs &, int, int, const KernelConfig &, hipStream_t) { return hipSuccess; }
hipError_t launch_sources(const SparseArgs &, hipStream_t)
{
    ++fake::source_launches;
    return hipSuccess;
}
hipError_t launch_receivers(const SparseArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_fill(float *, int64_t, float, hipStream_t) { return hipSuccess; }
hipError_t launch_check(const float *, const Geometry &, float, int *, hipStream_t) { return hipSuccess; }
hipError_t launch_set_counter(long long *c, long long v, hipStream_t)
{
    *c = v;
    return hipSuccess;
}
hipError_t launch_pack(const PlaneSet &, const Geometry &, float *, hipStream_t)
{
    ++fake::packs;
    return hipSuccess;
}
hipError_t launch_unpack(const PlaneSet &, const Geometry &, const float *, hipStream_t)
{
    ++fake::unpacks;
    return hipSuccess;
}
hipError_t launch_medium(const MediumArgs &, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_stream_probe(int, void *, uint64_t, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_batch_step(const BatchTable *, int, int tile, unsigned, hipStream_t)
{
    if (tile != kBatchTakeSteps) fake::batch_tile = tile;
    return hipSuccess;
}
hipError_t claim_static_batch_table(int, BatchTable **, bool *) { return hipErrorNoDevice; }
void release_static_batch_table(int) {}
hipError_t launch_adjoint_step(const StepArgs &, const SparseArgs &, const SparseArgs &, int, const float *,
                               const float *, const AdjointBuffers &, long long, bool, const float *, hipStream_t,
                               bool *)
{
    return hipErrorNoDevice;
}
hipError_t launch_adjoint_gradient(const StepArgs &, const AdjointBuffers &, hipStream_t) { return hipErrorNoDevice; }

}  // namespace fw2

#define CHECK(cond)                                                         \
    do {                                                                    \
        if (!(cond)) {                                                      \
            std::printf("check failed line %d: %s\n", __LINE__, #cond);     \
            ++g_fail;                                                       \
        }                                                                   \
    } while (0)

// A descriptor of a uniform medium, with the maps it points at.
struct Uniform {
    float *c = nullptr, *rho = nullptr, *beta = nullptr;
    double table[2 + 4 * 8];
    fw2_domain_desc d;

    Uniform(int64_t nx, int64_t ny, int64_t nz, int L)
    {
        std::memset(&d, 0, sizeof(d));
        d.ndim = nz > 1 ? 3 : 2;
        d.n_relax = L;
        d.n[0] = nx;
        d.n[1] = ny;
        d.n[2] = nz;
        d.h = 5e-5;
        d.dt = 0.3 * 5e-5 / 1600.0;
        d.pml_Rc = 1e-3;
        d.pml_npoly = 2;
        d.relax_scheme = FW2_RELAX_CENTRED;
        const size_t n = (size_t)(nx * ny * nz);
        c = new float[3 * n];
        rho = c + n;
        beta = rho + n;
        for (size_t i = 0; i < n; ++i) {
            c[i] = 1540.0f;
            rho[i] = 1000.0f;
            beta[i] = 3.5f;
        }
        for (double &t : table) t = 1e4;
        table[0] = table[1] = 1.0;
        d.c = c;
        d.rho = rho;
        d.beta = beta;
        d.n_labels = 1;
        d.relax_table = table;
    }
    ~Uniform() { delete[] c; }
};
