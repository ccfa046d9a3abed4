// noalloc.hip -- the FP64 direct sum of eq. 1 without any device allocation.
//
// bltc_direct keeps the partial sums of its source pieces in a buffer it
// allocates per call.  bltc_direct_noalloc runs the same kernels with that
// buffer in a file-scope device array of fixed size (or with the sources in it,
// where the potentials are written over an input and outnumber the array), so
// that callers that cannot allocate (code under HIP graph capture,
// serving loops, harnesses that forbid hipMalloc) can use it.  Every GPU the
// library runs on holds its own copy of the array until the process ends; the
// host side keeps each device's address of it (hipGetSymbolAddress, once per
// device with that device current) and passes that address to the kernels.
// The array's name is never used as a device address on the host.
#include "bltc.h"
#include "internal.hpp"
#include "kernels.hpp"

#include <mutex>

namespace {

// largest source count; the partial sums (32 MiB per device) hold any split
constexpr int64_t kNoAllocSources = int64_t(1) << 20;
__device__ __align__(256) double scratch[bltc::kDirectPartials];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};

// This device's address of `scratch`, looked up on its first use.
int scratch_for_current_device(double** out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return bltc_detail::fail(BLTC_EUNSUPPORTED, "device index %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return bltc_detail::hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol,
                                         "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return BLTC_OK;
}

}  // namespace

extern "C" int bltc_direct_noalloc(const bltc_params* p, int64_t nt, const double* tx,
                                   const double* ty, const double* tz, int64_t ns,
                                   const double* sx, const double* sy, const double* sz,
                                   const double* q, int32_t num_q, int64_t q_ld, double* phi,
                                   int64_t phi_ld, void* stream)
{
    using bltc_detail::fail;
    int rc = bltc_internal_check_direct(p, nt, tx, ty, tz, ns, sx, sy, sz, q, num_q, phi);
    if (rc != BLTC_OK)
        return rc;
    if (ns > kNoAllocSources)
        return fail(BLTC_EUNSUPPORTED,
                    "bltc_direct_noalloc takes at most %lld sources (its fixed array); "
                    "%lld given: use bltc_direct",
                    static_cast<long long>(kNoAllocSources), static_cast<long long>(ns));
    if (nt == 0)
        return BLTC_OK;
    double* part = nullptr;
    rc = scratch_for_current_device(&part);
    if (rc != BLTC_OK)
        return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // partial sums as in bltc_direct (no sources: the sum writes zeros)
    const bltc::DirectSplit split = bltc::direct_split(nt, ns);
    const bool fits = split.pieces * nt * std::min(num_q, bltc::kDirectVectors) <=
                      bltc::kDirectPartials;
    const bool overlap = bltc_internal_direct_overlap(nt, tx, ty, tz, ns, sx, sy, sz, q, num_q, q_ld,
                                                      phi, phi_ld);
    if (split.pieces > 1 || (overlap && fits)) {
        if (!fits)
            return fail(BLTC_EINTERNAL, "direct-sum partials exceed the fixed array");
        return bltc_internal_direct(p, nt, tx, ty, tz, ns, sx, sy, sz, q, num_q, q_ld, phi, phi_ld,
                                    split, part, s);
    }
    if (!overlap)
        return bltc_internal_direct(p, nt, tx, ty, tz, ns, sx, sy, sz, q, num_q, q_ld, phi, phi_ld,
                                    split, nullptr, s);
    // potentials written over an input, and too many of them for the array: it
    // holds the sources and one charge vector at a time instead, and a target's
    // coordinates are read by the workgroup that writes its potential
    static_assert(4 * kNoAllocSources <= bltc::kDirectPartials, "x, y, z and charges fit");
    double* const staged[4] = {part, part + ns, part + 2 * ns, part + 3 * ns};
    const double* const xyz[3] = {sx, sy, sz};
    for (int l = 0; l < 3 && ns > 0; ++l)
        HIP_TRY(hipMemcpyAsync(staged[l], xyz[l], ns * sizeof(double), hipMemcpyDeviceToDevice, s));
    for (int32_t m = 0; m < num_q; ++m) {
        if (ns > 0)
            HIP_TRY(hipMemcpyAsync(staged[3], q + m * q_ld, ns * sizeof(double),
                                   hipMemcpyDeviceToDevice, s));
        rc = bltc_internal_direct(p, nt, tx, ty, tz, ns, staged[0], staged[1], staged[2], staged[3], 1,
                                  ns, phi + m * phi_ld, phi_ld, split, nullptr, s);
        if (rc != BLTC_OK)
            return rc;
    }
    return BLTC_OK;
}
