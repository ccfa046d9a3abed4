// kernels_multi.hip -- FP64 batch/cluster interactions for up to 8 charge vectors
// (eqs. 9 and 11 with a matrix of charges), on the vector units.
//
// The kernel values do not depend on the charge vector: each is formed once and
// multiplied into the accumulators of M vectors.  One target per lane, lists,
// grids, sources and charges wave-uniform through the scalar cache, the lists of
// 64 targets shared by the waves of a workgroup (device_split.hpp), as in the
// one-vector kernel.
//
// Why not the matrix cores: v_mfma_f64_16x16x4 contracts 64 kernel values with 16
// vectors in 70 SIMD cycles, the M fused multiply-adds of a lane take 4.4 cycles
// each, and the two units do not issue at the same time.  The vector form pays for
// the vectors there are, and its far field forms r^2 with one addition per value
// (separable grid in registers).  At 16 vectors the contraction costs the same and
// the matrix-core kernel needs no row loads: 10^6 uniform points, n = 8, 2000 a leaf,
// 16 vectors 167 ms here, 147 there; 8 vectors 104 ms here.
//
// Charges: through the scalar cache (8 M bytes per value and wave) they bound the
// kernel at its miss rate; 16 records in the 16 lanes of a row cost one vector
// load per 16 values, and v_fmac_f64 takes its operand from any lane of the row.
//
// Measured (150,001 uniform points, n = 8, 293 a leaf; Coulomb): 3 vectors 14.4 ms
// on matrix-core tiles of one wave per 64 targets, 5.4 here, 8 vectors 7.0; the FP64
// issue cost of the terms is 4.1 and 5.1 ms at full lanes (the leaves fill 91% of
// them).
#include <type_traits>

#include "device_common.hpp"
#include "device_split.hpp"
#include "kernels.hpp"

namespace bltc {
namespace {

using namespace dev;

// terms of a sum held in registers before they go to the sum in LDS
constexpr int kBlockTerms = 256;

struct MultiArgs {
    const int32_t* group_batch;
    const int64_t* group_first;
    const int64_t* batch_end;
    const int32_t* far_off;
    const int32_t* near_off;
    double* phi;
    int64_t phi_ld;
    KernelConst kc;
    int32_t log_w, mc;
};

// acc[m] += g * (q[m] of lane K of this lane's row of 16 lanes): the charges of 16
// records sit in the 16 lanes of every row, and the multiply-add takes its
// operand from one of them (DPP row_newbcast, no extra instruction).  The wait
// states cover a write of q just before the block.
template <int K, int M>
__device__ __forceinline__ void fma_row(double (&acc)[M], const double (&q)[M], double g)
{
    static_assert(K < 16, "a row has 16 lanes");
    if constexpr (M == 2) {
        asm("s_nop 1\n\t"
            "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %1, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
            : "+v"(acc[0]), "+v"(acc[1])
            : "v"(q[0]), "v"(q[1]), "v"(g), "n"(K));
    } else {
        static_assert(M % 4 == 0, "");
#pragma unroll
        for (int m = 0; m < M; m += 4)
            asm("s_nop 1\n\t"
                "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
                : "+v"(acc[m]), "+v"(acc[m + 1]), "+v"(acc[m + 2]), "+v"(acc[m + 3])
                : "v"(q[m]), "v"(q[m + 1]), "v"(q[m + 2]), "v"(q[m + 3]), "v"(g), "n"(K));
    }
}

template <int M>
__device__ __forceinline__ void load_row(const double* __restrict__ q, double (&v)[M])
{
#pragma unroll
    for (int m = 0; m < M; ++m)
        v[m] = q[m];
}

// K, K + 1, ..., K + COUNT - 1 as compile-time constants
template <int K, int COUNT, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (COUNT > 0) {
        f(std::integral_constant<int, K>{});
        static_for<K + 1, COUNT - 1>(f);
    }
}

// Planes [ka, kb) of a cluster's grid, all M vectors (doubled terms).  The
// charges of 16 / (n + 1) grid lines (k1, k2) at a time are one row of lanes,
// loaded a step ahead.
template <int N, int KER, int M>
__device__ __forceinline__ void far_planes(double x, double y, double z,
                                           const double* __restrict__ nd,
                                           const double* __restrict__ qh, int ka, int kb,
                                           const KernelArg& kappa, double (&acc)[M])
{
    constexpr int NP = N + 1;
    static_assert(NP <= 16, "a grid line fits a row of lanes");
    constexpr int L = 16 / NP;              // lines per row of lanes
    const int r = threadIdx.x & 15;
    const int line = r < L * NP ? r / NP : 0;
    const int lane_off = r < L * NP ? r - line * NP : 0;
    auto row = [&](int k1, int k2) {
        const int k = k2 + line < NP ? k2 + line : NP - 1;
        return qh + ((k1 * NP + k) * NP + lane_off) * M;
    };
    double c2[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const double dz = z - nd[2 * NP + k];
        c2[k] = dz * dz;
    }
    // a step covers the lines k2 .. k2 + L - 1 (the last step of a plane fewer)
    auto lines = [&](int k2, double (&yn)[L]) {
#pragma unroll
        for (int l = 0; l < L; ++l)
            yn[l] = nd[NP + (k2 + l < NP ? k2 + l : NP - 1)];
    };
    double next[M], y2[L];
    lines(0, y2);
    load_row<M>(row(ka, 0), next);
#pragma unroll 1
    for (int k1 = ka; k1 < kb; ++k1) {
        const double dx = x - nd[k1];
        const double a2 = dx * dx;
#pragma unroll 1
        for (int k2 = 0; k2 < NP; k2 += L) {
            double q[M];
#pragma unroll
            for (int m = 0; m < M; ++m)
                q[m] = next[m];
            const bool same = k2 + L < NP;
            const int n1 = same || k1 + 1 == kb ? k1 : k1 + 1;
            load_row<M>(row(n1, same ? k2 + L : 0), next);
            double ab2[L];
#pragma unroll
            for (int l = 0; l < L; ++l) {
                const double dy = y - y2[l];
                ab2[l] = __fma_rn(dy, dy, a2);
            }
            __builtin_amdgcn_sched_barrier(0);
            lines(k2 + L < NP ? k2 + L : 0, y2);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, L>([&](auto l) {
                if (k2 + l < NP) {
                    const double ab = ab2[l];
                    static_for<0, NP>([&](auto k3) {
                        const double g = green_far2_f64<KER>(ab + c2[k3], kappa);
                        fma_row<l * NP + k3, M>(acc, q, g);
                    });
                }
            });
        }
    }
}

// two source records as one scalar load (their unused fourth words with them:
// loads of 24 bytes each take three requests a record and bound the kernel)
typedef double rec2 __attribute__((ext_vector_type(8), aligned(32)));

// cnt sources from s with charges q, all M vectors (doubled terms): coordinates
// through the scalar cache, four sources at a time, the charges of 16 sources in
// a row of lanes.  The next four sources' loads go out as soon as this four's
// coordinates are consumed (scalar loads return in any order, so a wait covers
// every load in flight; issued before that point they would stall it).
template <int KER, int M>
__device__ __forceinline__ void near_run(double x, double y, double z,
                                         const double4* __restrict__ s,
                                         const double* __restrict__ q, int32_t cnt,
                                         const KernelArg& kappa, double (&acc)[M])
{
    const int r = threadIdx.x & 15;
    double next[M], v[M];
    rec2 p[2];
    auto quad = [&](int32_t j) {
        p[0] = *reinterpret_cast<const rec2*>(s + j);
        p[1] = *reinterpret_cast<const rec2*>(s + j + 2);
    };
    auto square = [&](double px, double py, double pz) {
        const double dx = x - px, dy = y - py, dz = z - pz;
        return __fma_rn(dz, dz, __fma_rn(dy, dy, dx * dx));
    };
    auto squares = [&](double (&r2)[4]) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            r2[2 * e] = square(p[e][0], p[e][1], p[e][2]);
            r2[2 * e + 1] = square(p[e][4], p[e][5], p[e][6]);
        }
    };
    load_row<M>(q + (r < cnt ? r : cnt - 1) * M, next);
    if (cnt >= 16)
        quad(0);
    int32_t j0 = 0;
#pragma unroll 1
    for (; j0 + 16 <= cnt; j0 += 16) {
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = next[m];
        const int32_t jn = j0 + 16 + r;
        load_row<M>(q + (jn < cnt ? jn : cnt - 1) * M, next);
        static_for<0, 4>([&](auto u) {
            double r2[4];
            squares(r2);
            __builtin_amdgcn_sched_barrier(0);
            // past the last whole block: this block's first sources again
            const int32_t jn = u < 3 ? j0 + 4 * u + 4 : j0 + 32 <= cnt ? j0 + 16 : j0;
            quad(jn);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, 4>([&](auto e) {
                fma_row<4 * u + e, M>(acc, v, green_near2_f64<KER>(r2[e], kappa));
            });
        });
    }
    if (j0 < cnt) {
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = j0 + r < cnt ? next[m] : 0.0;   // lanes past the end: no charge
        static_for<0, 4>([&](auto u) {
            if (j0 + 4 * u < cnt) {
                double r2[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double4 t = s[j0 + 4 * u + e < cnt ? j0 + 4 * u + e : cnt - 1];
                    r2[e] = square(t.x, t.y, t.z);
                }
                static_for<0, 4>([&](auto e) {
                    fma_row<4 * u + e, M>(acc, v, green_near2_f64<KER>(r2[e], kappa));
                });
            }
        });
    }
}

template <int N, int KER, int M>
__global__ __launch_bounds__(64 * kMaxWaves) void interact_multi(
    const double4* __restrict__ tgt, const double4* __restrict__ src,
    const double* __restrict__ qm, const double* __restrict__ slot_nodes,
    const double* __restrict__ qhat16, const int32_t* __restrict__ far_slot,
    const int64_t* __restrict__ near_begin, const int64_t* __restrict__ near_count, MultiArgs a)
{
    constexpr int NP = N + 1;
    constexpr int P = NP * NP * NP;
    extern __shared__ double lds[];
    __shared__ double exp_tab[kExpTable];
    if constexpr (KER == 1)
        fill_exp2_table(exp_tab);
    const KernelArg kappa{a.kc.kappa, a.kc.delta2, exp_tab};
    const int g = blockIdx.x;
    const int b = a.group_batch[g];
    if (b < 0)
        return;  // empty slot of the per-die schedule
    const int64_t first = a.group_first[g];
    const int64_t end = a.batch_end[b];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int64_t i = first + lane;
    const bool valid = i < end;
    if (!valid)
        i = end - 1;
    const double4 t = tgt[i];
    // the lane's sums: kBlockTerms terms or a cluster or leaf at a time in
    // registers, then in LDS, so that a long list is not one chain of roundings
    double* const sums = lds + w * (M * 64) + lane;
    double acc[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        acc[m] = 0.0;
        sums[64 * m] = 0.0;
    }
    int terms = 0;
    auto flush = [&](int count) {
        terms += count;
        if (terms < kBlockTerms)
            return;
        terms = 0;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            sums[64 * m] += acc[m];
            acc[m] = 0.0;
        }
    };

    const int f0 = a.far_off[b];
    const int n1 = a.near_off[b + 1];
    const ListPart part = list_part<NP, NP * NP, KER, false>(
        w, a.log_w, a.far_off[b + 1] - f0, a.near_off[b], n1, near_count, 0, 0);
    int f = part.plane0 / NP, ka = part.plane0 - f * NP;
    for (int pl = part.plane0; pl < part.plane1; ++f) {
        const int64_t slot = far_slot[f0 + f];
        const int kb = ka + part.plane1 - pl < NP ? ka + part.plane1 - pl : NP;
        far_planes<N, KER, M>(t.x, t.y, t.z, slot_nodes + slot * 3 * NP,
                              qhat16 + slot * (P * M), ka, kb, kappa, acc);
        flush((kb - ka) * NP * NP);
        pl += kb - ka;
        ka = 0;
    }
    for_direct_runs<false>(part, n1, near_begin, near_count, [&](int64_t j, int32_t cnt, int32_t) {
        for (int32_t k = 0; k < cnt; k += 4 * kBlockTerms) {
            const int32_t c = cnt - k < 4 * kBlockTerms ? cnt - k : 4 * kBlockTerms;
            near_run<KER, M>(t.x, t.y, t.z, src + j + k, qm + (j + k) * M, c, kappa, acc);
            flush(c);
        }
    });
    flush(kBlockTerms);
    // the waves' sums in wave order, vector m by wave m mod W
    __syncthreads();
    const int64_t orig = caller_index(t);
    for (int m = w; m < a.mc; m += 1 << a.log_w) {
        double v = 0.0;
        for (int u = 0; u < (1 << a.log_w); ++u)
            v += lds[(u * M + m) * 64 + lane];
        if (valid)
            a.phi[m * a.phi_ld + orig] = 0.5 * v;   // the terms are doubled
    }
}

template <int N, int KER, int M>
hipError_t run_multi(const DevicePlan& d, const MultiArgs& a, const GroupLaunch& gl, hipStream_t s)
{
    hipLaunchKernelGGL((interact_multi<N, KER, M>), dim3(gl.blocks), dim3(64u << gl.log_w),
                       sizeof(double) * M * (64u << gl.log_w), s, d.tgt, d.src, d.qm, d.slot_nodes,
                       d.qhat16, d.far_slot, d.near_begin, d.near_count, a);
    return hipGetLastError();
}

template <int N, int KER>
hipError_t run_multi_m(const DevicePlan& d, const MultiArgs& a, const GroupLaunch& gl,
                       hipStream_t s)
{
    switch (multi_ld(0, N, a.mc)) {
    case 2: return run_multi<N, KER, 2>(d, a, gl, s);
    case 4: return run_multi<N, KER, 4>(d, a, gl, s);
    case 8: return run_multi<N, KER, 8>(d, a, gl, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_interact_multi(const DevicePlan& d, const KernelParams& kp, double* phi,
                                 int64_t phi_ld, int32_t mc, hipStream_t s)
{
    if (d.ngroups == 0)
        return hipSuccess;
    if (!d.qm || !d.qhat16 || mc < 1 || mc > 8)
        return hipErrorInvalidValue;
    const GroupLaunch gl = group_launch(d);
    const MultiArgs a{d.group_batch, d.group_first, d.batch_end, d.far_off, d.near_off,
                      phi, phi_ld, kp.kconst(), gl.log_w, mc};
    switch (d.degree) {
#define X(n)                                                             \
    case n:                                                              \
        return kp.kernel == 1 ? run_multi_m<n, 1>(d, a, gl, s)           \
             : kp.kernel == 2 ? run_multi_m<n, 2>(d, a, gl, s)           \
                              : run_multi_m<n, 0>(d, a, gl, s);
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace bltc
