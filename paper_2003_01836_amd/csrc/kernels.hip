// kernels.hip -- gfx950 kernels of the barycentric Lagrange treecode.
//
// Mapping (CDNA4, wave64):
//  * interactions: one target per lane, 64 targets of one batch per
//    workgroup; every lane of a wave walks the same interaction list (the MAC
//    is applied per batch, Sec. III-B), so source particles, Chebyshev points
//    and modified charges are wave-uniform and are read through the scalar
//    data cache into SGPRs -- no LDS staging.  The waves of a workgroup share
//    the lists of its targets (device_split.hpp); phi is written exactly once,
//    in caller order, without atomics.
//  * the upward pass lives in kernels_upward.hip (matrix cores).
#include <algorithm>

#include "kernels.hpp"
#include "device_common.hpp"
#include "device_split.hpp"

namespace bltc {
namespace {

using namespace dev;

// ---------------------------------------------------------------------------
// Batch/cluster approximation (eq. 11): sum_k G(x, s_k) qhat_k over the planes
// k1 in [ka, kb) of the (n+1)^3 tensor grid.  With the grid separable, r^2 = a_k1 + b_k2 + c_k3
// where a, b, c are the squared 1-D distances, formed once per target.
// `nd` ([3][n+1] points) and `qh` ([P] charges) are wave-uniform.
// ---------------------------------------------------------------------------
template <int N, int KER>
__device__ __forceinline__ double far_sum_f64(double x, double y, double z,
                                              const double* __restrict__ nd,
                                              const double* __restrict__ qh, int ka, int kb,
                                              const KernelArg& kappa)
{
    constexpr int NP = N + 1;
    double b2[NP], c2[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const double dy = y - nd[NP + k];
        const double dz = z - nd[2 * NP + k];
        b2[k] = dy * dy;
        c2[k] = dz * dz;
    }
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll 1
    for (int k1 = ka; k1 < kb; ++k1) {
        const double dx = x - nd[k1];
        const double a2 = dx * dx;
        const double* __restrict__ q1 = qh + k1 * NP * NP;
#pragma unroll
        for (int k2 = 0; k2 < NP; ++k2) {
            const double ab = a2 + b2[k2];
#pragma unroll
            for (int k3 = 0; k3 < NP; ++k3) {
                const double r2 = ab + c2[k3];
                const double g = green_far2_f64<KER>(r2, kappa);
                if ((k2 + k3) & 1)
                    acc1 = __fma_rn(g, q1[k2 * NP + k3], acc1);
                else
                    acc0 = __fma_rn(g, q1[k2 * NP + k3], acc0);
            }
        }
    }
    return 0.5 * (acc0 + acc1);   // the terms are doubled (green_far2_f64)
}

// ---------------------------------------------------------------------------
// Interactions of one workgroup: 64 consecutive targets of one batch, their
// lists shared by the workgroup's waves.
// ---------------------------------------------------------------------------
template <int N, int KER>
__global__ __launch_bounds__(64 * kMaxWaves) void interact_f64(
    int32_t log_w, const double4* __restrict__ tgt,
    const double4* __restrict__ src, const int32_t* __restrict__ group_batch,
    const int64_t* __restrict__ group_first, const int64_t* __restrict__ batch_end,
    const int32_t* __restrict__ far_off, const int32_t* __restrict__ far_slot,
    const int32_t* __restrict__ near_off, const int64_t* __restrict__ near_begin,
    const int64_t* __restrict__ near_count, const double* __restrict__ slot_nodes,
    const double* __restrict__ qhat,
    const int32_t* __restrict__ pc_off, const int64_t* __restrict__ pc_base,
    const double* __restrict__ pair_out, const int64_t* __restrict__ batch_begin,
    double* __restrict__ phi, KernelConst kc)
{
    constexpr int NP = N + 1;
    constexpr int P = NP * NP * NP;
    extern __shared__ double lds[];
    __shared__ double exp_tab[kExpTable];
    if constexpr (KER == 1)
        fill_exp2_table(exp_tab);
    const KernelArg kappa{kc.kappa, kc.delta2, exp_tab};
    const int g = blockIdx.x;
    const int b = group_batch[g];
    if (b < 0)
        return;  // empty slot of the per-die schedule
    const int64_t first = group_first[g];
    const int64_t end = batch_end[b];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int64_t i = first + lane;
    const bool valid = i < end;
    if (!valid)
        i = end - 1;
    const double4 t = tgt[i];
    double acc = 0.0;

    const int f0 = far_off[b];
    const int n1 = near_off[b + 1];
    const ListPart part =
        list_part<NP, NP * NP, KER, false>(w, log_w, far_off[b + 1] - f0, near_off[b], n1, near_count,
                               pc_off ? pc_off[b] : 0, pc_off ? pc_off[b + 1] : 0);
    int f = part.plane0 / NP, ka = part.plane0 - f * NP;
    for (int pl = part.plane0; pl < part.plane1; ++f) {
        const int64_t slot = far_slot[f0 + f];
        const int kb = ka + part.plane1 - pl < NP ? ka + part.plane1 - pl : NP;
        acc += far_sum_f64<N, KER>(t.x, t.y, t.z, slot_nodes + slot * 3 * NP, qhat + slot * P, ka,
                                   kb, kappa);
        pl += kb - ka;
        ka = 0;
    }
    for_direct_runs<false>(part, n1, near_begin, near_count, [&](int64_t j, int32_t cnt, int32_t) {
        acc += near_sum_f64<KER>(t.x, t.y, t.z, src + j, cnt, kappa);
    });
    if (pc_off) {
        // mutual leaf pairs: this target's row or column sums of each unit
        acc += pair_results(part, pc_base, pair_out, i - batch_begin[b]);
    }
    acc = sum_waves(acc, w, log_w, lds);
    if (w == 0 && valid)
        phi[caller_index(t)] = acc;
}

__global__ __launch_bounds__(256) void gather_charges(double4* __restrict__ src,
                                                      float4* __restrict__ src32,
                                                      const int64_t* __restrict__ order,
                                                      const double* __restrict__ q, int64_t ns)
{
    const int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j < ns) {
        const double v = q[order[j]];
        src[j].w = v;
        if (src32)
            src32[j].w = static_cast<float>(v);
    }
}

// ---------------------------------------------------------------------------
// Direct sum of eq. 1: 64 targets (one per lane) per workgroup, whose four
// waves each take a quarter of the workgroup's run of sources, wave-uniform
// and read in place through the scalar cache; a kernel value serves all M
// charge vectors.  Bound: FP64 issue (about 60 SIMD cycles per value and 64
// targets).  With few targets the sources are cut into gridDim.y pieces
// (launch_direct): 1000 targets against 2 10^6 sources took 188 ms with one
// lane per target and every source in it (16 waves on the chip), 1.12 ms so.
// Sums run in a fixed order: within a wave, over the waves, over the pieces.
// ---------------------------------------------------------------------------
constexpr int kDirectWaves = 4;

template <int KER, int M>
__global__ __launch_bounds__(64 * kDirectWaves) void direct_f64(
    int64_t nt, const double* __restrict__ tx, const double* __restrict__ ty,
    const double* __restrict__ tz, int64_t ns, const double* __restrict__ sx,
    const double* __restrict__ sy, const double* __restrict__ sz, const double* __restrict__ q,
    int64_t q_ld, int64_t per, double* __restrict__ out, int64_t out_ld, int64_t out_piece,
    KernelConst kc)
{
    __shared__ double exp_tab[kExpTable];
    __shared__ double part[kDirectWaves][M][64];
    if constexpr (KER == 1)
        fill_exp2_table(exp_tab);
    const KernelArg ka{kc.kappa, kc.delta2, exp_tab};
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    const int64_t it = i < nt ? i : nt - 1;
    const double x = tx[it], y = ty[it], z = tz[it];
    const int64_t j0 = (static_cast<int64_t>(blockIdx.y) * kDirectWaves + w) * per;
    const int64_t j1 = j0 + per < ns ? j0 + per : ns;
    // the terms are doubled (green_near2_f64) and halved once per sum
    constexpr int U = 4;
    double acc[M][U];
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int u = 0; u < U; ++u)
            acc[m][u] = 0.0;
    auto term = [&](int64_t j, int u) {
        const double dx = x - sx[j], dy = y - sy[j], dz = z - sz[j];
        const double r2 = __fma_rn(dz, dz, __fma_rn(dy, dy, dx * dx));
        const double g = green_near2_f64<KER>(r2, ka);
#pragma unroll
        for (int m = 0; m < M; ++m)
            acc[m][u] = __fma_rn(g, q[m * q_ld + j], acc[m][u]);
    };
    int64_t j = j0;
    for (; j + U <= j1; j += U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            term(j + u, u);
    }
    for (; j < j1; ++j)
        term(j, 0);
#pragma unroll
    for (int m = 0; m < M; ++m)
        part[w][m][lane] = 0.5 * ((acc[m][0] + acc[m][1]) + (acc[m][2] + acc[m][3]));
    __syncthreads();
    // wave w adds up vectors w, w + 4, ...
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if ((m % kDirectWaves) != w || i >= nt)
            continue;
        double v = part[0][m][lane];
#pragma unroll
        for (int u = 1; u < kDirectWaves; ++u)
            v += part[u][m][lane];
        out[blockIdx.y * out_piece + m * out_ld + i] = v;
    }
}

// phi[m phi_ld + i] = the pieces' partial sums of (m, i) in piece order
__global__ __launch_bounds__(256) void sum_direct(const double* __restrict__ part, int64_t nt,
                                                  int32_t m_count, int32_t pieces, int64_t k0,
                                                  double* __restrict__ phi, int64_t phi_ld)
{
    const int64_t k = k0 + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (k >= nt * m_count)
        return;
    double v = part[k];
    for (int32_t p = 1; p < pieces; ++p)
        v += part[p * nt * m_count + k];
    const int64_t m = k / nt;
    phi[m * phi_ld + (k - m * nt)] = v;
}

template <int KER>
void run_direct(int m, dim3 grid, hipStream_t s, int64_t nt, const double* tx, const double* ty,
                const double* tz, int64_t ns, const double* sx, const double* sy, const double* sz,
                const double* q, int64_t q_ld, int64_t per, double* out, int64_t out_ld,
                int64_t out_piece, KernelConst kc)
{
    const dim3 block(64 * kDirectWaves);
    switch (m) {
#define X(M)                                                                                     \
    case M:                                                                                      \
        hipLaunchKernelGGL((direct_f64<KER, M>), grid, block, 0, s, nt, tx, ty, tz, ns, sx, sy,  \
                           sz, q, q_ld, per, out, out_ld, out_piece, kc);                        \
        break;
        X(1) X(2) X(3) X(4)
#undef X
    }
}

// ---------------------------------------------------------------------------
// dispatch over the interpolation degree
// ---------------------------------------------------------------------------

template <int N, int KER>
hipError_t run_interact(const DevicePlan& d, double* phi, KernelConst kc, hipStream_t s)
{
    if (d.ngroups == 0)
        return hipSuccess;
    const NearLists nl = near_lists(d);
    const GroupLaunch gl = group_launch(d, kMaxWaves, true);
    hipLaunchKernelGGL((interact_f64<N, KER>), dim3(gl.blocks), dim3(64u << gl.log_w),
                       gl.log_w ? sizeof(double) * (64u << gl.log_w) : 0, s,
                       gl.log_w, d.tgt, d.src, d.group_batch,
                       d.group_first, d.batch_end, d.far_off, d.far_slot, nl.off, nl.begin,
                       nl.count, d.slot_nodes, d.qhat, nl.pc_off, nl.pc_base, nl.pair_out,
                       nl.batch_begin, phi, kc);
    return hipGetLastError();
}

#define BLTC_DEGREE_CASES(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

}  // namespace

hipError_t launch_gather_charges(const DevicePlan& d, const double* q, hipStream_t s)
{
    if (d.ns == 0)
        return hipSuccess;
    hipLaunchKernelGGL(gather_charges, dim3(static_cast<unsigned>((d.ns + 255) / 256)), dim3(256),
                       0, s, d.src, d.src32, d.src_order, q, d.ns);
    return hipGetLastError();
}

hipError_t launch_interact(const DevicePlan& d, const KernelParams& kp, double* phi,
                           hipStream_t s)
{
    const KernelConst kc = kp.kconst();
    switch (d.degree) {
#define X(n)                                                                   \
    case n:                                                                    \
        return kp.kernel == 1 ? run_interact<n, 1>(d, phi, kc, s)              \
             : kp.kernel == 2 ? run_interact<n, 2>(d, phi, kc, s)              \
                              : run_interact<n, 0>(d, phi, kc, s);
        BLTC_DEGREE_CASES(X)
#undef X
    default:
        return hipErrorInvalidValue;
    }
}

// Pieces the sources are cut into: enough workgroups that the last round of
// waves on the chip is short (8192 of four waves, four times what is resident
// at once), pieces of at least 64 sources per wave, one piece when the targets
// alone give that many workgroups.  1000 targets, 2 10^6 sources: 188 ms in
// one piece, 1.12 ms cut.
DirectSplit direct_split(int64_t nt, int64_t ns)
{
    DirectSplit d;
    const int64_t groups = (nt + 63) / 64;
    const int64_t want = (8192 + groups - 1) / std::max<int64_t>(1, groups);
    const int64_t most = (ns + 64 * kDirectWaves - 1) / (64 * kDirectWaves);
    const int64_t pieces = std::max<int64_t>(1, std::min(want, most));
    // whole quads of sources per wave; every piece non-empty
    d.per = std::max<int64_t>(4, ((ns + pieces * kDirectWaves - 1) / (pieces * kDirectWaves) + 3) / 4 * 4);
    d.pieces = static_cast<int32_t>(
        std::max<int64_t>(1, (ns + d.per * kDirectWaves - 1) / (d.per * kDirectWaves)));
    return d;
}

hipError_t launch_direct(int64_t nt, const double* tx, const double* ty, const double* tz,
                         int64_t ns, const double* sx, const double* sy, const double* sz,
                         const double* q, int32_t m, int64_t q_ld, const KernelParams& kp,
                         const DirectSplit& split, double* part, double* phi, int64_t phi_ld,
                         hipStream_t s)
{
    if (nt == 0)
        return hipSuccess;
    if (m < 1 || m > kDirectVectors || split.pieces > 65535 || (!part && split.pieces > 1))
        return hipErrorInvalidValue;
    const KernelConst kc = kp.kconst();
    double* out = part ? part : phi;
    const int64_t out_ld = part ? nt : phi_ld;
    const auto run = kp.kernel == 1 ? run_direct<1> : kp.kernel == 2 ? run_direct<2> : run_direct<0>;
    constexpr int64_t kTargets = kLaunchThreads / (64 * kDirectWaves) * 64;
    for (int64_t t0 = 0; t0 < nt; t0 += kTargets) {
        const int64_t n = std::min(kTargets, nt - t0);
        const dim3 grid(static_cast<unsigned>((n + 63) / 64), static_cast<unsigned>(split.pieces));
        run(m, grid, s, n, tx + t0, ty + t0, tz + t0, ns, sx, sy, sz, q, q_ld, split.per, out + t0,
            out_ld, nt * m, kc);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    if (!part)
        return hipSuccess;
    const int64_t total = nt * m;
    for (int64_t k0 = 0; k0 < total; k0 += kLaunchThreads) {
        const int64_t n = std::min(kLaunchThreads, total - k0);
        hipLaunchKernelGGL(sum_direct, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s,
                           part, nt, m, split.pieces, k0, phi, phi_ld);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace bltc
