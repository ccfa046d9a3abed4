// device_split.hpp -- how the waves of an interaction workgroup share the
// interaction lists of their targets.
//
// A workgroup holds 64 targets of one batch, one per lane, in each of its W
// waves (W = 1, 2, 4, 8 or 16, chosen per launch: group_log_waves).  Wave w
// takes the w-th of W parts of equal estimated work of the batch's lists laid
// end to end -- the (n+1) planes of every approximated cluster, the direct
// entries in blocks of kSplitBlock sources, the mutual-pair results -- and the
// waves' sums are added in wave order through LDS (fixed order, no atomics, no
// memory beyond LDS).  Lists stay wave-uniform in every wave.  Cuts fall only
// where the FP32-mixed sums go to FP64 anyway (a plane, 128 sources), so the
// split changes nothing but the order of FP64 additions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bltc {
namespace dev {

// sources of a block of the direct entries: FP32-mixed the flush length of its
// sums, FP64 a length that divides the few hundred sources of a small problem's
// leaves evenly among 16 waves
template <bool MIXED>
constexpr int kSplitBlock = MIXED ? 128 : 32;

struct ListPart {
    int32_t plane0, plane1;   // planes f (n+1) + k1 of the batch's far list
    int32_t entry;            // first direct entry, the block it starts with,
    int32_t skip;             // and how many blocks from there
    int32_t blocks;
    int32_t pc0, pc1;         // mutual-pair results
};

// Cost of a direct value in far-field kernel values of the same kernel and
// precision: three differences and squares, against one addition, beside the
// reciprocal square root (and, Yukawa, the exponential) that both form.
template <int KER, bool MIXED>
constexpr int kDirectCost = MIXED ? (KER == 1 ? 180 : 220) : (KER == 1 ? 130 : 180);   // percent

// Part w of 2^log_w of far entries [0, nf) with NP planes of PLANE far-field
// kernel values, direct entries [n0, n1) in blocks and pair results [p0, p1).
template <int NP, int PLANE, int KER, bool MIXED>
__device__ __forceinline__ ListPart list_part(int w, int log_w, int32_t nf, int32_t n0, int32_t n1,
                                              const int64_t* __restrict__ near_count, int32_t p0,
                                              int32_t p1)
{
    ListPart r;
    if (log_w == 0) {
        r.plane0 = 0;
        r.plane1 = nf * NP;
        r.entry = n0;
        r.skip = 0;
        r.blocks = INT32_MAX;
        r.pc0 = p0;
        r.pc1 = p1;
        return r;
    }
    constexpr int kPairCost = 4;   // a load and an addition
    constexpr int kBlock = kSplitBlock<MIXED>;
    constexpr int BLOCK = kDirectCost<KER, MIXED> * kBlock / 100;
    const int lane = threadIdx.x & 63;
    int32_t mine = 0;
    for (int32_t e = n0 + lane; e < n1; e += 64)
        mine += static_cast<int32_t>((near_count[e] + (kBlock - 1)) / kBlock);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        mine += __shfl_xor(mine, m);
    const int64_t nb = __builtin_amdgcn_readfirstlane(mine);
    const int64_t npl = static_cast<int64_t>(nf) * NP;
    const int64_t npc = p1 - p0;
    const int64_t far_cost = npl * PLANE, near_cost = nb * BLOCK;
    const int64_t total = far_cost + near_cost + npc * kPairCost;
    int32_t pl[2], bl[2], pc[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        // the cut at k = w or w + 1 parts, rounded to whole planes and blocks
        const int64_t a = (total * (w + k)) >> log_w;
        pl[k] = static_cast<int32_t>(a < far_cost ? (a + PLANE / 2) / PLANE : npl);
        const int64_t a1 = a - far_cost;
        bl[k] = a1 <= 0 ? 0
                        : static_cast<int32_t>(a1 < near_cost ? (a1 + BLOCK / 2) / BLOCK : nb);
        const int64_t a2 = a1 - near_cost;
        pc[k] = a2 <= 0 ? 0
                        : static_cast<int32_t>(a2 < npc * kPairCost ? (a2 + kPairCost / 2) / kPairCost
                                                                    : npc);
    }
    r.plane0 = pl[0];
    r.plane1 = pl[1];
    r.pc0 = p0 + pc[0];
    r.pc1 = p0 + pc[1];
    r.blocks = bl[1] - bl[0];
    r.entry = n1;
    r.skip = 0;
    if (r.blocks > 0) {
        // the entry that holds block bl[0]
        int32_t base = 0;
        for (int32_t e0 = n0; e0 < n1; e0 += 64) {
            const int32_t e = e0 + lane;
            const int32_t own =
                e < n1 ? static_cast<int32_t>((near_count[e] + (kBlock - 1)) / kBlock) : 0;
            int32_t upto = own;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int32_t v = __shfl_up(upto, m);
                upto += lane >= m ? v : 0;
            }
            const uint64_t past = __ballot(base + upto > bl[0]);
            if (past) {
                const int at = __builtin_ctzll(past);
                r.entry = __builtin_amdgcn_readfirstlane(e0 + at);
                r.skip = __builtin_amdgcn_readfirstlane(
                    bl[0] - (base + __shfl(upto, at) - __shfl(own, at)));
                break;
            }
            base += __builtin_amdgcn_readlane(upto, 63);
        }
    }
    return r;
}

// Direct entries of a part: sum(first source of the run, its length, entry).
template <bool MIXED, class F>
__device__ __forceinline__ void for_direct_runs(const ListPart& part, int32_t n1,
                                                const int64_t* __restrict__ near_begin,
                                                const int64_t* __restrict__ near_count, F&& sum)
{
    int32_t left = part.blocks, skip = part.skip;
    for (int32_t e = part.entry; left > 0 && e < n1; ++e) {
        constexpr int kBlock = kSplitBlock<MIXED>;
        const int32_t j0 = skip * kBlock;
        const int32_t avail = static_cast<int32_t>(near_count[e]) - j0;
        const int32_t have = (avail + (kBlock - 1)) / kBlock;
        const int32_t cnt = left < have ? left * kBlock : avail;
        sum(near_begin[e] + j0, cnt, e);
        left -= have;
        skip = 0;
    }
}

// Mutual-pair results of a part for the target at position pos of its batch.
__device__ __forceinline__ double pair_results(const ListPart& part,
                                               const int64_t* __restrict__ pc_base,
                                               const double* __restrict__ pair_out, int64_t pos)
{
    double v = 0.0;
#pragma unroll 4
    for (int e = part.pc0; e < part.pc1; ++e)
        v += pair_out[pc_base[e] + pos];
    return v;
}

// LDS written by a lane and read by others of the same wave: LDS operations of a
// wave run in order, so no workgroup barrier is needed (waves of a workgroup
// walk different lists and must not meet one).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sum of the waves' values per lane, in wave order; valid in wave 0.  `red`:
// 64 doubles per wave of LDS that no wave reads or writes for anything else
// after it has entered.
__device__ __forceinline__ double sum_waves(double v, int w, int log_w, double* red)
{
    if (log_w == 0)
        return v;
    const int lane = threadIdx.x & 63;
    __syncthreads();   // the LDS may have held staged charges
    if (w > 0)
        red[64 * w + lane] = v;
    __syncthreads();
    if (w == 0)
        for (int u = 1; u < (1 << log_w); ++u)
            v += red[64 * u + lane];
    return v;
}

}  // namespace dev
}  // namespace bltc
