// kernels.hpp -- launch wrappers of the gfx950 kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

namespace bltc {

constexpr int kMaxDegree = 16;
constexpr int kMaxHermiteDegree = 10;   // Hermite treecode: 8 (n+1)^3 charges per cluster
// Targets of an interaction workgroup, one per lane of each of its waves.  No
// workgroup of a launch is empty but a few at the end of a die's queue: a
// schedule of 256-target groups with a workgroup per 64 of them left a regular
// pattern of empty ones, which put 4 to 64 waves on a CU (even: 36 to 44) and
// a third of the CUs idle.
constexpr int kGroupSize = 64;
constexpr int kMaxWaves = 16;        // waves of an interaction workgroup
// A grid has fewer than 2^32 threads a dimension (more are cut off without an error):
// larger element-wise launches go in parts of this many.
constexpr int64_t kLaunchThreads = int64_t(1) << 31;

// The direct lists the single-vector interaction kernels walk: the plan's own,
// or, when mutual leaf pairs are evaluated by launch_near_pairs, the reduced
// lists plus per batch the unit results to add (pc_off == nullptr: none).
struct NearLists {
    const int32_t* off;
    const int64_t* begin;
    const int64_t* count;
    const int32_t* leaf;
    const int32_t* pc_off;
    const int64_t* pc_base;
    const double* pair_out;
    const int64_t* batch_begin;
};

// A sub-unit of a mutual pair of leaves (B, C) of a plan whose targets are
// its sources: nb of B's particles at tree positions [tb, tb + nb) against
// C's particles at [sb, sb + nc); row sums (potential at those B targets from
// C's sources) to out[roff + i], column sums (at C's targets from those B
// sources) to out[coff + j].
struct SymUnit {
    int64_t tb, sb, roff, coff;
    int32_t nb, nc;
    int32_t batch;    // B's batch (batch_info)
    int32_t leaf;     // C's node (node_info)
    int32_t apart;    // 1: no pair of the unit is at zero distance (SymPlan::apart)
    int32_t pad;
};

// Device-side view of a plan (all device pointers).
struct DevicePlan {
    int32_t degree = 0;
    int32_t hermite = 0;              // Hermite interpolation: 8 (n+1)^3 values per slot
    int64_t nt = 0, ns = 0, nslots = 0, nchunks = 0, ngroups = 0, nbatches = 0;
    int64_t groups = 0;               // of the ngroups workgroups, those with targets
    void set_groups(const std::vector<int32_t>& batch)   // the schedule's group_batch
    {
        ngroups = static_cast<int64_t>(batch.size());
        groups = ngroups - std::count(batch.begin(), batch.end(), -1);
    }
    // sources in tree order: x, y, z, charge of the current vector
    double4* src = nullptr;
    // targets in batch order: x, y, z, caller index (int64 bits)
    double4* tgt = nullptr;
    const int64_t* src_order = nullptr; // caller index of each tree position
    // FP32-mixed path: sources relative to the center of their leaf
    float4* src32 = nullptr;          // x - c_x, y - c_y, z - c_z, q (tree order)
    double4* node_info = nullptr;     // per source node: box center, radius
    double4* batch_info = nullptr;    // per batch: box center, radius
    // lists
    int32_t* group_batch = nullptr;
    int64_t* group_first = nullptr;
    int64_t* batch_end = nullptr;
    int32_t* far_off = nullptr;
    int32_t* far_slot = nullptr;
    int32_t* near_off = nullptr;
    int64_t* near_begin = nullptr;
    int64_t* near_count = nullptr;
    int32_t* near_leaf = nullptr;
    // upward pass
    double* slot_nodes = nullptr;     // [slot][3][n+1]
    int32_t* chunk_slot = nullptr;
    int64_t* chunk_begin = nullptr;
    int64_t* chunk_count = nullptr;
    int32_t* slot_chunk_off = nullptr;
    int64_t* chunk_dst = nullptr;     // output row of each chunk (slot, or nslots + partial)
    double* qhat = nullptr;           // [slot][P] or [slot][P][16], then partial rows
    int64_t qhat_rows = 0;            // nslots + partial rows
    float* qhat32 = nullptr;          // [slot][P] (mixed precision; Hermite [slot][(n+1)^3][8])
    // several charge vectors at once (16 per pass)
    int32_t* slot_cluster = nullptr;  // cluster id of each slot
    double* qm = nullptr;             // [ns][16] charges in tree order
    float* qm32 = nullptr;            // [ns][16] (mixed precision)
    double* qhat16 = nullptr;         // [slot][P][16] (same storage as qhat)
    double4* proxies = nullptr;       // [slot][P] expanded Chebyshev grid (x, y, z, -)
    float4* proxies32 = nullptr;      // [slot][P] grid relative to the cluster center
    float* qhat16f = nullptr;         // [slot][P][16] (mixed precision)
    // Hermite: modified charges regrouped per grid point, [slot][(n+1)^3][8]
    double* qhat_h = nullptr;
    // symmetric near field (one charge vector): mutual leaf pairs evaluated once
    // by launch_near_pairs; the interaction kernels then take the reduced direct
    // lists and add, per target, the unit results listed in sym_pc_*
    int32_t sym = 0;
    int64_t sym_units = 0;            // sub-units
    // lanes per target asked for (waves of an interaction workgroup, at least)
    int32_t threads_per_target = 1;
    SymUnit* sym_unit = nullptr;
    double* sym_out = nullptr;
    int32_t* sym_near_off = nullptr;
    int64_t* sym_near_begin = nullptr;
    int64_t* sym_near_count = nullptr;
    int32_t* sym_near_leaf = nullptr;
    int32_t* sym_pc_off = nullptr;
    int64_t* sym_pc_base = nullptr;
    int64_t* batch_begin = nullptr;
    // results of the mutual pairs in several rounds through a bounded
    // workspace (sym_rounds > 1): each round's results are folded into
    // sym_acc (one FP64 value per target, tree order), and the interaction
    // kernels read sym_acc through one entry per batch
    int32_t sym_rounds = 0;
    double* sym_acc = nullptr;
};

// Launch of an interaction kernel: a workgroup of 1 << log_w waves per group of the
// schedule.
//
// Waves per workgroup: a target's lists are one serial chain per lane, so a
// problem of few targets leaves the chip (1024 SIMDs, up to 8 waves each: 8192
// resident) idle, and one of many ends in a tail as long as its heaviest workgroup.
// 16 waves leave slots of a CU unused when the registers allow fewer than 32, 2 were
// not faster than 1 and 4 anywhere.  One evaluation at 1, 2, 4, 8, 16 waves, ms:
//   512 groups (30,011 regularized targets) 14.0 at 1, 3.2 at 16; 3.5 10^3 groups
//   (2 10^5 Yukawa targets, n = 6) 21.4 at 1, 16.3 at 8, 17.5 at 16
//   8100 (5 10^5 points, n = 4) FP64 5.82 5.76 5.68 5.96 7.01, eight vectors 11.9 12.0
//   11.4 11.3 13.0
//   20,480 (1.1 10^6) FP64 12.85 12.77 12.76 13.06, three vectors 22.6 22.9 22.1 22.1
//   32,768 (2 10^6) FP64 30.3 30.4 30.3 31.8, three vectors 50.3 51.0 49.8 49.8
// So the FP64 one-vector and the Hermite kernels (`early`) go from 8 to 4 waves a
// little below the resident waves, in groups; the others at as many full groups.
// Groups less than half full on average (small leaves) have lists of many short
// entries, and every wave's search for its cuts weighs more, so fewer waves share:
//   1.3 10^3 groups (3 10^4 points, 64 a leaf) FP32-mixed 0.235 0.201 0.187 0.153 0.126,
//   FP64 0.260 0.209 0.169 0.152 0.168
//   3.7 10^3 (3 10^4 points, 32 a leaf) FP32-mixed 0.286 0.267 0.282 0.305 0.311, FP64
//   0.417 0.392 0.374 0.359 0.423
//   3.1 10^4 (10^5 points, 8 a leaf) FP32-mixed 3.15 3.16 3.39 4.10 5.41
constexpr int64_t kWavesWanted = 32768;
constexpr int64_t kWavesResident = 8192;
constexpr int64_t kGroupsFill = kWavesResident * 7 / 8;   // groups that nearly fill the chip
inline int32_t group_log_waves(int64_t targets, int64_t groups, int32_t asked, int32_t max_waves,
                               bool early)
{
    const int64_t full = (targets + 63) / 64;   // groups if all were full
    int32_t log_w;
    if (full < 512 && groups < 1536)
        log_w = 4;
    else if (groups > 2 * full)
        log_w = groups < kWavesResident / 4 ? 3 : groups < kGroupsFill ? 2 : 0;
    else if (early ? groups < kGroupsFill : full < kWavesResident)
        log_w = 3;
    else
        log_w = full < kWavesWanted ? 2 : 0;
    while ((1 << log_w) > max_waves)
        --log_w;
    while ((1 << log_w) < asked && (2 << log_w) <= max_waves)
        ++log_w;
    // within the threads of a grid (an eighth left for the schedule's empty slots)
    while (log_w > 0 && (groups << (6 + log_w)) > 2 * kLaunchThreads / 8 * 7)
        --log_w;
    return log_w;
}
struct GroupLaunch {
    uint32_t blocks;
    int32_t log_w;
};
inline GroupLaunch group_launch(const DevicePlan& d, int32_t max_waves = kMaxWaves,
                                bool early = false)
{
    return GroupLaunch{static_cast<uint32_t>(d.ngroups),
                       group_log_waves(d.nt, d.groups, d.threads_per_target, max_waves, early)};
}

// Hermite kernels: up to 256 VGPRs a wave (the larger degrees need over 128).  The
// FP32-mixed one stages the charges of a cluster in LDS at n = 3 to 5.
constexpr int kHermiteWaves = 8;
constexpr bool stage_hermite(int32_t degree) { return degree >= 3 && degree <= 5; }
// Charges through the scalar cache: waves of different clusters evict each other's,
// so the lists are shared by fewer waves the more of the chip (8192 waves) the
// groups fill by themselves.  1, 2, 4, 8 waves, ms: 2048 groups (10^5 points, n = 2)
// 1.76 1.15 0.83 0.64; 3584 (2 10^5, n = 6) 4.81 4.49 4.35 4.59; 5632 (3.5 10^5)
// n = 6 7.09 6.74 6.99 7.31, n = 7 8.35 7.80 8.11 8.51; 8100 (5 10^5) n = 1 1.47 1.53
// 1.54 1.58, n = 2 2.93 2.99 3.01 3.16, n = 6 11.8 11.9 12.4 12.7, n = 7 13.0 13.3 13.9
// 14.5, n = 8 16.2 16.1 17.0 17.9, but 7872 n = 9 33.7 31.1 31.2 31.7; 10^6 points n = 6
// to 10 5% less at 1 than at 4.
inline int32_t hermite_mixed_waves(const DevicePlan& d)
{
    return stage_hermite(d.degree) || d.groups < 3072 ? kHermiteWaves : d.groups < 8000 ? 4 : 1;
}

// Waves that the one-vector kernel of a plan takes when no lanes are asked for (the
// FP32-mixed one may take 16 for 8).  Lanes asked for up to this many change nothing.
inline int32_t one_vector_waves(const DevicePlan& d, int32_t precision)
{
    const int32_t most = d.hermite && precision == 1 ? hermite_mixed_waves(d) : kHermiteWaves;
    return 1 << group_log_waves(d.nt, d.groups, 1, most, d.hermite || precision == 0);
}

// Constants of the kernel G passed to the interaction kernels: kappa of the
// Yukawa kernel and delta^2 of the regularized Coulomb kernel.
struct KernelConst {
    double kappa;
    double delta2;
};

// Everything the multi-vector interaction of one system needs (passed by value
// to a kernel, or as an array for the work-queue kernel).
struct MrhsDesc {
    const double4* tgt;
    const double4* src;
    const float4* src32;
    const double* qm;
    const float* qm32;
    const double4* node_info;
    const double4* batch_info;
    const int32_t* group_batch;
    const int64_t* group_first;
    const int64_t* batch_end;
    const int32_t* far_off;
    const int32_t* far_slot;
    const int32_t* near_off;
    const int64_t* near_begin;
    const int64_t* near_count;
    const int32_t* near_leaf;
    const int32_t* slot_cluster;
    const double4* proxies;
    const float4* proxies32;
    const double* qhat16;
    const float* qhat16f;
    double* phi;
    int64_t phi_ld;
    int32_t np;
    int32_t mc;
    KernelConst kc;
};

struct KernelParams {
    int32_t kernel = 0;     // 0 Coulomb, 1 Yukawa, 2 regularized Coulomb
    int32_t precision = 0;  // 0 FP64, 1 FP32-mixed
    double kappa = 0.0;
    double delta = 0.0;
    KernelConst kconst() const { return KernelConst{kappa, delta * delta}; }
};

// src[j].w = q[order[j]] (and src32[j].w when present), j < ns: charges into tree order
hipError_t launch_gather_charges(const DevicePlan& d, const double* q, hipStream_t s);
// upward pass, eqs. 14-15, on the matrix cores (kernels_upward.hip): mw = 1 (charges in
// src[j].w, result buf[slot][k]) or 2, 4, 8 (FP64), 16 (charges in qm[ns][mw], result
// buf[slot][k][mw]);
// buf holds nslots final rows followed by the partial rows of multi-chunk slots
hipError_t launch_upward_mfma(const DevicePlan& d, int32_t mw, double* buf, float* qhat32,
                              hipStream_t s);
// pieces of the same for many systems in one launch (unit = system, chunk)
struct UpwardDesc {
    const double4* src;
    const double* qm;
    const float* qm32;                // FP32 copies of the charges (FP32-mixed plans)
    const int32_t* chunk_slot;
    const int64_t* chunk_begin;
    const int64_t* chunk_count;
    const int64_t* chunk_dst;
    const double* slot_nodes;
    double* buf;
    int32_t np;
};
// nf: factors per dimension (np, or 2 np for the Hermite interpolation)
size_t upward_lds_bytes(int32_t np, int32_t mw, int32_t nf);
int32_t upward_passes(int32_t nf, int32_t mw);
hipError_t upward_prepare(size_t lds);
hipError_t launch_upward_many(const UpwardDesc* descs, const int2* units, int32_t nunits,
                              int32_t mw, int32_t passes, size_t lds, hipStream_t s);
// the 16-vector Lagrange kernel of n + 1 = np <= 9 for systems of one degree:
// whether it applies, and its launch (FP32 matrix-core products when f32)
bool upward_many_multi(int32_t np, int32_t mw);
hipError_t launch_upward_many_multi(const UpwardDesc* descs, const int2* units, int32_t nunits,
                                    int32_t np, bool f32, hipStream_t s);
hipError_t launch_upward_reduce(const DevicePlan& d, int32_t mw, double* buf, float* qhat32,
                                hipStream_t s, int32_t ranges = 1);
// (with d.hermite the upward pass forms 8 (n+1)^3 charges per slot and the
// reduction writes them to d.qhat_h, [slot][k][a], and their FP32 copy to
// qhat32 when given; mw must be 1)
// Hermite approximation and direct sums (kernels_hermite.hip), FP64 or
// FP32-mixed as kp.precision, n <= 10
hipError_t launch_interact_hermite(const DevicePlan& d, const KernelParams& kp, double* phi,
                                   hipStream_t s);
inline NearLists near_lists(const DevicePlan& d)
{
    if (d.sym)
        return NearLists{d.sym_near_off, d.sym_near_begin, d.sym_near_count, d.sym_near_leaf,
                         d.sym_pc_off,   d.sym_pc_base,
                         d.sym_rounds > 1 ? d.sym_acc : d.sym_out,            d.batch_begin};
    return NearLists{d.near_off, d.near_begin, d.near_count, d.near_leaf,
                     nullptr,    nullptr,      nullptr,      nullptr};
}
// near field of the mutual leaf pairs (kernels_sym.hip): sub-units
// d.sym_unit[first .. first + count) into d.sym_out, FP64 or FP32-mixed as
// kp.precision
hipError_t launch_near_pairs(const DevicePlan& d, int64_t first, int64_t count,
                             const KernelParams& kp, hipStream_t s);
// one round of mutual-pair results folded into the per-target sums: for batch
// b (targets at [begin[b], end[b])) and target position p of the batch,
// acc[begin[b] + p] = (first ? 0 : acc[...]) + sum over e in [off[b], off[b + 1])
// of out[base[e] + p], in that order
hipError_t launch_fold_pairs(int64_t nbatches, const int64_t* begin, const int64_t* end,
                             const int32_t* off, const int64_t* base, const double* out,
                             double* acc, bool first, hipStream_t s);
// B targets per sub-unit of launch_near_pairs (one wave holds them all in
// registers, 64 per chunk): FP32-mixed and FP64
constexpr int64_t kSymTargetsMixed = 512;
constexpr int64_t kSymTargetsF64 = 512;
// the FP32-mixed path computes the kernel values of pairs closer than
// kMixedTauRel * (distance of the box centers + r_B + 2 r_C) from FP64 coordinates
constexpr double kMixedTauRel = 2.4e-2;
// side of the largest box of points the FP32-mixed path takes: squared FP32
// distances stay below 3 * 2^120, finite
constexpr double kMixedMaxExtent = 0x1p60;
// batch/cluster interactions: eqs. 9 and 11, phi written in caller order
hipError_t launch_interact(const DevicePlan& d, const KernelParams& kp, double* phi,
                           hipStream_t s);
// the same in FP32-mixed arithmetic (kernels_mixed.hip)
hipError_t launch_interact_mixed(const DevicePlan& d, const KernelParams& kp, double* phi,
                                 hipStream_t s);
// several charge vectors: mc of them at a time, mc <= 16, in tree order in
// d.qm/d.qm32 ([ns][ld], zero padded), their modified charges in d.qhat16
// ([slot][P][ld]); ld = multi_ld(precision, mc).  phi[m * phi_ld + i], m < mc.
//
// FP64 passes of at most 8 vectors with n <= 15 run on the vector units, a grid line
// of n + 1 <= 16 points per row of lanes, their charges packed to the next of 2, 4, 8
// a source; the others run on the matrix cores, whose tiles have 16 columns.  One
// evaluation of 10^6 points, n = 8, 2000 a leaf, FP64 (10^4 points, n = 4, 500 a
// leaf): 8 vectors 104 ms (0.13) on the vector units, 9 to 16 vectors 147 (0.17) on
// the matrix cores against 163-167 (0.22) on the vector units.
constexpr int32_t kMultiMaxDegree = 15;
inline int32_t multi_ld(int32_t precision, int32_t degree, int32_t mc)
{
    return precision == 0 && degree <= kMultiMaxDegree && mc <= 8 ? (mc <= 2 ? 2 : mc <= 4 ? 4 : 8) : 16;
}
hipError_t launch_gather_charges_multi(const DevicePlan& d, const double* q, int64_t q_ld,
                                       int32_t mc, int32_t ld, hipStream_t s);
// on the matrix cores, ld = 16 (kernels_mrhs.hip)
hipError_t launch_interact_mrhs(const DevicePlan& d, const KernelParams& kp, double* phi,
                                int64_t phi_ld, int32_t mc, hipStream_t s);
// in FP64 on the vector units, n <= kMultiMaxDegree, ld <= 8 (kernels_multi.hip)
hipError_t launch_interact_multi(const DevicePlan& d, const KernelParams& kp, double* phi,
                                 int64_t phi_ld, int32_t mc, hipStream_t s);
MrhsDesc make_mrhs_desc(const DevicePlan& d, const KernelParams& kp, double* phi, int64_t phi_ld,
                        int32_t mc);
// work queue over (system, group) units of many systems; counter reset first
hipError_t launch_reset_counter(int32_t* counter, hipStream_t s);
// (persistent workgroups of 1 << log_w waves: as many as the chip holds)
struct QueueLaunch {
    int32_t workgroups = 0, log_w = 0;
};
hipError_t plan_interact_queue(const KernelParams& kp, int32_t nunits, QueueLaunch* q);
hipError_t launch_interact_queue(const MrhsDesc* descs, const int2* units, int32_t nunits,
                                 int32_t* counter, const KernelParams& kp, QueueLaunch q,
                                 hipStream_t s);
// GPU direct sum (eq. 1) of all targets against all sources, m <= kDirectVectors
// charge vectors at once.  split = direct_split(nt, ns); `part` holds the
// pieces' partial sums (pieces * m * nt values; NULL: one piece, phi written
// by the sum itself).
constexpr int32_t kDirectVectors = 4;
// partial sums of one call: a split beyond one piece has fewer than
// 8192 + nt / 64 + 1 target groups times pieces
constexpr int64_t kDirectPartials = int64_t(1) << 22;
struct DirectSplit {
    int32_t pieces = 1;
    int64_t per = 0;        // sources per wave
};
DirectSplit direct_split(int64_t nt, int64_t ns);
hipError_t launch_direct(int64_t nt, const double* tx, const double* ty, const double* tz,
                         int64_t ns, const double* sx, const double* sy, const double* sz,
                         const double* q, int32_t m, int64_t q_ld, const KernelParams& kp,
                         const DirectSplit& split, double* part, double* phi, int64_t phi_ld,
                         hipStream_t s);

}  // namespace bltc
