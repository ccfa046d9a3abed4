// internal.hpp -- definitions shared by the C-ABI sources (not installed).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "bltc.h"
#include "device_pool.hpp"
#include "kernels.hpp"
#include "planner.hpp"

namespace bltc_detail {

inline std::string& last_error()
{
    static thread_local std::string msg;
    return msg;
}

inline int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    last_error() = buf;
    return code;
}

// why the last allocation of the calling thread failed, when a plan's
// workspace limit refused it (empty otherwise)
inline std::string& limit_note()
{
    static thread_local std::string msg;
    return msg;
}

// A failed HIP call: BLTC_ENOMEM for allocations (the device's or a plan's
// workspace limit), BLTC_EHIP otherwise.
inline int hip_fail(hipError_t e, const char* what)
{
    if (e == hipErrorOutOfMemory) {
        std::string note;
        note.swap(limit_note());
        return fail(BLTC_ENOMEM, "%s: %s", what,
                    note.empty() ? "out of device memory" : note.c_str());
    }
    return fail(BLTC_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// device copy of a host vector (memory not owned by a plan)
template <class T>
hipError_t upload(T** dst, const std::vector<T>& v, hipStream_t s)
{
    const size_t bytes = std::max<size_t>(1, v.size()) * sizeof(T);
    hipError_t e = bltc::device_malloc(reinterpret_cast<void**>(dst), bytes);
    if (e != hipSuccess)
        return e;
    if (!v.empty())
        e = hipMemcpyAsync(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s);
    return e;
}

// device record of a target: position, and its caller index in the fourth word
inline double4 target_record(double x, double y, double z, int64_t index)
{
    double w;
    std::memcpy(&w, &index, sizeof(w));
    return make_double4(x, y, z, w);
}

// the caller indices of n target records on the device (whole records, a block at
// a time: a strided copy of the fourth words goes row by row, 6.7 s for 10^6 targets
// against 9 ms)
inline hipError_t copy_target_order(int64_t* out, const double4* tgt, int64_t n)
{
    constexpr int64_t kBlock = int64_t(1) << 18;   // 8 MiB
    const std::unique_ptr<double4[]> rec(new (std::nothrow) double4[std::min(n, kBlock)]);
    if (!rec)
        return hipErrorOutOfMemory;
    for (int64_t i = 0; i < n; i += kBlock) {
        const int64_t m = std::min(kBlock, n - i);
        const hipError_t e = hipMemcpy(rec.get(), tgt + i, m * sizeof(double4), hipMemcpyDeviceToHost);
        if (e != hipSuccess)
            return e;
        for (int64_t k = 0; k < m; ++k)
            std::memcpy(out + i + k, &rec[k].w, sizeof(int64_t));
    }
    return hipSuccess;
}

}  // namespace bltc_detail

// Device memory for the results of mutual leaf pairs when the whole result
// array does not fit: at most this many bytes per round (a plan's
// workspace_limit can lower it).  Pairs whose results alone exceed a quarter
// of it stay in the plain direct lists.
constexpr int64_t kPairWorkspaceBytes = int64_t(16) << 30;

#define HIP_TRY(call)                                              \
    do {                                                           \
        hipError_t e_ = (call);                                    \
        if (e_ != hipSuccess)                                      \
            return bltc_detail::hip_fail(e_, #call);               \
    } while (0)

struct bltc_plan {
    bltc_params prm{};
    int32_t max_q = 1;
    bltc::HostPlan hp;
    // true when the trees were built on the device: the per-particle arrays
    // (positions, orders, local coordinates) exist only in device memory
    bool device_particles = false;
    // true when the interaction lists were built on the device
    bool device_lists = false;
    int64_t n_items = 0;                 // interaction items (device lists)
    int32_t* item_batch = nullptr;       // device copies of the items (device lists)
    int32_t* item_cluster = nullptr;
    int32_t* item_kind = nullptr;
    // host copies for bltc_plan_view_get (device-built plans)
    mutable std::vector<int64_t> view_src_order, view_tgt_order;
    mutable std::vector<int32_t> view_item_batch, view_item_cluster, view_item_kind;
    mutable std::vector<double> view_batch_lo, view_batch_hi;
    // cluster-particle plans (method BLTC_CLUSTER_PARTICLE): host plan, the
    // proxy-potential and direct launches, interpolation lists, proxy potentials
    bool cp = false;
    bltc::CpPlan cpp;
    bltc::DevicePlan dprox, ddir;
    int32_t* cp_path_off = nullptr;
    int32_t* cp_path_slot = nullptr;
    double* cp_slot_nodes = nullptr;
    double* cp_phat = nullptr;
    // cluster-cluster plans (method BLTC_CLUSTER_CLUSTER): host plan; the
    // interaction launches, interpolation lists and proxy potentials use the
    // members above, the upward pass uses d
    bool cc = false;
    bltc::CcPlan ccp;
    bool uploaded = false;
    int device = -1;
    bltc::DevicePlan d;
    bltc::DeviceBlocks memory;           // released with the plan
    bool timing = false;
    int32_t last_q = 0;                  // charge vectors of the last execution
    int32_t last_ld = 16;                // and the row length of its last pass's charges
    int32_t timed_q = 0;                 // charge vectors covered by the recorded events
    int64_t sym_pair_evals = 0;          // kernel values of the mutual leaf pairs (each serving
                                         // two direct terms), once uploaded
    std::vector<hipEvent_t> events;      // 4 per charge vector
    hipEvent_t ev_pairs = nullptr;       // after the mutual-pair launch (timing)
    bool timed_pairs = false;            // ev_pairs belongs to the recorded execution
    // device memory the plan holds (requested bytes) and its limit (0: none)
    int64_t bytes = 0;
    int64_t limit = 0;
    // Mutual leaf pairs (d.sym): planned with the direct lists, their result
    // workspace and sub-units sized once the rest of the device side exists
    // (bltc_internal_finish_pairs), in one round when the whole result array
    // fits under the workspace cap, else in rounds folded into per-target sums.
    struct Pairs {
        bltc::DevicePlan* d = nullptr;   // the view whose direct lists hold the pairs
        bltc::SymPlan sp;                // every mutual pair taken
        std::vector<int64_t> batch_begin, batch_count;
        std::vector<int32_t> batch_node;
        bool pending = false;
        int64_t count = 0;               // mutual pairs evaluated once
        int32_t rounds = 0;
        int64_t workspace_bytes = 0;     // result workspace (and per-target sums)
        std::vector<int32_t> round_unit; // rounds + 1 sub-unit offsets
        int32_t* fold_off = nullptr;     // [rounds][batches + 1]
        int64_t* fold_base = nullptr;
        int64_t* batch_end = nullptr;    // device copy of begin + count per batch
    } pairs;

    ~bltc_plan()
    {
        for (hipEvent_t e : events)
            (void)hipEventDestroy(e);
        if (ev_pairs)
            (void)hipEventDestroy(ev_pairs);
    }

    // every device allocation of the plan: counted against its limit
    // (padding, which the plan's own layout adds, is not)
    hipError_t alloc_bytes(void** dst, size_t bytes_wanted, size_t padding = 0)
    {
        const size_t n = std::max<size_t>(1, bytes_wanted);
        if (limit > 0 && bytes + static_cast<int64_t>(n) > limit) {
            char buf[160];
            std::snprintf(buf, sizeof(buf),
                          "workspace_limit of %lld bytes reached (%lld held, %lld more needed)",
                          static_cast<long long>(limit), static_cast<long long>(bytes),
                          static_cast<long long>(n));
            bltc_detail::limit_note() = buf;
            return hipErrorOutOfMemory;
        }
        hipError_t e = memory.get(dst, n + padding);
        if (e == hipSuccess)
            bytes += static_cast<int64_t>(n);
        return e;
    }

    template <class T>
    hipError_t put(T** dst, const std::vector<T>& v, hipStream_t s)
    {
        hipError_t e = alloc_bytes(reinterpret_cast<void**>(dst), v.size() * sizeof(T));
        if (e == hipSuccess && !v.empty())
            e = hipMemcpyAsync(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s);
        return e;
    }

    // as put, a small table with the others of the pack when that is sent
    template <class T>
    hipError_t put(T** dst, const std::vector<T>& v, bltc::Pack& pack, hipStream_t s)
    {
        return pack.add(dst, v) ? hipSuccess : put(dst, v, s);
    }

    hipError_t send(const bltc::Pack& pack, hipStream_t s)
    {
        if (pack.bytes() == 0)
            return hipSuccess;
        void* block = nullptr;
        hipError_t e = alloc_bytes(&block, pack.wanted(), pack.bytes() - pack.wanted());
        return e == hipSuccess ? pack.send(block, s) : e;
    }

    template <class T>
    hipError_t alloc(T** dst, size_t count)
    {
        return alloc_bytes(reinterpret_cast<void**>(dst), count * sizeof(T));
    }
};


// device side of a plan (uploads on first use); synchronises the stream
int bltc_internal_upload_plan(bltc_plan* plan, hipStream_t s);

// Mutual direct pairs of one-tree direct lists evaluated once (see
// plan_symmetric): plans them, uploads the reduced lists and the per-batch
// result offsets into d (d.sym = 1), lowers the lists' batch_cost in *cost to
// the work left to the batches, and leaves the result workspace and the
// sub-units to bltc_internal_finish_pairs.  Returns BLTC_OK and leaves d alone
// when no pair qualifies.  d must be a member of *plan (d or ddir).
int bltc_internal_upload_symmetric(bltc_plan* plan, bltc::DevicePlan& d,
                                   const bltc::DirectLists& dl, std::vector<int64_t>* cost,
                                   hipStream_t s);
// The result workspace of the planned mutual pairs, sized from what the
// plan's workspace limit leaves once every other device array exists: one
// round when all results fit (at most kPairWorkspaceBytes), else rounds.
// BLTC_ENOMEM when the limit leaves no room for the largest pair.
int bltc_internal_finish_pairs(bltc_plan* plan, hipStream_t s);
// Enqueues the mutual-pair launches of d (every round, each folded into the
// per-target sums when there are several).
int bltc_internal_pairs(bltc_plan* plan, const bltc::DevicePlan& d, const bltc::KernelParams& kp,
                        hipStream_t s);

// Parameters left to the tuner (leaf_size = batch_size = 0, or threads per
// target 0 for a one-vector BLTC or Hermite plan) filled in by timing plans
// on the device (autotune.cpp; results cached as bltc_autotune's).  *out = *p
// when nothing is open.
int bltc_internal_tune(const bltc_params* p, int64_t nt, const double* tx, const double* ty,
                       const double* tz, int64_t ns, const double* sx, const double* sy,
                       const double* sz, int32_t max_q, bltc_params* out, void* stream);

// BLTC_EUNSUPPORTED for an FP32-mixed plan whose points do not fit in a box of
// side kMixedMaxExtent (capi.cpp); BLTC_OK otherwise.
int bltc_internal_check_mixed_extent(const bltc_plan* plan);

// Argument checks of bltc_direct and bltc_direct_noalloc (capi.cpp).
int bltc_internal_check_direct(const bltc_params* p, int64_t nt, const double* tx,
                               const double* ty, const double* tz, int64_t ns, const double* sx,
                               const double* sy, const double* sz, const double* q, int32_t num_q,
                               const double* phi);

// The launches of bltc_direct and bltc_direct_noalloc: every charge vector's
// direct sum, with room in `part` for the partial sums of one launch (NULL:
// split has one piece and phi is written directly).
int bltc_internal_direct(const bltc_params* p, int64_t nt, const double* tx, const double* ty,
                         const double* tz, int64_t ns, const double* sx, const double* sy,
                         const double* sz, const double* q, int32_t num_q, int64_t q_ld,
                         double* phi, int64_t phi_ld, const bltc::DirectSplit& split, double* part,
                         hipStream_t s);
// Whether phi shares memory with an input (potentials written over the
// charges).  The sums of a launch then go through `part`, so that it reads its
// sources and its up to kDirectVectors charge vectors before it writes a
// potential; potentials over what a later launch reads (coordinates, later
// charge vectors) change what that launch computes.
bool bltc_internal_direct_overlap(int64_t nt, const double* tx, const double* ty, const double* tz,
                                  int64_t ns, const double* sx, const double* sy, const double* sz,
                                  const double* q, int32_t num_q, int64_t q_ld, const double* phi,
                                  int64_t phi_ld);

// cluster-particle plans (cp.cpp)
namespace bltc_cp {
int create_host(bltc_plan* plan, const bltc::PlanParams& pp, int64_t nt, const double* tx,
                const double* ty, const double* tz, int64_t ns, const double* sx, const double* sy,
                const double* sz);
int create_device(bltc_plan* plan, const bltc::PlanParams& pp, int64_t nt, const double* tx,
                  const double* ty, const double* tz, int64_t ns, const double* sx,
                  const double* sy, const double* sz, hipStream_t s);
int upload(bltc_plan* plan, hipStream_t s);
int execute(bltc_plan* plan, const double* q, int32_t num_q, double* phi, hipStream_t s);
int proxy_potentials(bltc_plan* plan, int64_t cluster, double* out, hipStream_t s);
void stats(const bltc_plan* plan, bltc_stats* out);
int view(const bltc_plan* plan, bltc_plan_view* out);
// Pieces of the proxy-potential lists off/count (one list per slot, entries
// = source ranges): runs of whole entries of one slot with at most
// max(8192, listed / 16384) sources, so that the heaviest clusters do not set
// the run time of launch_proxy_potentials.  A slot's only piece writes the
// slot's row, several pieces write partial rows past the slots (summed by
// launch_upward_reduce).  Uploads d.chunk_slot / chunk_begin (first entry) /
// chunk_count (entries) / chunk_dst (row) / slot_chunk_off, sets d.nchunks
// and d.nslots, and returns the number of rows in *rows.
int upload_pieces(bltc_plan* plan, bltc::DevicePlan& d, const std::vector<int32_t>& off,
                  const std::vector<int64_t>& count, int64_t* rows, hipStream_t s);
}  // namespace bltc_cp

// cluster-cluster plans (cc.cpp)
namespace bltc_cc {
int create_host(bltc_plan* plan, const bltc::PlanParams& pp, int64_t nt, const double* tx,
                const double* ty, const double* tz, int64_t ns, const double* sx, const double* sy,
                const double* sz);
int create_device(bltc_plan* plan, const bltc::PlanParams& pp, int64_t nt, const double* tx,
                  const double* ty, const double* tz, int64_t ns, const double* sx,
                  const double* sy, const double* sz, hipStream_t s);
int upload(bltc_plan* plan, hipStream_t s);
int execute(bltc_plan* plan, const double* q, int32_t num_q, double* phi, hipStream_t s);
int proxy_potentials(bltc_plan* plan, int64_t cluster, double* out, hipStream_t s);
void stats(const bltc_plan* plan, bltc_stats* out);
int view(const bltc_plan* plan, bltc_plan_view* out);
}  // namespace bltc_cc
