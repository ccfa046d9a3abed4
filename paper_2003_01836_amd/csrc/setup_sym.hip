// setup_sym.hip -- planning of the mutual leaf pairs on the GPU.
//
// Two leaves in each other's direct lists are evaluated once for both directions
// (kernels_sym.hip).  Finding the pairs, cutting them into sub-units and taking
// them out of the lists is work on 10^5 to 10^7 list entries: one wave per batch
// here, over the direct lists that are on the device anyway.
//
//  1. match: for every entry (b, leaf c) the entry (c, leaf b), if there is one
//     (c's list bisected by the lane: the lists are in depth-first order, so the
//     first sources of their leaves ascend), and per-batch counts;
//  2. the host adds up the counts of the batches and sizes the arrays;
//  3. fill: the entries that stay, in list order; for the lower batch of a pair its
//     sub-units and the offsets of its rows and column blocks;
//  4. results: per batch, in list order, the offsets it adds up.
//
// Sub-units are placed heaviest first (a counting sort over kBuckets weights; the
// order within a weight does not matter to the results): in batch order the pair
// launch's tail cost the 10^6-point FP64 step 4%.
//
// 10^6 points (1093 batches, 25,100 pairs, 72,000 sub-units): 0.2 ms here, 6.5 ms
// on 16 host threads; 10^4 points: 20 us, 0.8 ms (starting the threads).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "kernels.hpp"
#include "planner.hpp"
#include "setup_gpu.hpp"

namespace bltc {
namespace {

constexpr int kSymWaves = 4;   // batches per workgroup

struct SymBatch {
    int64_t begin, count;
    double lo[3], hi[3];
    int32_t node;
    int32_t off;          // first direct entry
};

struct SymCount {
    int64_t out;          // result values of the batch's units (as their lower batch)
    int64_t evals;
    int64_t cut;          // direct evaluations per target taken out of its lists
    int64_t largest;      // result values of its largest unit
    int32_t kept, units, results;
    int32_t bad;          // an entry that is no batch's leaf, or out of order
};

struct SymOffsets {
    int64_t out;                   // result values
    int32_t kept, results;         // entries that stay, result offsets
};

// bucket of a sub-unit of `weight` kernel values, heaviest in bucket 0
constexpr int kBuckets = 1024;
__device__ __forceinline__ int weight_bucket(int64_t weight, double scale)
{
    const int k = static_cast<int>(static_cast<double>(weight) * scale);
    return kBuckets - 1 - (k < kBuckets ? k : kBuckets - 1);
}

__device__ __forceinline__ int64_t subs_of(int64_t count, int64_t sub)
{
    return (count + sub - 1) / sub;
}

__device__ __forceinline__ int64_t wave_total(long long v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        v += __shfl_xor(v, m);
    return v;
}

// sum over the lanes below; `total` over all
__device__ __forceinline__ int64_t wave_before(long long v, int64_t& total)
{
    const int lane = threadIdx.x % 64;
    long long upto = v;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const long long u = __shfl_up(upto, m);
        upto += lane >= m ? u : 0;
    }
    total = __shfl(upto, 63);
    return upto - v;
}

__global__ void __launch_bounds__(256) clear_buckets(int32_t* __restrict__ hist)
{
    hist[blockIdx.x * 256 + threadIdx.x] = 0;
}

__global__ void __launch_bounds__(64 * kSymWaves)
match_pairs(int32_t nb, const SymBatch* __restrict__ batches, const int32_t* __restrict__ near_leaf,
            const int64_t* __restrict__ near_begin, const int32_t* __restrict__ batch_of, int64_t sub,
            double scale,
            int32_t* __restrict__ match, SymCount* __restrict__ counts, int32_t* __restrict__ hist)
{
    const int32_t b = blockIdx.x * kSymWaves + threadIdx.x / 64;
    if (b >= nb)
        return;
    const int lane = threadIdx.x % 64;
    const SymBatch B = batches[b];
    const int32_t end = batches[b + 1].off;
    long long out = 0, evals = 0, cut = 0, largest = 0, kept = 0, units = 0, results = 0, bad = 0;
    for (int32_t e = B.off + lane; e < end; e += 64) {
        const int32_t c = batch_of[near_leaf[e]];
        int32_t at = -1;
        if (c < 0 || (e > B.off && near_begin[e] <= near_begin[e - 1])) {
            bad = 1;
        } else if (c != b) {
            int32_t k = batches[c].off, last = batches[c + 1].off;
            while (k < last) {
                const int32_t mid = k + (last - k) / 2;
                if (near_begin[mid] < B.begin)
                    k = mid + 1;
                else
                    last = mid;
            }
            if (k < batches[c + 1].off && near_leaf[k] == B.node)
                at = k;
        }
        match[e] = at;
        if (at < 0) {
            ++kept;
            continue;
        }
        const int64_t nc = batches[c].count;
        if (c > b) {
            const int64_t size = B.count + subs_of(B.count, sub) * nc;
            ++units;
            out += size;
            largest = max(largest, static_cast<long long>(size));
            evals += B.count * nc;
            const int32_t full = static_cast<int32_t>(B.count / sub);
            if (full > 0)
                atomicAdd(hist + weight_bucket(sub * nc, scale), full);
            if (B.count % sub)
                atomicAdd(hist + weight_bucket(B.count % sub * nc, scale), 1);
            results += 1;
            cut += nc - 1;          // one read instead of |C| evaluations
        } else {
            const int64_t ns = subs_of(nc, sub);
            results += ns;
            cut += nc - ns;
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        largest = max(largest, __shfl_xor(largest, m));
    SymCount r;
    r.out = wave_total(out);
    r.evals = wave_total(evals);
    r.cut = wave_total(cut);
    r.largest = largest;
    r.kept = static_cast<int32_t>(wave_total(kept));
    r.units = static_cast<int32_t>(wave_total(units));
    r.results = static_cast<int32_t>(wave_total(results));
    r.bad = static_cast<int32_t>(wave_total(bad));
    if (lane == 0)
        counts[b] = r;
}

__global__ void __launch_bounds__(64 * kSymWaves)
fill_pairs(int32_t nb, const SymBatch* __restrict__ batches, const SymOffsets* __restrict__ offs,
           const int32_t* __restrict__ near_leaf, const int32_t* __restrict__ batch_of,
           const int32_t* __restrict__ match, int64_t sub, double scale,
           int32_t* __restrict__ next, int32_t* __restrict__ leaf2, int64_t* __restrict__ begin2, int64_t* __restrict__ count2,
           const int64_t* __restrict__ near_begin, const int64_t* __restrict__ near_count,
           SymUnit* __restrict__ units, int64_t* __restrict__ rows)
{
    const int32_t b = blockIdx.x * kSymWaves + threadIdx.x / 64;
    if (b >= nb)
        return;
    const int lane = threadIdx.x % 64;
    const SymBatch B = batches[b];
    const int32_t end = batches[b + 1].off;
    const SymOffsets o = offs[b];
    const int64_t ns = subs_of(B.count, sub);
    int64_t kept0 = o.kept, out0 = o.out;
    for (int32_t e0 = B.off; e0 < end; e0 += 64) {
        const int32_t e = e0 + lane;
        const bool on = e < end;
        const int32_t leaf = on ? near_leaf[e] : -1;
        const int32_t c = on ? batch_of[leaf] : -1;
        const bool mutual = on && match[e] >= 0;
        const bool lower = mutual && c > b;
        const int64_t nc = lower ? batches[c].count : 0;
        int64_t nkept, nout;
        const int64_t k = kept0 + wave_before(on && !mutual ? 1 : 0, nkept);
        const int64_t roff = out0 + wave_before(lower ? B.count + ns * nc : 0, nout);
        if (on && !mutual) {
            leaf2[k] = leaf;
            begin2[k] = near_begin[e];
            count2[k] = near_count[e];
        }
        if (lower) {
            rows[e] = roff;
            const SymBatch C = batches[c];
            double gap = -INFINITY;
            for (int l = 0; l < 3; ++l)
                gap = fmax(gap, fmax(C.lo[l] - B.hi[l], B.lo[l] - C.hi[l]));
            for (int64_t q = 0; q < ns; ++q) {
                SymUnit su;
                su.tb = B.begin + q * sub;
                su.sb = C.begin;
                su.roff = roff + q * sub;
                su.coff = roff + B.count + q * C.count;
                su.nb = static_cast<int32_t>(min(sub, B.count - q * sub));
                su.nc = static_cast<int32_t>(C.count);
                su.batch = b;
                su.leaf = C.node;
                su.apart = gap >= 0x1p-500 ? 1 : 0;
                su.pad = 0;
                const int64_t weight = static_cast<int64_t>(su.nb) * su.nc;
                units[atomicAdd(next + weight_bucket(weight, scale), 1)] = su;
            }
        }
        kept0 += nkept;
        out0 += nout;
    }
}

__global__ void __launch_bounds__(64 * kSymWaves)
pair_results(int32_t nb, const SymBatch* __restrict__ batches, const SymOffsets* __restrict__ offs,
             const int32_t* __restrict__ near_leaf, const int32_t* __restrict__ batch_of,
             const int32_t* __restrict__ match, int64_t sub, const int64_t* __restrict__ rows,
             int64_t* __restrict__ base)
{
    const int32_t b = blockIdx.x * kSymWaves + threadIdx.x / 64;
    if (b >= nb)
        return;
    const int lane = threadIdx.x % 64;
    const int32_t first = batches[b].off, end = batches[b + 1].off;
    const int64_t count = batches[b].count;
    int64_t at = offs[b].results;
    for (int32_t e0 = first; e0 < end; e0 += 64) {
        const int32_t e = e0 + lane;
        const int32_t m = e < end ? match[e] : -1;
        const int32_t c = m >= 0 ? batch_of[near_leaf[e]] : -1;
        // lower batch of the pair: its rows; upper: a column block per sub-unit
        const int64_t nc = m >= 0 ? batches[c].count : 0;
        const int64_t n = m < 0 ? 0 : c > b ? 1 : subs_of(nc, sub);
        int64_t total;
        const int64_t k = at + wave_before(n, total);
        if (m >= 0) {
            if (c > b) {
                base[k] = rows[e];
            } else {
                const int64_t coff = rows[m] + nc;
                for (int64_t q = 0; q < n; ++q)
                    base[k + q] = coff + q * count;
            }
        }
        at += total;
    }
}

#define SYM_TRY(call)              \
    do {                           \
        hipError_t e_ = (call);    \
        if (e_ != hipSuccess)      \
            return e_;             \
    } while (0)

// device scratch of one call
struct Scratch {
    DeviceBlocks mem;
    template <class T>
    hipError_t get(T** p, size_t n)
    {
        return mem.get(reinterpret_cast<void**>(p), n * sizeof(T));
    }
    template <class T>
    hipError_t put(T** p, const std::vector<T>& v, hipStream_t s)
    {
        hipError_t e = get(p, v.size());
        if (e == hipSuccess && !v.empty())
            e = hipMemcpyAsync(*p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s);
        return e;
    }
    // a small table goes with the others of the pack when that is sent
    template <class T>
    hipError_t put(T** p, const std::vector<T>& v, Pack& pack, hipStream_t s)
    {
        return pack.add(p, v) ? hipSuccess : put(p, v, s);
    }
    hipError_t send(const Pack& pack, hipStream_t s)
    {
        if (pack.bytes() == 0)
            return hipSuccess;
        void* block = nullptr;
        hipError_t e = mem.get(&block, pack.bytes());
        return e == hipSuccess ? pack.send(block, s) : e;
    }
};

}  // namespace

hipError_t plan_symmetric_device(const DirectLists& dl, const DevicePlan& lists, int64_t sub,
                                 int64_t max_bytes, int64_t max_unit, const DeviceAlloc& alloc,
                                 SymDevice& out, hipStream_t s)
{
    out = SymDevice();
    const Tree& S = *dl.tree;
    const std::vector<int32_t>& near_off = *dl.near_off;
    const int64_t nb = static_cast<int64_t>(dl.batch_node->size());
    const int64_t ne = nb > 0 ? near_off[nb] : 0;
    if (ne == 0 || nb >= INT32_MAX) {
        out.planned = ne == 0;
        return hipSuccess;
    }
    std::vector<int32_t> batch_of(S.nodes(), -1);
    std::vector<SymBatch> batches(static_cast<size_t>(nb) + 1);
    for (int64_t b = 0; b < nb; ++b) {
        const int32_t u = (*dl.batch_node)[b];
        batch_of[u] = static_cast<int32_t>(b);
        SymBatch& t = batches[b];
        t.begin = (*dl.batch_begin)[b];
        t.count = (*dl.batch_count)[b];
        for (int l = 0; l < 3; ++l) {
            t.lo[l] = S.lo[3 * u + l];
            t.hi[l] = S.hi[3 * u + l];
        }
        t.node = u;
        t.off = near_off[b];
    }
    batches[nb] = SymBatch();
    batches[nb].off = near_off[nb];
    Scratch mem;
    int32_t *batch_of_d, *match;
    SymBatch* batches_d;
    SymCount* counts_d;
    Pack tables;
    SYM_TRY(mem.put(&batch_of_d, batch_of, tables, s));
    SYM_TRY(mem.put(&batches_d, batches, tables, s));
    SYM_TRY(mem.send(tables, s));
    SYM_TRY(mem.get(&match, ne));
    // the counts of the batches and the sub-units of each weight, one copy back
    std::vector<SymCount> counts(static_cast<size_t>(nb) +
                                 (kBuckets * sizeof(int32_t) + sizeof(SymCount) - 1) / sizeof(SymCount));
    SYM_TRY(mem.get(&counts_d, counts.size()));
    int32_t* const hist_d = reinterpret_cast<int32_t*>(counts_d + nb);
    clear_buckets<<<kBuckets / 256, 256, 0, s>>>(hist_d);
    SYM_TRY(hipGetLastError());
    int64_t most = 1;
    for (int64_t b = 0; b < nb; ++b)
        most = std::max(most, batches[b].count);
    const double scale = kBuckets / (static_cast<double>(std::min(sub, most)) * most + 1.0);
    const uint32_t grid = static_cast<uint32_t>((nb + kSymWaves - 1) / kSymWaves);
    const int32_t n = static_cast<int32_t>(nb);
    match_pairs<<<grid, 64 * kSymWaves, 0, s>>>(n, batches_d, lists.near_leaf, lists.near_begin, batch_of_d,
                                                sub, scale, match, counts_d, hist_d);
    SYM_TRY(hipGetLastError());
    SYM_TRY(hipMemcpyAsync(counts.data(), counts_d, counts.size() * sizeof(SymCount),
                           hipMemcpyDeviceToHost, s));
    SYM_TRY(hipStreamSynchronize(s));

    std::vector<SymOffsets> offs(static_cast<size_t>(nb));
    std::vector<int32_t> off2(static_cast<size_t>(nb) + 1), pc_off(off2.size());
    int64_t values = 0, kept = 0, results = 0, largest = 0, bad = 0, nsub = 0;
    out.cut.resize(static_cast<size_t>(nb));
    for (int64_t b = 0; b < nb; ++b) {
        const SymCount& c = counts[b];
        offs[b] = {values, static_cast<int32_t>(kept), static_cast<int32_t>(results)};
        off2[b] = static_cast<int32_t>(kept);
        pc_off[b] = static_cast<int32_t>(results);
        values += c.out;
        kept += c.kept;
        results += c.results;
        largest = std::max(largest, c.largest);
        bad += c.bad;
        out.units += c.units;
        out.pair_evals += c.evals;
        out.cut[b] = c.cut;
    }
    std::vector<int32_t> first(kBuckets);
    const int32_t* const hist = reinterpret_cast<const int32_t*>(counts.data() + nb);
    for (int k = 0; k < kBuckets; ++k) {
        first[k] = static_cast<int32_t>(nsub);
        nsub += hist[k];
    }
    const int64_t out_bytes = values * static_cast<int64_t>(sizeof(double));
    if (bad || results > INT32_MAX || largest > max_unit || nsub > INT32_MAX ||
        out_bytes + nsub * static_cast<int64_t>(sizeof(SymUnit)) > max_bytes)
        return hipSuccess;   // not planned: the host takes the pairs in rounds, or leaves some
    out.planned = true;
    if (out.units == 0)
        return hipSuccess;
    off2[nb] = static_cast<int32_t>(kept);
    pc_off[nb] = static_cast<int32_t>(results);

    auto get = [&](auto** p, int64_t count) -> hipError_t {
        return alloc(reinterpret_cast<void**>(p), static_cast<size_t>(count) * sizeof(**p));
    };
    SYM_TRY(get(&out.near_off, nb + 1));
    SYM_TRY(get(&out.near_begin, kept));
    SYM_TRY(get(&out.near_count, kept));
    SYM_TRY(get(&out.near_leaf, kept));
    SYM_TRY(get(&out.pc_off, nb + 1));
    SYM_TRY(get(&out.pc_base, results));
    SYM_TRY(get(&out.batch_begin, nb));
    SYM_TRY(get(&out.unit, nsub));
    SYM_TRY(get(&out.out, values));
    out.sub_units = nsub;
    out.workspace_bytes = std::max<int64_t>(1, out_bytes) + nsub * static_cast<int64_t>(sizeof(SymUnit));
    SYM_TRY(hipMemcpyAsync(out.near_off, off2.data(), off2.size() * sizeof(int32_t),
                           hipMemcpyHostToDevice, s));
    SYM_TRY(hipMemcpyAsync(out.pc_off, pc_off.data(), pc_off.size() * sizeof(int32_t),
                           hipMemcpyHostToDevice, s));
    SYM_TRY(hipMemcpyAsync(out.batch_begin, dl.batch_begin->data(), nb * sizeof(int64_t),
                           hipMemcpyHostToDevice, s));
    SymOffsets* offs_d;
    int64_t* rows;
    int32_t* next_d;
    Pack offsets;
    SYM_TRY(mem.put(&offs_d, offs, offsets, s));
    SYM_TRY(mem.put(&next_d, first, offsets, s));
    SYM_TRY(mem.send(offsets, s));
    SYM_TRY(mem.get(&rows, ne));
    fill_pairs<<<grid, 64 * kSymWaves, 0, s>>>(n, batches_d, offs_d, lists.near_leaf, batch_of_d, match,
                                               sub, scale, next_d, out.near_leaf, out.near_begin,
                                               out.near_count, lists.near_begin, lists.near_count,
                                               out.unit, rows);
    SYM_TRY(hipGetLastError());
    pair_results<<<grid, 64 * kSymWaves, 0, s>>>(n, batches_d, offs_d, lists.near_leaf, batch_of_d,
                                                 match, sub, rows, out.pc_base);
    SYM_TRY(hipGetLastError());
    // the tables and the scratch are freed on return: finish first
    return hipStreamSynchronize(s);
}

}  // namespace bltc
