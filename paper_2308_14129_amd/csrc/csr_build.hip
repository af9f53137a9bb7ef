// Graph validation and construction of the temporal adjacency (once, in tig_init).
//
// The history of a node before time t (the set E_t of the paper's Notations section restricted
// to the node) must be searchable by time.  Events arrive in chronological order, so listing
// every event under both of its endpoints in event-id order yields per-node lists that are
// already ordered by (time, event id).  A stable radix sort of the 2E (endpoint, entry) pairs
// by endpoint id produces exactly that grouping.
#include <cstring>

#include <hip/hip_runtime.h>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include "tig_internal.h"

namespace tig {

namespace {

constexpr int kThreads = 256;

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Endpoint of entry i = 2 * eid + role: what the sort reads as its keys (no array of pairs is written first).
struct EntryNode {
    const int32_t *src, *dst;
    __device__ uint32_t operator()(uint32_t i) const { return (uint32_t)((i & 1u) ? dst : src)[i >> 1]; }
};

// The event as one 16-byte record, so that an adjacency entry costs one random read.
struct __attribute__((aligned(16))) EventRecord {
    int32_t src, dst;
    double ts;
};

// Also checks the graph: flags[0] an id out of range, [1] times that decrease, [2] a self-loop.  (A pass of its own over
// the same three arrays took 60 us for 12.7 M events.)
__global__ void k_event_records(const int32_t *__restrict__ src, const int32_t *__restrict__ dst,
                                const double *__restrict__ ts, int64_t num_events, int64_t num_nodes,
                                EventRecord *__restrict__ rec, int32_t *flags)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < num_events; e += stride) {
        const int32_t s = src[e], d = dst[e];
        const double t = ts[e], before = ts[e > 0 ? e - 1 : 0];
        rec[e] = EventRecord{s, d, t};
        if (s < 0 || s >= num_nodes || d < 0 || d >= num_nodes)
            flags[0] = 1;
        if (e > 0 && !(before <= t))
            flags[1] = 1;
        if (s == d)
            flags[2] = 1;
    }
}

// 0.65 ms for 25 M entries.  Bound by the random accesses: beyond the few heaviest nodes, consecutive entries of a list are events far
// apart, so every entry is a memory line of its own for its event and another for its `pos`.  The sorted values and the
// entries pass by the caches (read and written once; they would push the records and `pos` out of them: 0.81 ms for 25 M).
__global__ void k_fill_csr(const EventRecord *__restrict__ rec, int64_t num_entries,
                           const uint32_t *__restrict__ vals_sorted, CsrEntry *__restrict__ csr,
                           int32_t *__restrict__ pos)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < num_entries; p += stride) {
        const uint32_t i = __builtin_nontemporal_load(vals_sorted + p);
        const EventRecord r = rec[i >> 1];
        pos[i] = (int32_t)p;  // where entry 2*eid + role sits in the adjacency array
        typedef int32_t Entry __attribute__((ext_vector_type(4)));
        static_assert(sizeof(Entry) == sizeof(CsrEntry), "an entry is one 16-byte store");
        const Entry ent = {(i & 1) ? r.src : r.dst, (int32_t)(i >> 1), __double2loint(r.ts), __double2hiint(r.ts)};
        __builtin_nontemporal_store(ent, (Entry *)(csr + p));
    }
}

// indptr[n] = number of sorted keys smaller than n, n = 0..N
__global__ void k_indptr(const uint32_t *__restrict__ keys_sorted, int64_t num_entries,
                         int64_t num_nodes, int64_t *__restrict__ indptr)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n <= num_nodes; n += stride) {
        int64_t lo = 0, hi = num_entries;
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if ((int64_t)keys_sorted[mid] < n)
                lo = mid + 1;
            else
                hi = mid;
        }
        indptr[n] = lo;
    }
}

int grid_for(int64_t n)
{
    int64_t g = (n + kThreads - 1) / kThreads;
    if (g < 1)
        g = 1;
    if (g > 65536)
        g = 65536;
    return (int)g;
}

int key_bits(int64_t num_nodes)
{
    int bits = 1;
    while (bits < 32 && ((int64_t)1 << bits) < num_nodes)
        ++bits;
    return bits;
}

// Upper bound on rocPRIM's temporary storage for the pair sort: the second pair of arrays its passes
// alternate with and its per-block digit counters.  Checked against the real requirement in csr_build.
size_t sort_temp_bound(int64_t num_entries) { return (size_t)num_entries * 12 + ((size_t)64 << 20); }

using EntryIndex = rocprim::counting_iterator<uint32_t>;
using EntryKeys = rocprim::transform_iterator<EntryIndex, EntryNode, uint32_t>;

}  // namespace

size_t csr_build_scratch_bytes(int64_t num_events, int64_t num_nodes)
{
    (void)num_nodes;
    const int64_t n2 = 2 * num_events;
    if (n2 == 0)
        return 256;
    return 2 * align_up(sizeof(uint32_t) * (size_t)n2) + align_up(sort_temp_bound(n2));
}

hipError_t csr_build(const int32_t *src, const int32_t *dst, const double *ts, int64_t num_events,
                     int64_t num_nodes, int64_t *indptr, CsrEntry *csr, int32_t *pos, int32_t *flags, void *scratch,
                     size_t scratch_bytes, hipStream_t s)
{
    const int64_t n2 = 2 * num_events;
    if (n2 == 0)
        return launch_fill_zero(indptr, sizeof(int64_t) * (size_t)(num_nodes + 1), s);
    if (scratch_bytes < csr_build_scratch_bytes(num_events, num_nodes))
        return hipErrorInvalidValue;
    const int bits = key_bits(num_nodes);
    const size_t seg = align_up(sizeof(uint32_t) * (size_t)n2);
    char *base = (char *)scratch;
    uint32_t *const keys = (uint32_t *)base, *const vals = (uint32_t *)(base + seg);
    void *temp = base + 2 * seg;
    const EntryIndex entries(0u);
    const EntryKeys nodes(entries, EntryNode{src, dst});
    size_t temp_bytes = 0;
    hipError_t err = rocprim::radix_sort_pairs(nullptr, temp_bytes, nodes, keys, entries, vals, (size_t)n2, 0u,
                                               (unsigned)bits, s);
    if (err != hipSuccess)
        return err;
    if (temp_bytes > sort_temp_bound(n2) || sizeof(EventRecord) * (size_t)num_events > sort_temp_bound(n2))
        return hipErrorOutOfMemory;
    // stable: entries of one node keep their input order, i.e. ascending event id
    err = rocprim::radix_sort_pairs(temp, temp_bytes, nodes, keys, entries, vals, (size_t)n2, 0u, (unsigned)bits, s);
    if (err != hipSuccess)
        return err;
    EventRecord *const rec = (EventRecord *)temp;  // (the sort is done with it)
    hipLaunchKernelGGL(k_event_records, dim3(grid_for(num_events)), dim3(kThreads), 0, s, src, dst, ts, num_events, num_nodes,
                       rec, flags);
    hipLaunchKernelGGL(k_fill_csr, dim3(grid_for(n2)), dim3(kThreads), 0, s, rec, n2, vals, csr, pos);
    err = hipGetLastError();
    if (err != hipSuccess)
        return err;
    hipLaunchKernelGGL(k_indptr, dim3(grid_for(num_nodes + 1)), dim3(kThreads), 0, s,
                       (const uint32_t *)keys, n2, num_nodes, indptr);
    return hipGetLastError();
}

}  // namespace tig
