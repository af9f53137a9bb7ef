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

// ---- the adjacency by a sort of its own ----------------------------------------------------------------------------
//
// Up to 2^22 nodes the entries are sorted by node in one or two stable counting passes of kDigitBits at most, and what a
// pass moves is the adjacency entry itself: events are read once in stream order, the last pass writes the adjacency.
// (Sorting entry numbers by a library's sort and fetching every entry's event afterwards, as above, reads a memory line
// per entry beyond the few heaviest nodes, and writes another for its `pos`.)  An entry's place is followed
// instead of scattered: a pass leaves every entry's destination at its source position, where two
// passes are composed by a read whose neighbours go to neighbouring places (k_sort_pos).
// Per pass: digit counts per workgroup (k_sort_count), their prefix sums (k_sort_scan), and the move (k_sort_move), no workgroup
// waiting for another.  25 M entries of 0.5 M nodes (Zipf 1.5), with the times' and ids' check: 1.62 -> 1.11 ms (moves 486 and 282 us, counts
// 44 and 116, positions 125, bounds 40); a sub-graph's whole rebuilding 3.19 -> 2.65 ms.  More nodes than 2^22 would need a third pass and a second copy of the entries; they take the sort above.
constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64;
constexpr int kSortRounds = 16;                       // entries per lane and tile
constexpr int kSortTile = kSortThreads * kSortRounds;
constexpr int kSortBlocks = 1024;                     // four workgroups per compute unit, all resident
constexpr int kDigitBits = 11;

struct SortPass {
    // source: the event stream (FIRST), or entries in the order of the pass before, role kept beside the event id
    const int32_t *src, *dst;
    const double *ts;
    const CsrEntry *in;
    const uint32_t *node_in;
    CsrEntry *out;        // FIRST and LAST: the adjacency
    uint32_t *node_out;   // (not LAST)
    int32_t *place;       // destination of the entry at source position q (LAST after another pass: over node_in)
    uint32_t *counts;     // [workgroups][bins], then their prefix sums within a bin
    uint32_t *totals;     // [bins]
    int32_t *flags;
    int64_t n, num_nodes;
    int64_t chunk;        // entries per workgroup, whole tiles
    int shift;
};

typedef int32_t EntryWords __attribute__((ext_vector_type(4)));
static_assert(sizeof(EntryWords) == sizeof(CsrEntry), "an entry is one 16-byte store");

template <int BITS, bool FIRST>
__global__ void __launch_bounds__(kSortThreads) k_sort_count(SortPass p)
{
    constexpr int kBins = 1 << BITS, kTurn = 8;
    __shared__ uint32_t count[kBins];
    for (int d = threadIdx.x; d < kBins; d += kSortThreads)
        count[d] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * p.chunk, hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
    for (int64_t q0 = lo + threadIdx.x; q0 < hi; q0 += kTurn * kSortThreads) {
        uint32_t node[kTurn];
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const int64_t q = q0 + u * kSortThreads;
            const int64_t qc = q < hi ? q : hi - 1;
            node[u] = FIRST ? (uint32_t)((qc & 1) ? p.dst : p.src)[qc >> 1] : p.node_in[qc];
        }
#pragma unroll
        for (int u = 0; u < kTurn; ++u)
            if (q0 + u * kSortThreads < hi)
                atomicAdd(&count[(node[u] >> p.shift) & (kBins - 1)], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kBins; d += kSortThreads)
        p.counts[(size_t)blockIdx.x * kBins + d] = count[d];
}

// counts[b][d] -> sum over the workgroups before b, totals[d]: 32 bins per workgroup, 32 threads share a bin
__global__ void __launch_bounds__(1024) k_sort_scan(uint32_t *counts, uint32_t *totals, int blocks, int bins)
{
    __shared__ uint32_t part[32][33];
    const int c = threadIdx.x & 31, g = threadIdx.x >> 5, d = (int)blockIdx.x * 32 + c;
    const int per = (blocks + 31) / 32, lo = g * per, hi = lo + per < blocks ? lo + per : blocks;
    uint32_t sum = 0;
#pragma unroll 8
    for (int b = lo; b < hi; ++b)
        sum += counts[(size_t)b * bins + d];
    part[g][c] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int i = 0; i < g; ++i)
        run += part[i][c];
    if (g == 31)
        totals[d] = run + sum;
#pragma unroll 8
    for (int b = lo; b < hi; ++b) {
        const uint32_t x = counts[(size_t)b * bins + d];
        counts[(size_t)b * bins + d] = run;
        run += x;
    }
}

// The move of a workgroup's entries, a tile at a time, in order.  Every wavefront takes a run of the tile, 64 entries a
// round: lanes with the same digit find each other by a ballot per bit, the wavefront counts its digits in LDS, and
// the counts of the wavefronts before it complete an entry's rank.  FIRST also checks the graph: flags[0] an id out of
// range, [1] times that decrease, [2] a self-loop (whatever the ids, a digit is one of the bins).
template <int BITS, bool FIRST, bool LAST>
__global__ void __launch_bounds__(kSortThreads, 4) k_sort_move(SortPass p)
{
    constexpr int kBins = 1 << BITS;
    constexpr int kPer = (kBins + kSortThreads - 1) / kSortThreads;  // bins of a thread
    static_assert(kBins % kSortThreads == 0 || kBins < kSortThreads, "");
    __shared__ __attribute__((aligned(16))) uint16_t mine[kSortWaves][kBins];  // digits of a wavefront's run, then those of the wavefronts before it
    __shared__ uint32_t base[kBins];              // where the next entry of a digit goes
    __shared__ uint32_t wave_sum[kSortWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d0 = (int)threadIdx.x * kPer;
    {   // first place of every digit: the totals of the digits before it, and of this digit in the workgroups before
        uint32_t tot[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            tot[i] = d0 + i < kBins ? p.totals[d0 + i] : 0u;
            sum += tot[i];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off, 64);
            incl += lane >= off ? up : 0u;
        }
        if (lane == 63)
            wave_sum[wave] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (int w = 0; w < wave; ++w)
            run += wave_sum[w];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (d0 + i < kBins) {
                base[d0 + i] = run + p.counts[(size_t)blockIdx.x * kBins + d0 + i];
                run += tot[i];
            }
    }
    const int64_t lo = (int64_t)blockIdx.x * p.chunk, hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
    int bad = 0;  // bit f: flags[f]
    for (int64_t t0 = lo; t0 < hi; t0 += kSortTile) {  // (t0 is even)
        const int left = hi - t0 < kSortTile ? (int)(hi - t0) : kSortTile;
        int at0 = wave * (64 * kSortRounds) + lane;  // of the tile; beyond its end the last of the same role stands in
        asm volatile("" : "+v"(at0));                // (sixteen rounds' places, kept over the tiles, spill)
        const int stand_in = left - 2 + (lane & 1);
        const int32_t *const src = p.src + (t0 >> 1), *const dst = p.dst + (t0 >> 1);
        const int32_t *const own = (lane & 1) ? dst : src, *const opposite = (lane & 1) ? src : dst;
        const double *const ts = p.ts + (t0 >> 1);
        const uint32_t *const node_in = p.node_in + t0;
        for (int i = threadIdx.x; i < kSortWaves * kBins / 2; i += kSortThreads)
            ((uint32_t *)mine)[i] = 0;
        uint32_t node[kSortRounds];
        uint16_t rank[kSortRounds];
#pragma unroll
        for (int u = 0; u < kSortRounds; ++u) {
            const int at = at0 + 64 * u < left ? at0 + 64 * u : stand_in;
            node[u] = FIRST ? (uint32_t)own[(unsigned)at >> 1] : node_in[(unsigned)at];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSortRounds; ++u) {
            const bool on = at0 + 64 * u < left;
            const uint32_t d = (node[u] >> p.shift) & (kBins - 1);
            unsigned long long same = __ballot(on);
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                const bool bit = (d >> b) & 1u;
                const unsigned long long set = __ballot(bit);
                same &= bit ? set : ~set;
            }
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            const uint32_t all = (uint32_t)__popcll(same);
            const uint32_t had = mine[wave][d];
            rank[u] = (uint16_t)(had + before);
            if (on && before + 1 == all)
                mine[wave][d] = (uint16_t)(had + all);
        }
        __syncthreads();
        uint32_t tile[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            tile[i] = 0;
            if (d0 + i < kBins)
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) {
                    const uint32_t x = mine[w][d0 + i];
                    mine[w][d0 + i] = (uint16_t)tile[i];
                    tile[i] += x;
                }
        }
        __syncthreads();
        constexpr int kTurn = 4;  // rounds whose loads are in flight together
#pragma unroll
        for (int u0 = 0; u0 < kSortRounds; u0 += kTurn) {
            EntryWords e[kTurn];
            asm volatile("" : "+v"(at0), "+v"(bad) : : "memory");  // (a turn at a time: all turns' loads together spill)
#pragma unroll
            for (int v = 0; v < kTurn; ++v) {
                const int at = at0 + 64 * (u0 + v) < left ? at0 + 64 * (u0 + v) : stand_in;
                if (FIRST) {
                    const unsigned ev = (unsigned)at >> 1;
                    const bool some = t0 + at > 1;  // not the stream's first event
                    const int32_t me = (int32_t)node[u0 + v], other = opposite[ev];
                    const double t = ts[ev], earlier = (ts - (some ? 1 : 0))[ev];
                    bad |= (me < 0 || (int64_t)me >= p.num_nodes ? 1 : 0) | (some && !(earlier <= t) ? 2 : 0) | (me == other ? 4 : 0);
                    e[v] = EntryWords{other, (int32_t)((t0 + at) >> (LAST ? 1 : 0)), __double2loint(t), __double2hiint(t)};
                } else {
                    e[v] = ((const EntryWords *)(p.in + t0))[(unsigned)at];
                    e[v][1] = (int32_t)((uint32_t)e[v][1] >> 1);  // (the role has done its service)
                }
            }
#pragma unroll
            for (int v = 0; v < kTurn; ++v) {
                const int u = u0 + v, at = at0 + 64 * u;
                const uint32_t d = (node[u] >> p.shift) & (kBins - 1);
                const uint32_t to = base[d] + mine[wave][d] + rank[u];
                if (at < left) {
                    ((EntryWords *)p.out)[to] = e[v];
                    if (!LAST)
                        p.node_out[to] = node[u];
                    (p.place + t0)[(unsigned)at] = (int32_t)to;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (d0 + i < kBins)
                base[d0 + i] += tile[i];
    }
    if (FIRST) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (bad >> f & 1)
                p.flags[f] = 1;
    }
}

// pos[2 * eid + role]: the second pass's destination of where the first one put the entry
__global__ void __launch_bounds__(kThreads) k_sort_pos(int32_t *__restrict__ pos, const int32_t *__restrict__ place, int64_t n)
{
    constexpr int kTurn = 4;
    const int64_t i0 = ((int64_t)blockIdx.x * kThreads) * kTurn + threadIdx.x;
    int32_t at[kTurn];
#pragma unroll
    for (int u = 0; u < kTurn; ++u) {
        const int64_t i = i0 + u * kThreads;
        at[u] = pos[i < n ? i : n - 1];  // (beyond the end: any value, not used)
    }
#pragma unroll
    for (int u = 0; u < kTurn; ++u)
        at[u] = place[i0 + u * kThreads < n ? at[u] : 0];
#pragma unroll
    for (int u = 0; u < kTurn; ++u)
        if (i0 + u * kThreads < n)
            pos[i0 + u * kThreads] = at[u];
}

// indptr[n] = entries of nodes below n, n = 0..N, where the nodes are not kept beside the entries: an entry's node is its
// event's other endpoint
__global__ void k_indptr_of_entries(const CsrEntry *__restrict__ csr, const int32_t *__restrict__ src, const int32_t *__restrict__ dst,
                                    int64_t num_entries, int64_t num_nodes, int64_t *__restrict__ indptr)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n <= num_nodes; n += stride) {
        int64_t lo = 0, hi = num_entries;
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            const CsrEntry x = csr[mid];
            const int32_t s = src[x.eid], d = dst[x.eid];
            if ((int64_t)(s == x.nbr ? d : s) < n)
                lo = mid + 1;
            else
                hi = mid;
        }
        indptr[n] = lo;
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

template <int BITS>
hipError_t sort_passes(SortPass first, SortPass second, int blocks, int bits, hipStream_t s)
{
    const dim3 grid((unsigned)blocks), threads(kSortThreads);
    const auto scan = [&] {
        hipLaunchKernelGGL(k_sort_scan, dim3((1 << BITS) / 32), dim3(1024), 0, s, first.counts, first.totals, blocks, 1 << BITS);
    };
    hipLaunchKernelGGL((k_sort_count<BITS, true>), grid, threads, 0, s, first);
    scan();
    if (bits <= BITS) {
        first.out = second.out;
        hipLaunchKernelGGL((k_sort_move<BITS, true, true>), grid, threads, 0, s, first);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_sort_move<BITS, true, false>), grid, threads, 0, s, first);
    second.shift = BITS;
    hipLaunchKernelGGL((k_sort_count<BITS, false>), grid, threads, 0, s, second);
    scan();
    hipLaunchKernelGGL((k_sort_move<BITS, false, true>), grid, threads, 0, s, second);
    const int64_t turns = (first.n + 4 * kThreads - 1) / (4 * kThreads);
    hipLaunchKernelGGL(k_sort_pos, dim3((unsigned)turns), dim3(kThreads), 0, s, first.place, second.place, first.n);
    return hipGetLastError();
}

// scratch: [entries | nodes, then destinations | counts per workgroup and digit | totals], within csr_build_scratch_bytes
hipError_t sort_adjacency(const int32_t *src, const int32_t *dst, const double *ts, int64_t num_events, int64_t num_nodes,
                          int64_t *indptr, CsrEntry *csr, int32_t *pos, int32_t *flags, char *scratch, size_t scratch_bytes,
                          int bits, hipStream_t s)
{
    const int64_t n2 = 2 * num_events, tiles = (n2 + kSortTile - 1) / kSortTile;
    const int64_t per = (tiles + kSortBlocks - 1) / kSortBlocks;
    const int blocks = (int)((tiles + per - 1) / per);
    // two passes: the bits in halves; at least eight, so that few kernels are compiled
    const int half = bits <= kDigitBits ? bits : (bits + 1) / 2, digit = half < 8 ? 8 : half;
    const size_t entries = align_up(sizeof(CsrEntry) * (size_t)n2), nodes = align_up(sizeof(uint32_t) * (size_t)n2);
    const size_t counts = align_up(sizeof(uint32_t) * (size_t)blocks << digit);
    if (entries + nodes + counts + (sizeof(uint32_t) << digit) > scratch_bytes)
        return hipErrorOutOfMemory;
    SortPass a = {};
    a.src = src, a.dst = dst, a.ts = ts;
    a.out = (CsrEntry *)scratch;
    a.node_out = (uint32_t *)(scratch + entries);
    a.place = pos;
    a.counts = (uint32_t *)(scratch + entries + nodes);
    a.totals = (uint32_t *)(scratch + entries + nodes + counts);
    a.flags = flags;
    a.n = n2, a.num_nodes = num_nodes;
    a.chunk = per * kSortTile;
    SortPass b = a;
    b.in = a.out, b.node_in = a.node_out;
    b.out = csr, b.node_out = nullptr;
    b.place = (int32_t *)a.node_out;
    hipError_t e;
    switch (digit) {
    case 8: e = sort_passes<8>(a, b, blocks, bits, s); break;
    case 9: e = sort_passes<9>(a, b, blocks, bits, s); break;
    case 10: e = sort_passes<10>(a, b, blocks, bits, s); break;
    default: e = sort_passes<11>(a, b, blocks, bits, s); break;
    }
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_indptr_of_entries, dim3(grid_for(num_nodes + 1)), dim3(kThreads), 0, s, csr, src, dst, n2, num_nodes, indptr);
    return hipGetLastError();
}

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
    if (bits <= 2 * kDigitBits)
        return sort_adjacency(src, dst, ts, num_events, num_nodes, indptr, csr, pos, flags, (char *)scratch, scratch_bytes, bits, s);
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
