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
// Per pass: digit counts per workgroup (k_sort_count), their prefix sums (k_sort_scan), and the move (k_sort_events, k_sort_entries), no workgroup
// waiting for another.  31.7 M entries of 0.5 M nodes (Zipf 1.5), with the times' and ids' check: 1.62 -> 0.86 ms (moves 309 and 293 us, counts
// 41 and 45, positions 127, list bounds 22); a sub-graph's whole rebuilding 3.19 -> 2.41 ms.  More nodes than 2^22 would need a third pass and a second copy of the entries; they take the sort above.
constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64;
constexpr int kSortRounds = 16;                       // entries per lane and tile
constexpr int kSortTile = kSortThreads * kSortRounds;
// At most so many workgroups.  Registers leave two of either move to a compute unit (LDS two or three), so that 1024 are two
// rounds; the counts' fit four.  512, one round: 16 M Zipf events of 1 M and of 2.6 M nodes take 1.6% longer for the whole build, 4 M
// flat ones of 0.3 M nodes 2.4% less; 2048: the Zipf graphs 1.5% and 2% less, flat ones up to 1.4% less.
constexpr int kSortBlocks = 1024;
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
    uint32_t *bounds;     // [bins + 2] last pass: first entry of every digit, NULL otherwise
    uint32_t *sample;     // LAST after another pass: node of every entry whose place is a multiple of 2^sample_shift
    int sample_shift;
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
            if (q0 + u * kSortThreads < hi) {
                // the first lane's digit is counted at once: most lanes share it where a few nodes have most of the entries, and
                // additions to one address take turns (31.7 M entries of which 97% have one digit: 116 us a lane at a time)
                const uint32_t d = (node[u] >> p.shift) & (kBins - 1), lead = __builtin_amdgcn_readfirstlane(d);
                const unsigned long long same = __ballot(d == lead);
                if (d != lead)
                    atomicAdd(&count[d], 1u);
                else if (__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) == 0)
                    atomicAdd(&count[d], (uint32_t)__popcll(same));
            }
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

// Lanes with the same digit: entries of it in the lanes before, and in all of them (`on`: the lanes that count).
template <int BITS>
__device__ inline void match_digit(uint32_t d, bool on, uint32_t &before, uint32_t &all)
{
    unsigned long long same = __ballot(on);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (d >> b) & 1u;
        const unsigned long long set = __ballot(bit);
        same &= bit ? set : ~set;
    }
    before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    all = (uint32_t)__popcll(same);
}

// Orders a wavefront's own LDS accesses: what a lane has stored is what the other lanes load next.  (The counters of
// match_digit's rounds go from the digit's last lane to whichever lanes have it a round later; LDS operations of a
// wavefront are carried out in order anyway, so that this only binds the compiler: the same instructions, no wait added.)
__device__ inline void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Sum over the threads before this one; `sums`: [wavefronts] of LDS that nobody else uses, whose readers may still be
// reading on return.
__device__ inline uint32_t sum_before(uint32_t x, uint32_t *sums, int wave, int lane)
{
    uint32_t incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off, 64);
        incl += lane >= off ? up : 0u;
    }
    if (lane == 63)
        sums[wave] = incl;
    __syncthreads();
    uint32_t run = incl - x;
    for (int w = 0; w < wave; ++w)
        run += sums[w];
    return run;
}

template <int BITS>
struct SortBins {
    static constexpr int kBins = 1 << BITS;
    static constexpr int kPer = (kBins + kSortThreads - 1) / kSortThreads;  // bins of a thread
    static_assert(kBins % kSortThreads == 0 || kBins < kSortThreads, "");
    // where the workgroup's first entry of each of the thread's digits goes: behind all entries of smaller digits, and those of
    // the digit in the workgroups before
    static __device__ inline void first_places(const SortPass &p, uint32_t *sums, int wave, int lane, uint32_t (&place)[kPer])
    {
        const int d0 = (int)threadIdx.x * kPer;
        uint32_t tot[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            tot[i] = d0 + i < kBins ? p.totals[d0 + i] : 0u;
            sum += tot[i];
        }
        uint32_t run = sum_before(sum, sums, wave, lane);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            place[i] = 0;
            if (d0 + i < kBins) {
                place[i] = run + p.counts[(size_t)blockIdx.x * kBins + d0 + i];
                if (p.bounds && blockIdx.x == 0)
                    p.bounds[d0 + i] = run;
                run += tot[i];
            }
        }
        if (p.bounds && blockIdx.x == 0 && threadIdx.x < 2)
            p.bounds[kBins + threadIdx.x] = (uint32_t)p.n;
    }
};

// The move of a workgroup's entries, a tile at a time, in order.  Every wavefront takes a run of the tile, 64 entries a
// round: lanes with the same digit find each other by a ballot per bit, the wavefront counts its digits in LDS, and
// the counts of the wavefronts before it complete an entry's rank.
//
// The first pass, from the event stream: a tile's events stay in LDS, and its entries leave in the order of their
// digits, so that neighbouring lanes write neighbouring places (written from where they were read, 16 and 4 bytes a lane to as many
// places, 31.7 M entries of 0.5 M nodes took 486 us instead of 309).  Also checks the graph: flags[0] an id out of
// range, [1] times that decrease, [2] a self-loop (whatever the ids, a digit is one of the bins).
template <int BITS, bool LAST>
__global__ void __launch_bounds__(kSortThreads, 4) k_sort_events(SortPass p)
{
    using Bins = SortBins<BITS>;
    constexpr int kBins = Bins::kBins, kPer = Bins::kPer, kRounds = 8, kTile = kSortThreads * kRounds;
    static_assert(kSortTile % kTile == 0, "");
    __shared__ EntryWords event[kTile / 2];                              // src, dst, time
    __shared__ __attribute__((aligned(16))) uint16_t mine[kSortWaves][kBins];  // digits of a wavefront's run, then first ranks
    __shared__ uint16_t at_rank[kTile];
    __shared__ uint32_t shift_of[kBins];  // destination less rank, per digit  (two workgroups of 11 bits fill the unit's LDS)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d0 = (int)threadIdx.x * kPer;
    uint32_t place[kPer];
    Bins::first_places(p, shift_of, wave, lane, place);
    const int64_t lo = (int64_t)blockIdx.x * p.chunk, hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
    int bad = 0;  // bit f: flags[f]
    for (int64_t t0 = lo; t0 < hi; t0 += kTile) {  // (t0 and hi are even)
        const int left = hi - t0 < kTile ? (int)(hi - t0) : kTile;
        const int64_t e0 = t0 >> 1;
        constexpr int kEvents = kTile / 2 / kSortThreads;
        __syncthreads();  // (the tile before is done with)
        for (int i = threadIdx.x; i < kSortWaves * kBins / 2; i += kSortThreads)
            ((uint32_t *)mine)[i] = 0;
        int32_t s[kEvents], d[kEvents];
        double t[kEvents], earlier[kEvents];
#pragma unroll
        for (int u = 0; u < kEvents; ++u) {
            const int x = (int)threadIdx.x + u * kSortThreads, ev = 2 * x < left ? x : left / 2 - 1;
            s[u] = (p.src + e0)[(unsigned)ev];
            d[u] = (p.dst + e0)[(unsigned)ev];
            t[u] = (p.ts + e0)[(unsigned)ev];
            earlier[u] = p.ts[e0 + ev > 0 ? e0 + ev - 1 : 0];
        }
#pragma unroll
        for (int u = 0; u < kEvents; ++u) {
            const int x = (int)threadIdx.x + u * kSortThreads;
            bad |= (s[u] < 0 || s[u] >= p.num_nodes || d[u] < 0 || d[u] >= p.num_nodes ? 1 : 0) | (s[u] == d[u] ? 4 : 0);
            bad |= e0 + x > 0 && 2 * x < left && !(earlier[u] <= t[u]) ? 2 : 0;
            event[x] = EntryWords{s[u], d[u], __double2loint(t[u]), __double2hiint(t[u])};
        }
        __syncthreads();
        uint32_t node[kRounds], rank[kRounds];
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int at = wave * (64 * kRounds) + 64 * u + lane;
            node[u] = ((const uint32_t *)event)[4 * (at >> 1) + (at & 1)];
        }
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const bool on = wave * (64 * kRounds) + 64 * u + lane < left;
            const uint32_t dig = (node[u] >> p.shift) & (kBins - 1);
            uint32_t before, all;
            match_digit<BITS>(dig, on, before, all);
            const uint32_t had = mine[wave][dig];
            rank[u] = had + before;
            if (on && before + 1 == all)
                mine[wave][dig] = (uint16_t)(had + all);
            wave_lds_order();
        }
        __syncthreads();
        {   // ranks of the tile: digit by digit, within a digit wavefront by wavefront
            uint32_t tot[kPer], sum = 0;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                tot[i] = 0;
                if (d0 + i < kBins)
#pragma unroll
                    for (int w = 0; w < kSortWaves; ++w)
                        tot[i] += mine[w][d0 + i];
                sum += tot[i];
            }
            uint32_t run = sum_before(sum, shift_of, wave, lane);
            __syncthreads();  // (the sums have been read)
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (d0 + i < kBins) {
                    shift_of[d0 + i] = place[i] - run;
                    place[i] += tot[i];
#pragma unroll
                    for (int w = 0; w < kSortWaves; ++w) {
                        const uint32_t x = mine[w][d0 + i];
                        mine[w][d0 + i] = (uint16_t)run;
                        run += x;
                    }
                }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int at = wave * (64 * kRounds) + 64 * u + lane;
            const uint32_t dig = (node[u] >> p.shift) & (kBins - 1), r = mine[wave][dig] + rank[u];
            if (at < left) {
                at_rank[r] = (uint16_t)at;
                (p.place + t0)[(unsigned)at] = (int32_t)(shift_of[dig] + r);
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int r = (int)threadIdx.x + u * kSortThreads;
            if (r < left) {
                const int at = at_rank[r];
                const EntryWords x = event[at >> 1];
                const bool role = at & 1;
                const uint32_t me = (uint32_t)(role ? x[1] : x[0]);
                const uint32_t to = shift_of[(me >> p.shift) & (kBins - 1)] + (uint32_t)r;
                ((EntryWords *)p.out)[to] = EntryWords{role ? x[0] : x[1], (int32_t)((t0 + at) >> (LAST ? 1 : 0)), x[2], x[3]};
                if (!LAST)
                    p.node_out[to] = me;
            }
        }
    }
#pragma unroll
    for (int f = 0; f < 3; ++f)
        if (bad >> f & 1)
            p.flags[f] = 1;
}

// The second pass: entries that are in the order of their low digits already, so that those of one high digit leave in long runs
// by themselves where a few nodes have most of them.
template <int BITS>
__global__ void __launch_bounds__(kSortThreads, 4) k_sort_entries(SortPass p)
{
    using Bins = SortBins<BITS>;
    constexpr int kBins = Bins::kBins, kPer = Bins::kPer;
    __shared__ __attribute__((aligned(16))) uint16_t mine[kSortWaves][kBins];  // digits of a wavefront's run, then of those before it
    __shared__ uint32_t base[kBins];                                          // where the next entry of a digit goes
    __shared__ uint32_t sums[kSortWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d0 = (int)threadIdx.x * kPer;
    {
        uint32_t place[kPer];
        Bins::first_places(p, sums, wave, lane, place);
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (d0 + i < kBins)
                base[d0 + i] = place[i];
    }
    const int64_t lo = (int64_t)blockIdx.x * p.chunk, hi = lo + p.chunk < p.n ? lo + p.chunk : p.n;
    for (int64_t t0 = lo; t0 < hi; t0 += kSortTile) {
        const int left = hi - t0 < kSortTile ? (int)(hi - t0) : kSortTile;
        int at0 = wave * (64 * kSortRounds) + lane;  // of the tile; beyond its end the last entry stands in
        asm volatile("" : "+v"(at0));                // (sixteen rounds' places, kept over the tiles, spill)
        const uint32_t *const node_in = p.node_in + t0;
        for (int i = threadIdx.x; i < kSortWaves * kBins / 2; i += kSortThreads)
            ((uint32_t *)mine)[i] = 0;
        uint32_t node[kSortRounds];
        uint16_t rank[kSortRounds];
#pragma unroll
        for (int u = 0; u < kSortRounds; ++u)
            node[u] = node_in[(unsigned)(at0 + 64 * u < left ? at0 + 64 * u : left - 1)];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSortRounds; ++u) {
            const bool on = at0 + 64 * u < left;
            const uint32_t d = (node[u] >> p.shift) & (kBins - 1);
            uint32_t before, all;
            match_digit<BITS>(d, on, before, all);
            const uint32_t had = mine[wave][d];
            rank[u] = (uint16_t)(had + before);
            if (on && before + 1 == all)
                mine[wave][d] = (uint16_t)(had + all);
            wave_lds_order();
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
            asm volatile("" : "+v"(at0) : : "memory");  // (a turn at a time: all turns' loads together spill)
#pragma unroll
            for (int v = 0; v < kTurn; ++v) {
                const int at = at0 + 64 * (u0 + v);
                e[v] = ((const EntryWords *)(p.in + t0))[(unsigned)(at < left ? at : left - 1)];
                e[v][1] = (int32_t)((uint32_t)e[v][1] >> 1);  // (the role has done its service)
            }
#pragma unroll
            for (int v = 0; v < kTurn; ++v) {
                const int u = u0 + v, at = at0 + 64 * u;
                const uint32_t d = (node[u] >> p.shift) & (kBins - 1);
                const uint32_t to = base[d] + mine[wave][d] + rank[u];
                if (at < left) {
                    ((EntryWords *)p.out)[to] = e[v];
                    (p.place + t0)[(unsigned)at] = (int32_t)to;
                    if ((to & ((1u << p.sample_shift) - 1u)) == 0u)
                        p.sample[to >> p.sample_shift] = node[u];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (d0 + i < kBins)
                base[d0 + i] += tile[i];
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

// indptr[n] = entries of nodes below n, n = 0..N.  bounds: first entry of every value of the last pass's digit.  After one pass the
// digit is the node.  After two the nodes are not kept beside the entries: a list's bound is searched among those that the
// second pass left of every 2^sample_shift-th entry, and between two of them by the entries, whose node is their event's other
// endpoint.  Bound by these last steps' memory lines, which nobody else wants.  Flat endpoints of 16 M events over 2.6 M nodes: 234 us
// with the node of every fourth entry, which costs the second pass 70 (of every eighth 320 and 40; with all steps among the
// entries 624 us, which made the whole build slower than the library's sort, 2310 -> 2514 us; now 2180).  Zipf 1.5 over
// 1 M nodes: 38 -> 22 us.
__global__ void k_bounds_to_indptr(const uint32_t *__restrict__ bounds, int64_t num_nodes, int64_t *__restrict__ indptr)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n <= num_nodes)
        indptr[n] = bounds[n];
}

__global__ void k_indptr_of_entries(const CsrEntry *__restrict__ csr, const int32_t *__restrict__ src, const int32_t *__restrict__ dst,
                                    const uint32_t *__restrict__ bounds, const uint32_t *__restrict__ sample, int sample_shift, int shift,
                                    int64_t num_nodes, int64_t *__restrict__ indptr)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n <= num_nodes; n += stride) {
        int64_t lo = bounds[n >> shift], hi = bounds[(n >> shift) + 1];
        // the samples of the list: places first, first + 1, ... in units of 2^sample_shift, below hi
        const int64_t round = ((int64_t)1 << sample_shift) - 1, first = (lo + round) >> sample_shift;
        int64_t a = first, b = (hi + round) >> sample_shift;
        while (a < b) {
            const int64_t mid = a + ((b - a) >> 1);
            if ((int64_t)sample[mid] < n)
                a = mid + 1;
            else
                b = mid;
        }
        // sample a, if it lies in the list, is the first whose node is not below n; the one before it is below
        hi = (a << sample_shift) < hi ? a << sample_shift : hi;
        lo = a > first ? ((a - 1) << sample_shift) + 1 : lo;
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            const CsrEntry x = csr[mid];
            int32_t node = src[x.eid];
            if (node == x.nbr)
                node = dst[x.eid];
            if ((int64_t)node < n)
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
        first.bounds = second.bounds;
        hipLaunchKernelGGL((k_sort_events<BITS, true>), grid, threads, 0, s, first);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_sort_events<BITS, false>), grid, threads, 0, s, first);
    hipLaunchKernelGGL((k_sort_count<BITS, false>), grid, threads, 0, s, second);
    scan();
    hipLaunchKernelGGL(k_sort_entries<BITS>, grid, threads, 0, s, second);
    const int64_t turns = (first.n + 4 * kThreads - 1) / (4 * kThreads);
    hipLaunchKernelGGL(k_sort_pos, dim3((unsigned)turns), dim3(kThreads), 0, s, first.place, second.place, first.n);
    return hipGetLastError();
}

// scratch: [entries | nodes, then destinations | counts per workgroup and digit | totals | bounds | samples], within
// csr_build_scratch_bytes
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
    const size_t totals = align_up(sizeof(uint32_t) << digit), bounds = totals + 256;
    const size_t before = entries + nodes + counts + totals + bounds;
    // The samples take what is left of the scratch memory: every fourth entry up to some 55 million of them, and
    // every 256th of the 2^31 that there can be.  (Every second one: 1268 -> 1218 us for 8 M flat events over 4 M nodes, but
    // 533 -> 551 for 4 M over 0.3 M; every eighth 1328 and 534.)
    int sample_shift = 2;
    while (bits > digit && sample_shift < 30 && before + 4 * (((size_t)n2 >> sample_shift) + 1) > scratch_bytes)
        ++sample_shift;
    if (before + (bits > digit ? 4 * (((size_t)n2 >> sample_shift) + 1) : 0) > scratch_bytes)
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
    b.bounds = (uint32_t *)(scratch + entries + nodes + counts + totals);
    b.shift = digit;
    b.sample = (uint32_t *)(scratch + before);
    b.sample_shift = sample_shift;
    hipError_t e;
    switch (digit) {
    case 8: e = sort_passes<8>(a, b, blocks, bits, s); break;
    case 9: e = sort_passes<9>(a, b, blocks, bits, s); break;
    case 10: e = sort_passes<10>(a, b, blocks, bits, s); break;
    default: e = sort_passes<11>(a, b, blocks, bits, s); break;
    }
    if (e != hipSuccess)
        return e;
    if (bits <= digit)
        hipLaunchKernelGGL(k_bounds_to_indptr, dim3((unsigned)(num_nodes / kThreads + 1)), dim3(kThreads), 0, s, b.bounds, num_nodes, indptr);
    else
        hipLaunchKernelGGL(k_indptr_of_entries, dim3(grid_for(num_nodes + 1)), dim3(kThreads), 0, s, csr, src, dst, b.bounds, b.sample,
                           sample_shift, digit, num_nodes, indptr);
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
