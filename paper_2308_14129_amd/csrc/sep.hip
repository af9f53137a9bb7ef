// Streaming edge partitioner (paper Sec. II-B, Alg. 1): the preprocessing step that cuts a
// temporal interaction graph into the per-GPU sub-graphs the batch step runs on.  gfx950 only.
//   k_centrality   Eq. 1 on the device: Cent(i) = sum over i's events of exp(beta (t - t_max)).
//                  One pass over the event stream (16 bytes per event); every workgroup merges
//                  its chunk's contributions per node in LDS first (a hub node takes part in a
//                  large share of all events, and same-address device atomics serialise), then
//                  adds one fp64 value per distinct node and workgroup to the node array.
//   top-k hubs     the floor(k |V|) nodes of greatest centrality, ties towards the smaller id:
//                  a stable descending radix sort of (centrality bits, node id) pairs.
//   assign         the edge loop of Alg. 1 (cases 1-5, score C = C_REP + C_BAL, Eq. 2-6).  Every
//                  decision depends on all earlier ones, so this part is sequential by
//                  definition and runs on the host.
#include <hip/hip_runtime.h>
#include <rocprim/device/device_radix_sort.hpp>

#include <cmath>
#include <cstring>

#include "tig_internal.h"

namespace tig {

namespace {

constexpr int kCentThreads = 512;
constexpr int kCentPerThread = 128;                        // events per thread
constexpr int kCentChunk = kCentThreads * kCentPerThread;  // events per workgroup
constexpr int kCentSlots = 4096;                           // LDS table: node id + fp64 sum per slot
constexpr int kCentProbes = 8;

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

__device__ inline double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Adds w to node's sum in the workgroup's LDS table; a node that finds no slot within a few
// probes goes straight to the node array.
__device__ inline void table_add(int32_t *t_node, double *t_sum, double *cent, int32_t node, double w)
{
    uint32_t h = ((uint32_t)node * 2654435761u) >> 20;  // 12 bits
    for (int probe = 0; probe < kCentProbes; ++probe) {
        const int32_t prev = atomicCAS(&t_node[h], -1, node);
        if (prev == -1 || prev == node) {
            atomicAdd(&t_sum[h], w);
            return;
        }
        h = (h + 1) & (kCentSlots - 1);
    }
    unsafeAtomicAdd(&cent[node], w);
}

// The lanes of a wavefront that hold the node of the first active lane hand their sum to that
// lane and drop out (two rounds: the heaviest nodes of a power-law stream fill most lanes).
__device__ inline void merge_heavy(bool &active, int32_t node, double &w)
{
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const unsigned long long todo = __ballot(active);
        if (todo == 0ull)
            break;
        const int first = __ffsll((long long)todo) - 1;
        const int32_t n0 = __builtin_amdgcn_readlane(node, first);
        const bool mine = active && node == n0;
        const unsigned long long grp = __ballot(mine);
        if (__popcll(grp) > 1) {  // uniform
            const double s = wave_sum_f64(mine ? w : 0.0);
            if (mine) {
                if ((int)(threadIdx.x & 63) == first)
                    w = s;
                else
                    active = false;
            }
        }
    }
}

__global__ void __launch_bounds__(kCentThreads)
k_centrality(const int32_t *__restrict__ src, const int32_t *__restrict__ dst, const double *__restrict__ ts,
             int64_t num_events, int64_t num_nodes, double beta, double t_max, double *__restrict__ cent)
{
    __shared__ int32_t t_node[kCentSlots];
    __shared__ double t_sum[kCentSlots];
    for (int i = threadIdx.x; i < kCentSlots; i += kCentThreads) {
        t_node[i] = -1;
        t_sum[i] = 0.0;
    }
    __syncthreads();
    const int64_t e0 = (int64_t)blockIdx.x * kCentChunk;
    for (int it = 0; it < kCentPerThread; ++it) {
        const int64_t e = e0 + (int64_t)it * kCentThreads + threadIdx.x;  // coalesced
        const bool in = e < num_events;
        int32_t s = 0, d = 0;
        double w = 0.0;
        if (in) {
            s = src[e];
            d = dst[e];
            w = exp(beta * (ts[e] - t_max));
        }
        // ids were validated by the caller's graph checks or are checked here: out-of-range ids are skipped
        bool as = in && s >= 0 && (int64_t)s < num_nodes, ad = in && d >= 0 && (int64_t)d < num_nodes;
        double ws = w, wd = w;
        merge_heavy(as, s, ws);
        merge_heavy(ad, d, wd);
        if (as)
            table_add(t_node, t_sum, cent, s, ws);
        if (ad)
            table_add(t_node, t_sum, cent, d, wd);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCentSlots; i += kCentThreads)
        if (t_node[i] >= 0)
            unsafeAtomicAdd(&cent[t_node[i]], t_sum[i]);
}

__global__ void k_topk_keys(const double *__restrict__ cent, int64_t n, unsigned long long *keys, uint32_t *vals)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        // centralities are sums of positive terms: for non-negative doubles the bit pattern orders like the value
        const double c = cent[i];
        keys[i] = c > 0.0 ? (unsigned long long)__double_as_longlong(c) : 0ull;
        vals[i] = (uint32_t)i;
    }
}

__global__ void k_topk_flags(const uint32_t *__restrict__ vals_sorted, int64_t n_hubs, int32_t *hubs, uint8_t *is_hub)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_hubs; i += stride) {
        hubs[i] = (int32_t)vals_sorted[i];
        is_hub[vals_sorted[i]] = 1;
    }
}

struct TopkLayout {
    unsigned long long *keys_in, *keys_out;
    uint32_t *vals_in, *vals_out;
    void *temp;
    size_t temp_bytes, bytes;
};

TopkLayout topk_layout(int64_t n, void *base)
{
    TopkLayout L;
    char *p = (char *)base;
    size_t off = 0;
    auto take = [&](size_t b) {
        char *q = base ? p + off : nullptr;
        off += align_up(b);
        return q;
    };
    L.keys_in = (unsigned long long *)take(8 * (size_t)n);
    L.keys_out = (unsigned long long *)take(8 * (size_t)n);
    L.vals_in = (uint32_t *)take(4 * (size_t)n);
    L.vals_out = (uint32_t *)take(4 * (size_t)n);
    L.temp_bytes = 0;
    (void)rocprim::radix_sort_pairs_desc(nullptr, L.temp_bytes, (unsigned long long *)nullptr,
                                         (unsigned long long *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr,
                                         (size_t)n, 0, 64, (hipStream_t)0);
    L.temp = take(L.temp_bytes);
    L.bytes = off;
    return L;
}

int grid_for(int64_t n, int threads)
{
    int64_t b = (n + threads - 1) / threads;
    return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

}  // namespace

}  // namespace tig

using namespace tig;

extern "C" {

int tig_sep_centrality(const int32_t *src, const int32_t *dst, const double *ts, int64_t num_events,
                       int64_t num_nodes, double beta, double *cent_out, void *hip_stream)
{
    if (num_nodes < 1 || num_nodes > 0x7FFFFFFF || num_events < 0 || !cent_out || !(beta >= 0.0))
        return TIG_EINVAL;
    if (num_events > 0 && (!src || !dst || !ts))
        return TIG_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    hipError_t e = launch_fill_zero(cent_out, sizeof(double) * (size_t)num_nodes, s);
    if (e != hipSuccess)
        return TIG_EHIP;
    if (num_events == 0)
        return TIG_OK;
    // the stream is chronological: the last event carries t_max
    double t_max = 0.0;
    if (hipMemcpyAsync(&t_max, ts + (num_events - 1), sizeof(double), hipMemcpyDefault, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return TIG_EHIP;
    const int64_t blocks = (num_events + kCentChunk - 1) / kCentChunk;
    hipLaunchKernelGGL(k_centrality, dim3((unsigned)blocks), dim3(kCentThreads), 0, s, src, dst, ts, num_events,
                       num_nodes, beta, t_max, cent_out);
    return hipGetLastError() == hipSuccess ? TIG_OK : TIG_EHIP;
}

size_t tig_sep_topk_scratch_bytes(int64_t num_nodes)
{
    if (num_nodes < 1 || num_nodes > 0x7FFFFFFF)
        return 0;
    return topk_layout(num_nodes, nullptr).bytes;
}

int tig_sep_top_k(const double *cent, int64_t num_nodes, int64_t n_hubs, int32_t *hubs_out, uint8_t *is_hub_out,
                  void *scratch, size_t scratch_bytes, void *hip_stream)
{
    if (!cent || !is_hub_out || num_nodes < 1 || num_nodes > 0x7FFFFFFF || n_hubs < 0 || n_hubs > num_nodes ||
        (n_hubs > 0 && !hubs_out) || !scratch || ((uintptr_t)scratch & 255))
        return TIG_EINVAL;
    const TopkLayout L = topk_layout(num_nodes, scratch);
    if (scratch_bytes < L.bytes)
        return TIG_ENOSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    if (hipMemsetAsync(is_hub_out, 0, (size_t)num_nodes, s) != hipSuccess)
        return TIG_EHIP;
    if (n_hubs == 0)
        return TIG_OK;
    hipLaunchKernelGGL(k_topk_keys, dim3(grid_for(num_nodes, 256)), dim3(256), 0, s, cent, num_nodes, L.keys_in,
                       L.vals_in);
    size_t temp_bytes = L.temp_bytes;
    if (rocprim::radix_sort_pairs_desc(L.temp, temp_bytes, L.keys_in, L.keys_out, L.vals_in, L.vals_out,
                                       (size_t)num_nodes, 0, 64, s) != hipSuccess)
        return TIG_EHIP;
    hipLaunchKernelGGL(k_topk_flags, dim3(grid_for(n_hubs, 256)), dim3(256), 0, s, L.vals_out, n_hubs, hubs_out,
                       is_hub_out);
    return hipGetLastError() == hipSuccess ? TIG_OK : TIG_EHIP;
}

}  // extern "C"

#pragma clang fp contract(off)
namespace tig {

namespace {

// The edge loop of Alg. 1, fed with consecutive pieces of the stream.  A decision depends on all
// earlier ones, so what counts is the chain from one edge's partition to the next edge's, the branches
// that cannot be foreseen, and what the loop touches in memory.  Evaluating Eq. 3 for every partition of
// every edge (|P| divisions behind the sizes the edge before left) took 35 ns per edge at 8 partitions.
// Instead:
//  - the balance term takes one value per partition SIZE: the partitions are kept as bit sets by size
//    (level k: the partitions of size mn + k);
//  - the replica term takes one value per CLASS of partitions (with replicas of both endpoints, of one,
//    of none), so the arg max is in the lowest level of some class, and the lowest index among equals
//    is a count of trailing zeros;
//  - where the balance term stays below a replica's worth (Eq. 5: at least 1), "both" beats "one" beats
//    "none" without any arithmetic: nine edges in ten of a power-law stream end in "both", a chain of
//    and / count zeros / exclusive or over the two lowest levels, which stay in registers.  "Both" needs no look at the
//    hub flags either: where a non-hub is an endpoint, its one partition is all that "both" can be.  The branches that are left
//    are foreseen most of the time; without them (conditional moves, levels in memory) the chain is twice as long.  An edge
//    that is not "both" has one more, whether it leaves the sets: in a flat stream none can be foreseen.
//    Sets and hub flags are requested some edges ahead, one edge's with every decision, so that their misses run beside it.
// Terms that are evaluated are the IEEE operations of Eq. 3-6 in their order, so the partitions are the
// same bit for bit; an edge that the sets do not cover (sizes spread over kLevels values or more, terms
// so close that rounding could make two sizes equal, centralities that are not finite and non-negative)
// is decided by the plain evaluation (best_plain), and while the sizes are spread that far only their extremes are
// kept.  Nothing is allocated, so that the C entries have no exception to hold back.  Measured per edge (Xeon at 2.7 GHz), with every level in memory
// and no test for "both", with ids checked and sets requested 64 edges at a time ahead of 64 decisions, and now: 4 M events, 1 M nodes
// (Zipf 1.5), 8 partitions 12.0, 5.6, 5.1 ns; 16 partitions, 5% hubs 12.2, 5.8, 5.3; 2 M events of 2.6 M nodes (Zipf 1.1), 8
// partitions 20.4, 25.7, 15.1; 0.6 M events of 1 M nodes (Zipf 0.8) 25.7, 40.8, 22.8.
class EdgeLoop {
public:
    EdgeLoop(const tig_sep_config &cfg, int64_t num_nodes, const double *cent, const uint8_t *is_hub, uint64_t *A)
        : P_(cfg.num_parts), lam_(cfg.lambda), eps_(cfg.epsilon), N_(num_nodes), cent_(cent), A_(A), is_hub_(is_hub)
    {
        int odd = 0;
        for (int64_t i = 0; i < N_; ++i)
            odd |= !(cent_[i] >= 0.0 && cent_[i] <= 1e300);
        memset(A_, 0, sizeof(uint64_t) * (size_t)N_);
        plain_ = odd || !(lam_ <= 1e100);
        // mx < 2^31: eps moves the denominator of Eq. 6 by at least 7e-7, so the balance term of a gap below
        // kLevels is below 1 - 1e-9 * 40, and neighbouring sizes' terms are at least 9e-7 apart
        easy_ = !plain_ && lam_ >= 1e-3 && lam_ <= 1.0 && eps_ >= 1e-6 && eps_ <= 1e3;
        all_ = P_ == 64 ? ~0ull : (1ull << P_) - 1ull;
        for (int p = 0; p < P_; ++p)
            size_[p] = 0;
        for (int g = 0; g < kLevels; ++g)
            terms_[g].den = -1.0;
        for (uint64_t &l : level_)
            l = 0;
        base_ = 0;
        mx_ = mn_ = 0;
        levels_from_sizes();
    }

    // decides `n` further edges; false: an endpoint is outside 0..N-1 (the edges before it are decided)
    bool run(const int32_t *src, const int32_t *dst, int64_t n, int32_t *part_out)
    {
        constexpr int64_t kAhead = 24;  // edges whose endpoints' sets and hub flags are requested early
        uint64_t *const A = A_;
        const uint8_t *const hub = is_hub_;
        // (whatever the ids are: a request is a hint, and an address of nothing is passed over)
        const auto request = [A, hub](int32_t i, int32_t j) {
            const uintptr_t a = (uintptr_t)A, h = (uintptr_t)hub, u = (uint32_t)i, v = (uint32_t)j;
            __builtin_prefetch((const void *)(a + sizeof(uint64_t) * u));
            __builtin_prefetch((const void *)(a + sizeof(uint64_t) * v));
            __builtin_prefetch((const void *)(h + u));
            __builtin_prefetch((const void *)(h + v));
        };
        const uint64_t N = (uint64_t)N_, all = all_;
        const bool easy = easy_ && mx_ + n < ((int64_t)1 << 31);
        int64_t e = 0;
        while (e < n) {
            // as long as the sizes fit the sets: the candidates of the edge as one set, and the lowest index of
            // its lowest level.  The two lowest levels are kept in registers: the chain from one edge to the next is
            // these few operations.
            uint64_t *lev = level_ + base_;
            int64_t mx = mx_, mn = mn_;
            uint64_t l0 = lev[0], l1 = lev[1];
            const int64_t stop = !easy || mx - mn >= kLevels ? e : n;
            for (; e < stop; ++e) {
                if (e + kAhead < n)
                    request(src[e + kAhead], dst[e + kAhead]);
                const uint32_t i = (uint32_t)src[e], j = (uint32_t)dst[e];
                if (i >= N || j >= N)
                    break;
                const uint64_t ai = A[i], aj = A[j], both = ai & aj;
                uint64_t set = both;
                // (a resident non-hub has one partition: where it is an endpoint, `both` is that partition or empty)
                if (__builtin_expect(!both, 0)) {
                    const uint64_t any = ai | aj;
                    // the partition of a resident non-hub is the only candidate; two of them: Case 3
                    const uint64_t x = ai & ((uint64_t)(hub[i] != 0) - 1u), y = aj & ((uint64_t)(hub[j] != 0) - 1u), xy = x | y;
                    // (two non-hubs apart; hubs on partitions of their own: the replicas' worths have to be compared)
                    const bool two = (x != 0) & (y != 0), apart = (ai != 0) & (aj != 0) & (xy == 0);
                    if (two | apart)
                        break;
                    set = any ? any : all;
                    set = xy ? xy : set;
                }
                const uint64_t m0 = set & l0;
                uint64_t bit;
                int64_t k = 0;
                if (__builtin_expect(m0 != 0, 1)) {
                    bit = m0 & (0ull - m0);
                    l0 ^= bit;
                    l1 |= bit;
                } else {
                    uint64_t m = set & l1;
                    if (m) {
                        k = 1;
                        bit = m & (0ull - m);
                        l1 ^= bit;
                        lev[2] |= bit;
                    } else {
                        k = 2;
                        while (!(m = set & lev[k]))
                            ++k;
                        bit = m & (0ull - m);
                        lev[k] ^= bit;
                        lev[k + 1] |= bit;
                    }
                }
                const int p = __builtin_ctzll(bit);
                part_out[e] = p;
                if (!both) {
                    A[i] = ai | 1ull << p;
                    A[j] |= 1ull << p;
                }
                ++size_[p];
                mx += mn + k == mx;
                if (l0 == 0) {  // (the smallest size had one partition left)
                    ++mn;
                    *lev++ = 0;
                    l0 = l1;
                    l1 = lev[1];
                    if (__builtin_expect(lev >= level_ + kRing, 0)) {
                        ++e;
                        break;
                    }
                }
                if (__builtin_expect(mx - mn >= kLevels, 0)) {
                    ++e;
                    break;
                }
            }
            lev[0] = l0;
            lev[1] = l1;
            mx_ = mx;
            mn_ = mn;
            base_ = (int)(lev - level_);
            if (base_ >= kRing && mx_ - mn_ < kLevels)
                levels_from_sizes();
            // one edge of any kind, or all of them while the sizes are too far apart for the sets
            while (e < n) {
                if (e + kAhead < n)
                    request(src[e + kAhead], dst[e + kAhead]);
                const int64_t i = src[e], j = dst[e];
                if (i < 0 || i >= N_ || j < 0 || j >= N_)
                    return false;
                const int p = decide(i, j);
                part_out[e] = p;
                if (p >= 0) {
                    A[i] |= 1ull << p;
                    A[j] |= 1ull << p;
                    grow(p);
                }
                ++e;
                if (easy && mx_ - mn_ < kLevels)
                    break;
            }
        }
        return true;
    }

    void sizes(int64_t *out) const
    {
        for (int p = 0; p < P_; ++p)
            out[p] = size_[p];
    }

private:
    static constexpr int kLevels = 16;
    static constexpr int kRing = 1024;  // the sets move up one place whenever mn grows; moved back after so many
    struct Terms {          // balance terms (Eq. 6) of sizes mn .. mx, mx - mn = g
        double den;         // their denominator, -1: not computed yet
        double of[kLevels];
        bool distinct;      // terms of different sizes stay apart when a replica term is added
    };

    int decide(int64_t i, int64_t j)
    {
        const bool hi = is_hub_[i] != 0, hj = is_hub_[j] != 0;
        const uint64_t ai = A_[i], aj = A_[j];
        if (ai && aj) {
            if (hi != hj)                                     // Case 1: where the non-hub resides
                return __builtin_ctzll(hi ? aj : ai);
            if (hi)                                           // Case 2
                return best(i, j, ai, aj);
            return ai == aj ? __builtin_ctzll(ai) : -1;       // Case 3
        }
        if (ai && !hi)                                        // Case 4 & 5: a resident non-hub is not replicated
            return __builtin_ctzll(ai);
        if (aj && !hj)
            return __builtin_ctzll(aj);
        return best(i, j, ai, aj);
    }

    // arg max over all partitions of C(i, j, p) = C_REP + C_BAL (Eq. 3), lowest index among equals
    int best(int64_t i, int64_t j, uint64_t ai, uint64_t aj)
    {
        const int64_t gap = mx_ - mn_;
        if (gap >= kLevels || plain_)
            return best_plain(i, j, ai, aj);
        const Terms &t = terms(gap);
        if (!t.distinct)
            return best_plain(i, j, ai, aj);
        double h_i, h_j;
        replica_worth(i, j, h_i, h_j);
        const uint64_t cls[4] = {ai & aj, ai & ~aj, aj & ~ai, all_ & ~(ai | aj)};
        const double rep[4] = {h_i + h_j, h_i + 0.0, 0.0 + h_j, 0.0 + 0.0};
        double top = -1.0;
        uint64_t arg = 0;
        for (int c = 0; c < 4; ++c) {
            if (!cls[c])
                continue;
            const uint64_t *lev = level_ + base_;
            int k = 0;
            while (!(cls[c] & lev[k]))
                ++k;
            const double v = rep[c] + t.of[k];
            if (v > top) {
                top = v;
                arg = cls[c] & lev[k];
            } else if (v == top) {
                arg |= cls[c] & lev[k];
            }
        }
        return __builtin_ctzll(arg);
    }

    int best_plain(int64_t i, int64_t j, uint64_t ai, uint64_t aj) const
    {
        double h_i, h_j;
        replica_worth(i, j, h_i, h_j);
        const double den = (eps_ + (double)mx_) - (double)mn_;
        int arg = 0;
        double top = 0.0;
        for (int p = 0; p < P_; ++p) {
            const double c_rep = (((ai >> p) & 1u) ? h_i : 0.0) + (((aj >> p) & 1u) ? h_j : 0.0);  // Eq. 4
            const double c_bal = lam_ * (double)(mx_ - size_[p]) / den;                            // Eq. 6
            const double c = c_rep + c_bal;
            if (p == 0 || c > top) {
                top = c;
                arg = p;
            }
        }
        return arg;
    }

    void replica_worth(int64_t i, int64_t j, double &h_i, double &h_j) const  // Eq. 5
    {
        const double tot = cent_[i] + cent_[j];
        const double th_i = tot == 0.0 ? 0.5 : cent_[i] / tot;
        const double th_j = tot == 0.0 ? 0.5 : cent_[j] / tot;
        h_i = 1.0 + (1.0 - th_i);
        h_j = 1.0 + (1.0 - th_j);
    }

    const Terms &terms(int64_t gap)
    {
        Terms &t = terms_[gap];
        // (compared, not recomputed: the denominator of a gap changes where eps meets another power of two)
        const double den = (eps_ + (double)mx_) - (double)mn_;
        if (t.den != den) {
            t.den = den;
            t.distinct = true;
            for (int k = 0; k <= (int)gap; ++k) {
                t.of[k] = lam_ * (double)(gap - k) / den;
                if (k > 0 && !(t.of[k - 1] - t.of[k] > 1e-9 * (4.0 + t.of[0])))
                    t.distinct = false;
            }
            if (!(t.of[0] >= 0.0))
                t.distinct = false;  // (an eps lost against the sizes: 0 / 0)
        }
        return t;
    }

    void grow(int p)
    {
        const int64_t sz = size_[p]++;
        if (mx_ - mn_ >= kLevels) {  // only the extremes, until the sizes are close enough for the sets again
            mx_ = sz + 1 > mx_ ? sz + 1 : mx_;
            if (sz == mn_) {
                mn_ = size_[0];
                for (int q = 1; q < P_; ++q)
                    mn_ = size_[q] < mn_ ? size_[q] : mn_;
                if (mx_ - mn_ < kLevels)
                    levels_from_sizes();
            }
            return;
        }
        uint64_t *lev = level_ + base_;
        const int64_t k = sz - mn_;
        lev[k] ^= 1ull << p;
        lev[k + 1] |= 1ull << p;
        mx_ += sz == mx_;
        if (lev[0] == 0) {
            ++mn_;
            if (++base_ >= kRing && mx_ - mn_ < kLevels)
                levels_from_sizes();
        }
    }

    // the sets of sizes that lie within kLevels values (mx_ and mn_ are kept by the callers)
    void levels_from_sizes()
    {
        for (int k = 0; k <= kLevels; ++k)  // (all others are zero)
            level_[base_ + k] = 0;
        base_ = 0;
        for (int p = 0; p < P_; ++p)
            level_[size_[p] - mn_] |= 1ull << p;
    }

    const int P_;
    const double lam_, eps_;
    const int64_t N_;
    const double *const cent_;
    uint64_t *const A_;
    const uint8_t *const is_hub_;
    bool plain_, easy_;
    uint64_t all_, level_[kRing + kLevels + 1];  // level k: level_[base_ + k], 0 <= k <= kLevels; all zero above
    int base_;
    int64_t size_[64], mx_, mn_;
    Terms terms_[kLevels];
};

bool sep_config_ok(const tig_sep_config *cfg)
{
    return cfg && cfg->struct_size == sizeof(tig_sep_config) && cfg->num_parts >= 1 && cfg->num_parts <= 64 &&
           cfg->lambda > 0.0 && cfg->epsilon > 0.0;
}

}  // namespace

}  // namespace tig

extern "C" {

int tig_sep_assign(const tig_sep_config *cfg, const int32_t *src, const int32_t *dst, int64_t num_events,
                   int64_t num_nodes, const double *cent, const uint8_t *is_hub, int32_t *edge_part_out,
                   uint64_t *node_parts_out, int64_t *part_edges_out)
{
    if (!sep_config_ok(cfg))
        return TIG_EINVAL;
    if (num_nodes < 1 || num_events < 0 || !cent || !is_hub || !node_parts_out || !part_edges_out ||
        (num_events > 0 && (!src || !dst || !edge_part_out)))
        return TIG_EINVAL;
    EdgeLoop loop(*cfg, num_nodes, cent, is_hub, node_parts_out);
    if (!loop.run(src, dst, num_events, edge_part_out))
        return TIG_ERANGE;
    loop.sizes(part_edges_out);
    return TIG_OK;
}

size_t tig_sep_scratch_bytes(int64_t num_nodes)
{
    const size_t t = tig_sep_topk_scratch_bytes(num_nodes);
    if (t == 0)
        return 0;
    // [centrality | hub flags | hub list | top-k scratch]
    return align_up(8 * (size_t)num_nodes) + align_up((size_t)num_nodes) + align_up(4 * (size_t)num_nodes) + t;
}

int tig_sep_partition(const tig_sep_config *cfg, const int32_t *src, const int32_t *dst, const double *ts,
                      int64_t num_events, int64_t num_nodes, void *scratch, size_t scratch_bytes, void *hip_stream,
                      double *cent_out, uint8_t *is_hub_out, int32_t *edge_part_out, uint64_t *node_parts_out,
                      int64_t *part_edges_out)
{
    if (!cfg || cfg->struct_size != sizeof(tig_sep_config) || !(cfg->top_k >= 0.0) || !(cfg->top_k <= 1.0) ||
        !cent_out || !is_hub_out || !scratch || ((uintptr_t)scratch & 255))
        return TIG_EINVAL;
    const size_t need = tig_sep_scratch_bytes(num_nodes);
    if (need == 0)
        return TIG_EINVAL;
    if (scratch_bytes < need)
        return TIG_ENOSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    char *base = (char *)scratch;
    double *cent_d = (double *)base;
    uint8_t *hub_d = (uint8_t *)(base + align_up(8 * (size_t)num_nodes));
    int32_t *list_d = (int32_t *)((char *)hub_d + align_up((size_t)num_nodes));
    void *topk = (char *)list_d + align_up(4 * (size_t)num_nodes);
    int rc = tig_sep_centrality(src, dst, ts, num_events, num_nodes, cfg->beta, cent_d, hip_stream);
    if (rc != TIG_OK)
        return rc;
    const int64_t n_hubs = (int64_t)std::floor(cfg->top_k * (double)num_nodes);
    rc = tig_sep_top_k(cent_d, num_nodes, n_hubs, list_d, hub_d, topk, tig_sep_topk_scratch_bytes(num_nodes),
                       hip_stream);
    if (rc != TIG_OK)
        return rc;
    // the centralities and hub flags go to the caller; the endpoints pass through a pinned buffer in pieces,
    // the next piece's copy beside the edge loop over this one
    if (hipMemcpyAsync(cent_out, cent_d, 8 * (size_t)num_nodes, hipMemcpyDefault, s) != hipSuccess ||
        hipMemcpyAsync(is_hub_out, hub_d, (size_t)num_nodes, hipMemcpyDefault, s) != hipSuccess)
        return TIG_EHIP;
    if (!sep_config_ok(cfg) || num_events < 0 || !node_parts_out || !part_edges_out ||
        (num_events > 0 && (!src || !dst || !edge_part_out)))
        return hipStreamSynchronize(s) == hipSuccess ? TIG_EINVAL : TIG_EHIP;
    PinnedStage stage;
    if (!stage.ptr)
        return TIG_ENOMEM;
    struct Events {
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events()
        {
            for (hipEvent_t x : e)
                if (x)
                    (void)hipEventDestroy(x);
        }
    } ready;
    for (hipEvent_t &x : ready.e)
        if (hipEventCreateWithFlags(&x, hipEventDisableTiming) != hipSuccess)
            return TIG_EHIP;
    const int64_t piece = (int64_t)(kPinnedStageBytes / (4 * sizeof(int32_t)));  // two buffers of two arrays
    int32_t *const buf = (int32_t *)stage.ptr;
    auto request = [&](int64_t k) -> hipError_t {
        const int64_t e0 = k * piece, n = num_events - e0 < piece ? num_events - e0 : piece;
        if (n <= 0)
            return hipSuccess;
        int32_t *const d = buf + (k & 1) * 2 * piece;
        hipError_t e = hipMemcpyAsync(d, src + e0, 4 * (size_t)n, hipMemcpyDefault, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(d + piece, dst + e0, 4 * (size_t)n, hipMemcpyDefault, s);
        return e == hipSuccess ? hipEventRecord(ready.e[k & 1], s) : e;
    };
    hipError_t he = hipStreamSynchronize(s);  // the centralities are here
    if (he == hipSuccess)
        he = request(0);
    int status = TIG_OK;
    EdgeLoop loop(*cfg, num_nodes, cent_out, is_hub_out, node_parts_out);
    for (int64_t k = 0; he == hipSuccess && status == TIG_OK && k * piece < num_events; ++k) {
        if ((he = request(k + 1)) != hipSuccess || (he = hipEventSynchronize(ready.e[k & 1])) != hipSuccess)
            break;
        const int64_t e0 = k * piece, n = num_events - e0 < piece ? num_events - e0 : piece;
        const int32_t *const d = buf + (k & 1) * 2 * piece;
        if (!loop.run(d, d + piece, n, edge_part_out + e0))
            status = TIG_ERANGE;
    }
    loop.sizes(part_edges_out);
    // (nothing is in flight into the pinned buffer when it is given back)
    const hipError_t last = hipStreamSynchronize(s);
    return he != hipSuccess || last != hipSuccess ? TIG_EHIP : status;
}

}  // extern "C"
