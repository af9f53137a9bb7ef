// Other instances of the general architecture (paper Sec. II-C "Training approach for TIGs": the
// messages of a node within a batch "can be aggregated by ... mean message", the state update "can
// be chosen from ... GRU, RNN", the embedding function f is "identity, time projection or
// attention"; Sec. II-A: nodes may carry static features), device side.  gfx950 only, fp32.
//
// A context with an attached module selection runs its state update in k_gru (message build and gates on
// the matrix cores; the plain recurrent cell is a one-gate product there) and, with attention and no node
// features, the fused embedding (two layers: k_two_*, then one launch per layer) and closing launches of the
// headline instance.  The rest:
//   k_mod_msgsum / k_mod_mean   mean aggregator: sums of all the node's messages of the batch (either role,
//                  every one built from the memory at the start of the step), then their means
//   k_mod_final    the last launch of a step without the fused ones: identity / time-projection embedding of
//                  sixteen events' queries (or their rows out of the attention layers), both logits on the
//                  matrix cores, beside it the memory overwrite and the preparation of the batch expected next
//   k_mod_commit   memory overwrite M <- s_i(t) and last_update ahead of attention layers that read the table
//   k_mr_items / k_mr_attn + k_rowgemm   attention embedding with node features, or second-layer rows that
//                  do not fit the fused kernel's tiles: every layer product as one contraction over all items of the layer, the
//                  attention core per item in its re-associated form (stated above k_mr_items); a
//                  negative's neighbours are looked up by k_mr_items
//   k_mod_hop2     two stacked attention layers (the embedding module's sum over the 2-hop temporal
//                  neighbourhood): the K most recent events, before the QUERY's time, of every
//                  neighbour of every distinct query; the first layer then runs over each used
//                  (query, neighbour) pair and each query itself, the second layer over those rows
#include <hip/hip_runtime.h>

#include "kernels_common.h"
#include "prepare.h"
#include "rowgemm.h"
#include "winners.h"

namespace tig {

namespace {

constexpr int kModThreads = 256;
constexpr int kModWaves = kModThreads / kWave;

struct ModDims {
    int M, T, F, E, K, H, da, dh, dkv;
    int Ep, Ek;  // E padded to the decoder's output tiles / to its k-blocks
    int emb;
};

// The dimensions the second layer sees: its input rows are E wide.
ModDims second_layer_dims(ModDims d)
{
    d.M = d.E;
    d.da = d.E + d.T;
    d.dkv = d.E + d.F + d.T;
    d.dh = d.da / d.H;
    return d;
}

ModDims mod_dims(const Dims &d, const ModParams &p)
{
    return ModDims{d.M, d.T, d.F, d.E, d.K, d.H, d.da, d.dh, d.dkv, d.Ep, d.Ek, p.emb};
}

// r_i(t): the state row the embedding module reads for node v (memory row plus the static feature
// row), element j; a node id outside the graph reads as a zero row
__device__ inline float repr_elem(const StepArgs &a, const ModParams &p, int M, int32_t v, int j)
{
    if (v < 0 || (int64_t)v >= a.num_nodes)
        return 0.0f;
    float x = a.mem[(size_t)v * M + j];
    if (p.node_feat)
        x += p.node_feat[(size_t)v * M + j];
    return x;
}

// ------------------------------------------------------------------------------------------
// Mean aggregator, first half: one wavefront per (event, role) entry of the applied batch adds the
// columns of its message that differ between a node's messages -- [s'_other | Phi(dt) | e] -- to the
// accumulation row of the entry that won the node's last message (named by the node's key), in
// double.  A hub node collects thousands of messages per batch, and additions to one address queue
// up: a workgroup first collects its kMsgEntries entries' rows in an LDS table of kMsgSlots rows
// (direct-mapped by accumulation row; a row whose place is taken goes to memory directly) and adds
// every table row to memory once, dealt out over the node's kAccCopies copies.  The rows in memory
// are all zero between steps: k_mod_mean clears what it has read.
constexpr int kMsgThreads = 1024, kMsgEntries = 64, kMsgSlots = 16;

__global__ void __launch_bounds__(kMsgThreads) k_mod_msgsum(StepArgs a, ModDims d, ModParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int M = d.M, T = d.T, F = d.F, rest = M + T + F;
    double *acc = (double *)smem;                    // [slots x rest]
    int *tag = (int *)(acc + kMsgSlots * rest);      // [slots] accumulation row held by the slot, -1: none
    int *cnt = tag + kMsgSlots;                      // [slots] messages collected in it
    for (int i = threadIdx.x; i < kMsgSlots * rest; i += kMsgThreads)
        acc[i] = 0.0;
    if (threadIdx.x < kMsgSlots) {
        tag[threadIdx.x] = -1;
        cnt[threadIdx.x] = 0;
    }
    __syncthreads();
    const int lane = lane_id();
    const int i_end = ((int)blockIdx.x + 1) * kMsgEntries < 2 * a.msg_count ? ((int)blockIdx.x + 1) * kMsgEntries : 2 * a.msg_count;
    for (int i = (int)blockIdx.x * kMsgEntries + wave_id(); i < i_end; i += kMsgThreads / kWave) {
        const int64_t e = a.msg_first_eid + (i >> 1);
        const int32_t u = (i & 1) ? a.dst[e] : a.src[e];
        const int32_t o = (i & 1) ? a.src[e] : a.dst[e];
        if (u < 0 || (int64_t)u >= a.num_nodes)
            continue;
        const int32_t ref = ref_of_key(ref_ctx(a), u, a.msg_key[u]);
        if (ref >= 0 || ref == kRefNone)
            continue;  // (not reachable: every node of the applied batch has a winning entry in it)
        const int row = ~ref;
        const bool ok = o >= 0 && (int64_t)o < a.num_nodes;
        const double dt = a.ts[e] - a.lu[u];
        const int slot = row & (kMsgSlots - 1);
        int old = 0;
        if (lane == 0)
            old = atomicCAS(&tag[slot], -1, row);
        old = __shfl(old, 0);
        const bool in_lds = old == -1 || old == row;
        double *dst = in_lds ? acc + (size_t)slot * rest
                             : p.acc + ((size_t)row * kAccCopies + ((i >> 1) & (kAccCopies - 1))) * rest;
        for (int j = lane; j < rest; j += kWave) {
            float v;
            if (j < M)
                v = ok ? a.mem[(size_t)o * M + j] : 0.0f;
            else if (j < M + T)
                v = time_enc(p.time_w_rev[j - M], p.time_b_rev[j - M], dt);
            else
                v = a.edge_feat[(size_t)e * F + (j - M - T)];
            if (in_lds)
                atomicAdd(&dst[j], (double)v);
            else
                unsafeAtomicAdd(&dst[j], (double)v);
        }
        if (lane == 0) {
            if (in_lds)
                atomicAdd(&cnt[slot], 1);
            else
                atomicAdd(&p.acc_cnt[row], 1);
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < kMsgSlots * rest; idx += kMsgThreads) {
        const int slot = idx / rest, j = idx - slot * rest;
        const int row = tag[slot];
        if (row < 0 || row >= 2 * a.msg_count)
            continue;
        unsafeAtomicAdd(&p.acc[((size_t)row * kAccCopies + ((int)blockIdx.x & (kAccCopies - 1))) * rest + j], acc[idx]);
        if (j == 0)
            atomicAdd(&p.acc_cnt[row], cnt[slot]);
    }
}

// Mean aggregator, second half: the means of one updated node's message columns (one wavefront per winner).
__global__ void __launch_bounds__(kModThreads) k_mod_mean(StepArgs a, ModDims d, ModParams p)
{
    const int rest = d.M + d.T + d.F;
    int n_win = *a.n_win;
    n_win = n_win < 2 * a.msg_count ? n_win : 2 * a.msg_count;
    const int r = (int)blockIdx.x * kModWaves + wave_id();
    if (r >= n_win)
        return;
    const int entry = a.win[r].entry;
    if (entry < 0 || entry >= 2 * a.msg_count)
        return;  // (not a descriptor of this batch)
    double *acc = p.acc + (size_t)entry * kAccCopies * rest;
    const int n = p.acc_cnt[entry];
    const double inv = 1.0 / (double)(n > 0 ? n : 1);
    for (int j = lane_id(); j < rest; j += kWave) {
        double sum = 0.0;
#pragma unroll
        for (int c = 0; c < kAccCopies; ++c)  // (fixed order: the result does not depend on the adds' order beyond fp64 rounding)
            sum += acc[(size_t)c * rest + j];
#pragma unroll
        for (int c = 0; c < kAccCopies; ++c)
            acc[(size_t)c * rest + j] = 0.0;
        p.mean_msg[(size_t)entry * rest + j] = (float)(sum * inv);
    }
    if (lane_id() == 0)
        p.acc_cnt[entry] = 0;
}

__global__ void __launch_bounds__(kModThreads) k_mod_commit(StepArgs a, int M)
{
    overwrite_memory(a, M, (int)(blockIdx.x * kModWaves + threadIdx.x / kWave), (int)(gridDim.x * kModWaves));
}

// ------------------------------------------------------------------------------------------
// Two layers: the neighbour tables of the second hop.  One workgroup per query row (distinct source /
// destination queries, then the negatives, whose own table is looked up first): wavefront w takes the
// neighbours k = w, w + waves, ... and looks up the K most recent events of neighbour k before the
// QUERY's time into row q * K + k of the second-hop tables.
__global__ void __launch_bounds__(kModThreads) k_mod_hop2(StepArgs a, ModDims d, ModParams p, int msg_count, int n_commit)
{
    __shared__ int s_cnt;
    if ((int)blockIdx.x < n_commit) {  // the memory overwrite (nothing of this launch reads the memory)
        StepArgs c = a;
        c.msg_count = msg_count;
        overwrite_memory(c, d.M, (int)(blockIdx.x * kModWaves + threadIdx.x / kWave), n_commit * kModWaves);
        return;
    }
    int n_u = *a.qs.n_u;
    n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
    const int n_rows = n_u + (a.roles == 3 ? a.count : 0);
    const int x = (int)blockIdx.x - n_commit;
    if (x >= n_rows)
        return;
    const int K = d.K;
    const int q = x < n_u ? x : 2 * a.count + (x - n_u);
    if (x >= n_u && threadIdx.x < kWave) {
        int32_t rf, ee;
        double ts_k;
        (void)finish_negative(a, K, x - n_u, rf, ee, ts_k);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int c = a.qs.cnt[q];
        s_cnt = c < 0 ? 0 : (c > K ? K : c);
    }
    __syncthreads();
    const int cnt = s_cnt;
    const double t_q = a.qs.t[q];
    for (int k = wave_id(); k < cnt; k += kModWaves) {
        int32_t nb, ee;
        double tt;
        (void)nbr_lookup_wave(a, K, a.qs.nbr[(size_t)q * K + k], t_q, -1, p.hop2, q * K + k, nb, ee, tt);
    }
}

// ------------------------------------------------------------------------------------------
// Two layers without node features: the rows of the first layer -- every distinct (node, time) among the queries
// and their neighbours at the queries' times -- as a query set of their own, so that either layer is one launch
// of the embedding kernel (embed_tile.h, LAYER; the second with the first's rows as its "memory").  4000 events of
// 100 columns: 337 -> 128 us a step (48 + 40 us of it the layers); with the products of both layers as launches over
// all rows (k_mr_*, below, which remain for node features and for rows that the embedding kernel's tiles do not hold) every
// intermediate of every row went through memory, and the host issued 22 launches a step.
//   k_two_negatives  memory overwrite; the negatives' own neighbours, one wavefront each
//   k_two_claim      equal pairs merged, one wavefront per query: the rows' (node, time), and for every (query,
//                    slot) its row or the (query, slot) that represents the pair
//   k_two_lookup     the rows' neighbours, one wavefront each; the references of the queries' slots into the rows
// Bound by chains of dependent reads (claims; the search for t in a hub's list): as many wavefronts as the
// chip holds, and none waits for another's chain.
constexpr int kTwoWaves = 8, kTwoThreads = kTwoWaves * kWave;

__device__ inline int two_rows(const StepArgs &a, int &n_u)
{
    n_u = *a.qs.n_u;
    n_u = n_u < 0 ? 0 : (n_u < 2 * a.count ? n_u : 2 * a.count);
    return n_u + (a.roles == 3 ? a.count : 0);
}

__device__ inline int two_query_row(const StepArgs &a, int n_u, int x) { return x < n_u ? x : 2 * a.count + (x - n_u); }

__device__ inline int two_slots(const StepArgs &a, int K, int q)
{
    const int c = a.qs.cnt[q];
    return c < 0 ? 0 : (c > K ? K : c);
}

__global__ void __launch_bounds__(kTwoThreads) k_two_negatives(StepArgs a, int M, int K, int n_commit)
{
    int x = (int)blockIdx.x;
    if (x < n_commit) {
        if (x == 0 && threadIdx.x == 0 && a.rows_seen)
            a.rows_seen[1] = *a.n_win;  // (a hint for the host)
        overwrite_memory(a, M, x * kTwoWaves + wave_id(), n_commit * kTwoWaves);
        return;
    }
    const int b = (x - n_commit) * kTwoWaves + wave_id();
    if (b >= a.count)
        return;
    const int32_t u = a.neg[b];
    int32_t nbr, eid;
    double ts;
    (void)nbr_lookup_wave(a, K, u, a.ts[a.first_eid + b], -1, a.qs, 2 * a.count + b, nbr, eid, ts);
}

// Pair (u, t) of (query x, slot j) = index `dense` claims a place of the table (open addressing; a place
// changes once per epoch); returns the index that represents the pair.
__device__ inline int two_claim(const StepArgs &a, const ModParams &p, int K, int n_u, int n_rows, uint32_t epoch, int dense, int32_t u, double t)
{
    const unsigned long long mine = ((unsigned long long)epoch << 32) | (uint32_t)dense;
    uint32_t h = query_hash(u, t) & p.claim_mask;
    for (uint32_t probes = 0; probes <= p.claim_mask; ++probes) {
        unsigned long long cur = __hip_atomic_load(&p.claim[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(cur >> 32) != epoch) {
            const unsigned long long old = atomicCAS(&p.claim[h], cur, mine);
            if (old == cur)
                return dense;
            cur = old;
        }
        const int other = (int)(uint32_t)cur;
        const int xo = other / (K + 1), jo = other - xo * (K + 1);
        if (other >= 0 && xo < n_rows) {
            const int qo = two_query_row(a, n_u, xo);
            const int32_t uo = jo < K ? a.qs.nbr[(size_t)qo * K + jo] : a.qs.node[qo];
            if (uo == u && a.qs.t[qo] == t)
                return other;
        }
        h = (h + 1) & p.claim_mask;
    }
    return dense;
}

__global__ void __launch_bounds__(kTwoThreads) k_two_claim(StepArgs a, ModParams p, int K, uint32_t epoch)
{
    __shared__ int s_items[kTwoWaves], s_base;
    int n_u;
    const int n_rows = two_rows(a, n_u), lane = lane_id(), wave = wave_id();
    int32_t *counter = p.it.n_u + (epoch & 1u);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        p.it.n_u[(epoch & 1u) ^ 1u] = 0;  // (the next step's)
    const int x = (int)blockIdx.x * kTwoWaves + wave;
    const bool valid = x < n_rows;  // (uniform over the wavefront)
    const int q = valid ? two_query_row(a, n_u, x) : 0;
    const int cnt = valid ? two_slots(a, K, q) : 0;
    // lane j < cnt: slot j; lane K: the query itself
    const bool cand = valid && (lane < cnt || lane == K);
    const double t = a.qs.t[q];
    int32_t u = -1;
    int rep = -1;
    const int dense = x * (K + 1) + lane;
    if (cand)
        u = lane < K ? a.qs.nbr[(size_t)q * K + lane] : a.qs.node[q];
    // A node that a query has several times (where few nodes have most of the events: its partner of all its recent ones) is claimed
    // once, by its first lane: the wavefront's lanes have one time.  Three nodes are looked for this way, first lanes first; lanes
    // that then remain claim for themselves.  A step over 4000 events of a partition of 2.6 M nodes 112.6 -> 111.1 us, over 1000 66.9 ->
    // 65.5; over 200 to 700 of small graphs without such nodes at most 0.3 us more, of 61 to 105.  (Every lane compared with each of
    // the query's slots: 111.8 and 65.7; with conditions in the place of keys the launch alone took 0.4 to 0.7 us more there.)
    const int32_t key = cand ? u : -1 - lane;  // (a value of its own for a lane that claims nothing)
    int first = lane;
    unsigned long long todo = __ballot(cand);
    for (int turn = 0; turn < 3 && todo; ++turn) {
        const int lead = __builtin_ctzll(todo);
        const unsigned long long same = __ballot(key == __builtin_amdgcn_readlane(key, lead));
        first = (same >> lane) & 1ull ? lead : first;
        todo &= ~same;
    }
    if (cand && first == lane)
        rep = two_claim(a, p, K, n_u, n_rows, epoch, dense, u, t);
    rep = __shfl(rep, first, kWave);
    const bool is_row = cand && rep == dense;
    const unsigned long long m = __ballot(is_row);
    if (lane == 0)
        s_items[wave] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
        for (int i = 0; i < kTwoWaves; ++i)
            total += s_items[i];
        s_base = total > 0 ? atomicAdd(counter, total) : 0;
    }
    __syncthreads();
    int row = s_base + __popcll(m & ((1ull << lane) - 1ull));
    for (int i = 0; i < wave; ++i)
        row += s_items[i];
    if (is_row && row >= 0 && row < 3 * a.count * (K + 1)) {  // (always, with a counter that started at 0)
        p.it.node[row] = u;
        p.it.t[row] = t;
        p.mr_ci[dense] = row;
    } else if (cand) {
        p.mr_ci[dense] = -rep - 1;
    }
}

__global__ void __launch_bounds__(kTwoThreads) k_two_lookup(StepArgs a, ModParams p, int K, uint32_t epoch, int n_refs)
{
    int n_u;
    const int n_rows = two_rows(a, n_u), most = 3 * a.count * (K + 1);
    if ((int)blockIdx.x < n_refs) {  // the references, a thread each
        const int n = n_rows * (K + 1);
        for (int i = (int)blockIdx.x * kTwoThreads + (int)threadIdx.x; i < n; i += n_refs * kTwoThreads) {
            const int x = i / (K + 1), j = i - x * (K + 1), q = two_query_row(a, n_u, x);
            if (j < K && j >= two_slots(a, K, q))
                continue;
            int c = p.mr_ci[i];
            if (c < 0 && -c - 1 < n)
                c = p.mr_ci[-c - 1];
            c = c >= 0 && c < most ? c : 0;
            if (j < K)
                p.ref2[(size_t)q * K + j] = c;
            else
                p.self2[q] = c;
        }
        return;
    }
    int n = p.it.n_u[epoch & 1u];
    n = n < 0 ? 0 : (n < most ? n : most);
    const int step = ((int)gridDim.x - n_refs) * kTwoWaves;
    for (int r = ((int)blockIdx.x - n_refs) * kTwoWaves + wave_id(); r < n; r += step) {
        int32_t nbr, eid;
        double ts;
        (void)nbr_lookup_wave(a, K, p.it.node[r], p.it.t[r], -1, p.it, r, nbr, eid, ts);
    }
}

// ------------------------------------------------------------------------------------------
// With node features: the attention embedding as contractions over all ITEMS of a layer at once (an item is a distinct
// query or, in the first of two layers, neighbour j of a distinct query at the query's time): every
// layer product is one k_rowgemm launch over the items instead of one pass over the weight matrices
// per item (forty thousand workgroups streaming 0.7 MB each from L2 bounded the per-item kernel),
// and the attention core runs in the re-associated form that is the same function in exact
// arithmetic -- q~_h = W_K,h^T Qv_h, score <q~_h, kv_k> / sqrt(d_h) (the key bias adds a constant
// over the slots that the softmax cancels), head output W_V,h (sum_k p_hk kv_k) + b_V,h -- so that no
// product runs over neighbour slots and the raw key / value rows [row of the neighbour | e |
// Phi(t - t_k)] are never stored: the attention kernel forms them in registers.
//   k_mr_items   one wavefront per distinct query: the item list (first of two layers: the used
//                (query, slot) pairs and the queries themselves, packed in the order the workgroups
//                arrive), query rows [own row | Phi(0)] and the own row as the tail of the merge
//                layer's input
//   k_mr_attn    one wavefront per item: scores, softmax, weighted sums of the raw rows
enum MrMode { kMrSingle = 0, kMrFirst = 1, kMrSecond = 2 };
constexpr int kMrWaves = 16;
constexpr int kMrCH = 4;   // slots per register chunk
constexpr int kMrCC = 8;   // 64-column pieces of a raw row a lane can hold at most: rows of up to 512 columns
constexpr int kMrMaxHeads = 4;

// The item of (query row x, slot j) once the item list is complete: an index, or the pair's
// representative's.
__device__ inline int mr_item_of(const ModParams &p, size_t dense)
{
    int c = p.mr_ci[dense];
    if (c < 0)
        c = p.mr_ci[(size_t)(-c - 1)];
    return c < 0 ? 0 : c;
}

// First of two layers: equal (node, t) pairs -- a hub is a neighbour of most queries of a second, and
// is a query itself -- are one item.  Pair (u, t) of (x, j) index `dense` claims a slot of the table
// (open addressing; a slot changes once per step, from empty to claimed); returns the index that
// represents the pair: its own, or the first claimant's.
__device__ inline int mr_claim(const StepArgs &a, const ModParams &p, int K, int n_u, int dense, int32_t u, double t)
{
    uint32_t h = query_hash(u, t) & p.mr_tab_mask;
    for (uint32_t probes = 0; probes <= p.mr_tab_mask; ++probes) {
        uint32_t cur = __hip_atomic_load(&p.mr_tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == 0u) {
            const uint32_t old = atomicCAS(&p.mr_tab[h], 0u, (uint32_t)dense + 1u);
            if (old == 0u)
                return dense;
            cur = old;
        }
        const int other = (int)(cur - 1u);
        const int xo = other / (K + 1), jo = other - xo * (K + 1);
        if (xo < n_u + a.count) {
            const int qo = xo < n_u ? xo : 2 * a.count + (xo - n_u);
            const int32_t uo = jo < K ? a.qs.nbr[(size_t)qo * K + jo] : a.qs.node[qo];
            if (uo == u && a.qs.t[qo] == t)
                return other;
        }
        h = (h + 1) & p.mr_tab_mask;
    }
    return dense;
}

// One wavefront per distinct query row x; its items are the used slots j < cnt of its neighbour table
// and -- slot K -- the query itself (one layer, and the second of two: that one only).
template <int MODE>
__global__ void __launch_bounds__(kMrWaves *kWave) k_mr_items(StepArgs a, ModDims d, ModParams p)
{
    __shared__ int wg_items[kMrWaves], wg_base;
    int n_u = *a.qs.n_u;
    n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
    const int n_rows = n_u + (a.roles == 3 ? a.count : 0);
    const int M = d.M, E = d.E, K = d.K, da = d.da;
    const int lane = lane_id();
    const int x = (int)blockIdx.x * kMrWaves + wave_id();
    const bool valid = x < n_rows;  // (uniform over the wavefront; every wavefront reaches the barriers)
    const int q = x < n_u ? x : 2 * a.count + (x - n_u);
    int cnt_x = 0;
    if (valid) {
        if (MODE == kMrSingle && x >= n_u) {  // a negative: its neighbours are looked up here
            int32_t rf, ee;
            double ts_k;
            cnt_x = finish_negative(a, K, x - n_u, rf, ee, ts_k);
        } else {
            cnt_x = a.qs.cnt[q];
        }
        cnt_x = cnt_x < 0 ? 0 : (cnt_x > K ? K : cnt_x);
    }
    const int32_t u_self = !valid ? -1 : (MODE == kMrSingle && x >= n_u ? a.neg[x - n_u] : a.qs.node[q]);
    // lane `it` of the wavefront: candidate item `it` of the row (slots first, the query itself last)
    const int n_cand = !valid ? 0 : (MODE == kMrFirst ? cnt_x + 1 : 1);
    const int my_j = MODE == kMrFirst && lane < cnt_x ? lane : K;
    int32_t my_u = u_self;
    bool is_item = lane < n_cand;
    if (MODE == kMrFirst && lane < n_cand) {
        if (my_j < K)
            my_u = a.qs.nbr[(size_t)q * K + my_j];
        const int dense = x * (K + 1) + my_j;
        const int rep = mr_claim(a, p, K, n_u, dense, my_u, a.qs.t[q]);
        is_item = rep == dense;
        if (!is_item)
            p.mr_ci[dense] = -rep - 1;
    }
    const unsigned long long items = __ballot(is_item);
    const int n_it = __popcll(items);
    int ci0 = x;
    if (MODE == kMrFirst) {  // the items are packed in the order the workgroups arrive: one addition per workgroup
        if (lane == 0)
            wg_items[wave_id()] = n_it;
        __syncthreads();
        if (threadIdx.x == 0) {
            int total = 0;
            for (int i = 0; i < kMrWaves; ++i)
                total += wg_items[i];
            wg_base = total > 0 ? atomicAdd(p.mr_n, total) : 0;
        }
        __syncthreads();
        ci0 = wg_base;
        for (int i = 0; i < wave_id(); ++i)
            ci0 += wg_items[i];
        if (ci0 < 0 || ci0 + n_it > 3 * a.count * (K + 1))
            return;  // (not reachable while the counter is cleared every step)
    }
    int rank = 0;
    for (unsigned long long left = items; left != 0ull; left &= left - 1ull, ++rank) {
        const int it = __ffsll((long long)left) - 1;  // (uniform)
        const int j = __shfl(my_j, it);
        const int32_t u = __shfl(my_u, it);
        const int ci = ci0 + rank;
        const bool hop = j < K;
        int cnt_item = cnt_x;
        if (hop) {
            const int c = p.hop2.cnt[(size_t)q * K + j];
            cnt_item = c < 0 ? 0 : (c > K ? K : c);
        }
        if (lane == 0) {
            p.mr_itq[ci] = q;
            p.mr_itj[ci] = j;
            p.mr_has[ci] = cnt_item > 0 ? 1 : 0;
            if (MODE == kMrFirst)
                p.mr_ci[(size_t)x * (K + 1) + j] = ci;
        }
        // the item's own row: the node's state row (+ features), or -- second layer -- its first-layer row
        const float *own1 = MODE == kMrSecond ? p.h1 + (size_t)mr_item_of(p, (size_t)x * (K + 1) + K) * E : nullptr;
        for (int jj = lane; jj < da; jj += kWave) {
            float v;
            if (jj >= M)
                v = time_enc(p.time_w_rev[jj - M], p.time_b_rev[jj - M], 0.0);
            else
                v = MODE == kMrSecond ? own1[jj] : repr_elem(a, p, M, u, jj);
            p.mr_qin[(size_t)ci * da + jj] = v;
            if (jj < M)
                p.mr_x1[(size_t)ci * (da + M) + da + jj] = v;
        }
    }
}

// CC: 64-column pieces of a raw row (dkv <= 64 CC)
template <int MODE, int HT, int CC>
__global__ void __launch_bounds__(kModThreads) k_mr_attn(StepArgs a, ModDims d, ModParams p)
{
    int n_u = *a.qs.n_u;
    n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
    const int n_rows = n_u + (a.roles == 3 ? a.count : 0);
    int n_items = n_rows;
    if (MODE == kMrFirst) {
        n_items = *p.mr_n;
        const int most = 3 * a.count * (d.K + 1);
        n_items = n_items < 0 ? 0 : (n_items < most ? n_items : most);
    }
    const int ci = (int)blockIdx.x * kModWaves + wave_id();
    if (ci >= n_items)
        return;
    const int lane = lane_id();
    const int M = d.M, F = d.F, E = d.E, K = d.K, H = d.H, dh = d.dh, dkv = d.dkv;
    const int q = p.mr_itq[ci], j = p.mr_itj[ci];
    const bool hop = MODE == kMrFirst && j < K;
    const QuerySet &tab = hop ? p.hop2 : a.qs;
    const size_t trow = hop ? (size_t)q * K + j : (size_t)q;
    int cnt = tab.cnt[trow];
    cnt = cnt < 0 ? 0 : (cnt > K ? K : cnt);
    float *kvb = p.mr_kvb + (size_t)ci * H * dkv;
    if (cnt == 0) {
        for (int i = lane; i < H * dkv; i += kWave)
            kvb[i] = 0.0f;
        return;
    }
    const double t_q = a.qs.t[q];
    // lane k < cnt: slot k of the item's table
    int32_t my_nbr = -1, my_eid = -1, my_src = 0;
    double my_dt = 0.0;
    if (lane < cnt) {
        my_nbr = tab.nbr[trow * K + lane];
        my_eid = tab.eid[trow * K + lane];
        my_dt = t_q - tab.ts[trow * K + lane];
        if (MODE == kMrSecond)  // (second layer: item ci is query row x = ci; its slot's first-layer row)
            my_src = mr_item_of(p, (size_t)ci * (K + 1) + lane);
    }
    // kvr[u][c] = column c * 64 + lane of the raw row [row of the neighbour | e | Phi(t - t_k)] of slot k0 + u
    auto load_chunk = [&](float (&kvr)[kMrCH][CC], int k0) {
#pragma unroll
        for (int u = 0; u < kMrCH; ++u) {
            const int k = k0 + u < cnt ? k0 + u : cnt - 1;  // (uniform; the shuffles are executed by every lane)
            const int32_t nb = __shfl(my_nbr, k), ee = __shfl(my_eid, k), sr = __shfl(my_src, k);
            const int dlo = __shfl(__double2loint(my_dt), k), dhi = __shfl(__double2hiint(my_dt), k);
            const double dt = __hiloint2double(dhi, dlo);
#pragma unroll
            for (int c = 0; c < CC; ++c) {
                const int i = c * kWave + lane;
                float v = 0.0f;
                if (c * kWave < dkv && i < dkv) {  // (the first test is uniform)
                    if (i < M)
                        v = MODE == kMrSecond ? p.h1[(size_t)sr * E + i] : repr_elem(a, p, M, nb, i);
                    else if (i < M + F)
                        v = ee >= 0 ? a.edge_feat[(size_t)ee * F + (i - M)] : 0.0f;
                    else
                        v = time_enc(p.time_w_rev[i - M - F], p.time_b_rev[i - M - F], dt);
                }
                kvr[u][c] = v;
            }
        }
    };
    const float scale = 1.0f / sqrtf((float)dh);
    float sc = -INFINITY;  // lane h * K + k: score of slot k under head h
    {
        float qtr[HT][CC];
        const float *qt = p.mr_qt + (size_t)ci * H * dkv;
#pragma unroll
        for (int h = 0; h < HT; ++h)
#pragma unroll
            for (int c = 0; c < CC; ++c) {
                const int i = c * kWave + lane;
                qtr[h][c] = h < H && c * kWave < dkv && i < dkv ? qt[(size_t)h * dkv + i] : 0.0f;
            }
        for (int k0 = 0; k0 < cnt; k0 += kMrCH) {
            float kvr[kMrCH][CC];
            load_chunk(kvr, k0);
#pragma unroll
            for (int u = 0; u < kMrCH; ++u)
#pragma unroll
                for (int h = 0; h < HT; ++h)
                    if (h < H && k0 + u < cnt) {  // (uniform)
                        float part = 0.0f;
#pragma unroll
                        for (int c = 0; c < CC; ++c)
                            part += qtr[h][c] * kvr[u][c];
                        const float sum = wave_sum_uniform(part) * scale;
                        if (lane == h * K + k0 + u)
                            sc = sum;
                    }
        }
    }
    // softmax over the filled slots of the lane's head (every lane walks the head of lane % (H * K))
    const int hl = (lane % (H * K)) / K;
    float mx = -INFINITY;
    for (int k = 0; k < cnt; ++k)
        mx = fmaxf(mx, __shfl(sc, hl * K + k));
    const bool mine = lane < H * K && lane - hl * K < cnt;
    const float ex = mine ? expf(sc - mx) : 0.0f;
    float sum = 0.0f;
    for (int k = 0; k < cnt; ++k)
        sum += __shfl(ex, hl * K + k);
    const float pr = mine ? ex / sum : 0.0f;
    float acc[HT][CC];
#pragma unroll
    for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int c = 0; c < CC; ++c)
            acc[h][c] = 0.0f;
    for (int k0 = 0; k0 < cnt; k0 += kMrCH) {
        float kvr[kMrCH][CC];
        load_chunk(kvr, k0);
#pragma unroll
        for (int u = 0; u < kMrCH; ++u)
#pragma unroll
            for (int h = 0; h < HT; ++h)
                if (h < H && k0 + u < cnt) {  // (uniform: the shuffles are executed by every lane)
                    const float pk = __shfl(pr, h * K + k0 + u);
#pragma unroll
                    for (int c = 0; c < CC; ++c)
                        acc[h][c] += pk * kvr[u][c];
                }
    }
#pragma unroll
    for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int c = 0; c < CC; ++c)
            if (h < H && c * kWave + lane < dkv)
                kvb[(size_t)h * dkv + c * kWave + lane] = acc[h][c];
}

// ------------------------------------------------------------------------------------------
__device__ inline int mod_row_of_entry(const QuerySet &qs, int i, int entries)
{
    int s = qs.slot[i];
    if (s < 0) {
        const int rep = -s - 1;
        s = rep < entries ? qs.slot[rep] : 0;
    }
    return s >= 0 && s < entries ? s : 0;
}

// The last launch of a step: the preparation of the batch expected next (workgroups of 1024 threads, as
// winners_block and dedup_block want), the memory overwrite, and workgroups of sixteen events (embedding
// rows into LDS and out, both logits).
//   ROWS   the embeddings are the distinct rows of the query set (attention layers; the memory has been
//          overwritten by an earlier launch)
//   else   identity / time projection: emb = r_u(t), or (1 + (t - last_update[u]) w_p) * r_u(t), from the
//          state as this step leaves it -- the staged row and the winning event's time for a node
//          the step updates (the overwrite runs beside this), the memory row and last_update for the others
// First decoder layer on the matrix cores: the sixteen sources against the weights' first half, the
// sixteen destinations and sixteen negatives against the second, an output tile of sixteen columns per
// wavefront.  Bound by latency (ids -> keys -> rows, then the weights' first touch): 1000 events of 100
// columns in 7 us; a workgroup of eight events with the weights read once per event column took 24 us
// after a launch of 4 us for the rows.
constexpr int kFinEvents = 16, kFinThreads = 1024, kFinWaves = kFinThreads / kWave;

struct FinalParams {
    int n_side;    // workgroups that prepare the next batch (first: they take the longest)
    int n_commit;  // then: of the memory overwrite; the ones beyond take sixteen events each
    int applied;   // events of the applied batch (0: none)
    int ldr;       // LDS row stride of the embedding rows, bytes
    int32_t *clear;  // a counter that block 0 sets to 0, or NULL
};

template <bool ROWS>
__global__ void __launch_bounds__(kFinThreads) k_mod_final(StepArgs a, ModDims d, ModParams p, PackedWeights w, FinalParams f)
{
    using P = Prec<TIG_FP32>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int x = (int)blockIdx.x;
    if (x == 0 && threadIdx.x == 0) {
        if (f.clear)
            *f.clear = 0;
        if (a.rows_seen && f.applied > 0)
            a.rows_seen[1] = *a.n_win;  // (a hint for the host)
    }
    if (x < f.n_side) {
        if (a.sel.count > 0) {
            if (x == 0) {
                winners_block(a, a.sel, smem);
                return;
            }
            --x;
        }
        if (a.ded.count > 0 && x < a.ded.n_wgs)
            dedup_block(a, a.ded, d.K, x, smem);
        return;
    }
    x -= f.n_side;
    if (x < f.n_commit) {
        overwrite_memory(a, d.M, x * kFinWaves + wave_id(), f.n_commit * kFinWaves);
        return;
    }
    x -= f.n_commit;
    const int E = d.E, B = a.count, roles = a.roles;
    char *em = smem;                                              // [3 roles x 16 events] rows of ldr bytes
    int32_t *row_ref = (int32_t *)(em + (size_t)3 * kFinEvents * f.ldr);  // [48] row to read
    int32_t *row_node = row_ref + 3 * kFinEvents;                 // [48] node, or -1
    double *row_dt = (double *)(row_node + 3 * kFinEvents);       // [48] t - last_update
    float *part = (float *)(row_dt + 3 * kFinEvents);             // [output tiles][2][16]
    const int b0 = x * kFinEvents;
    const int lane = lane_id(), wave = wave_id();
    if ((int)threadIdx.x < 3 * kFinEvents) {
        const int role = (int)threadIdx.x / kFinEvents, b = b0 + (int)threadIdx.x % kFinEvents;
        int32_t ref = kRefNone, u = -1;
        double dt = 0.0;
        if (b < B && role < roles) {
            if (ROWS) {
                ref = role < 2 ? mod_row_of_entry(a.qs, 2 * b + role, 2 * B) : 2 * B + b;
            } else {
                const int64_t e = a.first_eid + b;
                u = role == 0 ? a.src[e] : (role == 1 ? a.dst[e] : a.neg[b]);
                const double t = a.ts[e];
                if (u < 0 || (int64_t)u >= a.num_nodes)
                    u = -1;
                if (u >= 0) {
                    const unsigned long long key = a.msg_count > 0 ? a.msg_key[u] : 0ull;
                    const double lu = a.lu[u];
                    ref = ref_of_key(ref_ctx(a), u, key);
                    dt = t - (ref >= 0 ? lu : a.ts[a.msg_first_eid + (~ref >> 1)]);
                }
            }
            if (role < 2 && a.out_is_winner && a.win_flags)
                a.out_is_winner[2 * b + role] = a.win_flags[2 * b + role];
        }
        row_ref[threadIdx.x] = ref;
        row_node[threadIdx.x] = u;
        row_dt[threadIdx.x] = dt;
    }
    __syncthreads();
    for (int j0 = 0; j0 < d.Ek; j0 += 2 * kWave) {  // (all of a wavefront's rows in flight together)
        float v[3][2], nf[3][2];
        int32_t node[3];
        double dt[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int32_t ref = __builtin_amdgcn_readfirstlane(row_ref[wave + i * kFinWaves]);
            node[i] = __builtin_amdgcn_readfirstlane(row_node[wave + i * kFinWaves]);
            dt[i] = row_dt[wave + i * kFinWaves];
            const float *row = ROWS ? a.emb_u + (size_t)(ref > 0 ? ref : 0) * E
                                    : (ref >= 0 ? a.mem + (size_t)ref * E : a.staging + (size_t)(ref == kRefNone ? 0 : ~ref) * E);
            const __amdgpu_buffer_rsrc_t rr =
                __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, ref == kRefNone ? 0 : E * 4, kBufferFlags);
            const bool has_nf = !ROWS && p.node_feat && node[i] >= 0;  // (uniform)
            const float *feat = has_nf ? p.node_feat + (size_t)node[i] * E : row;
            const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void *)feat, 0, has_nf ? E * 4 : 0, kBufferFlags);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                v[i][k] = buffer_load_f32(rr, (uint32_t)(j0 + lane + kWave * k) * 4u);
                nf[i][k] = ROWS ? 0.0f : buffer_load_f32(rf, (uint32_t)(j0 + lane + kWave * k) * 4u);
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int r = wave + i * kFinWaves, b = b0 + wave;  // (kFinWaves = kFinEvents: row i of the wavefront has role i)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int j = j0 + lane + kWave * k;
                float y = ROWS ? v[i][k] : v[i][k] + nf[i][k];
                if (!ROWS && d.emb == TIG_EMB_TIME_PROJECTION && node[i] >= 0 && j < E)
                    y = (float)((1.0 + dt[i] * (double)p.time_proj_w[j]) * (double)y);
                if (j < d.Ek)
                    P::store_a(em + (size_t)r * f.ldr, j, y);
                if (j < E && b < B && i < roles)
                    a.emb[((size_t)i * B + b) * E + j] = y;
            }
        }
    }
    __syncthreads();
    const int nE = d.Ep / 16, kb = d.Ek / P::KB;
    for (int nt = wave; nt < nE; nt += kFinWaves) {
        floatx4 src[1] = {floatx4{0, 0, 0, 0}}, oth[2] = {floatx4{0, 0, 0, 0}, floatx4{0, 0, 0, 0}};
        const int col = nt * 16 + (lane & 15);
        const float b1 = w.dec_b1[col], w2 = w.dec_w2[col];  // (0 in the padding)
        tile_gemm<TIG_FP32, 1, 4>(src, em, f.ldr, 0, w.dec_W, kb, 0, kb, nt);
        tile_gemm<TIG_FP32, 2, 4>(oth, em + (size_t)kFinEvents * f.ldr, f.ldr, 0, w.dec_W, kb, 0, kb, nE + nt);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float y = row_sum_all(w2 * fmaxf(src[0][v] + oth[q][v] + b1, 0.0f));
                if ((lane & 15) == 0)
                    part[(nt * 2 + q) * kFinEvents + 4 * (lane >> 4) + v] = y;
            }
    }
    __syncthreads();
    if ((int)threadIdx.x < 2 * kFinEvents) {
        const int q = (int)threadIdx.x / kFinEvents, ev = (int)threadIdx.x % kFinEvents;
        float sum = w.dec_b2[0];
        for (int nt = 0; nt < nE; ++nt)
            sum += part[(nt * 2 + q) * kFinEvents + ev];
        if (b0 + ev < B && q == 0)
            a.score_pos[b0 + ev] = sum;
        else if (b0 + ev < B && roles == 3)
            a.score_neg[b0 + ev] = sum;
    }
}

__global__ void k_mod_transpose(float *dst, const float *src, int rows, int cols)  // dst[c][r] = src[r][c]
{
    const size_t n = (size_t)rows * cols, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const size_t r = i / cols, c = i - r * cols;
        dst[c * rows + r] = src[i];
    }
}

__global__ void k_mod_revolutions(double *out, const float *in, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = (double)in[i] / 6.283185307179586476925286766559;
}

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

int msgsum_lds(const ModDims &d) { return kMsgSlots * (d.M + d.T + d.F) * 8 + 2 * kMsgSlots * 4; }

int final_lds(const ModDims &d)
{
    return 3 * kFinEvents * lds_row_bytes(d.Ek) + 3 * kFinEvents * 16 + d.Ep / 16 * 2 * kFinEvents * 4;
}

}  // namespace

constexpr int kModLdsLimit = 160 * 1024;

// The dimensions the second layer sees (embedding part): its input rows are E wide.
static Dims second_layer_dims(const Dims &d)
{
    Dims o = d;
    o.M = d.E;
    o.da = o.M + o.T;
    o.dh = o.da / o.H;
    o.dkv = o.M + o.F + o.T;
    o.dkvp = round_up(o.dkv, o.KB);
    o.Mq = round_up(o.M, o.KB);
    o.N1 = o.H * o.dkvp;
    o.K2 = o.N1 + o.Mq;
    return o;
}

bool two_layers_fused(const ModParams &p) { return p.fused_embed && p.layers == 2; }

// Layout of the attached workspace: [vectors | transposed matrices | raw staging of one matrix |
// node features].  Fills `p` when base != NULL.
static size_t mod_layout(const Dims &d, int agg, int upd, int emb, int layers, bool node_feat, int64_t num_nodes, char *base,
                         ModParams *p, float **raw_stage, float **nf_dst, void **pack2 = nullptr, void **fold2 = nullptr,
                         float **raw2 = nullptr)
{
    size_t off = 0;
    auto take = [&](size_t count, size_t elem) -> void * {
        void *q = base ? base + off : nullptr;
        off += align_up(count * elem);
        return q;
    };
    const size_t M = d.M, T = d.T, E = d.E;
    const bool attn = emb == TIG_EMB_ATTENTION;
    ModParams q = {};
    q.agg = agg;
    q.upd = upd;
    q.emb = emb;
    q.layers = layers == 2 ? 2 : 1;
    q.fused_embed = attn && !node_feat && q.layers == 1;
    q.time_w_rev = (const double *)take(T, 8);
    q.time_b_rev = (const double *)take(T, 8);
    size_t biggest = T;
    const Dims d2 = second_layer_dims(d);
    if (attn && !node_feat && q.layers == 2) {
        q.d2 = d2;
        q.mt[0] = layer_tiles(d, kModLdsLimit);
        q.mt[1] = layer_tiles(d2, kModLdsLimit);
        q.fused_embed = q.mt[0] > 0 && q.mt[1] > 0;
    }
    if (attn) {
        for (int l = 0; l < q.layers && !q.fused_embed; ++l) {
            // layer l reads rows of width in_w: the state width, then the first layer's width
            const size_t in_w = l == 0 ? M : E, a_w = in_w + T, kv_w = in_w + d.F + T;
            AttnLayer &A = q.L[l];
            A.b_Q = (const float *)take(a_w, 4);
            A.b_K = (const float *)take(a_w, 4);
            A.b_V = (const float *)take(a_w, 4);
            A.b_O = (const float *)take(a_w, 4);
            A.b_m1 = (const float *)take(E, 4);
            A.b_m2 = (const float *)take(E, 4);
            A.T_K = (const float *)take(kv_w * a_w, 4);
            A.N_Q = (const float *)take(a_w * a_w, 4);
            A.N_V = (const float *)take(a_w * kv_w, 4);
            A.N_O = (const float *)take(a_w * a_w, 4);
            A.N_m1 = (const float *)take(E * (a_w + in_w), 4);
            A.N_m2 = (const float *)take(E * E, 4);
            biggest = kv_w * a_w > biggest ? kv_w * a_w : biggest;
        }
        if (q.layers == 2 && q.fused_embed) {
            const size_t R = (size_t)3 * d.max_batch, items = R * (d.K + 1);
            QuerySet &it = q.it;
            it.node = it.self_ref = (int32_t *)take(items, 4);  // (no batch is applied any more: a reference is the node)
            it.t = (double *)take(items, 8);
            it.cnt = (int32_t *)take(items, 4);
            it.nbr = it.ref = (int32_t *)take(items * d.K, 4);
            it.eid = (int32_t *)take(items * d.K, 4);
            it.ts = (double *)take(items * d.K, 8);
            it.n_u = (int32_t *)take(64, 4);  // two counters: a step's, by its epoch's parity, and the next one's
            q.h1 = (float *)take(items * E, 4);
            q.mr_ci = (int32_t *)take(items, 4);
            q.ref2 = (int32_t *)take(R * d.K, 4);
            q.self2 = (int32_t *)take(R, 4);
            size_t slots = 1024;
            while (slots < 2 * items)
                slots *= 2;
            q.claim = (unsigned long long *)take(slots, 8);
            q.claim_mask = (uint32_t)(slots - 1);
            void *packed = take(packed_weights_bytes(d2), 1);
            void *fold = take(pack_scratch_bytes(d2), 1);
            // the layer's weights as given, each padded to 64 floats
            const size_t a2 = d2.da, raw = 2 * a2 * a2 + 2 * a2 * d2.dkv + E * (a2 + E) + 3 * E * E + 4 * a2 + 4 * E + 1 + 2 * T + 18 * 64;
            float *as_given = (float *)take(raw, 4);
            if (pack2)
                *pack2 = packed, *fold2 = fold, *raw2 = as_given;
            q.fused_embed = true;
        } else if (q.layers == 2) {
            const size_t R2 = (size_t)3 * d.max_batch * d.K;  // rows of the second-hop tables
            q.hop2.node = (int32_t *)take(R2, 4);
            q.hop2.t = (double *)take(R2, 8);
            q.hop2.cnt = (int32_t *)take(R2, 4);
            q.hop2.nbr = (int32_t *)take(R2 * d.K, 4);
            q.hop2.eid = (int32_t *)take(R2 * d.K, 4);
            q.hop2.ts = (double *)take(R2 * d.K, 8);
            q.h1 = (float *)take((size_t)3 * d.max_batch * (d.K + 1) * E, 4);
            q.mr_ci = (int32_t *)take((size_t)3 * d.max_batch * (d.K + 1), 4);
            size_t slots = 1024;
            while (slots < (size_t)2 * 3 * d.max_batch * (d.K + 1))
                slots *= 2;
            q.mr_tab = (uint32_t *)take(slots, 4);
            q.mr_tab_mask = (uint32_t)(slots - 1);
        }
        if (!q.fused_embed) {  // the items' matrices: widths of the wider layer
            const size_t items = (size_t)3 * d.max_batch * (q.layers == 2 ? d.K + 1 : 1);
            const size_t in_w = q.layers == 2 && E > M ? E : M, a_w = in_w + T, kv_w = in_w + d.F + T;
            q.mr_qin = (float *)take(items * a_w, 4);
            q.mr_qv = (float *)take(items * a_w, 4);
            q.mr_qt = (float *)take(items * d.H * kv_w, 4);
            q.mr_kvb = (float *)take(items * d.H * kv_w, 4);
            q.mr_o = (float *)take(items * a_w, 4);
            q.mr_x1 = (float *)take(items * (a_w + in_w), 4);
            q.mr_h1 = (float *)take(items * E, 4);
            q.mr_has = (int32_t *)take(items, 4);
            q.mr_itq = (int32_t *)take(items, 4);
            q.mr_itj = (int32_t *)take(items, 4);
            q.mr_n = (int32_t *)take(64, 4);
        }
    }
    if (emb == TIG_EMB_TIME_PROJECTION)
        q.time_proj_w = (const float *)take(M, 4);
    if (agg == TIG_AGG_MEAN) {
        q.acc = (double *)take((size_t)2 * d.max_batch * kAccCopies * (M + T + d.F), 8);
        q.acc_cnt = (int32_t *)take((size_t)2 * d.max_batch, 4);
        q.mean_msg = (float *)take((size_t)2 * d.max_batch * (M + T + d.F), 4);
    }
    float *stage = (float *)take(biggest, 4);
    float *nf = node_feat ? (float *)take((size_t)num_nodes * M, 4) : nullptr;
    q.node_feat = nf;
    if (p)
        *p = q;
    if (raw_stage)
        *raw_stage = stage;
    if (nf_dst)
        *nf_dst = nf;
    return off;
}

size_t modules_workspace_bytes(const Dims &d, const tig_modules &m, int64_t num_nodes)
{
    return mod_layout(d, m.aggregator, m.updater, m.embedding, m.num_layers, m.node_feat != nullptr, num_nodes, nullptr,
                      nullptr, nullptr, nullptr);
}

bool modules_supported(const Dims &d, const tig_modules &m)
{
    ModParams p = {};
    p.agg = m.aggregator;
    p.upd = m.updater;
    p.emb = m.embedding;
    const ModDims md = mod_dims(d, p);
    if (m.embedding != TIG_EMB_ATTENTION && d.E != d.M)
        return false;
    if (m.num_layers == 2 && (m.embedding != TIG_EMB_ATTENTION || (d.E + d.T) % d.H != 0 || d.K + 1 > kWave))
        return false;
    return d.prec == TIG_FP32 && msgsum_lds(md) <= 64 * 1024 && final_lds(md) <= 160 * 1024 && d.K <= kModThreads &&
           (m.embedding != TIG_EMB_ATTENTION || (d.H <= kMrMaxHeads && d.H * d.K <= kWave && d.dkv <= kMrCC * kWave &&
                                                  d.E + d.F + d.T <= kMrCC * kWave));
}

hipError_t modules_attach(const Dims &d, const tig_modules &m, const tig_weights &w, int64_t num_nodes, void *workspace,
                          ModParams *out, hipStream_t s)
{
    ModParams p;
    float *stage = nullptr, *nf = nullptr;
    void *packed2 = nullptr, *fold2 = nullptr;
    float *raw2 = nullptr;
    mod_layout(d, m.aggregator, m.updater, m.embedding, m.num_layers, m.node_feat != nullptr, num_nodes, (char *)workspace, &p,
               &stage, &nf, &packed2, &fold2, &raw2);
    const ModDims md = mod_dims(d, p);
    const int M = d.M, T = d.T, E = d.E;
    hipError_t e;
    auto vec = [&](const float *dst, const float *src, size_t n) -> hipError_t {
        return hipMemcpyAsync((void *)dst, src, 4 * n, hipMemcpyDefault, s);
    };
    // a matrix goes through the staging area (the source may be host memory) and is transposed from there
    auto mat = [&](const float *dst_t, const float *src, int rows, int cols) -> hipError_t {
        const size_t n = (size_t)rows * cols;
        hipError_t e2 = hipMemcpyAsync(stage, src, 4 * n, hipMemcpyDefault, s);
        if (e2 != hipSuccess)
            return e2;
        hipLaunchKernelGGL(k_mod_transpose, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (float *)dst_t, stage, rows, cols);
        return hipGetLastError();
    };
    auto rev = [&](const double *dst, const float *src) -> hipError_t {
        hipError_t e2 = hipMemcpyAsync(stage, src, 4 * (size_t)T, hipMemcpyDefault, s);
        if (e2 != hipSuccess)
            return e2;
        hipLaunchKernelGGL(k_mod_revolutions, dim3((T + 255) / 256), dim3(256), 0, s, (double *)dst, stage, T);
        return hipGetLastError();
    };
#define MOD_TRY(x)            \
    if ((e = (x)) != hipSuccess) \
        return e
    MOD_TRY(rev(p.time_w_rev, w.time_w));
    MOD_TRY(rev(p.time_b_rev, w.time_b));
    if (m.embedding == TIG_EMB_ATTENTION && !p.fused_embed) {
        // the second layer's matrices have the first layer's roles with E-wide input rows
        tig_layer_weights first = {};
        first.W_Q = w.W_Q, first.b_Q = w.b_Q, first.W_K = w.W_K, first.b_K = w.b_K, first.W_V = w.W_V, first.b_V = w.b_V;
        first.W_O = w.W_O, first.b_O = w.b_O, first.W_m1 = w.W_m1, first.b_m1 = w.b_m1, first.W_m2 = w.W_m2, first.b_m2 = w.b_m2;
        for (int l = 0; l < p.layers; ++l) {
            const tig_layer_weights &src = l == 0 ? first : *m.layer2;
            const AttnLayer &A = p.L[l];
            const int in_w = l == 0 ? M : E, a_w = in_w + T, kv_w = in_w + d.F + T;
            MOD_TRY(vec(A.b_Q, src.b_Q, a_w));
            MOD_TRY(vec(A.b_K, src.b_K, a_w));
            MOD_TRY(vec(A.b_V, src.b_V, a_w));
            MOD_TRY(vec(A.b_O, src.b_O, a_w));
            MOD_TRY(vec(A.b_m1, src.b_m1, E));
            MOD_TRY(vec(A.b_m2, src.b_m2, E));
            MOD_TRY(mat(A.T_K, src.W_K, a_w, kv_w));
            MOD_TRY(vec(A.N_Q, src.W_Q, (size_t)a_w * a_w));
            MOD_TRY(vec(A.N_V, src.W_V, (size_t)a_w * kv_w));
            MOD_TRY(vec(A.N_O, src.W_O, (size_t)a_w * a_w));
            MOD_TRY(vec(A.N_m1, src.W_m1, (size_t)E * (a_w + in_w)));
            MOD_TRY(vec(A.N_m2, src.W_m2, (size_t)E * E));
        }
    }
    if (m.embedding == TIG_EMB_TIME_PROJECTION)
        MOD_TRY(vec(p.time_proj_w, m.time_proj_w, M));
    if (nf)
        MOD_TRY(hipMemcpyAsync(nf, m.node_feat, 4 * (size_t)num_nodes * M, hipMemcpyDefault, s));
    if (p.acc) {
        MOD_TRY(launch_fill_zero(p.acc, (size_t)2 * d.max_batch * kAccCopies * (M + T + d.F) * 8, s));
        MOD_TRY(launch_fill_zero(p.acc_cnt, (size_t)2 * d.max_batch * 4, s));
    }
    MOD_TRY(hipFuncSetAttribute((const void *)k_mod_msgsum, hipFuncAttributeMaxDynamicSharedMemorySize, msgsum_lds(md)));
    const int fin = final_lds(md) > kOneLds ? final_lds(md) : kOneLds;
    MOD_TRY(hipFuncSetAttribute((const void *)k_mod_final<true>, hipFuncAttributeMaxDynamicSharedMemorySize, fin));
    MOD_TRY(hipFuncSetAttribute((const void *)k_mod_final<false>, hipFuncAttributeMaxDynamicSharedMemorySize, fin));
    if (two_layers_fused(p)) {
        // the second layer's prepared weights: its matrices and the decoder's as given, through a device copy
        float *at = raw2;
        auto dev = [&](const float *src, size_t n) -> const float * {
            float *dst = at;
            at += align_up(n, 64);
            if (e == hipSuccess)
                e = vec(dst, src, n);
            return dst;
        };
        const tig_layer_weights &l = *m.layer2;
        const size_t da2 = p.d2.da, dkv2 = p.d2.dkv, E_ = E;
        tig_weights w2 = {};
        e = hipSuccess;
        w2.W_Q = dev(l.W_Q, da2 * da2), w2.b_Q = dev(l.b_Q, da2), w2.W_K = dev(l.W_K, da2 * dkv2), w2.b_K = dev(l.b_K, da2);
        w2.W_V = dev(l.W_V, da2 * dkv2), w2.b_V = dev(l.b_V, da2), w2.W_O = dev(l.W_O, da2 * da2), w2.b_O = dev(l.b_O, da2);
        w2.W_m1 = dev(l.W_m1, E_ * (da2 + E_)), w2.b_m1 = dev(l.b_m1, E_), w2.W_m2 = dev(l.W_m2, E_ * E_), w2.b_m2 = dev(l.b_m2, E_);
        w2.W_d1 = dev(w.W_d1, 2 * E_ * E_), w2.b_d1 = dev(w.b_d1, E_), w2.w_d2 = dev(w.w_d2, E_), w2.b_d2 = dev(w.b_d2, 1);
        w2.time_w = dev(w.time_w, T), w2.time_b = dev(w.time_b, T);
        if (e != hipSuccess)
            return e;
        MOD_TRY(launch_fill_zero(packed2, packed_weights_bytes(p.d2), s));
        MOD_TRY(pack_weights(p.d2, w2, packed2, fold2, &p.pw2, s, kPackEmbed));
        MOD_TRY(clear_two_layers(p, s));
        MOD_TRY(prepare_embed_layer(d, p.mt[0]));
        MOD_TRY(prepare_embed_layer(p.d2, p.mt[1]));
    }
#undef MOD_TRY
    *out = p;
    return hipStreamSynchronize(s);
}

// Mean aggregator: the message columns of the applied batch's nodes into p.mean_msg, ahead of k_gru.
hipError_t launch_mean_messages(const Dims &d, const StepArgs &a, const ModParams &p, hipStream_t s)
{
    const ModDims md = mod_dims(d, p);
    hipLaunchKernelGGL(k_mod_msgsum, dim3((2 * a.msg_count + kMsgEntries - 1) / kMsgEntries), dim3(kMsgThreads), msgsum_lds(md), s,
                       a, md, p);
    hipLaunchKernelGGL(k_mod_mean, dim3((2 * a.msg_count + kModWaves - 1) / kModWaves), dim3(kModThreads), 0, s, a, md, p);
    return hipGetLastError();
}

// Everything of a step after the state update (k_gru) of a selection that the fused launches do not
// cover: memory overwrite, embedding, decoder, inspection outputs, the next batch's preparation.
hipError_t launch_modules(const Dims &d, const LaunchPlan &plan, const PackedWeights &pw, const StepArgs &a,
                          const ModParams &p, hipStream_t s, int *launches)
{
    const ModDims md = mod_dims(d, p);
    hipError_t e;
    const int B = a.count;
    FinalParams fp = {};
    const int n_events = (B + kFinEvents - 1) / kFinEvents;
    fp.ldr = lds_row_bytes(d.Ek);
    fp.applied = a.msg_count;
    const int side = fp.n_side = (a.sel.count > 0 ? 1 : 0) + (a.ded.count > 0 ? a.ded.n_wgs : 0);
    const int fin_lds = side > 0 && final_lds(md) < kOneLds ? kOneLds : final_lds(md);
    // about four winners per wavefront at the winner count recent steps had
    const int most = 2 * a.msg_count;
    const int wins = a.wins_est > 0 && a.wins_est < most ? a.wins_est : most;
    // from here on the attention layers read every state row from the memory table: nothing is "applied" any more
    StepArgs b = a;
    b.msg_count = 0;
    if (p.emb == TIG_EMB_ATTENTION) {
        const int n_commit = a.msg_count > 0 ? 64 : 0;
        if (n_commit > 0 && p.layers != 2) {
            hipLaunchKernelGGL(k_mod_commit, dim3(n_commit), dim3(kModThreads), 0, s, a, d.M);
            if ((e = hipGetLastError()) != hipSuccess)
                return e;
        }
        // one attention layer + merge MLP over all items of `mode`: item list and query rows, the layer's
        // products as contractions over the items, the attention core per item in between
        auto layer_pass = [&](const ModDims &ld, const AttnLayer &A, int mode) {
            const int items_max = 3 * B * (mode == kMrFirst ? d.K + 1 : 1);
            const RowCount rc = mode == kMrFirst ? RowCount{p.mr_n, 0, 1, items_max}
                                                 : RowCount{b.qs.n_u, b.roles == 3 ? B : 0, 1, items_max};
            const int da = ld.da, dh = ld.dh, dkv = ld.dkv, M_ = ld.M, E_ = ld.E, H = ld.H;
            const dim3 g_items((3 * B + kMrWaves - 1) / kMrWaves), g_attn((items_max + kModWaves - 1) / kModWaves);
            auto prod = [&](float *C, int ldc, const float *X, int lda, const float *W, int ldw, const float *bias, int N, int Kd) {
                RowGemm g = {};
                g.A = X, g.lda = lda, g.W = W, g.ldw = ldw, g.bias = bias, g.C = C, g.ldc = ldc, g.N = N, g.Kd = Kd, g.rc = rc;
                g.vecA = rowgemm_vec_ok(X, lda), g.vecW = rowgemm_vec_ok(W, ldw);
                return g;
            };
            if (mode == kMrSingle)
                hipLaunchKernelGGL(k_mr_items<kMrSingle>, g_items, dim3(kMrWaves * kWave), 0, s, b, ld, p);
            else if (mode == kMrFirst)
                hipLaunchKernelGGL(k_mr_items<kMrFirst>, g_items, dim3(kMrWaves * kWave), 0, s, b, ld, p);
            else
                hipLaunchKernelGGL(k_mr_items<kMrSecond>, g_items, dim3(kMrWaves * kWave), 0, s, b, ld, p);
            launch_rowgemm(prod(p.mr_qv, da, p.mr_qin, da, A.N_Q, da, A.b_Q, da, da), 1, s);
            {   // q~_h = W_K,h^T Qv_h, every head in one launch
                RowGemm g = prod(p.mr_qt, H * dkv, p.mr_qv, da, A.T_K, da, nullptr, dkv, dh);
                g.zA = dh, g.zW = dh, g.zC = dkv;
                g.vecA = g.vecA && dh % 4 == 0, g.vecW = g.vecW && dh % 4 == 0;
                launch_rowgemm(g, H, s);
            }
#define MR_ATTN(MODE)                                                                                             \
    do {                                                                                                          \
        if (H <= 2 && dkv <= 256)                                                                                 \
            hipLaunchKernelGGL((k_mr_attn<MODE, 2, 4>), g_attn, dim3(kModThreads), 0, s, b, ld, p);               \
        else if (H <= 2)                                                                                          \
            hipLaunchKernelGGL((k_mr_attn<MODE, 2, kMrCC>), g_attn, dim3(kModThreads), 0, s, b, ld, p);           \
        else                                                                                                      \
            hipLaunchKernelGGL((k_mr_attn<MODE, kMrMaxHeads, kMrCC>), g_attn, dim3(kModThreads), 0, s, b, ld, p); \
    } while (0)
            if (mode == kMrSingle)
                MR_ATTN(kMrSingle);
            else if (mode == kMrFirst)
                MR_ATTN(kMrFirst);
            else
                MR_ATTN(kMrSecond);
#undef MR_ATTN
            {   // o_h = W_V,h KVB_h + b_V,h
                RowGemm g = prod(p.mr_o, da, p.mr_kvb, H * dkv, A.N_V, dkv, A.b_V, dh, dkv);
                g.zA = dkv, g.zW = dh * dkv, g.zC = dh, g.zBias = dh;
                g.vecA = g.vecA && dkv % 4 == 0, g.vecW = g.vecW && (dh * dkv) % 4 == 0;
                launch_rowgemm(g, H, s);
            }
            {   // attn = W_O o + b_O into the head of the merge layer's input; the zero vector without neighbours
                RowGemm g = prod(p.mr_x1, da + M_, p.mr_o, da, A.N_O, da, A.b_O, da, da);
                g.rowmask = p.mr_has;
                launch_rowgemm(g, 1, s);
            }
            {
                RowGemm g = prod(p.mr_h1, E_, p.mr_x1, da + M_, A.N_m1, da + M_, A.b_m1, E_, da + M_);
                g.relu = 1;
                launch_rowgemm(g, 1, s);
            }
            if (mode == kMrFirst) {  // the first layer's rows, one per item
                launch_rowgemm(prod(p.h1, E_, p.mr_h1, E_, A.N_m2, E_, A.b_m2, E_, E_), 1, s);
            } else {                 // the embedding rows of the query set
                RowGemm g = prod(b.emb_u, E_, p.mr_h1, E_, A.N_m2, E_, A.b_m2, E_, E_);
                g.remap_nu = b.qs.n_u, g.remap_2b = 2 * B;
                launch_rowgemm(g, 1, s);
            }
        };
        if (p.layers == 2) {
            const ModDims md2 = second_layer_dims(md);
            if ((e = launch_fill_zero(p.mr_n, 4, s)) != hipSuccess ||
                (e = launch_fill_zero(p.mr_tab, ((size_t)p.mr_tab_mask + 1) * 4, s)) != hipSuccess)
                return e;
            hipLaunchKernelGGL(k_mod_hop2, dim3(3 * B + n_commit), dim3(kModThreads), 0, s, b, md, p, a.msg_count, n_commit);
            layer_pass(md, p.L[0], kMrFirst);
            layer_pass(md2, p.L[1], kMrSecond);
        } else {
            layer_pass(md, p.L[0], kMrSingle);
        }
        fp.clear = b.qs.n_u;  // (for the set's next preparation)
        hipLaunchKernelGGL(k_mod_final<true>, dim3(side + n_events), dim3(kFinThreads), fin_lds, s, b, md, p, pw, fp);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        *launches += p.layers == 2 ? 2 + 1 + 2 * 8 + 1 : (n_commit > 0 ? 1 : 0) + 8 + 1;
        if (wants_inspection(a)) {  // (the winner flags are out)
            StepArgs c = b;
            c.out_is_winner = nullptr;
            if (wants_inspection(c)) {
                *launches += 1;
                return launch_closing(d, plan, pw, c, GruAhead{}, s, false);
            }
        }
        return hipSuccess;
    }
    fp.n_commit = a.msg_count > 0 ? (wins + 4 * kFinWaves - 1) / (4 * kFinWaves) : 0;
    fp.n_commit = fp.n_commit > 16 ? 16 : fp.n_commit;
    hipLaunchKernelGGL(k_mod_final<false>, dim3(side + fp.n_commit + n_events), dim3(kFinThreads), fin_lds, s, a, md, p, pw, fp);
    *launches += 1;
    return hipGetLastError();
}

hipError_t clear_two_layers(const ModParams &p, hipStream_t s)
{
    const hipError_t e = launch_fill_zero(p.it.n_u, 64 * 4, s);
    return e != hipSuccess ? e : launch_fill_zero(p.claim, ((size_t)p.claim_mask + 1) * 8, s);
}

hipError_t launch_two_layers(const Dims &d, int num_cus, const PackedWeights &pw, const StepArgs &a, const ModParams &p, uint32_t epoch,
                             hipStream_t s, int *launches)
{
    const int B = a.count, K = d.K;
    const int rows = a.roles * B, cus = num_cus > 0 ? num_cus : 256;
    // a wavefront of the overwrite takes about four winners, at the winner count recent steps had
    const int most = 2 * a.msg_count;
    const int wins = a.wins_est > 0 && a.wins_est < most ? a.wins_est : most;
    const int n_commit = (wins + 4 * kTwoWaves - 1) / (4 * kTwoWaves);
    const int n_neg = a.roles == 3 ? (B + kTwoWaves - 1) / kTwoWaves : 0;
    if (n_commit + n_neg > 0)
        hipLaunchKernelGGL(k_two_negatives, dim3(n_commit + n_neg), dim3(kTwoThreads), 0, s, a, d.M, K, n_commit);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_two_claim, dim3((rows + kTwoWaves - 1) / kTwoWaves), dim3(kTwoThreads), 0, s, a, p, K, epoch);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    const int n_refs = cus / 4 > 0 ? cus / 4 : 1;
    hipLaunchKernelGGL(k_two_lookup, dim3(n_refs + 3 * cus), dim3(kTwoThreads), 0, s, a, p, K, epoch, n_refs);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    // the first layer reads the memory as overwritten; the next batch's preparation runs beside it
    const int items = rows * (K + 1);
    StepArgs one = a;
    one.msg_count = 0;
    one.qs = p.it;
    one.qs.n_u = p.it.n_u + (epoch & 1u);
    one.count = (items + 1) / 2;
    one.roles = 2;
    one.emb_u = p.h1;
    one.dec_a = one.dec_b = nullptr;
    LaunchPlan plan = {};
    plan.num_cus = cus;
    const int side = winners_in_one_launch(B) ? embed_spare_workgroups(d, plan, a.roles, B) : 0;
    if ((e = launch_embed_layer(d, p.mt[0], num_cus, side, pw, one, s)) != hipSuccess)
        return e;
    StepArgs two = a;
    two.msg_count = 0;
    two.mem = p.h1;
    two.num_nodes = items;
    two.qs.ref = p.ref2;
    two.qs.self_ref = p.self2;
    two.sel.count = two.ded.count = 0;
    *launches += 3 + (n_commit + n_neg > 0 ? 1 : 0);  // (beyond embedding and closing launch)
    return launch_embed_layer(p.d2, p.mt[1], num_cus, 0, p.pw2, two, s);
}

}  // namespace tig
