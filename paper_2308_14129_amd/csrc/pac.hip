// Epoch machinery of parallel training on partitions (paper Sec. II-C "Distributed Parallel
// Training", Alg. 2), device side.  gfx950 only.
//   sub-graph of a (combined) partition   E_k = {(i, j, t) in E | i, j in V_k}: an order-preserving
//       compaction of the event stream by a per-node membership test (count per workgroup, scan of
//       the counts, write), and the same compaction over the nodes for the local ids;
//   gather of the sub-graph's event arrays with endpoints relabelled to local ids;
//   memory synchronisation of the shared nodes across the partitions resident on this GPU.
#include <hip/hip_runtime.h>

#include "kernels_common.h"
#include "tig_internal.h"

namespace tig {

namespace {

constexpr int kCompThreads = 256;
constexpr int kCompPer = 8;                           // consecutive items per thread
constexpr int kCompBlock = kCompThreads * kCompPer;   // items per workgroup
constexpr int kScanThreads = 1024;

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// A node with replicas in more than one part resides in every part (node loop of Alg. 1).
__device__ inline bool is_member(uint64_t parts, uint64_t group)
{
    return __popcll(parts) > 1 ? group != 0ull : (parts & group) != 0ull;
}

__device__ inline bool inside(int32_t v, int64_t num_nodes) { return v >= 0 && (int64_t)v < num_nodes; }

// Consecutive items of a thread, tested together: all ids are there in two loads, and all their masks on their way before the first is
// looked at (one item after the other, two dependent reads each, 16 M events took 114 us; with the counts' scan in wavefronts and one wait for both
// compactions a sub-graph's rebuilding takes 2305 instead of 2408 us).
struct __attribute__((packed, aligned(4))) EightIds {
    int32_t v[kCompPer];
};

struct EventPred {
    const int32_t *src, *dst;
    const uint64_t *node_parts;
    int64_t num_nodes;
    uint64_t group;
    __device__ unsigned operator()(int64_t i0, int64_t n) const
    {
        EightIds s, d;
        if (i0 + kCompPer <= n) {
            s = *(const EightIds *)(src + i0);
            d = *(const EightIds *)(dst + i0);
        } else {
            for (int u = 0; u < kCompPer; ++u) {
                s.v[u] = i0 + u < n ? src[i0 + u] : -1;
                d.v[u] = i0 + u < n ? dst[i0 + u] : -1;
            }
        }
        uint64_t ms[kCompPer], md[kCompPer];
#pragma unroll
        for (int u = 0; u < kCompPer; ++u) {
            ms[u] = node_parts[inside(s.v[u], num_nodes) ? s.v[u] : 0];
            md[u] = node_parts[inside(d.v[u], num_nodes) ? d.v[u] : 0];
        }
        unsigned bits = 0;
#pragma unroll
        for (int u = 0; u < kCompPer; ++u)
            if (inside(s.v[u], num_nodes) && inside(d.v[u], num_nodes) && is_member(ms[u], group) && is_member(md[u], group))
                bits |= 1u << u;
        return bits;
    }
};

struct NodePred {
    const uint64_t *node_parts;
    uint64_t group;
    __device__ unsigned operator()(int64_t i0, int64_t n) const
    {
        unsigned bits = 0;
#pragma unroll
        for (int u = 0; u < kCompPer; ++u) {
            const uint64_t m = node_parts[i0 + u < n ? i0 + u : n - 1];
            if (i0 + u < n && is_member(m, group))
                bits |= 1u << u;
        }
        return bits;
    }
};

// The count pass also leaves the verdicts of a thread's 8 consecutive items as one byte, so the
// write pass neither re-reads the items nor repeats the test.
template <class Pred>
__global__ void __launch_bounds__(kCompThreads) k_comp_count(Pred pred, int64_t n, int32_t *block_counts,
                                                             uint8_t *keep_bits)
{
    __shared__ int total;
    if (threadIdx.x == 0)
        total = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kCompBlock + (int64_t)threadIdx.x * kCompPer;
    if (i0 < n) {
        const unsigned bits = pred(i0, n);
        keep_bits[i0 / kCompPer] = (uint8_t)bits;
        if (bits)
            atomicAdd(&total, __popc(bits));
    }
    __syncthreads();
    if (threadIdx.x == 0)
        block_counts[blockIdx.x] = total;
}

// exclusive scan of the workgroup counts (one workgroup; the counts of ~1e5 workgroups at most)
__global__ void __launch_bounds__(kScanThreads) k_comp_scan(const int32_t *block_counts, int64_t n_blocks,
                                                            int64_t *block_offsets, int64_t *total)
{
    __shared__ int64_t part[kScanThreads / kWave];
    const int64_t per = (n_blocks + kScanThreads - 1) / kScanThreads;
    const int64_t lo = (int64_t)threadIdx.x * per;
    const int64_t hi = lo + per < n_blocks ? lo + per : n_blocks;
    int64_t s = 0;
    for (int64_t b = lo; b < hi; ++b)
        s += block_counts[b];
    // (one thread adding up the threads' sums was 15 of 18 us)
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int64_t incl = s;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int64_t up = __shfl_up(incl, off, kWave);
        if (lane >= off)
            incl += up;
    }
    if (lane == kWave - 1)
        part[wave] = incl;
    __syncthreads();
    int64_t run = incl - s;
    for (int w = 0; w < wave; ++w)
        run += part[w];
    if (threadIdx.x == kScanThreads - 1)
        *total = run + s;
    for (int64_t b = lo; b < hi; ++b) {
        block_offsets[b] = run;
        run += block_counts[b];
    }
}

// kept items, in index order, to out[offset ..]; `rank_of` (may be NULL) gets every item's position or -1
__global__ void __launch_bounds__(kCompThreads) k_comp_write(const uint8_t *keep_bits, int64_t n,
                                                             const int64_t *block_offsets, int64_t capacity,
                                                             int32_t *out, int32_t *rank_of)
{
    __shared__ int wave_tot[kCompThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t i0 = (int64_t)blockIdx.x * kCompBlock + (int64_t)threadIdx.x * kCompPer;
    static_assert(kCompPer == 8, "one byte of verdicts per thread");
    const unsigned bits = i0 < n ? keep_bits[i0 / kCompPer] : 0u;
    bool keep[kCompPer];
#pragma unroll
    for (int u = 0; u < kCompPer; ++u)
        keep[u] = (bits >> u) & 1u;
    const int c = __popc(bits);
    int incl = c;  // inclusive scan over the wavefront
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off)
            incl += up;
    }
    if (lane == kWave - 1)
        wave_tot[wave] = incl;
    __syncthreads();
    int base = 0;
    for (int w2 = 0; w2 < wave; ++w2)
        base += wave_tot[w2];
    int64_t pos = block_offsets[blockIdx.x] + base + incl - c;
#pragma unroll
    for (int u = 0; u < kCompPer; ++u) {
        if (i0 + u < n) {
            if (keep[u]) {
                if (out && pos < capacity)
                    out[pos] = (int32_t)(i0 + u);
                if (rank_of)
                    rank_of[i0 + u] = (int32_t)pos;
                ++pos;
            } else if (rank_of) {
                rank_of[i0 + u] = -1;
            }
        }
    }
}

// Event arrays of a sub-graph, 256 events per workgroup and turn: a thread gathers one event's endpoints,
// time and local ids, then the workgroup copies the tile's feature rows as one flat range of V-float
// pieces (V = 4, 2 or 1, the widest that row length and addresses allow), four pieces in flight per
// thread.  Bound by memory: event ids ascend, so rows are read almost in stream order.  One wavefront per
// event, a lane per feature, left three lanes in four idle at 16 features and waited for a chain of three
// dependent reads per event: 12.7 M events of 16 features took 3.95 ms, now 0.5 ms (4.3 TB/s read + written).
constexpr int kGatherThreads = 256, kGatherTurn = 4;

template <int V>
__global__ void __launch_bounds__(kGatherThreads)
k_pac_gather(const int32_t *__restrict__ src, const int32_t *__restrict__ dst, const double *__restrict__ ts,
             const float *__restrict__ feat, int F, const int32_t *__restrict__ eid, int64_t n,
             const int32_t *__restrict__ local, int32_t *__restrict__ src_out, int32_t *__restrict__ dst_out,
             double *__restrict__ ts_out, float *__restrict__ feat_out)
{
    typedef float piece __attribute__((ext_vector_type(V)));
    __shared__ int32_t s_eid[kGatherThreads];
    const int tid = (int)threadIdx.x;
    const int pieces = F / V;  // of one row
    const int row_step = kGatherThreads / pieces, col_step = kGatherThreads - row_step * pieces;
    const int row_first = tid / pieces, col_first = tid - row_first * pieces;
    for (int64_t w0 = (int64_t)blockIdx.x * kGatherThreads; w0 < n; w0 += (int64_t)gridDim.x * kGatherThreads) {
        const int rows = n - w0 < kGatherThreads ? (int)(n - w0) : kGatherThreads;
        __syncthreads();  // (the previous turn's pieces have been read)
        if (tid < rows) {
            const int32_t e = eid[w0 + tid];
            s_eid[tid] = e;
            const int32_t u = src[e], v = dst[e];
            const double t = ts[e];
            src_out[w0 + tid] = local[u];
            dst_out[w0 + tid] = local[v];
            ts_out[w0 + tid] = t;
        }
        __syncthreads();
        const int total = rows * pieces;
        piece *const out = (piece *)(feat_out + w0 * F);
        int row = row_first, col = col_first;
        for (int idx = tid; idx < total; idx += kGatherThreads * kGatherTurn) {
            piece v[kGatherTurn];
#pragma unroll
            for (int u = 0; u < kGatherTurn; ++u) {
                const int r = row < rows ? row : rows - 1;  // (beyond the tile: a valid row, the piece is dropped)
                v[u] = ((const piece *)(feat + (int64_t)s_eid[r] * F))[col];
                row += row_step;
                col += col_step;
                if (col >= pieces) {
                    col -= pieces;
                    ++row;
                }
            }
#pragma unroll
            for (int u = 0; u < kGatherTurn; ++u)
                if (idx + u * kGatherThreads < total)
                    out[idx + u * kGatherThreads] = v[u];
        }
    }
}

__global__ void __launch_bounds__(256) k_sync_shared(SyncArgs a)
{
    const int64_t s = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (s >= a.n_shared)
        return;
    int32_t row[kMaxSyncParts];
    double t_star = 0.0;
    int win = -1;
    for (int k = 0; k < a.n_parts; ++k) {
        row[k] = a.ids[k][s];
        if (row[k] < 0 || (int64_t)row[k] >= a.num_nodes[k])
            return;  // not a row of that partition: the node is left alone everywhere
    }
    for (int k = 0; k < a.n_parts; ++k) {
        const double t = a.lu[k][row[k]];
        if (win < 0 || t > t_star) {  // the lowest partition among equal times
            t_star = t;
            win = k;
        }
    }
    for (int j = lane; j < a.M; j += kWave) {
        float v;
        if (a.mode == 0) {
            v = a.mem[win][(size_t)row[win] * a.M + j];
        } else {
            v = a.mem[0][(size_t)row[0] * a.M + j];
            for (int k = 1; k < a.n_parts; ++k)
                v += a.mem[k][(size_t)row[k] * a.M + j];
            v /= (float)a.n_parts;
        }
        for (int k = 0; k < a.n_parts; ++k)
            a.mem[k][(size_t)row[k] * a.M + j] = v;
    }
    if (lane == 0)
        for (int k = 0; k < a.n_parts; ++k)
            a.lu[k][row[k]] = t_star;
}

struct CompScratch {
    int32_t *block_counts;
    int64_t *block_offsets;
    int64_t *total;
    uint8_t *keep_bits;
    size_t bytes;
};

CompScratch comp_scratch(int64_t n_max, void *base)
{
    const int64_t nb = (n_max + kCompBlock - 1) / kCompBlock + 1;
    CompScratch c;
    char *p = (char *)base;
    size_t off = 0;
    c.block_counts = base ? (int32_t *)(p + off) : nullptr;
    off += align_up(4 * (size_t)nb);
    c.block_offsets = base ? (int64_t *)(p + off) : nullptr;
    off += align_up(8 * (size_t)nb);
    c.total = base ? (int64_t *)(p + off) : nullptr;
    off += 256;
    c.keep_bits = base ? (uint8_t *)(p + off) : nullptr;
    off += align_up((size_t)nb * kCompThreads);  // one byte per thread of every workgroup
    c.bytes = off;
    return c;
}

// (enqueues; *total is device memory)
template <class Pred>
hipError_t compact(Pred pred, int64_t n, const CompScratch &c, int64_t capacity, int32_t *out, int32_t *rank_of,
                   int64_t *total, hipStream_t s)
{
    const int64_t nb = (n + kCompBlock - 1) / kCompBlock;
    if (nb == 0)
        return launch_fill_zero(total, sizeof(int64_t), s);
    hipLaunchKernelGGL(k_comp_count<Pred>, dim3((unsigned)nb), dim3(kCompThreads), 0, s, pred, n, c.block_counts,
                       c.keep_bits);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_comp_scan, dim3(1), dim3(kScanThreads), 0, s, c.block_counts, nb, c.block_offsets, total);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_comp_write, dim3((unsigned)nb), dim3(kCompThreads), 0, s, c.keep_bits, n, c.block_offsets,
                       capacity, out, rank_of);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sync_shared(const SyncArgs &a, hipStream_t s)
{
    if (a.n_shared == 0)
        return hipSuccess;
    const int64_t blocks = (a.n_shared * kWave + 255) / 256;
    hipLaunchKernelGGL(k_sync_shared, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace tig

using namespace tig;

extern "C" {

size_t tig_pac_scratch_bytes(int64_t num_events, int64_t num_nodes)
{
    if (num_events < 0 || num_nodes < 1)
        return 0;
    return comp_scratch(num_events > num_nodes ? num_events : num_nodes, nullptr).bytes;
}

int tig_pac_subgraph(const int32_t *src, const int32_t *dst, int64_t num_events, const uint64_t *node_parts,
                     int64_t num_nodes, uint64_t group, int32_t *eid_out, int32_t *local_out, int64_t *counts_out,
                     void *scratch, size_t scratch_bytes, void *hip_stream)
{
    if (num_events < 0 || num_events > 0x7FFFFFFF || num_nodes < 1 || num_nodes > 0x7FFFFFFF || !node_parts ||
        !local_out || !counts_out || !scratch || ((uintptr_t)scratch & 255) ||
        (num_events > 0 && (!src || !dst || !eid_out)))
        return TIG_EINVAL;
    if (scratch_bytes < tig_pac_scratch_bytes(num_events, num_nodes))
        return TIG_ENOSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    const CompScratch c = comp_scratch(num_events > num_nodes ? num_events : num_nodes, scratch);
    hipError_t e = compact(EventPred{src, dst, node_parts, num_nodes, group}, num_events, c, num_events, eid_out,
                           nullptr, c.total, s);
    if (e != hipSuccess)
        return fail_global("tig_pac_subgraph: event compaction", e);
    e = compact(NodePred{node_parts, group}, num_nodes, c, 0, nullptr, local_out, c.total + 1, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(counts_out, c.total, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    return e == hipSuccess ? TIG_OK : fail_global("tig_pac_subgraph: node compaction", e);
}

int tig_pac_gather(const int32_t *src, const int32_t *dst, const double *ts, const float *edge_feat, int32_t feat_dim,
                   const int32_t *eid, int64_t n, const int32_t *local, int32_t *src_out, int32_t *dst_out,
                   double *ts_out, float *feat_out, void *hip_stream)
{
    if (n < 0 || feat_dim < 1 || (n > 0 && (!src || !dst || !ts || !edge_feat || !eid || !local || !src_out ||
                                             !dst_out || !ts_out || !feat_out)))
        return TIG_EINVAL;
    if (n == 0)
        return TIG_OK;
    int64_t blocks = (n + kGatherThreads - 1) / kGatherThreads;
    blocks = blocks > (1 << 20) ? (1 << 20) : blocks;  // (the kernel strides over the events)
    const auto aligned = [&](int V) {  // rows of both arrays start on V-float boundaries
        return feat_dim % V == 0 && (((uintptr_t)edge_feat | (uintptr_t)feat_out) & (4 * (uintptr_t)V - 1)) == 0;
    };
#define PAC_GATHER(V)                                                                                                \
    hipLaunchKernelGGL(k_pac_gather<V>, dim3((unsigned)blocks), dim3(kGatherThreads), 0, (hipStream_t)hip_stream, src, dst, \
                       ts, edge_feat, (int)feat_dim, eid, n, local, src_out, dst_out, ts_out, feat_out)
    if (aligned(4))
        PAC_GATHER(4);
    else if (aligned(2))
        PAC_GATHER(2);
    else
        PAC_GATHER(1);
#undef PAC_GATHER
    return hipGetLastError() == hipSuccess ? TIG_OK : TIG_EHIP;
}

int tig_pac_combine(const int32_t *order, int32_t num_parts, int32_t num_groups, uint64_t *group_masks_out)
{
    if (!order || !group_masks_out || num_parts < 1 || num_parts > 64 || num_groups < 1 || num_parts % num_groups)
        return TIG_EINVAL;
    uint64_t seen = 0;
    for (int i = 0; i < num_parts; ++i) {
        if (order[i] < 0 || order[i] >= num_parts || ((seen >> order[i]) & 1u))
            return TIG_EINVAL;  // not a permutation of the parts
        seen |= 1ull << order[i];
    }
    const int w = num_parts / num_groups;
    for (int g = 0; g < num_groups; ++g) {
        uint64_t m = 0;
        for (int i = g * w; i < (g + 1) * w; ++i)
            m |= 1ull << order[i];
        group_masks_out[g] = m;
    }
    return TIG_OK;
}

}  // extern "C"
