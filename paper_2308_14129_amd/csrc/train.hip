// Training step (paper Sec. II-C: the decoder's edge probabilities "provide the self-supervised
// signals for training"; Alg. 2: "Training and compute loss", "Backward and Optimize"): layout, weight
// gradients, update, host side.  gfx950 only, fp32.
//
// The forward pass is the embedding kernel of an ordinary step (embed_tile.h, TRAIN), which runs on
// FOLDED weights (pack.hip): q~ = A1 s_u + a1, h1 = relu(P kvbar + R s_u + c), decoder halves from h1.  The
// backward pass (train_back.hip) goes through the same foldings, so every product over rows runs over
// the distinct queries and the narrow state rows; the gradients of the folded matrices are then taken apart
// into those of the master weights by small products over the weights alone.  One step, on the context's
// stream:
//   k_gru, k_embed<TRAIN>                  state update (gates kept), forward pass
//   k_tr_decode, k_tr_back, k_tr_gru_back  loss and backward pass (train_back.hip)
//   k_tr_wgrad    every contraction over rows, dW = D^T X, in one launch
//   k_tr_small    products over weights: gradients of folded matrices -> of the masters (two launches), and
//                 after the update the foldings themselves, straight into the layouts of the kernels (two)
//   k_tr_update   memory overwrite, sum of the loss terms, SGD on the fp32 masters
// (The step in direct form, layer by layer over all rows, was 43 launches with the weight gradients on a second
// stream: 350 us at 200 events of 172 columns, most of it the host launching; 450 us at 4000 events.)
#include <hip/hip_runtime.h>

#include <cstring>

#include "train.h"
#include "winners.h"

namespace tig {

namespace {

// ------------------------------------------------------------------------------------------
// acc[i][j] += sum over k < n of a(k, i) b(k, j): the block of row 16 MI x 32 whose row MI r + i and column 2 c + j are
// row r and column c of the 16 x 16 block (i, j), so that a lane's operand values are adjacent in memory and come in
// one load each.  a(k, i) = A[k * sa + ao + i], b(k, j) = B[k * sb + bo + j]; A, B, sa, sb are uniform and ao, bo this
// lane's first elements for k = lane / 16: every load of a step is a scalar address plus an offset that does not
// change, and the vector unit has nothing to do beside the products (with an address per lane and 4-byte loads the
// instructions for these were what bound these kernels).  Rows and columns beyond a matrix may read any element
// in bounds; they reach results that nobody stores.
// sum[i]: the sums of a's values, per lane.  Products are summed sixteen rows at a time and those sums added up (in one
// chain over a wavefront's 150 rows gradients were up to 1.6 times as far from 64 bits as in the step in direct form;
// in parts, with the column sums in double, they are below it everywhere).
template <int N>
struct __attribute__((packed, aligned(4))) Floats {
    float v[N];
};

// A and B are read through buffer descriptors whose extent is the n rows: a k beyond the end reads zeros.  Where a width is no
// multiple of a lane's two or four columns, its load of the last row reaches beyond the extent: such loads are checked dword
// by dword, so that the columns inside arrive and those outside, which are no columns of the matrix, read zero; nothing behind
// an array is read.  Two groups of kU k-steps take turns, one on its way while the other is multiplied; where the rows end with the
// first group, nothing more is asked for (three groups of loads for the few rows of 16 events: k_tr_wgrad 5.7 instead of 5.1 us).
template <int MI, int kU>  // kU: k-steps of 4 whose loads are issued together
__device__ inline void multiply(const float *A, const float *B, int sa, int sb, int ao, int bo, int n, floatx4 (&acc)[MI][2],
                                double (&sum)[MI])
{
    constexpr int kPart = 4;  // k-steps whose products are summed on their own
    using VA = Floats<MI>;
    using VB = Floats<2>;
    struct Group {
        VA a[kU];
        VB b[kU];
    };
    uint32_t at_a[kU], at_b[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        at_a[u] = 4u * (uint32_t)(ao + 4 * u * sa);
        at_b[u] = 4u * (uint32_t)(bo + 4 * u * sb);
    }
    auto request = [&](Group &q, int k) {
        const int left = n - k < 4 * kU ? (n > k ? n - k : 0) : 4 * kU;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc((void *)(A + (size_t)k * sa), 0, left * sa * 4, kBufferFlags);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc((void *)(B + (size_t)k * sb), 0, left * sb * 4, kBufferFlags);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if constexpr (MI == 4)
                q.a[u] = __builtin_bit_cast(VA, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)at_a[u], 0, 0));
            else
                q.a[u] = __builtin_bit_cast(VA, __builtin_amdgcn_raw_buffer_load_b64(ra, (int)at_a[u], 0, 0));
            q.b[u] = __builtin_bit_cast(VB, __builtin_amdgcn_raw_buffer_load_b64(rb, (int)at_b[u], 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);  // (sunk to their use otherwise)
    };
    auto products = [&](const Group &q, int k) {
#pragma unroll
        for (int u0 = 0; u0 < kU; u0 += kPart) {
            if (k + 4 * u0 >= n)  // (uniform)
                break;
            floatx4 part[MI][2] = {};
            float ps[MI] = {};
#pragma unroll
            for (int u = u0; u < u0 + kPart; ++u)
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    ps[i] += q.a[u].v[i];
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        part[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(q.a[u].v[i], q.b[u].v[j], part[i][j], 0, 0, 0);
                }
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                sum[i] += (double)ps[i];
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] += part[i][j];
            }
        }
    };
    Group x, y;
    request(x, 0);
#pragma unroll 1
    for (int k = 0; k < n; k += 8 * kU) {
        request(y, k + 4 * kU);
        products(x, k);
        if (k + 4 * kU >= n)  // (uniform)
            break;
        request(x, k + 8 * kU);
        products(y, k + 4 * kU);
    }
}

// ------------------------------------------------------------------------------------------
// C[Mo x No] = A[rows x Mo]^T B[rows x No] for several products in one launch: a workgroup of four
// wavefronts takes one block of 16 * MI x 32 of one C over all of its rows (no atomics, no cleared targets), the
// wavefronts split the rows and add their blocks up in LDS.  csum: also the column sums of A (the bias gradient
// that goes with a weight gradient), by the workgroups of the first block column.
// The wavefronts' and XCDs' parts are added in double.
// Bound by the matrix units of the compute unit a block lies on: blocks of 64 rows where these fill the chip, of 32
// otherwise.  SPLIT: many rows and few blocks -- every XCD takes an eighth of the rows (and reads
// each of them once: with the blocks spread over the XCDs, every L2 fetched nearly all of the operands, 200 MB in
// 52 us at 5700 rows of 100 columns) and leaves its part of every block for k_tr_wgrad_sum.
constexpr int kWgWaves = 4;
constexpr int kPartFloats = 64 * 32 + 64;       // a partial block of 64 x 32 and its column sums
constexpr size_t kSplitRows = 2048;             // the sum costs about 5 us: what 2048 rows take one compute unit
constexpr int kSplitTiles = 512;
struct WgradJob {
    const float *A, *B;
    float *C, *C_hi, *csum;  // column n >= split of C goes to C_hi[m]
    int lda, ldb, ldc, Mo, No, split;
    int winners;             // rows: 0 = queries (two ranges of the query set's rows), 1 = applied winners
};
constexpr int kMaxWgrad = 8;
// first[i]: first workgroup of job i (beyond the last job: past every workgroup).  The array of them leads the
// arguments: a workgroup finds its job with one scalar load, not with a chain of loads from job to job.
struct WgradJobs {
    int first[kMaxWgrad];
    float *part;
    WgradJob j[kMaxWgrad];
};

template <int N>
__device__ inline int job_of_block(const int (&first)[N], int block)
{
    int ji = 0;
#pragma unroll
    for (int i = 1; i < N; ++i)
        ji += block >= first[i] ? 1 : 0;
    return ji;
}

constexpr int kXcds = 8;

// element e of a block: register v of lane l of the 16 x 16 block (i, j)
template <int MI>
__device__ inline void store_block(const WgradJob &q, int m0, int n0, int e, float x)
{
    const int l = e & (kWave - 1), v = (e / kWave) & 3, j = (e / (4 * kWave)) & 1, i = e / (8 * kWave);
    const int mm = m0 + MI * (4 * (l >> 4) + v) + i, nn = n0 + 2 * (l & 15) + j;
    if (mm < q.Mo && nn < q.No) {
        if (nn < q.split)
            q.C[(size_t)mm * q.ldc + nn] = x;
        else
            q.C_hi[mm] = x;
    }
}

// Registers: two groups of loads and 64 products' sums.  SPLIT launches more workgroups than fit at once: three wavefronts per
// SIMD, groups of four (135 registers); the others two, groups of eight (186).  With one group, asked for when the one before was used
// up, a training step took 212 us instead of 208.5 at 4000 events of 100 columns and 169 instead of 168 at 200 of 172.
template <int MI, bool SPLIT>
__global__ void __launch_bounds__(kWgWaves *kWave, SPLIT ? 3 : 2) k_tr_wgrad(StepArgs a, WgradJobs jobs)
{
    __shared__ float red[kWgWaves][MI * 512];
    __shared__ double reds[kWgWaves][MI][kWave];
    const int block = SPLIT ? (int)blockIdx.x / kXcds : (int)blockIdx.x;
    const int ji = job_of_block(jobs.first, block);
    const WgradJob q = jobs.j[ji];
    const int w = wave_id_uniform(), lane = lane_id();
    const int tiles_n = (q.No + 31) / 32, tile = block - jobs.first[ji];
    const int m0 = (tile / tiles_n) * (16 * MI), n0 = (tile % tiles_n) * 32;
    int rows, gap_at = 0x7fffffff, gap = 0;  // row r lies at r, or behind a gap
    if (q.winners) {
        rows = a.msg_count > 0 ? *a.n_win : 0;
        rows = rows < 2 * a.msg_count ? rows : 2 * a.msg_count;
    } else {
        int n_u = *a.qs.n_u;
        n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
        rows = n_u + a.count;
        gap_at = n_u;
        gap = 2 * a.count - n_u;
    }
    rows = __builtin_amdgcn_readfirstlane(rows);
    gap_at = __builtin_amdgcn_readfirstlane(gap_at);
    gap = __builtin_amdgcn_readfirstlane(gap);
    constexpr int kParts = SPLIT ? kWgWaves * kXcds : kWgWaves;
    const int sub = ((rows + kParts - 1) / kParts + 3) / 4 * 4;
    const int k_lo = (SPLIT ? (int)blockIdx.x % kXcds * kWgWaves + w : w) * sub, k_hi = k_lo + sub < rows ? k_lo + sub : rows;
    const bool with_sum = q.csum != nullptr && n0 == 0;  // (uniform over the workgroup)
    floatx4 acc[MI][2];
    double sum[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        sum[i] = 0.0;
        acc[i][0] = acc[i][1] = floatx4{0, 0, 0, 0};
    }
    const int c = lane & 15, g = lane >> 4, mm = m0 + MI * c, nn = n0 + 2 * c;
    const int ao = g * q.lda + (mm < q.Mo ? mm : 0), bo = g * q.ldb + (nn < q.No ? nn : 0);
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {  // before and behind the gap
        const int lo = part ? (k_lo > gap_at ? k_lo : gap_at) : k_lo, hi = part ? k_hi : (k_hi < gap_at ? k_hi : gap_at);
        if (lo >= hi)
            continue;
        const size_t row = (size_t)lo + (part ? gap : 0);
        const float *A = q.A + row * q.lda, *B = q.B + row * q.ldb;
        multiply<MI, SPLIT ? 4 : 8>(A, B, q.lda, q.ldb, ao, bo, hi - lo, acc, sum);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[w][((i * 2 + j) * 4 + v) * kWave + lane] = acc[i][j][v];
        reds[w][i][lane] = sum[i];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < MI * 512; e += kWgWaves * kWave) {
        double sum_e = 0.0;
#pragma unroll
        for (int ww = 0; ww < kWgWaves; ++ww)
            sum_e += (double)red[ww][e];
        const float x = (float)sum_e;
        if (SPLIT)
            jobs.part[(size_t)blockIdx.x * kPartFloats + e] = x;
        else
            store_block<MI>(q, m0, n0, e, x);
    }
    if (with_sum && threadIdx.x < 16 * MI && m0 + (int)threadIdx.x < q.Mo) {
        double sum_m = 0.0;
#pragma unroll
        for (int ww = 0; ww < kWgWaves; ++ww)
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
                sum_m += reds[ww][threadIdx.x % MI][16 * gg + threadIdx.x / MI];
        const float x = (float)sum_m;
        if (SPLIT)
            jobs.part[(size_t)blockIdx.x * kPartFloats + 512 * MI + threadIdx.x] = x;
        else
            q.csum[m0 + threadIdx.x] = x;
    }
}

// The parts of a block from k_tr_wgrad<4, true>, added up.
__global__ void __launch_bounds__(512) k_tr_wgrad_sum(WgradJobs jobs)
{
    const int block = (int)blockIdx.x, ji = job_of_block(jobs.first, block);
    const WgradJob q = jobs.j[ji];
    const int tiles_n = (q.No + 31) / 32, tile = block - jobs.first[ji];
    const int m0 = (tile / tiles_n) * 64, n0 = (tile % tiles_n) * 32;
    const float *part = jobs.part + (size_t)block * kXcds * kPartFloats;
    const int e = 4 * threadIdx.x;
    float4 p[kXcds];
#pragma unroll
    for (int x = 0; x < kXcds; ++x)
        p[x] = *(const float4 *)(part + (size_t)x * kPartFloats + e);
    double sum[4] = {};
#pragma unroll
    for (int x = 0; x < kXcds; ++x)
        sum[0] += (double)p[x].x, sum[1] += (double)p[x].y, sum[2] += (double)p[x].z, sum[3] += (double)p[x].w;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        store_block<4>(q, m0, n0, e + v, (float)sum[v]);
    if (q.csum && n0 == 0 && threadIdx.x < 64 && m0 + (int)threadIdx.x < q.Mo) {
        double x = 0.0;
#pragma unroll
        for (int i = 0; i < kXcds; ++i)
            x += (double)part[(size_t)i * kPartFloats + 2048 + threadIdx.x];
        q.csum[m0 + threadIdx.x] = (float)x;
    }
}

// ------------------------------------------------------------------------------------------
// Products over the weights: C[m][n] = alpha sum_k A(m, k) B(k, n) (+ u[m] v[n]) (+ add[m]), a workgroup of eight
// wavefronts per 32 x 32 block of a C, the wavefronts split k.  Results go to a plain matrix and / or, as
// element (r, c) of a prepared operand or of its transpose, straight into the kernels' lane-ordered layout.
// Beside them plain copies into such layouts.  Latency: a launch is one round of loads and two LDS steps.
// Products and sums in double: the foldings are what every row of the next step is multiplied by, and a gradient passes
// through two of these products (in single precision, 35 instead of 43 us for the four launches at 172 state columns and 25
// instead of 29 at 100, gradients came out up to 1.7 times as far from 64 bits).
//
// Columns of a key / value row have two orders: the model's [s | e | Phi] and the kernels' [Phi | s | e];
// a job names, per operand index, which way it is mapped.
enum IndexMap { kAsIs = 0, kToModel = 1, kToKernel = 2 };
struct SmallJob {
    const float *A, *B, *u, *v, *add;
    float *C, *C_hi;           // column n >= split goes to C_hi[m]
    float *pk, *pkT;           // element (pk_r + m, pk_c + n) of pk, element (pkT_r + n, pkT_c + m) of pkT
    int ars, acs, brs, bcs, us, vs, ldc, split;
    int m, n, k;
    double alpha, u_scale;
    int pk_kbs, pk_r, pk_c, pkT_kbs, pkT_r, pkT_c;  // (no narrow fields: those are not scalar loads)
    int am, bn;                // IndexMap of A's row, of B's column (and of v)
    int k_at;                  // A's k is k + a_k[0] and B's k + b_k[0] below this k, + [1] from it on
    int a_k[2], b_k[2];
};
constexpr int kMaxSmall = 17;
struct CopyJob {  // dst element (r, c), r < rows, c < cols, = src[r * rs + c * cs] (+ src2[r * rs2 + c] for c < cols2)
    float *dst;
    const float *src, *src2;
    int kbs;      // k-blocks per output tile of a prepared operand, 0: a plain vector (c only)
    int r0, c0, rows, cols, rs, cs, rs2, cols2;
};
constexpr int kMaxCopy = 22;
struct SmallJobs {
    int first[kMaxSmall];  // as in WgradJobs
    SmallJob j[kMaxSmall];
    int n, tiles;  // jobs, their workgroups
    int T, MF;     // key / value row: time encoding, state + features
};
// A thread takes four columns of a row (16 bytes of a prepared operand); first[i]: first workgroup of job i, as in WgradJobs.
struct CopyJobs {
    int first[kMaxCopy];
    CopyJob j[kMaxCopy];
    int n, blocks;
    const float *time_w, *time_b;
    double *time_w_rev, *time_b_rev;
    int T;
};

__device__ inline size_t packed_index(int r, int c, int kbs)  // fp32 operand, 16-deep k-blocks
{
    return ((((size_t)(r >> 4) * kbs + (c >> 4)) * kWave) + (size_t)((c & 15) >> 2) * 16 + (r & 15)) * 4 + (c & 3);
}

// element e of a block of k_tr_small
__device__ inline void element(int e, int m0, int n0, int &mm, int &nn)
{
    const int l = e & (kWave - 1), v = (e / kWave) & 3, j = (e / (4 * kWave)) & 1, i = e / (8 * kWave);
    mm = m0 + 16 * i + 4 * v + (l >> 4);  // (products of doubles: a lane's rows are four apart)
    nn = n0 + 16 * j + (l & 15);
}

__device__ inline int map_index(int i, int how, int T, int MF)
{
    if (how == kToModel)
        return i < T ? MF + i : i - T;
    if (how == kToKernel)
        return i < MF ? T + i : i - MF;
    return i;
}

constexpr int kSmallThreads = 512, kSmallWaves = kSmallThreads / kWave, kSmallPer = 1024 / kSmallThreads;

__device__ void copy_block(const CopyJobs &jobs, int block);

struct __attribute__((packed, aligned(4))) Four {
    float v[4];
};

// The wavefront's part k_lo <= k < k_hi of a block.  Of sixteen k, lane group g takes the four from 4 g on, so that an
// operand with consecutive k in memory (AV, BV: and with k in fours) is one load of 16 bytes where it would be four
// of 4 bytes in sixteen cache lines each, which bound these products (172 x 272 x 272: 9 us).
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <bool AV, bool BV>
__device__ inline void small_multiply(const SmallJob &q, const int (&ao)[2], const int (&bo)[2], int k_lo, int k_hi,
                                      doublex4 (&acc)[2][2])
{
    constexpr int kS = 2;  // steps of 16 k whose loads are issued together
    const int g = lane_id() >> 4;
#pragma unroll 1
    for (int k = k_lo; k < k_hi; k += 16 * kS) {
        Four av[kS][2], bv[kS][2];
#pragma unroll
        for (int u = 0; u < kS; ++u) {
            const int k4 = k + 16 * u + 4 * g;
            const auto index = [&](int kk, const int (&of)[2], int stride) {
                const int kc = kk < k_hi ? kk : k_lo;
                return (kc + (kc >= q.k_at ? of[1] : of[0])) * stride;
            };
            if (AV) {
                const int ka = index(k4, q.a_k, 1);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    av[u][i] = *(const Four *)(q.A + (unsigned)(ao[i] + ka));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int ka = index(k4 + e, q.a_k, q.acs);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        av[u][i].v[e] = q.A[(unsigned)(ao[i] + ka)];
                }
            }
            if (BV) {
                const int kb = index(k4, q.b_k, 1);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    bv[u][i] = *(const Four *)(q.B + (unsigned)(bo[i] + kb));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int kb = index(k4 + e, q.b_k, q.brs);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        bv[u][i].v[e] = q.B[(unsigned)(bo[i] + kb)];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kS; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool on = k + 16 * u + 4 * g + e < k_hi;
                double x[2], y[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    x[i] = (double)(on ? av[u][i].v[e] : 0.0f);
                    y[i] = (double)(on ? bv[u][i].v[e] : 0.0f);
                }
                if (k + 16 * u + e < k_hi)  // (uniform)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], acc[i][j], 0, 0, 0);
            }
    }
}

// The workgroups beyond the products' take the copies.
__global__ void __launch_bounds__(kSmallThreads, 4) k_tr_small(SmallJobs jobs, CopyJobs copies)
{
    __shared__ float red[kSmallWaves][1024];
    if ((int)blockIdx.x >= jobs.tiles) {
        copy_block(copies, (int)blockIdx.x - jobs.tiles);
        return;
    }
    const int block = (int)blockIdx.x;
    const int ji = job_of_block(jobs.first, block);
    const SmallJob q = jobs.j[ji];
    const int w = wave_id_uniform(), lane = lane_id(), c = lane & 15;
    const int T = jobs.T, MF = jobs.MF;
    const int tiles_n = (q.n + 31) / 32, tile = block - jobs.first[ji];
    const int m0 = (tile / tiles_n) * 32, n0 = (tile % tiles_n) * 32;
    int ao[2], bo[2];
    doublex4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        acc[i][0] = acc[i][1] = doublex4{0, 0, 0, 0};
        const int mm = m0 + 16 * i + c, nn = n0 + 16 * i + c;
        ao[i] = map_index(mm < q.m ? mm : 0, q.am, T, MF) * q.ars;
        bo[i] = map_index(nn < q.n ? nn : 0, q.bn, T, MF) * q.bcs;
    }
    // (values of the epilogue, on their way meanwhile)
    float eu[kSmallPer], ev[kSmallPer], ea[kSmallPer];
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        int mm, nn;
        element(threadIdx.x + r * kSmallThreads, m0, n0, mm, nn);
        mm = mm < q.m ? mm : 0;
        nn = nn < q.n ? nn : 0;
        eu[r] = (q.u ? q.u : q.A)[q.u ? mm * q.us : 0];
        ev[r] = (q.u ? q.v : q.A)[q.u ? map_index(nn, q.bn, T, MF) * q.vs : 0];
        ea[r] = (q.add ? q.add : q.A)[q.add ? mm : 0];
    }
    const int per = ((q.k + kSmallWaves - 1) / kSmallWaves + 3) / 4 * 4;
    const int k_lo = w * per, k_hi = k_lo + per < q.k ? k_lo + per : q.k;
    const bool wide = q.k % 4 == 0 && (q.k_at >= q.k || q.k_at % 4 == 0);
    if (wide && q.acs == 1 && q.brs == 1)
        small_multiply<true, true>(q, ao, bo, k_lo, k_hi, acc);
    else if (wide && q.acs == 1)
        small_multiply<true, false>(q, ao, bo, k_lo, k_hi, acc);
    else
        small_multiply<false, false>(q, ao, bo, k_lo, k_hi, acc);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[w][((i * 2 + j) * 4 + v) * kWave + lane] = (float)acc[i][j][v];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const int e = threadIdx.x + r * kSmallThreads;
        int mm, nn;
        element(e, m0, n0, mm, nn);
        if (mm >= q.m || nn >= q.n)
            continue;
        double total = 0.0;
#pragma unroll
        for (int ww = 0; ww < kSmallWaves; ++ww)
            total += (double)red[ww][e];
        total *= q.alpha;
        if (q.u)
            total += q.u_scale * (double)eu[r] * (double)ev[r];
        if (q.add)
            total += (double)ea[r];
        const float sum = (float)total;
        if (q.C) {
            if (nn < q.split)
                q.C[(size_t)mm * q.ldc + nn] = sum;
            else
                q.C_hi[mm] = sum;
        }
        if (q.pk)
            q.pk[packed_index(q.pk_r + mm, q.pk_c + nn, q.pk_kbs)] = sum;
        if (q.pkT)
            q.pkT[packed_index(q.pkT_r + nn, q.pkT_c + mm, q.pkT_kbs)] = sum;
    }
}

// One group of four per thread, all of its loads together (a fixed number of workgroups per matrix, element by element, was a chain of
// seven loads and scattered stores for the widest ones; with the order of the unfolding's jobs, a training step of 200 events of 172
// columns 168 -> 164.5 us, of 4000 of 100 as before).
__device__ void copy_block(const CopyJobs &jobs, int block)
{
    const int y = job_of_block(jobs.first, block);
    if (y >= jobs.n) {  // the time encoding's parameters in revolutions
        const int i = (block - jobs.first[y]) * kSmallThreads + (int)threadIdx.x;
        if (i < 2 * jobs.T) {
            const bool phase = i >= jobs.T;
            const int j = phase ? i - jobs.T : i;
            (phase ? jobs.time_b_rev : jobs.time_w_rev)[j] = (double)(phase ? jobs.time_b : jobs.time_w)[j] / 6.283185307179586476925286766559;
        }
        return;
    }
    const CopyJob q = jobs.j[y];
    const int groups = (q.cols + 3) / 4, i = (block - jobs.first[y]) * kSmallThreads + (int)threadIdx.x;
    if (i >= q.rows * groups)
        return;
    // (the faster index of the source varies fastest)
    const int r = q.cs == 1 ? i / groups : i % q.rows, c = 4 * (q.cs == 1 ? i % groups : i / q.rows);
    floatx4 v, v2 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ce = c + e < q.cols ? c + e : c;
        v[e] = q.src[(size_t)r * q.rs + (size_t)ce * q.cs];
        if (q.src2)
            v2[e] = q.src2[(size_t)r * q.rs2 + (ce < q.cols2 ? ce : 0)];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] += q.src2 && c + e < q.cols2 ? v2[e] : 0.0f;
    float *const dst = q.dst + (q.kbs ? packed_index(q.r0 + r, q.c0 + c, q.kbs) : (size_t)c);
    if (q.kbs && c + 4 <= q.cols) {
        *(floatx4 *)dst = v;  // (c0 is a multiple of four: one lane's share of an operand)
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < q.cols)
                dst[e] = v[e];
    }
}

// The memory overwrite (the GRU's backward read the memory as the step found it), the sum of the loss
// terms (one workgroup, if loss_out != NULL), and -- the workgroups beyond -- the gradients that were
// collected outside the gradient buffer (time encoding, second decoder layer) and the SGD update, which share
// nothing; the step's query set is empty again afterwards (its counter is cleared for the set's next
// preparation).
struct UpdateJob {
    int M, T, E, commit_blocks;
    const float *terms;
    int n_terms;
    float *loss_out;
    float *P, *G;
    size_t n_params;
    float lr;
    double *TACC;
    float *WACC;
    float *phi0;         // [T] Phi(0), which the query row carries
    const float *dphi0;  // [T] its gradient
};

__global__ void __launch_bounds__(256) k_tr_update(StepArgs a, UpdateJob u)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *a.qs.n_u = 0;
    if ((int)blockIdx.x < u.commit_blocks) {
        overwrite_memory(a, u.M, (int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave),
                         (int)(u.commit_blocks * (blockDim.x / kWave)));
        return;
    }
    const int loss_blocks = u.loss_out ? 1 : 0;
    if ((int)blockIdx.x >= u.commit_blocks + loss_blocks) {
        const size_t i = (size_t)((int)blockIdx.x - u.commit_blocks - loss_blocks) * blockDim.x + threadIdx.x;
        if (i >= u.n_params)
            return;
        float g = u.G[i];
        const size_t T = (size_t)u.T, tail = u.n_params - (size_t)(u.E + 1);
        if (i < 2 * T) {  // the first two arrays: frequencies, phases (Phi(0)_j = cos(b_j))
            double sum = 0.0, part[kSumCopies];
#pragma unroll
            for (int c = 0; c < kSumCopies; ++c)
                part[c] = u.TACC[c * 2 * T + i];
#pragma unroll
            for (int c = 0; c < kSumCopies; ++c) {
                sum += part[c];
                u.TACC[c * 2 * T + i] = 0.0;
            }
            g = (float)(sum - (i >= T ? sin((double)u.P[i]) * (double)u.dphi0[i - T] : 0.0));
            u.G[i] = g;
        } else if (i >= tail) {  // the last two: w_d2, b_d2
            const size_t n = (size_t)(u.E + 1);
            float part[kSumCopies];
            double sum = 0.0;
#pragma unroll
            for (int c = 0; c < kSumCopies; ++c)
                part[c] = u.WACC[c * n + i - tail];
#pragma unroll
            for (int c = 0; c < kSumCopies; ++c) {
                sum += (double)part[c];
                u.WACC[c * n + i - tail] = 0.0f;
            }
            g = (float)sum;
            u.G[i] = g;
        }
        float x = u.P[i];
        if (u.lr != 0.0f) {
            x -= u.lr * g;
            u.P[i] = x;
        }
        if (i >= T && i < 2 * T)
            u.phi0[i - T] = (float)cos((double)x);
        return;
    }
    __shared__ float red[256];
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int i = threadIdx.x; i < u.n_terms; i += 4 * 256)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            acc[v] += i + v * 256 < u.n_terms ? u.terms[i + v * 256] : 0.0f;
    red[threadIdx.x] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st)
            red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        *u.loss_out = red[0];
}

__global__ void k_tr_phi0(const float *time_b, float *phi0, int T)
{
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < T)
        phi0[i] = (float)cos((double)time_b[i]);
}

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

}  // namespace

// ---- host side ---------------------------------------------------------------------------------

struct TrainLayout {
    float *P, *G;       // master weights and their gradients, the fields of tig_weights in order
    size_t n_params;
    tig_weights w, g;   // pointers into P and G
    TrainArrays t;
    // folded intermediates and the gradients of the folded matrices
    float *Gm;          // [E x da]   W_m1[:, :da] W_O
    float *cQ, *cO;     // [da], [E]  W_Q[:, M:] Phi(0) + b_Q;  b_m1 + W_m1[:, :da] b_O
    float *gP, *gA1;    // [E x N1], [N1 x (M + 1)] (last column: gradient of a1)
    float *gG, *gc;     // [E x da], [E] (gradient of the bias c of rows with neighbours)
    float *phi0, *dphi0;  // [T] Phi(0) = cos(time_b), and its gradient
    float *part;        // partial blocks of the contractions whose rows are split over workgroups
    void *pack_scratch;
    size_t zero_lo, zero_hi;  // byte range that train_attach clears
    size_t bytes;
};

static int wgrad_job_tiles(int Mo, int No, int mi) { return ((Mo + 16 * mi - 1) / (16 * mi)) * ((No + 31) / 32); }

// blocks of all contractions over rows (launch_train's list)
static int wgrad_tiles(const Dims &d, int mi)
{
    const int M = d.M, E = d.E;
    return wgrad_job_tiles(d.N1, M + 1, mi) + wgrad_job_tiles(E, d.N1, mi) + wgrad_job_tiles(E, M + 1, mi) +
           3 * wgrad_job_tiles(E, E, mi) + wgrad_job_tiles(3 * M, d.Dmsg, mi) + wgrad_job_tiles(3 * M, M, mi);
}

static TrainLayout train_layout(const Dims &d, void *base)
{
    TrainLayout L;
    memset(&L, 0, sizeof(L));
    char *p = (char *)base;
    size_t off = 0;
    auto take = [&](size_t n_floats) -> float * {
        float *q = base ? (float *)(p + off) : nullptr;
        off += align_up(4 * (n_floats ? n_floats : 1));
        return q;
    };
    const size_t M = d.M, T = d.T, E = d.E, da = d.da, dkv = d.dkv, D = d.Dmsg, N1 = d.N1;
    const size_t B = d.max_batch, R = 3 * B, U = 2 * B;
    const size_t counts[22] = {T, T, 3 * M * D, 3 * M, 3 * M * M, 3 * M, da * da, da, da * dkv, da, da * dkv, da,
                               da * da, da, E * (da + M), E, E * E, E, E * 2 * E, E, E, 1};
    size_t n = 0;
    for (size_t c : counts)
        n += c;
    L.n_params = n;
    L.P = take(n);
    L.zero_lo = off;
    L.G = take(n);
    TrainArrays &t = L.t;
    t.TACC = (double *)take(kSumCopies * 2 * 2 * T);
    t.WACC = take(kSumCopies * (E + 1));
    t.Wd1T = take((size_t)d.Ep * 2 * d.Ek);
    t.Wm2T = take((size_t)d.Ep * d.Ek);
    t.PRT = take((size_t)d.K2 * d.Ek);
    t.A1T = take((size_t)d.Mq * N1);
    t.WiT = take((T + 15) / 16 * 16 * ((3 * M + 15) / 16 * 16));
    L.zero_hi = off;
    const float **wf[22] = {&L.w.time_w, &L.w.time_b, &L.w.W_i, &L.w.b_i, &L.w.W_h, &L.w.b_h, &L.w.W_Q, &L.w.b_Q,
                            &L.w.W_K, &L.w.b_K, &L.w.W_V, &L.w.b_V, &L.w.W_O, &L.w.b_O, &L.w.W_m1, &L.w.b_m1,
                            &L.w.W_m2, &L.w.b_m2, &L.w.W_d1, &L.w.b_d1, &L.w.w_d2, &L.w.b_d2};
    const float **gf[22] = {&L.g.time_w, &L.g.time_b, &L.g.W_i, &L.g.b_i, &L.g.W_h, &L.g.b_h, &L.g.W_Q, &L.g.b_Q,
                            &L.g.W_K, &L.g.b_K, &L.g.W_V, &L.g.b_V, &L.g.W_O, &L.g.b_O, &L.g.W_m1, &L.g.b_m1,
                            &L.g.W_m2, &L.g.b_m2, &L.g.W_d1, &L.g.b_d1, &L.g.w_d2, &L.g.b_d2};
    size_t o = 0;
    for (int i = 0; i < 22; ++i) {
        *wf[i] = L.P ? L.P + o : nullptr;
        *gf[i] = L.G ? L.G + o : nullptr;
        o += counts[i];
    }
    L.w.struct_size = L.g.struct_size = sizeof(tig_weights);
    t.S = take(R * (M + 1));
    t.QT = take(R * N1);
    t.KVB = take(R * N1);
    t.H1 = take(R * E);
    t.DA = take(R * E);
    t.DB = take(R * E);
    t.DEMB = take(R * E);
    t.DZ1 = take(R * E);
    t.DQT = take(R * N1);
    t.LOSS = take(U);
    t.MSG = take(U * D);
    t.GATES = take(U * 4 * M);
    t.DGI = take(U * 3 * M);
    t.DGH = take(U * 3 * M);
    t.D_STAG = take(U * M);
    L.Gm = take(E * da);
    L.cQ = take(da);
    L.cO = take(E);
    L.gP = take(E * N1);
    L.gA1 = take(N1 * (M + 1));
    L.gG = take(E * da);
    L.gc = take(E);
    L.phi0 = take(T);
    L.dphi0 = take(T);
    L.part = R >= kSplitRows && wgrad_tiles(d, 4) <= kSplitTiles ? take((size_t)wgrad_tiles(d, 4) * kXcds * kPartFloats) : nullptr;
    L.pack_scratch = base ? p + off : nullptr;
    off += align_up(pack_scratch_bytes(d));
    L.bytes = off;
    return L;
}

size_t train_workspace_bytes(const Dims &d) { return train_layout(d, nullptr).bytes; }

hipError_t prepare_train(const Dims &d, const LaunchPlan &plan)
{
    const hipError_t e = prepare_embed(d, plan, true);
    return e == hipSuccess ? prepare_train_back(d) : e;
}

bool train_supported(const Dims &d)
{
    return d.prec == TIG_FP32 && d.M <= 255 && d.H * d.K <= kWave && d.K < kWave && train_back_fits(d);
}

namespace {

struct SmallList {
    SmallJobs jobs = {};
    explicit SmallList(const Dims &d)
    {
        jobs.T = d.T;
        jobs.MF = d.M + d.F;
        for (int &f : jobs.first)
            f = 0x7fffffff;
    }
    // C[m x n] = alpha A B, A(i, k) = A[i * ars + k * acs], B(k, j) = B[k * brs + j * bcs]
    SmallJob &add(float *C, int ldc, const float *A, int ars, int acs, const float *B, int brs, int bcs, int m, int n, int k,
                  double alpha = 1.0)
    {
        jobs.first[jobs.n] = jobs.tiles;
        SmallJob &q = jobs.j[jobs.n++];
        q = SmallJob{};
        q.A = A, q.B = B, q.C = C;
        q.ars = ars, q.acs = acs, q.brs = brs, q.bcs = bcs, q.ldc = ldc, q.split = n;
        q.m = m, q.n = n, q.k = k, q.alpha = alpha, q.u_scale = 1.0, q.k_at = k;
        jobs.tiles += ((m + 31) / 32) * ((n + 31) / 32);
        return q;
    }
    // k in the kernels' column order, the operand's in the model's: [Phi | s | e] -> [s | e | Phi]
    void k_to_model(SmallJob &q, int (&of)[2]) const
    {
        q.k_at = jobs.T, of[0] = jobs.MF, of[1] = -jobs.T;
    }
    hipError_t launch(hipStream_t s, const CopyJobs *copies = nullptr) const
    {
        const CopyJobs none = {};
        const int blocks = jobs.tiles + (copies ? copies->blocks : 0);
        hipLaunchKernelGGL(k_tr_small, dim3(blocks), dim3(kSmallThreads), 0, s, jobs, copies ? *copies : none);
        return hipGetLastError();
    }
};

// The kernels' weights from the masters: foldings (in two stages) and copies, forward and transposed.
hipError_t fold_weights(const Dims &d, const TrainLayout &L, const PackedWeights &pw, hipStream_t s)
{
    const tig_weights &w = L.w;
    const TrainArrays &t = L.t;
    const int M = d.M, T = d.T, F = d.F, E = d.E, H = d.H, da = d.da, dh = d.dh, dkv = d.dkv, D = d.Dmsg;
    const int kbM = d.Mq / 16, kbN = d.N1 / 16, kbE = d.Ek / 16, kbK2 = d.K2 / 16, ld_m1 = da + M;
    const double scale = 1.0 / sqrt((double)dh);
    SmallList one(d), two(d);
    one.add(L.Gm, da, w.W_m1, ld_m1, 1, w.W_O, da, 1, E, da, da);
    for (int h = 0; h < H; ++h) {  // A1_h = scale W_K,h^T W_Q,h[:, :M]; rows in the kernels' column order
        SmallJob &q = one.add(nullptr, 0, w.W_K + (size_t)h * dh * dkv, 1, dkv, w.W_Q + (size_t)h * dh * da, da, 1, dkv, M, dh, scale);
        q.am = kToModel;
        q.pk = (float *)pw.emb_A1, q.pk_kbs = kbM, q.pk_r = (h * d.dkvp);
        q.pkT = t.A1T, q.pkT_kbs = kbN, q.pkT_c = (h * d.dkvp);
    }
    {   // cQ = W_Q[:, M:] Phi(0) + b_Q
        SmallJob &q = one.add(L.cQ, 1, w.W_Q + M, da, 1, L.phi0, 1, 1, da, 1, T);
        q.add = w.b_Q;
    }
    one.add(L.cO, 1, w.W_m1, ld_m1, 1, w.b_O, 1, 1, E, 1, da).add = w.b_m1;
    for (int half = 0; half < 2; ++half) {  // decoder halves through merge layer 2
        SmallJob &q = one.add(nullptr, 0, w.W_d1 + half * E, 2 * E, 1, w.W_m2, E, 1, E, E, E);
        q.pk = (float *)pw.dec_WF, q.pk_kbs = kbE, q.pk_r = (half * d.Ep);
    }
    {   // b_d1 + (W_d1[:, :E] + W_d1[:, E:]) b_m2
        SmallJob &q = one.add((float *)pw.dec_b1f, 1, w.W_d1, 2 * E, 1, w.b_m2, 1, 1, E, 1, 2 * E);
        q.k_at = E, q.b_k[1] = -E;
        q.add = w.b_d1;
    }
    for (int h = 0; h < H; ++h) {
        // P_h = G_h W_V,h; columns in the kernels' order
        SmallJob &q = two.add(nullptr, 0, L.Gm + h * dh, da, 1, w.W_V + (size_t)h * dh * dkv, dkv, 1, E, dkv, dh);
        q.bn = kToModel;
        q.pk = (float *)pw.emb_PR, q.pk_kbs = kbK2, q.pk_c = (h * d.dkvp);
        q.pkT = t.PRT, q.pkT_kbs = kbE, q.pkT_r = (h * d.dkvp);
        // a1_h = scale W_K,h^T cQ_h
        two.add((float *)pw.emb_a1 + h * d.dkvp, 1, w.W_K + (size_t)h * dh * dkv, 1, dkv, L.cQ + h * dh, 1, 1, dkv, 1, dh, scale).am =
            kToModel;
    }
    two.add((float *)pw.emb_c, 1, L.Gm, da, 1, w.b_V, 1, 1, E, 1, da).add = L.cO;
    CopyJobs c = {};
    auto mat = [&](const void *dst, int kbs, int r0, int c0, int rows, int cols, const float *src, int rs, int cs,
                   const float *src2 = nullptr, int rs2 = 0, int cols2 = 0) {
        c.j[c.n++] = CopyJob{(float *)dst, src, src2, kbs, r0, c0, rows, cols, rs, cs, rs2, cols2};
    };
    auto vec = [&](const float *dst, const float *src, int n, const float *src2 = nullptr) {
        c.j[c.n++] = CopyJob{(float *)dst, src, src2, 0, 0, 0, 1, n, 0, 1, 0, src2 ? n : 0};
    };
    // state update: the r and z gates' hidden weights folded onto the s_self columns (see k_pack_gru)
    const int kbG = d.Kg / 16, kbH = d.Khn / 16, kb3 = (3 * M + 15) / 16;
    mat(pw.gru_Wr, kbG, 0, 0, M, D, w.W_i, D, 1, w.W_h, M, M);
    mat(pw.gru_Wz, kbG, 0, 0, M, D, w.W_i + (size_t)M * D, D, 1, w.W_h + (size_t)M * M, M, M);
    mat(pw.gru_Win, kbG, 0, 0, M, D, w.W_i + (size_t)2 * M * D, D, 1);
    mat(pw.gru_Whn, kbH, 0, 0, M, M, w.W_h + (size_t)2 * M * M, M, 1);
    vec(pw.gru_br, w.b_i, M, w.b_h);
    vec(pw.gru_bz, w.b_i + M, M, w.b_h + M);
    vec(pw.gru_bin, w.b_i + 2 * M, M);
    vec(pw.gru_bhn, w.b_h + 2 * M, M);
    mat(t.WiT, kb3, 0, 0, T, 3 * M, w.W_i + 2 * M, 1, D);
    // merge layers and decoder
    mat(pw.emb_PR, kbK2, 0, d.N1, E, M, w.W_m1 + da, ld_m1, 1);
    mat(t.PRT, kbE, d.N1, 0, M, E, w.W_m1 + da, 1, ld_m1);
    mat(pw.emb_Wm2, kbE, 0, 0, E, E, w.W_m2, E, 1);
    mat(t.Wm2T, kbE, 0, 0, E, E, w.W_m2, 1, E);
    mat(t.Wd1T, 2 * kbE, 0, 0, E, E, w.W_d1, 1, 2 * E);
    mat(t.Wd1T, 2 * kbE, 0, d.Ek, E, E, w.W_d1 + E, 1, 2 * E);
    vec(pw.emb_c0, w.b_m1, E);
    vec(pw.emb_bm2, w.b_m2, E);
    vec(pw.dec_w2, w.w_d2, E);
    vec(pw.dec_b2, w.b_d2, 1);
    c.time_w = w.time_w, c.time_b = w.time_b, c.T = T;
    c.time_w_rev = (double *)pw.time_w_rev, c.time_b_rev = (double *)pw.time_b_rev;
    for (int i = 0; i < kMaxCopy; ++i) {
        c.first[i] = i <= c.n ? c.blocks : 0x7fffffff;
        const int items = i < c.n ? c.j[i].rows * ((c.j[i].cols + 3) / 4) : (i == c.n ? 2 * T : 0);
        c.blocks += (items + kSmallThreads - 1) / kSmallThreads;
    }
    (void)F;
    const hipError_t e = one.launch(s, &c);
    return e == hipSuccess ? two.launch(s) : e;
}

// Gradients of the masters from the contractions over rows and the gradients of the folded matrices.
hipError_t unfold_gradients(const Dims &d, const TrainLayout &L, hipStream_t s)
{
    const tig_weights &w = L.w, &g = L.g;
    const int M = d.M, T = d.T, E = d.E, H = d.H, da = d.da, dh = d.dh, dkv = d.dkv, ld_m1 = da + M, ldA = M + 1;
    const double scale = 1.0 / sqrt((double)dh);
    SmallList one(d), two(d);
    // Two workgroups fit a compute unit, and the first 256 spread over all: those of the longest sums (over key / value columns)
    // in the middle, so that the ones that share a unit with another, the first and the last, have the shorter sums.
    for (int h = 0; h < H; ++h) {   // dW_K,h = scale (W_Q,h[:, :M] dA1_h^T + cQ_h (x) da1_h)
        const float *WQ = w.W_Q + (size_t)h * dh * da, *gA = L.gA1 + (size_t)h * d.dkvp * ldA;
        SmallJob &q = one.add((float *)g.W_K + (size_t)h * dh * dkv, dkv, WQ, da, 1, gA, 1, ldA, dh, dkv, M, scale);
        q.bn = kToKernel;
        q.u = L.cQ + h * dh, q.us = 1, q.v = gA + M, q.vs = ldA;
        q.u_scale = scale;
    }
    for (int h = 0; h < H; ++h) {
        const float *WK = w.W_K + (size_t)h * dh * dkv, *WV = w.W_V + (size_t)h * dh * dkv;
        const float *gP = L.gP + h * d.dkvp, *gA = L.gA1 + (size_t)h * d.dkvp * ldA;
        {   // dG_h = dP_h W_V,h^T + dc (x) b_V,h
            SmallJob &q = one.add(L.gG + h * dh, da, gP, d.N1, 1, WV, 1, dkv, E, dh, dkv);
            one.k_to_model(q, q.b_k);
            q.u = L.gc, q.us = 1, q.v = w.b_V + h * dh, q.vs = 1;
        }
        {   // [dW_Q,h[:, :M] | d cQ_h] = scale W_K,h [dA1_h | da1_h];  d b_Q = d cQ
            SmallJob &q = one.add((float *)g.W_Q + (size_t)h * dh * da, da, WK, dkv, 1, gA, ldA, 1, dh, M + 1, dkv, scale);
            one.k_to_model(q, q.a_k);
            q.split = M, q.C_hi = (float *)g.b_Q + h * dh;
        }
    }
    for (int h = 0; h < H; ++h)     // dW_V,h = G_h^T dP_h
        one.add((float *)g.W_V + (size_t)h * dh * dkv, dkv, L.Gm + h * dh, 1, da, L.gP + h * d.dkvp, d.N1, 1, dh, dkv, E).bn = kToKernel;
    // d b_V = G^T dc
    one.add((float *)g.b_V, 1, L.Gm, 1, da, L.gc, 1, 1, da, 1, E);
    {   // dW_m1[:, :da] = dG W_O^T + dc (x) b_O
        SmallJob &q = two.add((float *)g.W_m1, ld_m1, L.gG, da, 1, w.W_O, 1, da, E, da, da);
        q.u = L.gc, q.us = 1, q.v = w.b_O, q.vs = 1;
    }
    two.add((float *)g.W_O, da, w.W_m1, 1, ld_m1, L.gG, da, 1, da, da, E);       // dW_O = W_m1a^T dG
    two.add((float *)g.b_O, 1, w.W_m1, 1, ld_m1, L.gc, 1, 1, da, 1, E);          // d b_O = W_m1a^T dc
    {   // dW_Q[:, M:] = d cQ (x) Phi(0)
        SmallJob &q = two.add((float *)g.W_Q + M, da, w.W_Q, 0, 0, w.W_Q, 0, 0, da, T, 0);
        q.u = g.b_Q, q.us = 1, q.v = L.phi0, q.vs = 1;
    }
    two.add(L.dphi0, 1, w.W_Q + M, 1, da, g.b_Q, 1, 1, T, 1, da);                // d Phi(0) = W_Q[:, M:]^T d cQ
    const hipError_t e = one.launch(s);
    return e == hipSuccess ? two.launch(s) : e;
}

}  // namespace

// Copies the caller's weights into the master buffer and prepares the kernels' weights.
hipError_t train_attach(const Dims &d, const tig_weights &w, void *workspace, void *packed, PackedWeights *pw,
                        hipStream_t s)
{
    const TrainLayout L = train_layout(d, workspace);
    const float *const src[22] = {w.time_w, w.time_b, w.W_i, w.b_i, w.W_h, w.b_h, w.W_Q, w.b_Q, w.W_K, w.b_K, w.W_V,
                                  w.b_V, w.W_O, w.b_O, w.W_m1, w.b_m1, w.W_m2, w.b_m2, w.W_d1, w.b_d1, w.w_d2, w.b_d2};
    const float *const dst[22] = {L.w.time_w, L.w.time_b, L.w.W_i, L.w.b_i, L.w.W_h, L.w.b_h, L.w.W_Q, L.w.b_Q,
                                  L.w.W_K, L.w.b_K, L.w.W_V, L.w.b_V, L.w.W_O, L.w.b_O, L.w.W_m1, L.w.b_m1,
                                  L.w.W_m2, L.w.b_m2, L.w.W_d1, L.w.b_d1, L.w.w_d2, L.w.b_d2};
    for (int i = 0; i < 22; ++i) {
        const size_t n = (i + 1 < 22 ? dst[i + 1] : L.P + L.n_params) - dst[i];
        hipError_t e = hipMemcpyAsync((void *)dst[i], src[i], 4 * n, hipMemcpyDefault, s);
        if (e != hipSuccess)
            return e;
    }
    hipError_t e = launch_fill_zero((char *)workspace + L.zero_lo, L.zero_hi - L.zero_lo, s);
    if (e == hipSuccess)
        e = pack_weights(d, L.w, packed, L.pack_scratch, pw, s);
    hipLaunchKernelGGL(k_tr_phi0, dim3((d.T + 255) / 256), dim3(256), 0, s, L.w.time_b, L.phi0, d.T);
    if (e == hipSuccess)
        e = hipGetLastError();
    // (for the backward pass's copies; the forward pass and ordinary steps start from foldings in double throughout, where
    // fold_weights rounds G and cQ once in between)
    if (e == hipSuccess)
        e = fold_weights(d, L, *pw, s);
    return e == hipSuccess ? pack_weights(d, L.w, packed, L.pack_scratch, pw, s, kPackEmbed) : e;
}

// The masters (or gradients) lie in one range: through a pinned buffer to host destinations in pieces (one
// copy per array from pageable memory took 0.6 ms for a model of 0.9 M weights).
hipError_t train_copy_out(const Dims &d, void *workspace, bool grads, const tig_weights &out, hipStream_t s)
{
    const TrainLayout L = train_layout(d, workspace);
    const tig_weights &src = grads ? L.g : L.w;
    const float *const sp[22] = {src.time_w, src.time_b, src.W_i, src.b_i, src.W_h, src.b_h, src.W_Q, src.b_Q,
                                 src.W_K, src.b_K, src.W_V, src.b_V, src.W_O, src.b_O, src.W_m1, src.b_m1,
                                 src.W_m2, src.b_m2, src.W_d1, src.b_d1, src.w_d2, src.b_d2};
    const float *const dp[22] = {out.time_w, out.time_b, out.W_i, out.b_i, out.W_h, out.b_h, out.W_Q, out.b_Q,
                                 out.W_K, out.b_K, out.W_V, out.b_V, out.W_O, out.b_O, out.W_m1, out.b_m1,
                                 out.W_m2, out.b_m2, out.W_d1, out.b_d1, out.w_d2, out.b_d2};
    const float *const base = grads ? L.G : L.P, *const end = base + L.n_params;
    const PinnedStage stage;
    bool host[22];
    hipError_t e = hipSuccess;
    for (int i = 0; i < 22; ++i) {
        hipPointerAttribute_t at;
        host[i] = dp[i] && stage.ptr && hipPointerGetAttributes(&at, dp[i]) == hipSuccess && at.type != hipMemoryTypeDevice &&
                  at.type != hipMemoryTypeManaged;
        (void)hipGetLastError();
        if (dp[i] && !host[i]) {
            const size_t n = (i + 1 < 22 ? sp[i + 1] : end) - sp[i];
            if ((e = hipMemcpyAsync((void *)dp[i], sp[i], 4 * n, hipMemcpyDefault, s)) != hipSuccess)
                return e;
        }
    }
    const size_t piece = kPinnedStageBytes / 4;
    for (size_t lo = 0; stage.ptr && lo < L.n_params; lo += piece) {
        const size_t hi = lo + piece < L.n_params ? lo + piece : L.n_params;
        size_t first = hi, last = lo;  // what of the piece is asked for
        for (int i = 0; i < 22; ++i) {
            const size_t a0 = (size_t)(sp[i] - base), a1 = (size_t)((i + 1 < 22 ? sp[i + 1] : end) - base);
            if (!host[i] || a0 >= hi || a1 <= lo)
                continue;
            first = a0 < first ? (a0 < lo ? lo : a0) : first;
            last = a1 > last ? (a1 > hi ? hi : a1) : last;
        }
        if (first >= last)
            continue;
        if ((e = hipMemcpyAsync(stage.ptr, base + first, 4 * (last - first), hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return e;
        for (int i = 0; i < 22; ++i) {
            const size_t a0 = (size_t)(sp[i] - base), a1 = (size_t)((i + 1 < 22 ? sp[i + 1] : end) - base);
            const size_t b0 = a0 > first ? a0 : first, b1 = a1 < last ? a1 : last;
            if (host[i] && b0 < b1)
                memcpy((float *)dp[i] + (b0 - a0), (const float *)stage.ptr + (b0 - first), 4 * (b1 - b0));
        }
    }
    return hipStreamSynchronize(s);
}

void train_step_args(const Dims &d, void *workspace, StepArgs *a)
{
    const TrainArrays t = train_layout(d, workspace).t;
    a->gru_gates = t.GATES;
    a->gru_msg = t.MSG;
    a->d_staging = t.D_STAG;
    a->tr = TrainFwd{t.S, t.QT, t.KVB, t.H1, t.DA, t.DB};
}

// Everything of a training step after the GRU launch.
hipError_t launch_train(const Dims &d, const LaunchPlan &plan, const StepArgs &a, void *workspace, const PackedWeights &pw, float lr,
                        float *loss_out, int *launches, hipStream_t s)
{
    const TrainLayout L = train_layout(d, workspace);
    const TrainArrays &t = L.t;
    const int M = d.M, E = d.E, da = d.da, D = d.Dmsg, ld_m1 = da + M;
    hipError_t e;
    if ((e = launch_embed(d, plan, pw, a, s)) != hipSuccess || (e = launch_train_decode(d, a, pw, t, s)) != hipSuccess ||
        (e = launch_train_back(d, plan, a, pw, t, s)) != hipSuccess)
        return e;
    if (a.msg_count > 0 && (e = launch_train_gru_back(d, plan, a, pw, t, s)) != hipSuccess)
        return e;
    *launches += a.msg_count > 0 ? 4 : 3;
    {
        WgradJobs w = {};
        int n = 0;
        auto add = [&](const float *C, int ldc, const float *A, int lda, int Mo, const float *B, int ldb, int No, const float *csum,
                       bool winners = false) -> WgradJob & {
            WgradJob &q = w.j[n++];
            q = WgradJob{A, B, (float *)C, nullptr, (float *)csum, lda, ldb, ldc, Mo, No, No, winners ? 1 : 0};
            return q;
        };
        add(L.gA1, M + 1, t.DQT, d.N1, d.N1, t.S, M + 1, M + 1, nullptr);  // [dA1 | da1] (d q~ is zero without neighbours)
        add(L.gP, d.N1, t.DZ1, E, E, t.KVB, d.N1, d.N1, nullptr);
        {   // the state part of merge layer 1, and the gradient of the bias of the rows with neighbours
            WgradJob &q = add(L.g.W_m1 + da, ld_m1, t.DZ1, E, E, t.S, M + 1, M + 1, L.g.b_m1);
            q.split = M, q.C_hi = L.gc;
        }
        add(L.g.W_m2, E, t.DEMB, E, E, t.H1, E, E, L.g.b_m2);
        add(L.g.W_d1, 2 * E, t.DA, E, E, a.emb_u, E, E, L.g.b_d1);
        add(L.g.W_d1 + E, 2 * E, t.DB, E, E, a.emb_u, E, E, nullptr);
        add(L.g.W_i, D, t.DGI, 3 * M, 3 * M, t.MSG, D, D, L.g.b_i, true);
        add(L.g.W_h, M, t.DGH, 3 * M, 3 * M, t.MSG, D, M, L.g.b_h, true);  // h = the first M columns of the message rows
        auto number = [&](int mi) {
            int tiles = 0;
            for (int i = 0; i < kMaxWgrad; ++i) {
                w.first[i] = i < n ? tiles : 0x7fffffff;
                tiles += i < n ? wgrad_job_tiles(w.j[i].Mo, w.j[i].No, mi) : 0;
            }
            return tiles;
        };
        w.part = L.part;
        const dim3 threads(kWgWaves * kWave);
        const size_t rows = (size_t)(a.rows_est > 0 && a.rows_est < 3 * a.count ? a.rows_est : 3 * a.count);
        int tiles = number(4);
        if (L.part && rows >= kSplitRows) {
            hipLaunchKernelGGL((k_tr_wgrad<4, true>), dim3(tiles * kXcds), threads, 0, s, a, w);
            ++*launches;
            hipLaunchKernelGGL(k_tr_wgrad_sum, dim3(tiles), dim3(512), 0, s, w);
        } else if (tiles >= plan.num_cus) {
            hipLaunchKernelGGL((k_tr_wgrad<4, false>), dim3(tiles), threads, 0, s, a, w);
        } else {
            tiles = number(2);
            hipLaunchKernelGGL((k_tr_wgrad<2, false>), dim3(tiles), threads, 0, s, a, w);
        }
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if ((e = unfold_gradients(d, L, s)) != hipSuccess)
        return e;
    UpdateJob u = {};
    u.M = M, u.T = d.T, u.E = E;
    u.commit_blocks = a.msg_count > 0 ? 32 : 0;  // (last: the GRU's backward read the memory as the step found it)
    u.terms = t.LOSS, u.n_terms = 2 * a.count, u.loss_out = loss_out;
    u.P = L.P, u.G = L.G, u.n_params = L.n_params, u.lr = lr;
    u.TACC = t.TACC, u.WACC = t.WACC, u.phi0 = L.phi0, u.dphi0 = L.dphi0;
    const int blocks = u.commit_blocks + (loss_out ? 1 : 0) + (int)((L.n_params + 255) / 256);
    hipLaunchKernelGGL(k_tr_update, dim3(blocks), dim3(256), 0, s, a, u);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    *launches += lr != 0.0f ? 6 : 4;  // contractions, two of k_tr_small, update; two of k_tr_small
    return lr != 0.0f ? fold_weights(d, L, pw, s) : hipSuccess;
}

hipError_t train_refold_embed(const Dims &d, void *workspace, void *packed, PackedWeights *pw, hipStream_t s)
{
    const TrainLayout L = train_layout(d, workspace);
    return pack_weights(d, L.w, packed, L.pack_scratch, pw, s, kPackEmbed);
}

}  // namespace tig
