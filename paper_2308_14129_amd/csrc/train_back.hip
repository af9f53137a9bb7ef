// The backward pass of a training step (paper Sec. II-C: the decoder's edge probabilities "provide the
// self-supervised signals for training"; Alg. 2 "Backward and Optimize"), device side.  gfx950 only, fp32.
//
// It runs over the same rows as the forward pass -- the DISTINCT queries of the batch -- and through the
// same foldings (pack.hip, embed_tile.h), as three launches that keep every intermediate of their rows in
// LDS and leave per row only what the weight gradients contract over:
//   k_tr_decode    per event: logits, loss terms, and the gradients of the two decoder halves' pre-activations
//                  added to their rows (a row is shared by every event that asked for the same query)
//   k_tr_back      4 to 32 query rows per workgroup: decoder halves -> embedding -> merge MLP -> attention ->
//                  folded query, as matrix-core products and one wavefront per row for the attention (two in tiles of four); the
//                  gradients of state rows that this step's GRU wrote are collected in an LDS table
//   k_tr_gru_back  4 to 16 applied winners per workgroup: gradients of the gates' pre-activations, time encoding
// (Layer by layer as products over all rows in memory, with the key / value rows and their gradients
// stored per slot, the same pass was two dozen launches: half of a step of 200 events was the host launching
// them.)
#include "prepare.h"
#include "train.h"
#include "winners.h"

namespace tig {

#ifdef TIG_PHASE_CLOCKS
static __device__ unsigned long long g_phase_clocks[8192 * 8];
extern "C" __attribute__((visibility("default"))) int tig_debug_phase_clocks_back(unsigned long long *out, int n)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_clocks), sizeof(unsigned long long) * (size_t)n);
}
#endif

namespace {

__device__ inline int row_of_entry_tr(const QuerySet &qs, int i, int entries)
{
    int s = qs.slot[i];
    if (s < 0) {
        const int rep = -s - 1;
        s = rep < entries ? qs.slot[rep] : 0;
    }
    return s >= 0 && s < entries ? s : 0;
}

// ------------------------------------------------------------------------------------------
// One wavefront per event, sixteen consecutive events per workgroup.  y = W_a emb_src + W_b emb_other + b1 comes from
// the per-row halves that the forward pass left; d y goes to the source's row of DA and the other's row
// of DB (a negative's row belongs to its event alone: stored, not added).
// MERGE: events of one moment share a hub's row, and additions to one row take turns.  An eighth of the batch per XCD, so that a
// row's come from one of them, and a workgroup adds each of its rows once (merge_rows: when).
constexpr int kDecThreads = 1024, kDecWaves = kDecThreads / kWave;
constexpr int kDecCols = 8;  // 64-column pieces of a row at most
constexpr int kDecXcds = 8;

template <bool MERGE>
__global__ void __launch_bounds__(kDecThreads) k_tr_decode(StepArgs a, PackedWeights w, TrainArrays t, int E, int Ep)
{
    extern __shared__ float wsum[];  // [waves x (E + 1)] the wavefronts' shares of the gradients of w_d2 and b_d2
    float *const share = wsum + kDecWaves * (E + 1);  // MERGE: [2][waves x E] what the events add to DA, to DB
    __shared__ int s_row[2][kDecWaves];
    const int B = a.count, lane = lane_id(), wave = wave_id_uniform();
    const int per_xcd = ((int)gridDim.x + kDecXcds - 1) / kDecXcds;  // (a launch's workgroups go round the XCDs)
    const int block = MERGE ? (int)blockIdx.x % kDecXcds * per_xcd + (int)blockIdx.x / kDecXcds : (int)blockIdx.x;
    const int b = block * kDecWaves + wave;
    if (MERGE && block * kDecWaves >= B)  // (the grid is whole rounds over the XCDs)
        return;
    const bool on = b < B;  // (uniform over the wavefront)
    const int bb = on ? b : 0;
    const int row[3] = {row_of_entry_tr(a.qs, 2 * bb, 2 * B), row_of_entry_tr(a.qs, 2 * bb + 1, 2 * B), 2 * B + bb};
    float g[2][kDecCols], w2[kDecCols], part[2] = {0.0f, 0.0f};
    for (int c = 0; c < kDecCols; ++c)
        if (c * kWave < E) {  // (uniform)
            const int j = c * kWave + lane, jc = j < E ? j : 0;
            const float x = a.dec_a[(size_t)row[0] * Ep + jc] + w.dec_b1f[jc];
            const float y0 = a.dec_b[(size_t)row[1] * Ep + jc], y1 = a.dec_b[(size_t)row[2] * Ep + jc];
            float em[3];
#pragma unroll
            for (int r = 0; r < 3; ++r)
                em[r] = a.emb_u[(size_t)row[r] * E + jc];
            const float ww = w.dec_w2[jc];
            w2[c] = j < E ? ww : 0.0f;
            g[0][c] = j < E ? fmaxf(x + y0, 0.0f) : 0.0f;
            g[1][c] = j < E ? fmaxf(x + y1, 0.0f) : 0.0f;
            part[0] += w2[c] * g[0][c];
            part[1] += w2[c] * g[1][c];
            if (on && j < E)
#pragma unroll
                for (int r = 0; r < 3; ++r)
                    a.emb[((size_t)r * B + b) * E + j] = em[r];
        }
    const float b2 = w.dec_b2[0];
    float dl[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        // d softplus(sign * logit) / d logit = sign * sigmoid(sign * logit), averaged over the batch
        const float sign = p == 0 ? -1.0f : 1.0f;
        const float logit = wave_sum_uniform(part[p]) + b2;
        const float z = sign * logit;
        dl[p] = on ? sign / (1.0f + expf(-z)) / (float)B : 0.0f;
        if (on && lane == 0) {
            (p == 0 ? a.score_pos : a.score_neg)[b] = logit;
            t.LOSS[p * B + b] = (z > 0.0f ? z + log1pf(expf(-z)) : log1pf(expf(z))) / (float)B;
        }
    }
    for (int c = 0; c < kDecCols; ++c)
        if (c * kWave < E) {
            const int j = c * kWave + lane;
            if (j < E) {
                wsum[wave * (E + 1) + j] = dl[0] * g[0][c] + dl[1] * g[1][c];
                const float dp = g[0][c] > 0.0f ? dl[0] * w2[c] : 0.0f, dn = g[1][c] > 0.0f ? dl[1] * w2[c] : 0.0f;
                if (MERGE) {
                    share[wave * E + j] = dp + dn;
                    share[(kDecWaves + wave) * E + j] = dp;
                } else if (on) {
                    atomicAdd(&t.DA[(size_t)row[0] * E + j], dp + dn);
                    atomicAdd(&t.DB[(size_t)row[1] * E + j], dp);
                }
                if (on)
                    t.DB[(size_t)row[2] * E + j] = dn;
            }
        }
    if (lane == 0) {
        wsum[wave * (E + 1) + E] = dl[0] + dl[1];
        if (MERGE) {
            s_row[0][wave] = on ? row[0] : -1;
            s_row[1][wave] = on ? row[1] : -1;
        }
    }
    __syncthreads();
    // the first event of the workgroup with a row adds for all of them
#pragma unroll
    for (int p = 0; MERGE && p < 2; ++p) {
        const int mine = __builtin_amdgcn_readfirstlane(s_row[p][wave]);
        const int theirs = lane < kDecWaves ? s_row[p][lane] : -1;
        const unsigned long long same = __ballot(theirs == mine && lane < kDecWaves);
        if (mine < 0 || __builtin_ctzll(same) != wave)
            continue;
        float *const dst = (p == 0 ? t.DA : t.DB) + (size_t)mine * E;
        for (int j = lane; j < E; j += kWave) {
            float sum = 0.0f;
            for (unsigned long long m = same; m; m &= m - 1)  // (uniform)
                sum += share[(p * kDecWaves + __builtin_ctzll(m)) * E + j];
            atomicAdd(&dst[j], sum);
        }
    }
    for (int j = threadIdx.x; j <= E; j += kDecThreads) {
        float sum = 0.0f;
        for (int v = 0; v < kDecWaves; ++v)
            sum += wsum[v * (E + 1) + j];
        atomicAdd(&t.WACC[(blockIdx.x % kSumCopies) * (E + 1) + j], sum);
    }
}

// ------------------------------------------------------------------------------------------
// maximum over the 64 lanes, wave-uniform (lanes a step shifts in from outside keep their own value)
__device__ inline float wave_max_uniform(float v)
{
#define TIG_MAX_STEP(CTRL, ROWS_)                                                                                            \
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROWS_, 0xf, false)));
    TIG_MAX_STEP(0x111, 0xf)
    TIG_MAX_STEP(0x112, 0xf)
    TIG_MAX_STEP(0x114, 0xf)
    TIG_MAX_STEP(0x118, 0xf)
    TIG_MAX_STEP(0x142, 0xa)
    TIG_MAX_STEP(0x143, 0xc)
#undef TIG_MAX_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Eight wavefronts of up to 256 registers: a row's q~, d kvbar and d q~ for all heads and ten neighbour rows stay in
// registers (sixteen wavefronts of 128 spilled up to 160 of them: 84 instead of 12 us for the attention phase of sixteen
// rows of 444 columns and two heads).
constexpr int kBackThreads = 512;
// A tile of four rows has two wavefronts for each, which take every other neighbour slot: the attention of one row of ten
// 444-column slots 13.4 -> 7.8 us (one wavefront's registers also spilled, 47 of them).
template <int NPL, int H, int ROWS>
struct BackShape {
    static constexpr int KC = NPL >= 6 && (H >= 4 || ROWS == 4) ? 6 : 10;  // neighbour rows in registers at a time
};

// acc[j] += A[the tile's rows][k-blocks a_kb0 .. + n) x W[nt[j]]^T over W's k-blocks [w_kb0, w_kb0 + n), for NT output tiles
// that share the reads of A.  With eight wavefronts on a unit a product is as long as its round trips to L2, so DEPTH
// blocks of every tile's weights are requested together (a block beyond n repeats the last and is not used), the next
// DEPTH while these are multiplied.
// Products are summed two blocks (32 terms) at a time, see tile_gemm's PARTS.
template <int MT, int RG, int NT, int DEPTH>
__device__ inline void tile_gemm_deep(floatx4 (&acc)[NT][MT + RG], const char *A, int lda, int a_kb0, const void *W, int w_kblocks,
                                      int w_kb0, int n, const int (&nt)[NT])
{
    using P = Prec<TIG_FP32>;
    using TR = TileRows<TIG_FP32, MT, RG>;
    using frag = typename P::frag;
    const int lane = lane_id();
    const TR rows(A, lda);
    auto request = [&](frag (&b)[NT][DEPTH], int kb) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int kc = kb + u < n ? kb + u : n - 1;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                b[j][u] = P::load_w(W, ((size_t)nt[j] * w_kblocks + w_kb0 + kc) * kWave + lane);
        }
    };
    auto multiply = [&](const frag (&b)[NT][DEPTH], int kb) {
#pragma unroll
        for (int u0 = 0; u0 < DEPTH; u0 += 2) {
            if (kb + u0 >= n)  // (uniform)
                break;
            floatx4 part[NT][TR::kAcc] = {};
#pragma unroll
            for (int u = u0; u < u0 + 2 && u < DEPTH; ++u)
                if (kb + u < n) {  // (uniform)
#pragma unroll
                    for (int i = 0; i < TR::kAcc; ++i) {
                        const frag a = rows.load(i, a_kb0 + kb + u);
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            TR::mma(i, part[j][i], a, b[j][u]);
                    }
                }
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < TR::kAcc; ++i)
                    acc[j][i] += part[j][i];
        }
    };
    frag b0[NT][DEPTH], b1[NT][DEPTH];
    request(b0, 0);
    for (int kb = 0; kb < n; kb += 2 * DEPTH) {
        if (kb + DEPTH < n)  // (uniform)
            request(b1, kb + DEPTH);
        multiply(b0, kb);
        if (kb + DEPTH >= n)
            break;
        if (kb + 2 * DEPTH < n)
            request(b0, kb + 2 * DEPTH);
        multiply(b1, kb + DEPTH);
    }
}

// NPHI: 64-column pieces of a row that hold time-encoding columns (they come first).
template <int ROWS, int NPL, int NPHI, int H>
__global__ void __launch_bounds__(kBackThreads)
k_tr_back(StepArgs a, PackedWeights w, TrainArrays t, BackParams p)
{
    using P = Prec<TIG_FP32>;
    constexpr int kThreads = kBackThreads, kWaves = kThreads / kWave, KC = BackShape<NPL, H, ROWS>::KC;
    constexpr bool PAIR = ROWS == 4;  // two wavefronts share a row's attention
    static_assert(!PAIR || 2 * ROWS == kWaves, "");
    constexpr int MT = ROWS / 16, RG = ROWS % 16 / 4;
    using TR = TileRows<TIG_FP32, MT, RG>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char *X = smem, *Z = smem + p.off_z;
    double *row_t = (double *)(smem + p.off_meta);  // [ROWS] query time
    double *tw_tab = row_t + ROWS;                  // [T][2] time encoding (w_rev, b_rev)
    int *row_q = (int *)(tw_tab + 2 * p.T);         // [ROWS] row of the query set or -1
    int *row_cnt = row_q + ROWS;                    // [ROWS]
    int *row_ref = row_cnt + ROWS;                  // [ROWS] row reference of the node's own state
    int *next_row = row_ref + ROWS;                 // [1]
    // [slots x M] sums, in double: an LDS addition of doubles takes 8 clocks for a wavefront, one of floats 192
    double *tab = (double *)(smem + p.off_tab);
    int *tag = (int *)(tab + p.slots * p.M);        // [slots] staged row held by the table's row, -1: none
    float *pair_sd = (float *)(tag + p.slots);      // PAIR: [ROWS][2 H][64] scores and d p of every slot

    const int lane = lane_id(), wave = wave_id_uniform();
    int n_u = *a.qs.n_u;
    n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
    const int neg_row0 = 2 * a.count;
    const int n_rows = n_u + a.count;
    const int n_passes = (n_rows + p.rpt - 1) / p.rpt;
    const int pass = (int)blockIdx.x;
    if (pass >= n_passes)
        return;  // fewer distinct queries than the grid was sized for
    TIG_MARK(0);
    for (int i = threadIdx.x; i < p.slots; i += kThreads)
        tag[i] = -1;
    for (int i = threadIdx.x; i < p.slots * p.M; i += kThreads)
        tab[i] = 0.0;
    for (int j = threadIdx.x; j < p.T; j += kThreads) {
        tw_tab[2 * j] = w.time_w_rev[j];
        tw_tab[2 * j + 1] = w.time_b_rev[j];
    }
    if (threadIdx.x < ROWS) {
        const int x = pass + n_passes * (int)threadIdx.x;
        const bool on = (int)threadIdx.x < p.rpt;
        const int q = !on ? -1 : x < n_u ? x : (x < n_rows ? neg_row0 + (x - n_u) : -1), qq = q >= 0 ? q : 0;
        const int cnt = a.qs.cnt[qq];
        row_t[threadIdx.x] = a.qs.t[qq];
        row_ref[threadIdx.x] = q >= 0 ? a.qs.self_ref[qq] : kRefNone;
        row_cnt[threadIdx.x] = q < 0 || cnt < 0 ? 0 : (cnt < p.K ? cnt : p.K);
        row_q[threadIdx.x] = q;
    }
    if (threadIdx.x == 0)
        *next_row = 0;
    __syncthreads();
    // ---- 1. gradients of the decoder halves -> X = [DA | DB]
    for (int row = wave; row < ROWS; row += kWaves) {
        const int q = __builtin_amdgcn_readfirstlane(row_q[row]);
        float *x = (float *)(X + (size_t)row * p.row_bytes);
        const float *da = t.DA + (size_t)(q >= 0 ? q : 0) * p.E, *db = t.DB + (size_t)(q >= 0 ? q : 0) * p.E;
        for (int j = lane; j < p.Ek; j += kWave) {
            const float va = da[j < p.E ? j : 0], vb = db[j < p.E ? j : 0];
            const bool in = q >= 0 && j < p.E;
            x[j] = in ? va : 0.0f;
            x[p.Ek + j] = in ? vb : 0.0f;
        }
    }
    __syncthreads();
    auto clear = [&](auto &acc) {
        for (auto &tile : acc)
            for (floatx4 &x : tile)
                x = floatx4{0, 0, 0, 0};
    };
    const int kbE = p.Ek / P::KB;
    TIG_MARK(1);
    // ---- 2. d emb = W_d1[:, :E]^T DA + W_d1[:, E:]^T DB -> X behind them
    for (int nt = wave; nt < p.Ep / 16; nt += kWaves) {
        floatx4 acc[1][TR::kAcc];
        float d[TR::kOut];
        clear(acc);
        tile_gemm_deep<MT, RG, 1, 16>(acc, X, p.row_bytes, 0, t.Wd1T, 2 * kbE, 0, 2 * kbE, {nt});
        TR::results(acc[0], d);
        const int col = nt * 16 + (lane & 15);
#pragma unroll
        for (int o = 0; o < TR::kOut; ++o) {
            const int row = TR::row(o), q = row_q[row];
            ((float *)(X + (size_t)row * p.row_bytes))[2 * p.Ek + col] = d[o];
            if (q >= 0 && col < p.E)
                t.DEMB[(size_t)q * p.E + col] = d[o];
        }
    }
    __syncthreads();
    // ---- 3. d z1 = (W_m2^T d emb) where h1 > 0 -> Z
    for (int nt = wave; nt < p.Ep / 16; nt += kWaves) {
        floatx4 acc[1][TR::kAcc];
        float d[TR::kOut];
        clear(acc);
        const int col = nt * 16 + (lane & 15);
        float h1[TR::kOut];
#pragma unroll
        for (int o = 0; o < TR::kOut; ++o) {
            const int q = row_q[TR::row(o)];
            h1[o] = t.H1[(size_t)(q >= 0 ? q : 0) * p.E + (col < p.E ? col : 0)];
        }
        tile_gemm_deep<MT, RG, 1, 8>(acc, X, p.row_bytes, 2 * kbE, t.Wm2T, kbE, 0, kbE, {nt});
        TR::results(acc[0], d);
#pragma unroll
        for (int o = 0; o < TR::kOut; ++o) {
            const int row = TR::row(o), q = row_q[row];
            const float g = q >= 0 && col < p.E && h1[o] > 0.0f ? d[o] : 0.0f;
            ((float *)(Z + (size_t)row * p.ldz))[col] = g;
            if (q >= 0 && col < p.E)
                t.DZ1[(size_t)q * p.E + col] = g;
        }
    }
    __syncthreads();
    TIG_MARK(2);
    // ---- 4. [d kvbar | d s_u] = [P | R]^T d z1 -> X (no attention without neighbours)
    // (two output tiles per pass, the next pass's weights on their way while this one's are multiplied)
    {
        using frag = typename P::frag;
        constexpr int kDeep = 7;
        const int n_nt = p.K2 / 16;
        const TR rows(Z, p.ldz);
        auto request = [&](frag (&b)[2][kDeep], int nt, int kb0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = nt + j * kWaves < n_nt ? nt + j * kWaves : nt;
#pragma unroll
                for (int u = 0; u < kDeep; ++u) {
                    const int kc = kb0 + u < kbE ? kb0 + u : kbE - 1;
                    b[j][u] = P::load_w(t.PRT, ((size_t)n * kbE + kc) * kWave + lane);
                }
            }
        };
        frag cur[2][kDeep], nxt[2][kDeep];
        if (wave < n_nt)
            request(cur, wave, 0);
        for (int nt = wave; nt < n_nt; nt += 2 * kWaves) {
            floatx4 acc[2][TR::kAcc];
            clear(acc);
            const bool two = nt + kWaves < n_nt;  // (uniform)
            for (int kb = 0; kb < kbE; kb += kDeep) {
                const bool last = kb + kDeep >= kbE;
                request(nxt, last ? (nt + 2 * kWaves < n_nt ? nt + 2 * kWaves : nt) : nt, last ? 0 : kb + kDeep);
#pragma unroll
                for (int u = 0; u < kDeep; ++u)
                    if (kb + u < kbE) {  // (uniform)
#pragma unroll
                        for (int i = 0; i < TR::kAcc; ++i) {
                            const frag a = rows.load(i, kb + u);
#pragma unroll
                            for (int j = 0; j < 2; ++j)
                                if (j == 0 || two)
                                    TR::mma(i, acc[j][i], a, cur[j][u]);
                        }
                    }
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int u = 0; u < kDeep; ++u)
                        cur[j][u] = nxt[j][u];
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int col = (nt + j * kWaves) * 16 + (lane & 15);
                float d[TR::kOut];
                TR::results(acc[j], d);
                if (nt + j * kWaves < n_nt)  // (uniform)
#pragma unroll
                    for (int o = 0; o < TR::kOut; ++o) {
                        const int row = TR::row(o);
                        ((float *)(X + (size_t)row * p.row_bytes))[col] = col >= p.N1 || row_cnt[row] > 0 ? d[o] : 0.0f;
                    }
            }
        }
    }
    __syncthreads();
    // The table's row of staged row `srow` (claimed by open addressing with a few probes: a hub's row that lost its
    // place to another row would send all its additions to memory), or -1: additions go to memory.
    auto claim = [&](int srow) -> int {
        int h = (int)((((uint32_t)srow * 2654435761u) >> 16) * (uint32_t)p.slots >> 16);
        for (int probe = 0; probe < 8 && probe < p.slots; ++probe) {
            const int old = atomicCAS(&tag[h], -1, srow);
            if (old == -1 || old == srow)
                return h;
            h = h + 1 == p.slots ? 0 : h + 1;
        }
        return -1;
    };
    auto staged = [&](int32_t ref) -> int { return ref < 0 && ref != kRefNone && ~ref < 2 * a.msg_count ? ~ref : -1; };
    TIG_MARK(3);
    // time-encoding gradients of the lane's dims, over all rows of the wavefront (in double: some hundred terms, whose
    // sizes differ as the time differences do)
    double gw[NPHI], gb[NPHI];
    double tw_reg[NPHI], tb_reg[NPHI];  // ... and its parameters
#pragma unroll
    for (int n = 0; n < NPHI; ++n) {
        gw[n] = gb[n] = 0.0;
        const int j = lane + kWave * n < p.T ? lane + kWave * n : 0;
        tw_reg[n] = tw_tab[2 * j];
        tb_reg[n] = tw_tab[2 * j + 1];
    }
    // ---- 5. attention, one wavefront per row: scores and softmax again from q~ and the neighbour rows
    //      [Phi | s_v | e] (lane: dims lane + 64 n), then d p_hk = <d kvbar_h, kv_k>, d q~ and d kv_k
    {
        // The lane's element n of a neighbour row lies in the state row or in the feature row: one load from a lane's
        // own address, nothing conditional (a load behind a condition, even a uniform one, is waited for where its
        // value meets the other path's: the gather of a row was a chain of seventy round trips).  A time-encoding
        // element reads the state row's first.
        uint32_t off[NPL];  // byte offset from the state row, or from the feature row
        uint32_t from_e = 0, from_m = 0;  // bit n: a feature / a state element
#pragma unroll
        for (int n = 0; n < NPL; ++n) {
            const int jj = lane + kWave * n - p.T;
            const bool in_m = jj >= 0 && jj < p.M, in_e = jj >= p.M && jj < p.M + p.F;
            off[n] = in_m ? (uint32_t)jj * 4u : (in_e ? (uint32_t)(jj - p.M) * 4u : 0u);
            from_e |= in_e ? 1u << n : 0u;
            from_m |= in_m ? 1u << n : 0u;
        }
        // PAIR: wavefronts 2 r and 2 r + 1 take row r, once; slot k is the (k / 2)th of wavefront 2 r + k % 2.
        constexpr int STEP = PAIR ? 2 : 1;
        const int half = PAIR ? wave & 1 : 0;
        auto slot = [&](int i) { return STEP * i + half; };  // the wavefront's slot i
        while (true) {
            int r = wave >> 1;
            if constexpr (!PAIR) {
                r = 0;
                if (lane == 0)
                    r = atomicAdd(next_row, 1);
                r = __builtin_amdgcn_readfirstlane(r);
                if (r >= ROWS)
                    break;
            }
            const int q0 = __builtin_amdgcn_readfirstlane(row_q[r]), cnt = __builtin_amdgcn_readfirstlane(row_cnt[r]);
            if (!PAIR && q0 < 0)
                continue;
            const int q = q0 < 0 ? 0 : q0;
            const int own = (cnt - half + STEP - 1) / STEP;  // slots of this wavefront
            float *dq = t.DQT + (size_t)q * p.N1;
            if (!PAIR && cnt == 0) {
                for (int j = lane; j < p.N1; j += kWave)
                    dq[j] = 0.0f;
                continue;
            }
            // lane k < cnt: neighbour slot k
            int32_t nb_v = 0, nb_e = 0;
            double nb_dt = 0.0;
            int my_srow = -1, my_lds = -1;
            if (lane < cnt) {
                const size_t o = (size_t)q * p.K + lane;
                nb_v = a.qs.ref[o];
                nb_e = a.qs.eid[o];
                nb_dt = row_t[r] - a.qs.ts[o];
                my_srow = staged(nb_v);
                if (my_srow < 0 && (nb_v < 0 || (int64_t)nb_v >= a.num_nodes))
                    nb_v = 0;  // (not a row reference: only a corrupted table could hold it)
                nb_e = nb_e >= 0 ? nb_e : 0;
                if (my_srow >= 0 && (lane & (STEP - 1)) == half)
                    my_lds = claim(my_srow);
            }
            float *xrow = (float *)(X + (size_t)r * p.row_bytes);
            float qv[H][NPL], dv[H][NPL], acc[H][NPL];
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int n = 0; n < NPL; ++n) {
                    const int j = lane + kWave * n, jc = h * p.dkvp + (j < p.dkvp ? j : 0);
                    const float x = t.QT[(size_t)q * p.N1 + jc];
                    qv[h][n] = j < p.dkvp ? x : 0.0f;
                    dv[h][n] = j < p.dkvp ? xrow[jc] : 0.0f;
                    acc[h][n] = 0.0f;
                }
            float raw[KC][NPL];
            auto gather = [&](int c0) {  // the rows of the wavefront's slots c0 .. (the last one again beyond them)
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int k = slot(c0 + kk < own ? c0 + kk : own - 1);
                    const int32_t v = __builtin_amdgcn_readlane(nb_v, k), e = __builtin_amdgcn_readlane(nb_e, k);
                    const float *vrow = v >= 0 ? a.mem + (size_t)v * p.M : a.staging + (size_t)(~v) * p.M;
                    const float *erow = a.edge_feat + (size_t)e * p.F;
#pragma unroll
                    for (int n = 0; n < NPL; ++n)
                        raw[kk][n] = *(const float *)((const char *)((from_e >> n) & 1u ? erow : vrow) + off[n]);
                }
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int k = slot(c0 + kk < own ? c0 + kk : own - 1);
                    const double dt = readlane_f64(nb_dt, k);
#pragma unroll
                    for (int n = 0; n < NPHI; ++n) {
                        const float ph = time_enc(tw_reg[n], tb_reg[n], dt);
                        raw[kk][n] = lane + kWave * n < p.T ? ph : raw[kk][n];
                    }
                    // (the row's padding holds some state value: it meets zeros of q~ and d kvbar)
                }
            };
            float S[H], D[H];  // lane k: score of slot k, d p_hk
#pragma unroll
            for (int h = 0; h < H; ++h) {
                S[h] = -INFINITY;
                D[h] = 0.0f;
            }
            for (int c0 = 0; c0 < own; c0 += KC) {
                gather(c0);
#pragma unroll
                for (int kk = 0; kk < KC; ++kk)
                    if (c0 + kk < own) {  // (uniform)
                        float ps[H], pd[H];
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            ps[h] = pd[h] = 0.0f;
#pragma unroll
                            for (int n = 0; n < NPL; ++n) {
                                ps[h] += qv[h][n] * raw[kk][n];
                                pd[h] += dv[h][n] * raw[kk][n];
                            }
                        }
                        const bool mine = lane == slot(c0 + kk);
                        if constexpr (H % 2 == 0) {
#pragma unroll
                            for (int h = 0; h < H; h += 2) {
                                const float z = wave_sum_four(ps[h], ps[h + 1], pd[h], pd[h + 1]);
                                const float z0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), 15));
                                const float z1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), 31));
                                const float z2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), 47));
                                const float z3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), 63));
                                S[h] = mine ? z0 : S[h];
                                S[h + 1] = mine ? z1 : S[h + 1];
                                D[h] = mine ? z2 : D[h];
                                D[h + 1] = mine ? z3 : D[h + 1];
                            }
                        } else {
#pragma unroll
                            for (int h = 0; h < H; ++h) {
                                const float z0 = wave_sum_uniform(ps[h]), z2 = wave_sum_uniform(pd[h]);
                                S[h] = mine ? z0 : S[h];
                                D[h] = mine ? z2 : D[h];
                            }
                        }
                    }
            }
            if constexpr (PAIR) {  // every lane's score and d p from the wavefront that has its slot
                float *ex = pair_sd + (size_t)r * 2 * H * kWave;
#pragma unroll
                for (int h = 0; h < H; ++h)
                    if (lane < cnt && (lane & 1) == half) {
                        ex[h * kWave + lane] = S[h];
                        ex[(H + h) * kWave + lane] = D[h];
                    }
                __syncthreads();
#pragma unroll
                for (int h = 0; h < H; ++h)
                    if (lane < cnt) {
                        S[h] = ex[h * kWave + lane];
                        D[h] = ex[(H + h) * kWave + lane];
                    }
            }
            float pr[H], ds[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const float mx = wave_max_uniform(S[h]);
                const float ex = lane < cnt ? expf(S[h] - mx) : 0.0f;
                pr[h] = ex / wave_sum_uniform(ex);
                ds[h] = pr[h] * (D[h] - wave_sum_uniform(pr[h] * D[h]));  // gradient of <q~_h, kv_k>
            }
            for (int c0 = 0; c0 < own; c0 += KC) {
                if (own > KC)
                    gather(c0);
#pragma unroll
                for (int kk = 0; kk < KC; ++kk)
                    if (c0 + kk < own) {  // (uniform)
                        const int k = slot(c0 + kk);
                        float dk[NPL];  // d kv_k = sum_h p_hk d kvbar_h + d s_hk q~_h
#pragma unroll
                        for (int n = 0; n < NPL; ++n)
                            dk[n] = 0.0f;
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const float pk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr[h]), k));
                            const float dsk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ds[h]), k));
#pragma unroll
                            for (int n = 0; n < NPL; ++n) {
                                acc[h][n] += dsk * raw[kk][n];
                                dk[n] += pk * dv[h][n] + dsk * qv[h][n];
                            }
                        }
                        const int srow = __builtin_amdgcn_readlane(my_srow, k), trow = __builtin_amdgcn_readlane(my_lds, k);
                        if (trow >= 0) {  // the neighbour's state row was written by this step's GRU
#pragma unroll
                            for (int n = 0; n < NPL; ++n)
                                if ((from_m >> n) & 1u)
                                    atomicAdd((double *)((char *)(tab + trow * p.M) + 2 * off[n]), (double)dk[n]);
                        } else if (srow >= 0) {
#pragma unroll
                            for (int n = 0; n < NPL; ++n)
                                if ((from_m >> n) & 1u)
                                    atomicAdd((float *)((char *)(t.D_STAG + (size_t)srow * p.M) + off[n]), dk[n]);
                        }
                        const double dt = readlane_f64(nb_dt, k);
#pragma unroll
                        for (int n = 0; n < NPHI; ++n) {
                            const float v = -time_enc_sin(tw_reg[n], tb_reg[n], dt) * dk[n];
                            gw[n] += dt * (double)v;  // (lanes beyond T are dropped at the end)
                            gb[n] += (double)v;
                        }
                    }
            }
            if constexpr (PAIR) {  // (both have taken d kvbar from the row before the barrier above)
                if (half == 1)
#pragma unroll
                    for (int h = 0; h < H; ++h)
#pragma unroll
                        for (int n = 0; n < NPL; ++n)
                            if (lane + kWave * n < p.dkvp)
                                xrow[h * p.dkvp + lane + kWave * n] = acc[h][n];
                __syncthreads();
                if (half == 1)
                    break;
            }
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int n = 0; n < NPL; ++n) {
                    const int j = lane + kWave * n;
                    if (j < p.dkvp) {
                        const float both = PAIR ? acc[h][n] + xrow[h * p.dkvp + j] : acc[h][n];
                        const float x = j < p.dkv ? both : 0.0f;
                        xrow[h * p.dkvp + j] = x;
                        if (!PAIR || q0 >= 0)
                            dq[h * p.dkvp + j] = x;
                    }
                }
            if constexpr (PAIR)
                break;
        }
    }
    __syncthreads();
    TIG_MARK(4);
    // ---- 6. d s_u += A1^T d q~
    // (the tiles of the last, incomplete round are split over the wavefronts it leaves idle: eleven tiles of 172 columns
    // took two rounds where 1.4 are needed; with few results per lane only, the parts meet by LDS additions)
    {
        const int n_t = p.Mq / 16, kbN = p.N1 / P::KB, rem = n_t % kWaves, whole = n_t - rem;
        const int parts = ROWS <= 8 && rem > 0 && kbN >= kWaves ? kWaves / rem : 1;
        for (int u = wave; u < whole + rem * parts; u += kWaves) {
            const int nt = u < whole ? u : whole + (u - whole) % rem, part = u < whole ? 0 : (u - whole) / rem;
            const int of = u < whole ? 1 : parts, lo = kbN * part / of, hi = kbN * (part + 1) / of;
            floatx4 acc[1][TR::kAcc];
            float d[TR::kOut];
            clear(acc);
            tile_gemm_deep<MT, RG, 1, 14>(acc, X, p.row_bytes, lo, t.A1T, kbN, lo, hi - lo, {nt});
            TR::results(acc[0], d);
            const int col = p.N1 + nt * 16 + (lane & 15);
#pragma unroll
            for (int o = 0; o < TR::kOut; ++o) {
                float *x = (float *)(X + (size_t)TR::row(o) * p.row_bytes) + col;
                if (ROWS <= 8 && of > 1)  // (uniform)
                    atomicAdd(x, d[o]);
                else
                    *x += d[o];
            }
        }
    }
    __syncthreads();
    TIG_MARK(5);
    // ---- 7. the rows' own states
    for (int row = wave; row < ROWS; row += kWaves) {
        const int srow = __builtin_amdgcn_readfirstlane(row_q[row] >= 0 ? staged(row_ref[row]) : -1);
        if (srow < 0)
            continue;
        int trow = -1;
        if (lane == 0)
            trow = claim(srow);
        trow = __builtin_amdgcn_readfirstlane(trow);
        const float *g = (const float *)(X + (size_t)row * p.row_bytes) + p.N1;
        for (int j = lane; j < p.M; j += kWave) {
            if (trow >= 0)
                atomicAdd(tab + (size_t)trow * p.M + j, (double)g[j]);
            else
                atomicAdd(&t.D_STAG[(size_t)srow * p.M + j], g[j]);
        }
    }
    __syncthreads();
    // ---- 8. the table's rows and the time encoding's sums to memory
    for (int i = wave; i < p.slots; i += kWaves) {
        const int srow = __builtin_amdgcn_readfirstlane(tag[i]);
        for (int j = lane; srow >= 0 && j < p.M; j += kWave)
            atomicAdd(&t.D_STAG[(size_t)srow * p.M + j], (float)tab[i * p.M + j]);
    }
    double *red = (double *)X;  // [waves x T], frequencies first, then phases
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int n = 0; n < NPHI; ++n) {
            const int j = lane + kWave * n;
            if (j < p.T)
                red[wave * p.T + j] = half ? gb[n] : gw[n];
        }
        __syncthreads();
        for (int j = threadIdx.x; j < p.T; j += kThreads) {
            double sum = 0.0;
            for (int v = 0; v < kWaves; ++v)
                sum += red[v * p.T + j];
            atomicAdd(&t.TACC[((int)blockIdx.x % kSumCopies * 2 + half) * p.T + j], sum);
        }
        __syncthreads();
    }
    TIG_MARK(6);
}

// ------------------------------------------------------------------------------------------
// The GRU's backward pass over the applied winners, from the message rows and gates that the step's GRU launch
// left: gradients of the gate pre-activations, and through W_i's time columns the time encoding's gradient.
// A workgroup's chain (winners, gates, one product, the time encoding) is as long as its winners are many: tiles of 4, 8 or
// 16, the lowest that recent steps' winners fit one workgroup per compute unit in (200 events of 172 columns 15.5 -> 9.5 us,
// 4000 of 100 11.4 -> 8.4, both from 16 rows to 4); with more winners a workgroup takes tile after tile.
constexpr int kGbThreads = 512, kGbWaves = kGbThreads / kWave;
constexpr int kGbHeights[] = {4, 8, 16};

__device__ inline bool win_ok(const StepArgs &a, const WinDesc &w)
{
    return w.node >= 0 && (int64_t)w.node < a.num_nodes && w.other >= 0 && (int64_t)w.other < a.num_nodes &&
           w.entry >= 0 && w.entry < 2 * a.msg_count && w.b >= 0 && w.b < a.msg_count;
}

struct GruBackParams {
    int M, T, D, Kp, Tp;  // Kp: 3M padded to the k-blocks, Tp: T padded to output tiles
    int ldx, ldp;            // LDS bytes per row of the gate gradients / of d Phi
};

template <int ROWS>
__global__ void __launch_bounds__(kGbThreads) k_tr_gru_back(StepArgs a, PackedWeights w, TrainArrays t, GruBackParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char *X = smem, *DP = smem + ROWS * p.ldx;
    double *row_dt = (double *)(DP + ROWS * p.ldp);  // [rows]
    int n_win = *a.n_win;
    n_win = n_win < 2 * a.msg_count ? n_win : 2 * a.msg_count;
    const int lane = lane_id(), wave = wave_id_uniform();
    const int M = p.M, T = p.T, D = p.D;
    using TR = TileRows<TIG_FP32, ROWS / 16, ROWS % 16 / 4>;
    for (int r0 = (int)blockIdx.x * ROWS; r0 < n_win; r0 += (int)gridDim.x * ROWS) {
        if (r0 != (int)blockIdx.x * ROWS)
            __syncthreads();  // (the tile before is done with)
        for (int i = wave; i < ROWS; i += kGbWaves) {
            const int r = r0 + i;
            float *x = (float *)(X + (size_t)i * p.ldx);
            if (r >= n_win) {  // (uniform)
                for (int j = lane; j < p.Kp; j += kWave)
                    x[j] = 0.0f;
                if (lane == 0)
                    row_dt[i] = 0.0;
                continue;
            }
            const WinDesc d = a.win[r];
            const bool ok = win_ok(a, d);
            const double dt = ok ? d.t - a.lu[d.node] : 0.0;
            if (lane == 0)
                row_dt[i] = dt;
            const size_t entry = ok ? (size_t)d.entry : 0;
            const float *gt = t.GATES + (size_t)r * 4 * M;  // r, z, n, W_hn h + b_hn
            float *dgi = t.DGI + (size_t)r * 3 * M, *dgh = t.DGH + (size_t)r * 3 * M;
#pragma unroll 4
            for (int j = lane; j < M; j += kWave) {
                const float rg = gt[j], zg = gt[M + j], ng = gt[2 * M + j], ghn = gt[3 * M + j];
                const float dh0 = t.D_STAG[entry * M + j], h = t.MSG[(size_t)r * D + j];  // s_self leads the message
                const float dh = ok ? dh0 : 0.0f;
                const float dn = dh * (1.0f - zg);
                const float dz = dh * (h - ng);
                const float dpre_n = dn * (1.0f - ng * ng);
                const float dpre_r = dpre_n * ghn * rg * (1.0f - rg);
                const float dpre_z = dz * zg * (1.0f - zg);
                dgi[j] = x[j] = dpre_r;
                dgi[M + j] = x[M + j] = dpre_z;
                dgi[2 * M + j] = x[2 * M + j] = dpre_n;
                dgh[j] = dpre_r;
                dgh[M + j] = dpre_z;
                dgh[2 * M + j] = dpre_n * rg;
            }
            for (int j = 3 * M + lane; j < p.Kp; j += kWave)
                x[j] = 0.0f;
        }
        __syncthreads();
        for (int nt = wave; nt < p.Tp / 16; nt += kGbWaves) {
            floatx4 acc[1][TR::kAcc] = {};
            float d[TR::kOut];
            const int kb = p.Kp / Prec<TIG_FP32>::KB;
            tile_gemm_deep<ROWS / 16, ROWS % 16 / 4, 1, 12>(acc, X, p.ldx, 0, t.WiT, kb, 0, kb, {nt});
            TR::results(acc[0], d);
#pragma unroll
            for (int o = 0; o < TR::kOut; ++o)
                ((float *)(DP + (size_t)TR::row(o) * p.ldp))[nt * 16 + (lane & 15)] = d[o];
        }
        __syncthreads();
        for (int j = threadIdx.x; j < T; j += kGbThreads) {
            const double w_rev = w.time_w_rev[j], b_rev = w.time_b_rev[j];
            double gw = 0.0, gb = 0.0;
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {  // (rows beyond the winners hold zeros)
                const double dt = row_dt[i];
                const float v = -time_enc_sin(w_rev, b_rev, dt) * ((const float *)(DP + (size_t)i * p.ldp))[j];
                gw += dt * (double)v;
                gb += (double)v;
            }
            double *sums = t.TACC + (int)blockIdx.x % kSumCopies * 2 * T;
            atomicAdd(&sums[j], gw);
            atomicAdd(&sums[T + j], gb);
        }
    }
}

// ------------------------------------------------------------------------------------------
// host side

BackParams back_params(const Dims &d, int rows, int lds_limit, int *lds)
{
    BackParams p = {};
    p.M = d.M, p.T = d.T, p.F = d.F, p.E = d.E, p.K = d.K;
    p.dkv = d.dkv, p.dkvp = d.dkvp, p.Mq = d.Mq, p.N1 = d.N1, p.K2 = d.K2, p.Ep = d.Ep, p.Ek = d.Ek;
    const int wide = d.K2 > 3 * d.Ek ? d.K2 : 3 * d.Ek;
    p.row_bytes = lds_row_bytes(wide);
    p.ldz = lds_row_bytes(d.Ek);
    p.off_z = rows * p.row_bytes;
    p.off_meta = p.off_z + rows * p.ldz;
    // (the wavefronts' time-encoding sums take the place of both at the end)
    const int sums = (kBackThreads / kWave) * d.T * 8;
    p.off_meta = p.off_meta > sums ? p.off_meta : sums;
    p.off_tab = (p.off_meta + rows * 20 + d.T * 16 + 16 + 15) / 16 * 16;
    // as many table rows as fit: hubs are few, but every row that misses the table costs device atomics; at most two for
    // each that the tile can ask for
    const int slot_bytes = 8 * d.M + 4, pair_bytes = rows == 4 ? rows * 2 * (d.H <= 2 ? d.H : 4) * kWave * 4 : 0;
    const int most = 2 * rows * (d.K + 1) < 128 ? 2 * rows * (d.K + 1) : 128;
    p.slots = (lds_limit - p.off_tab - pair_bytes) / slot_bytes;
    p.slots = p.slots < 0 ? 0 : (p.slots > most ? most : p.slots);
    *lds = p.off_tab + p.slots * slot_bytes + pair_bytes;
    return p;
}

constexpr int kBackLds = 160 * 1024;

// 64-column pieces of a row the kernel is compiled for.  Above four, one too many costs: at 444 columns and two heads
// eight pieces spilled 69 registers, seven spill 31; six pieces fit.
int back_npl(const Dims &d)
{
    const int need = (d.dkvp + 63) / 64;
    return need <= 2 ? 2 : (need <= 4 ? 4 : (need <= 6 ? 6 : need));
}

template <int ROWS, int NPL, int NPHI>
const void *pick_back_h(int H)
{
    return H == 1   ? (const void *)k_tr_back<ROWS, NPL, NPHI, 1>
           : H == 2 ? (const void *)k_tr_back<ROWS, NPL, NPHI, 2>
                    : (const void *)k_tr_back<ROWS, NPL, NPHI, 4>;
}

template <int ROWS>
const void *pick_back(const Dims &d)
{
    const bool few = d.T <= 2 * kWave;
    switch (back_npl(d)) {
    case 2: return pick_back_h<ROWS, 2, 2>(d.H);
    case 4: return few ? pick_back_h<ROWS, 4, 2>(d.H) : pick_back_h<ROWS, 4, 4>(d.H);
    case 6: return few ? pick_back_h<ROWS, 6, 2>(d.H) : pick_back_h<ROWS, 8, 8>(d.H);
    case 7: return few ? pick_back_h<ROWS, 7, 2>(d.H) : pick_back_h<ROWS, 8, 8>(d.H);
    default: return few ? pick_back_h<ROWS, 8, 2>(d.H) : pick_back_h<ROWS, 8, 8>(d.H);
    }
}

// rows of a workgroup's tile the kernel is compiled for
constexpr int kBackHeights[] = {4, 8, 16, 32};

const void *back_kernel(const Dims &d, int rows)
{
    switch (rows) {
    case 4: return pick_back<4>(d);
    case 8: return pick_back<8>(d);
    case 16: return pick_back<16>(d);
    default: return pick_back<32>(d);
    }
}

// most rows per workgroup: a second block of sixteen only where the table keeps enough rows beside it
int back_most_rows(const Dims &d)
{
    int lds = 0;
    const BackParams p = back_params(d, 32, kBackLds, &lds);
    return lds <= kBackLds && p.slots >= 48 ? 32 : 16;
}

GruBackParams gru_back_params(const Dims &d)
{
    GruBackParams p;
    p.M = d.M, p.T = d.T, p.D = d.Dmsg;
    p.Kp = (3 * d.M + 15) / 16 * 16;
    p.Tp = (d.T + 15) / 16 * 16;
    p.ldx = lds_row_bytes(p.Kp);
    p.ldp = lds_row_bytes(p.Tp);
    return p;
}

int gru_back_lds(const Dims &d, int rows)
{
    const GruBackParams p = gru_back_params(d);
    return rows * (p.ldx + p.ldp + 8);
}

const void *gru_back_kernel(int rows)
{
    return rows == 4 ? (const void *)k_tr_gru_back<4> : (rows == 8 ? (const void *)k_tr_gru_back<8> : (const void *)k_tr_gru_back<16>);
}

int decode_lds_bytes(const Dims &d, bool merge) { return kDecWaves * ((merge ? 3 : 1) * d.E + 1) * 4; }

// Turns at shared rows count where they are more than the launch's latency hides: many events of wide rows, and few rows for
// them (by the steps before, whose rows are estimated up to an eighth high: a negative's for every event, and at most one
// more; then two to three endpoints ask for the same row).  And two workgroups have to fit a compute unit's LDS, up
// to 425 columns.  Every event on its own and merged, 100 columns, 44% of the endpoints at one node: 4000 events 12.1 and 10.2 us,
// 3000 10.5 and 9.4, 2000 9.1 and 8.9, 1000 7.7 and 8.8; of a quarter as many events a moment, 4000 10.4 and 10.2, 2000 7.9 and 8.8; a
// sixteenth, 4000 10.1 and 10.7; 32 columns, 4000 7.4 and 8.1; 400 columns, 2000 17.4 and 16.7; one workgroup a unit, 5000 events of 512 columns
// 33 and 43.
bool merge_rows(const Dims &d, const StepArgs &a)
{
    const size_t lds = (size_t)decode_lds_bytes(d, true) + 2 * kDecWaves * sizeof(int);
    return a.rows_est > 0 && a.rows_est <= 2 * a.count && (int64_t)a.count * d.E >= (1 << 18) && lds <= 80 * 1024;
}

}  // namespace

bool train_back_fits(const Dims &d)
{
    int lds = 0;
    (void)back_params(d, 16, kBackLds, &lds);
    return lds <= kBackLds && gru_back_lds(d, 16) <= kBackLds && d.E <= kDecCols * kWave && d.K <= kWave;
}

hipError_t prepare_train_back(const Dims &d)
{
    hipError_t e = hipFuncSetAttribute((const void *)k_tr_decode<false>, hipFuncAttributeMaxDynamicSharedMemorySize, decode_lds_bytes(d, false));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_tr_decode<true>, hipFuncAttributeMaxDynamicSharedMemorySize, decode_lds_bytes(d, true));
    for (const int h : kGbHeights)
        if (e == hipSuccess)
            e = hipFuncSetAttribute(gru_back_kernel(h), hipFuncAttributeMaxDynamicSharedMemorySize, gru_back_lds(d, h));
    for (const int h : kBackHeights) {
        if (h > back_most_rows(d) || e != hipSuccess)
            break;
        int lds = 0;
        (void)back_params(d, h, kBackLds, &lds);
        e = hipFuncSetAttribute(back_kernel(d, h), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    }
    return e;
}

hipError_t launch_train_decode(const Dims &d, const StepArgs &a, const PackedWeights &pw, const TrainArrays &t, hipStream_t s)
{
    const int blocks = (a.count + kDecWaves - 1) / kDecWaves;
    if (merge_rows(d, a))
        hipLaunchKernelGGL(k_tr_decode<true>, dim3((blocks + kDecXcds - 1) / kDecXcds * kDecXcds), dim3(kDecThreads), decode_lds_bytes(d, true), s,
                           a, pw, t, d.E, d.Ep);
    else
        hipLaunchKernelGGL(k_tr_decode<false>, dim3(blocks), dim3(kDecThreads), decode_lds_bytes(d, false), s, a, pw, t, d.E, d.Ep);
    return hipGetLastError();
}

hipError_t launch_train_back(const Dims &d, const LaunchPlan &plan, const StepArgs &a, const PackedWeights &pw,
                             const TrainArrays &t, hipStream_t s)
{
    // One round of workgroups: a compute unit's share of the rows that recent steps had (the estimate is up to an eighth
    // high, so that up to one unit in nine goes without: 221 of 256 at 5740 rows), in the lowest tile that takes it (the
    // products' time follows the tile's rows, see kHeights; the attention's the rows in use).
    const int most = 3 * a.count, rows = a.rows_est > 0 && a.rows_est < most ? a.rows_est : most;
    const int cus = plan.num_cus > 0 ? plan.num_cus : 256;
    const int even = (rows + cus - 1) / cus, tallest = back_most_rows(d);
    int height = tallest;
    for (const int h : kBackHeights)
        if (h >= even && h < height)
            height = h;
    int lds = 0;
    StepArgs aa = a;
    PackedWeights ww = pw;
    TrainArrays tt = t;
    BackParams p = back_params(d, height, kBackLds, &lds);
    p.rpt = even < 4 ? 4 : (even > height ? height : even);
    void *args[] = {&aa, &ww, &tt, &p};
    return hipLaunchKernel(back_kernel(d, height), dim3((most + p.rpt - 1) / p.rpt), dim3(kBackThreads), args, (size_t)lds, s);
}

hipError_t launch_train_gru_back(const Dims &d, const LaunchPlan &plan, const StepArgs &a, const PackedWeights &pw,
                                 const TrainArrays &t, hipStream_t s)
{
    const int most = 2 * a.msg_count, wins = a.wins_est > 0 && a.wins_est < most ? a.wins_est : most;
    const int cus = plan.num_cus > 0 ? plan.num_cus : 256;
    int height = 16;
    for (const int h : kGbHeights)
        if (h < height && (wins + h - 1) / h <= cus)
            height = h;
    const int tiles = (most + height - 1) / height;
    StepArgs aa = a;
    PackedWeights ww = pw;
    TrainArrays tt = t;
    GruBackParams p = gru_back_params(d);
    void *args[] = {&aa, &ww, &tt, &p};
    return hipLaunchKernel(gru_back_kernel(height), dim3(tiles < 2 * cus ? tiles : 2 * cus), dim3(kGbThreads), args,
                           (size_t)gru_back_lds(d, height), s);
}

}  // namespace tig
