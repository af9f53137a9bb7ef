// k_gru: message build and GRU state update (message module, state-update module and memory
// fetch of the paper's Sec. II-C) for the compacted winners of one batch.  gfx950 only.
// The same grid carries, in extra workgroups, work that depends on nothing the GRU produces:
//   - ahead of the embedding launch (a step whose batch was not prepared by the step before):
//     what is left of the query preparation (prepare.h), slots and row references;
//   - as the closing launch of a step (decode.h): the decoder scores and embedding rows of the
//     step's events and the finishing pass of the batch prepared for the next step -- and then
//     the GRU workgroups run for the batch the NEXT step applies (its winners were selected
//     beside the embedding launch), so that step starts with its embedding launch.
// All of these are chains of dependent memory round trips, so they hide each other.
//
// The number of winners is only known on the device (hub nodes make it a small fraction of the
// 2B entries), so the GRU workgroups are a fixed grid that divides the work itself: 16-row tiles
// of winners x slices of the gate columns, as many column slices per tile as keep the grid busy
// (every workgroup streams only its slice of the gate weights; all slices of a tile gather the
// same rows).  One work item (8 wavefronts):
//   1  row descriptors: node, partner, event, event time (dt = t - last_update[node] in step 2)
//   2  message rows [s_self | s_other | Phi(dt) | e] gathered from the batch-START memory into an
//      LDS tile (every element of every row is an independent load: one round of latency)
//   3  gate pre-activations on the matrix cores: the 8 wavefronts are 4 pairs, one wavefront of
//      a pair for the r and z gates, the other for the two halves of the n gate (input part over
//      the whole message, hidden part over s_self); the pairs split the item's column tiles and,
//      when there are fewer column tiles than pairs, the k range of each; partial sums meet in LDS
//   4  h' = (1 - z) n + z h  -> staging rows (memory is overwritten beside the embedding)
// W_hr and W_hz are folded onto the s_self columns of W_ir / W_iz at init (pack.hip).
#include <hip/hip_runtime.h>

#include "decode.h"
#include "gru_rules.h"
#include "kernels_common.h"
#include "prepare.h"

namespace tig {

#ifdef TIG_PHASE_CLOCKS
static __device__ unsigned long long g_phase_clocks[8192 * 8];
extern "C" __attribute__((visibility("default"))) int tig_debug_phase_clocks_gru(unsigned long long *out, int n)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_clocks), sizeof(unsigned long long) * (size_t)n);
}
#endif

namespace {

constexpr int kGruThreads = 512;  // two workgroups per compute unit: the finishing pass runs beside the GRU
constexpr int kGruWaves = kGruThreads / kWave;
constexpr int kPairs = kGruWaves / 2;  // wavefront pairs: (r, z) | n
constexpr int EC = 16;                 // winners per tile
constexpr int kPhi = 2;                // 64-column pieces of the time encoding whose parameters stay in registers

struct GruParams {
    int M, T, F, Dmsg;
    int Kg, Khn, Ng;
    int ldx;       // LDS row stride of the message tile, bytes
    int off_part;  // byte offset of the partial-sum buffer in LDS
    int n_gru;     // GRU workgroups (the first blocks of the grid)
    ColumnSlices guess;  // at the winner count that recent steps had
    int n_row_blocks;   // then: blocks that fix row references of this step's queries (grid-stride over the rows)
    int n_slot_blocks;  // then: blocks that fix their slots, one entry per thread
                        // then: the blocks of the closing work (decode.h)
    int32_t *clear;     // a counter block 0 sets to 0, or NULL
};

// The batch whose winners the GRU workgroups apply.
struct GruJob {
    int64_t first_eid;
    int32_t count;      // 0: nothing to apply
    const WinDesc *win;
    const int32_t *n_win;
};

// Products of a tile of winners with two weight streams that share the reads of A: acc1 += A W1[nt]^T over W1's k-blocks
// [kb_lo, kb_hi) and acc2 += A W2[nt]^T over W2's k-blocks [kb_lo, min(kb_hi, W2's number of blocks)).  A workgroup has
// eight wavefronts, so few loads in flight would make every block a round trip to L2 (the compiler moves a load down to its use:
// two in flight, 4.1 us for the 130 KB of an item of 172 columns that one compute unit can read in 0.9).  So kG blocks of both are
// requested together, the next kG while these are multiplied, and the first two groups (start) before the rows are there;
// the scheduler does not cross the barriers between.  A block beyond the last is the last again and is not used.
template <int PREC, int kG>
struct GateStream {
    using P = Prec<PREC>;
    using frag = typename P::frag;
    static constexpr int kBlock = kWave * P::kLaneBytes;
    const char *w1, *w2;  // block 0 of the output tile
    int kb_lo, kb_hi, kb_hi2, last2;
    frag a1[kG], a2[kG], b1[kG], b2[kG];

    __device__ inline void request(frag (&f1)[kG], frag (&f2)[kG], int kb) const
    {
        const unsigned lane_off = (unsigned)lane_id() * P::kLaneBytes;
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            const int k1 = kb + u < kb_hi ? kb + u : kb_hi - 1, k2 = k1 < last2 ? k1 : last2;
            f1[u] = P::load_w_at(w1 + (size_t)k1 * kBlock, lane_off);
            f2[u] = P::load_w_at(w2 + (size_t)k2 * kBlock, lane_off);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // (everything uniform; kb_lo < kb_hi)
    __device__ inline void start(const void *W1, const void *W2, int w1_kblocks, int w2_kblocks, int lo, int hi, int nt)
    {
        w1 = (const char *)W1 + (size_t)(nt * w1_kblocks) * kBlock;
        w2 = (const char *)W2 + (size_t)(nt * w2_kblocks) * kBlock;
        kb_lo = lo, kb_hi = hi, last2 = w2_kblocks - 1;
        kb_hi2 = hi < w2_kblocks ? hi : w2_kblocks;
        request(a1, a2, lo);
        request(b1, b2, lo + kG);
    }
    __device__ inline void multiply(const frag (&f1)[kG], const frag (&f2)[kG], int kb, const char *ap, floatx4 &acc1, floatx4 &acc2) const
    {
#pragma unroll
        for (int u = 0; u < kG; ++u)
            if (kb + u < kb_hi) {
                const frag a = P::load_a(ap, kb + u, lane_id() >> 4);
                P::mma(acc1, a, f1[u]);
                if (kb + u < kb_hi2)
                    P::mma(acc2, a, f2[u]);
            }
    }
    __device__ inline void run(floatx4 &acc1, floatx4 &acc2, const char *A, int lda)
    {
        const char *ap = A + (size_t)(lane_id() & 15) * lda;
        int kb = kb_lo;
        for (; kb + 2 * kG < kb_hi; kb += 2 * kG) {
            multiply(a1, a2, kb, ap, acc1, acc2);
            request(a1, a2, kb + 2 * kG);
            multiply(b1, b2, kb + kG, ap, acc1, acc2);
            request(b1, b2, kb + 3 * kG);
        }
        multiply(a1, a2, kb, ap, acc1, acc2);
        multiply(b1, b2, kb + kG, ap, acc1, acc2);
    }
};

// KIND: an ordinary step; the state update of a module selection (the plain recurrent cell, library exp / tanh), with last
// messages and with mean ones; a training step, which keeps what its backward pass reads.  Instances of their own, so that the
// ordinary one carries nothing of the others (in one kernel they cost a step 2 us and 1 us; last and mean messages in one
// instance spilled 104 scalar registers instead of 69 and 83, and steps of 200 to 2000 events took 0.5 to 1.3 us more: mean messages,
// GRU, attention 38.4 -> 37.7 at 200 narrow events, 63.2 -> 61.9 at 2000 of 100 columns; last, RNN, projection 14.3 -> 13.8).
// Spilled in the others: 35 scalar registers (bf16), 58 (fp32), 79 (training), to lanes of vector registers, and none of these: a
// wavefront's six row descriptors, the weights' bases and the closing work's arguments are alive together.  (Arguments read again
// where they are used, from a pointer that the compiler cannot see through: none spilled, and every step 0.8 to 1.4 us longer.)
enum GruKind { kGruPlain, kGruModules, kGruMeans, kGruTraining };
template <int PREC, GruKind KIND>
__global__ void __launch_bounds__(kGruThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))  // 128 registers: two workgroups per unit
k_gru(StepArgs a, GruJob gj, PackedWeights w, GruParams g, DecodeParams dp)
{
    constexpr bool means = KIND == kGruMeans, MOD = KIND == kGruModules || means, TRAIN = KIND == kGruTraining;
    TIG_MARK(0);
    if (blockIdx.x == 0 && threadIdx.x == 0 && g.clear)
        *g.clear = 0;
    if ((int)blockIdx.x >= g.n_gru) {
        int x = (int)blockIdx.x - g.n_gru;
        if (x < g.n_row_blocks) {  // finishing pass of this step's query preparation
            int n_u = *a.qs.n_u;
            n_u = n_u < 2 * a.count ? n_u : 2 * a.count;
            for (int row = x * kGruWaves + wave_id(); row < n_u; row += g.n_row_blocks * kGruWaves)
                finish_row(ref_ctx(a), a.qs, dp.K, row);
        } else if ((x -= g.n_row_blocks) < g.n_slot_blocks) {
            const int i = x * kGruThreads + (int)threadIdx.x;
            if (i < 2 * a.count)
                finish_slots(a.qs, i, 2 * a.count);
        } else {
            closing_block(a, w, dp, x - g.n_slot_blocks, kGruWaves);
        }
        TIG_MARK(1);
        return;
    }
    using P = Prec<PREC>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int *row_i = (int *)smem;                  // [EC] entry 2b + role
    int *row_u = row_i + EC;                   // [EC] node
    int *row_o = row_u + EC;                   // [EC] partner
    int *row_e = row_o + EC;                   // [EC] event id - first_eid
    double *row_t = (double *)(row_e + EC);    // [EC] event time
    char *X = smem + EC * 24;                  // [EC rows x ldx bytes]
    float *part = (float *)(smem + g.off_part);  // [2 halves][kPairs][2 streams][16 x 16]

    const int lane = lane_id();
    const int wave_u = wave_id_uniform();

    // the work: tiles x column slices.  The first item's descriptors are requested together with the winner
    // count, at the slice count that comes with the launch (slots beyond the count hold stale
    // descriptors of earlier batches or nothing: they are only used below the count).
    const int n_ct = g.Ng / 16;
    WinDesc d_first;
    {
        const int r = ((int)blockIdx.x / g.guess.slices) * EC + (int)threadIdx.x;
        if (threadIdx.x < EC && r < 2 * gj.count)
            d_first = gj.win[r];
    }
    int n_win = *gj.n_win;
    n_win = n_win < 2 * gj.count ? n_win : 2 * gj.count;  // (a list never holds more than the batch's entries)
    const int tiles = (n_win + EC - 1) / EC;
    if (tiles == 0)
        return;
    // (a product's sum is split where an item has few columns, so the slices follow the winners that there are: those
    // of earlier steps, which the launch knows, would show in the last bits.  Three divisions here took 0.35 us of every step)
    const int wide = winner_tiles(n_win, 2 * gj.count, EC);
    const bool foreseen = slices_hold(g.guess, g.n_gru, wide);
    const ColumnSlices now = foreseen ? g.guess : column_slices(n_ct, g.n_gru, wide);
    const int cs = now.slices, tpp = now.tiles;  // column tiles per item
    const int items = tiles * cs;
    const int kblocks = g.Kg / P::KB;
    const int kblocks_hn = g.Khn / P::KB;

    for (int item = (int)blockIdx.x; item < items; item += g.n_gru) {
        // 1. this item's slice of the compacted winner list
        const int r0 = (item / cs) * EC;
        const int ct_lo = (item % cs) * tpp;
        const int ct_hi = n_ct < ct_lo + tpp ? n_ct : ct_lo + tpp;
        const int n_rows = n_win - r0 < EC ? n_win - r0 : EC;
        if (threadIdx.x < EC) {
            const int r = threadIdx.x;
            int i = 0, u = 0, o = 0, b = 0;
            double t = 0.0;
            if (r < n_rows) {
                const WinDesc d0 = item == (int)blockIdx.x && foreseen ? d_first : gj.win[r0 + r];
                i = d0.entry;
                u = d0.node;
                o = d0.other;
                b = d0.b;
                t = d0.t;
            }
            row_i[r] = i;
            row_u[r] = u;
            row_o[r] = o;
            row_e[r] = b;
            row_t[r] = t;
        }
        lds_barrier();
        TIG_MARK(1);

        // The gates' weights.  A round covers up to kPairs column tiles; with fewer, the pairs also split k.
        GateStream<PREC, PREC == TIG_BF16_MFMA ? 1 : 2> gate;
        const int half = wave_u / kPairs;  // 0: r and z gates, 1: n gate (input part over the whole message, hidden part over s_self)
        const int pair = wave_u % kPairs;
        auto begin_round = [&](int base) {
            const int cts = ct_hi - base < kPairs ? ct_hi - base : kPairs;
            const int ksplit = cts == 1 ? 4 : (cts == 2 ? 2 : 1), ctl = pair / ksplit;
            const int per = (kblocks + ksplit - 1) / ksplit, kb_lo = pair % ksplit * per;
            const int kb_hi = kblocks < kb_lo + per ? kblocks : kb_lo + per;
            if (ctl >= cts || kb_lo >= kb_hi)
                return;
            if (half == 0)
                gate.start(w.gru_Wr, w.gru_Wz, kblocks, kblocks, kb_lo, kb_hi, base + ctl);
            else
                gate.start(w.gru_Win, w.gru_Whn, kblocks, kblocks_hn, kb_lo, kb_hi, base + ctl);
        };
        // (the plain recurrent cell has one gate, whose products go another way)
        const bool streams = !MOD || a.upd != kUpdModuleRnn;

        // 2. message rows [s_self | s_other | Phi(dt) | e] from batch-start memory (mean messages: [s_self | mean]).  One
        //    wavefront per row, segment by segment with the lanes from the segment's first column on, through buffer
        //    descriptors in scalar registers: a lane beyond the segment reads 0, no load is conditional (such a load
        //    is waited for at the condition's end) and no lane has an address to compute (with one per lane, chosen
        //    among the segments, it was 900 vector instructions a wavefront, 4.7 us for rows of 616 columns).  The loads of both
        //    of a wavefront's rows are requested before the first is stored, and behind them the first weights.
        {
            constexpr int kRowsPerWave = EC / kGruWaves, kPieces = 3;  // 192 columns of a segment at a time
            int lane = lane_id();
            asm volatile("" : "+v"(lane));  // (addresses are not taken out of the loop over the items: there are no registers for them)
            // (a mean's columns are taken as two segments, so that their loads are in flight together)
            const int mean = g.M + g.T + g.F, second = means ? (mean + 1) / 2 : g.M, third = means ? mean - second : g.F;
            const int wider = second > third ? second : third, widest = means && g.M > wider ? g.M : wider;
            __amdgpu_buffer_rsrc_t rs[kRowsPerWave], ro[kRowsPerWave], rf[kRowsPerWave];
            double since[kRowsPerWave];
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i) {
                const int r = wave_u + i * kGruWaves;
                const bool live = r < n_rows;  // (a row beyond reads 0)
                const int u = __builtin_amdgcn_readfirstlane(row_u[r]), o = __builtin_amdgcn_readfirstlane(row_o[r]);
                const int e = __builtin_amdgcn_readfirstlane(row_e[r]), entry = __builtin_amdgcn_readfirstlane(row_i[r]);
                const float *self = a.mem + (size_t)u * g.M;
                const float *other = means ? a.mean_msg + (size_t)entry * mean : a.mem + (size_t)o * g.M;
                const float *feat = means ? other + second : a.edge_feat + (size_t)(gj.first_eid + e) * g.F;
                rs[i] = __builtin_amdgcn_make_buffer_rsrc((void *)self, 0, live ? 4 * g.M : 0, kBufferFlags);
                ro[i] = __builtin_amdgcn_make_buffer_rsrc((void *)other, 0, live ? 4 * second : 0, kBufferFlags);
                rf[i] = __builtin_amdgcn_make_buffer_rsrc((void *)feat, 0, live ? 4 * third : 0, kBufferFlags);
                since[i] = means ? 0.0 : a.lu[u];
            }
            double tw_w[kPhi], tw_b[kPhi];  // time-encoding parameters of the lane's first columns
#pragma unroll
            for (int k = 0; k < kPhi; ++k) {
                const int j = lane + kWave * k < g.T ? lane + kWave * k : 0;
                tw_w[k] = w.time_w_rev[j];
                tw_b[k] = w.time_b_rev[j];
            }
            for (int c0 = 0; c0 < widest; c0 += kWave * kPieces) {
                float v[kRowsPerWave][3][kPieces];
#pragma unroll
                for (int i = 0; i < kRowsPerWave; ++i)
#pragma unroll
                    for (int k = 0; k < kPieces; ++k) {
                        const uint32_t at = 4u * (uint32_t)(c0 + lane + kWave * k);
                        v[i][0][k] = buffer_load_f32(rs[i], at);
                        v[i][1][k] = buffer_load_f32(ro[i], at);
                        v[i][2][k] = buffer_load_f32(rf[i], at);
                    }
                __builtin_amdgcn_sched_barrier(0);
                if (c0 == 0 && streams)
                    begin_round(ct_lo);
#pragma unroll
                for (int i = 0; i < kRowsPerWave; ++i) {
                    const int r = wave_u + i * kGruWaves;
                    char *const x = X + (size_t)r * g.ldx;
                    float *const keep = TRAIN && ct_lo == 0 && r < n_rows ? a.gru_msg + (size_t)(r0 + r) * g.Dmsg : nullptr;
#pragma unroll
                    for (int seg = 0; seg < 3; ++seg) {
                        const int width = seg == 0 ? g.M : (seg == 1 ? second : third);
                        const int at = seg == 0 ? 0 : (seg == 1 ? g.M : (means ? g.M + second : 2 * g.M + g.T));
#pragma unroll
                        for (int k = 0; k < kPieces; ++k) {
                            const int j = c0 + lane + kWave * k;
                            if (j < width) {
                                P::store_a(x, at + j, v[i][seg][k]);
                                if (TRAIN && keep)
                                    keep[at + j] = v[i][seg][k];
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i)
                since[i] = row_t[wave_u + i * kGruWaves] - since[i];  // since the node's last update
            auto phi = [&](int j, double w_rev, double b_rev) {
#pragma unroll
                for (int i = 0; i < kRowsPerWave; ++i) {
                    const int r = wave_u + i * kGruWaves;
                    // (uniform; what stands in a row beyond reaches no other.  Computed for all sixteen rows: steps of 1 to 16 events 0.2 us
                    // more; left out in the other instances, 0 to 0.4 us more)
                    if (KIND == kGruPlain && PREC == TIG_FP32 && r >= n_rows)
                        continue;
                    const float x = time_enc(w_rev, b_rev, since[i]);
                    P::store_a(X + (size_t)r * g.ldx, 2 * g.M + j, x);
                    if (TRAIN && ct_lo == 0 && r < n_rows)
                        a.gru_msg[(size_t)(r0 + r) * g.Dmsg + 2 * g.M + j] = x;
                }
            };
            if (!means) {
#pragma unroll
                for (int k = 0; k < kPhi; ++k)
                    if (lane + kWave * k < g.T)
                        phi(lane + kWave * k, tw_w[k], tw_b[k]);
                for (int j = lane + kWave * kPhi; j < g.T; j += kWave)
                    phi(j, w.time_w_rev[j], w.time_b_rev[j]);
            }
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i)  // the k-depth's padding
                if (lane < g.Kg - g.Dmsg)
                    P::store_a(X + (size_t)(wave_u + i * kGruWaves) * g.ldx, g.Dmsg + lane, 0.0f);
        }
        lds_barrier();
        TIG_MARK(2);

        // 3. + 4. gates
        for (int base = ct_lo; base < ct_hi; base += kPairs) {
            const int cts = ct_hi - base < kPairs ? ct_hi - base : kPairs;  // column tiles of this round
            const int ksplit = cts == 1 ? 4 : (cts == 2 ? 2 : 1);
            const int ctl = pair / ksplit;   // column tile of the round
            const int ks = pair % ksplit;    // k slice
            // gate biases of the element this thread finishes below, requested with the weights
            float pb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if ((int)threadIdx.x < cts * 256) {
                const int col = (base + ((int)threadIdx.x >> 8)) * 16 + ((int)threadIdx.x & 15);
                pb[0] = w.gru_br[col];
                pb[1] = w.gru_bz[col];
                pb[2] = w.gru_bin[col];
                pb[3] = w.gru_bhn[col];
            }
            floatx4 acc1 = floatx4{0, 0, 0, 0}, acc2 = floatx4{0, 0, 0, 0};
            {
                const int per = (kblocks + ksplit - 1) / ksplit;
                const int kb_lo = ks * per;
                const int kb_hi = kblocks < kb_lo + per ? kblocks : kb_lo + per;
                if (ctl < cts && kb_lo < kb_hi) {
                    if (!streams) {  // one gate: the halves of a pair split its k range once more
                        floatx4 one[1] = {acc1};
                        const int mid = kb_lo + (kb_hi - kb_lo + 1) / 2, lo = half ? mid : kb_lo, hi = half ? kb_hi : mid;
                        tile_gemm<PREC, 1, 4>(one, X, g.ldx, lo, w.gru_Wr, kblocks, lo, hi - lo, base + ctl);
                        acc1 = one[0];
                    } else {
                        if (base != ct_lo)
                            begin_round(base);
                        gate.run(acc1, acc2, X, g.ldx);
                    }
                }
            }
            {
                float *p1 = part + (size_t)((half * kPairs + pair) * 2) * 256;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int e = (4 * (lane >> 4) + v) * 16 + (lane & 15);
                    p1[e] = acc1[v];
                    p1[256 + e] = acc2[v];
                }
            }
            lds_barrier();
            TIG_MARK(3);
            for (int idx = threadIdx.x; idx < cts * 256; idx += kGruThreads) {
                const int ctl2 = idx >> 8, e = idx & 255;
                const int row = e >> 4, col = (base + ctl2) * 16 + (e & 15);
                if (row < n_rows && col < g.M) {
                    float sr = 0.0f, sz = 0.0f, sin_ = 0.0f, shn = 0.0f;
                    for (int k2 = 0; k2 < ksplit; ++k2) {
                        const float *q0 = part + (size_t)((ctl2 * ksplit + k2) * 2) * 256;
                        const float *q1 = part + (size_t)((kPairs + ctl2 * ksplit + k2) * 2) * 256;
                        sr += q0[e];
                        sz += q0[256 + e];
                        sin_ += q1[e];
                        shn += q1[256 + e];
                    }
                    const bool pre = idx < kGruThreads;  // the preloaded biases are this element's
                    const float br = pre ? pb[0] : w.gru_br[col], bz = pre ? pb[1] : w.gru_bz[col];
                    const float bin = pre ? pb[2] : w.gru_bin[col], bhn = pre ? pb[3] : w.gru_bhn[col];
                    const float h = P::load_elem(X + (size_t)row * g.ldx, col);  // s_self
                    float r, z, n;
                    if (!MOD) {
                        r = 1.0f / (1.0f + __expf(-(sr + br)));
                        z = 1.0f / (1.0f + __expf(-(sz + bz)));
                        const float x = sin_ + bin + r * (shn + bhn);
                        const float e2 = __expf(2.0f * x);          // tanh(x) = 1 - 2 / (e^{2x} + 1)
                        n = 1.0f - 2.0f / (e2 + 1.0f);
                    } else if (a.upd == kUpdModuleGru) {
                        r = 1.0f / (1.0f + expf(-(sr + br)));
                        z = 1.0f / (1.0f + expf(-(sz + bz)));
                        n = tanhf(sin_ + bin + r * (shn + bhn));
                    } else {  // s = tanh(W_i m + b_i + W_h s' + b_h): both halves' sums make up the one gate
                        r = z = 0.0f;
                        n = tanhf(sr + sin_ + br);
                    }
                    a.staging[(size_t)row_i[row] * g.M + col] = (1.0f - z) * n + z * h;
                    if (TRAIN) {
                        float *go = a.gru_gates + (size_t)(r0 + row) * 4 * g.M + col;
                        a.d_staging[(size_t)row_i[row] * g.M + col] = 0.0f;
                        go[0] = r;
                        go[g.M] = z;
                        go[2 * g.M] = n;
                        go[3 * g.M] = shn + bhn;
                    }
                }
            }
            lds_barrier();  // the partial sums (and, after the last round, the tile) are reused
        }
    }
    TIG_MARK(4);
}

GruParams gru_params(const Dims &d)
{
    GruParams g;
    g.M = d.M;
    g.T = d.T;
    g.F = d.F;
    g.Dmsg = d.Dmsg;
    g.Kg = d.Kg;
    g.Khn = d.Khn;
    g.Ng = d.Ng;
    g.ldx = lds_row_bytes(d.Kg);
    g.off_part = (EC * 24 + EC * g.ldx + 15) / 16 * 16;
    g.n_gru = 0;
    g.guess = ColumnSlices{1, 1, 0};
    g.n_row_blocks = 0;
    g.n_slot_blocks = 0;
    g.clear = nullptr;
    return g;
}

const void *gru_kernel(const Dims &d, int upd, bool means, bool train)
{
    if (train)
        return (const void *)k_gru<TIG_FP32, kGruTraining>;
    if (d.prec == TIG_BF16_MFMA)  // (module selections run in fp32 contexts)
        return (const void *)k_gru<TIG_BF16_MFMA, kGruPlain>;
    if (upd == kUpdGru)
        return (const void *)k_gru<TIG_FP32, kGruPlain>;
    return means ? (const void *)k_gru<TIG_FP32, kGruMeans> : (const void *)k_gru<TIG_FP32, kGruModules>;
}

// GRU workgroups and column slices for a batch of `count` events with about `wins_est` winners.
void size_gru(const Dims &d, const LaunchPlan &plan, int count, int wins_est, GruParams *g)
{
    // one workgroup per compute unit, but no more than the work of the largest possible winner
    // count (every entry a winner, every column tile its own item); none if nothing is applied
    const int cus = plan.num_cus > 0 ? plan.num_cus : 256;
    const int max_items = (2 * count + EC - 1) / EC * (d.Ng / 16);
    g->n_gru = max_items < cus ? max_items : cus;
    // (at the winner count that recent steps had: hub nodes make it a small share of the 2 * count entries)
    const int wins = wins_est > 0 ? wins_est - wins_est / 9 : 2 * count;  // (the estimate is an eighth above them)
    g->guess = column_slices(d.Ng / 16, g->n_gru, winner_tiles(wins, 2 * count, EC));
}

DecodeParams no_closing(const Dims &d)
{
    DecodeParams p;
    p.M = d.M;
    p.E = d.E;
    p.Ep = d.Ep;
    p.K = d.K;
    p.n_event_blocks = p.n_expand_blocks = p.n_fin_row_blocks = p.n_fin_slot_blocks = 0;
    return p;
}

}  // namespace

int gru_lds_bytes(const Dims &d)
{
    return gru_params(d).off_part + 2 * kPairs * 2 * 256 * 4;
}

hipError_t prepare_gru(const Dims &d, const LaunchPlan &plan)
{
    for (int i = 0; i < 4; ++i) {
        const void *const kernel = gru_kernel(d, i == 1 || i == 3 ? kUpdModuleGru : kUpdGru, i == 3, i == 2 && d.prec == TIG_FP32);
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, gru_lds_bytes(d));
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// Ahead of the embedding launch: the GRU of the batch this step applies and, if asked for, the
// finishing pass of this step's queries.
hipError_t launch_gru(const Dims &d, const LaunchPlan &plan, const PackedWeights &pw, const StepArgs &a,
                      hipStream_t s, bool gru_work)
{
    StepArgs aa = a;
    PackedWeights ww = pw;
    GruParams g = gru_params(d);
    GruJob gj = {a.msg_first_eid, gru_work ? a.msg_count : 0, a.win, a.n_win};
    DecodeParams dp = no_closing(d);
    size_gru(d, plan, gj.count, a.wins_est, &g);
    if (a.finish_here) {
        const int cus = plan.num_cus > 0 ? plan.num_cus : 256;
        const int rows = 2 * a.count;  // at most; a wavefront takes several rows if there are many
        g.n_row_blocks = (rows + kGruWaves - 1) / kGruWaves;
        if (g.n_row_blocks > 2 * cus)
            g.n_row_blocks = 2 * cus;
        g.n_slot_blocks = (2 * a.count + kGruThreads - 1) / kGruThreads;
    }
    const int blocks = g.n_gru + g.n_row_blocks + g.n_slot_blocks;
    if (blocks == 0)
        return hipSuccess;  // nothing to apply, nothing to finish
    void *args[] = {&aa, &gj, &ww, &g, &dp};
    return hipLaunchKernel(gru_kernel(d, a.upd, a.mean_msg != nullptr, a.gru_gates != nullptr), dim3(blocks), dim3(kGruThreads), args, (size_t)gru_lds_bytes(d), s);
}

// The closing launch of a step: scores and embedding rows of its events, inspection outputs, the
// finishing pass of the batch prepared ahead; its own query set's counter is cleared for the
// set's next preparation; and, if ahead.count > 0, the GRU of the batch the next step applies.
hipError_t launch_closing(const Dims &d, const LaunchPlan &plan, const PackedWeights &pw, const StepArgs &a,
                          const GruAhead &ahead, hipStream_t s, bool events)
{
    StepArgs aa = a;
    PackedWeights ww = pw;
    GruParams g = gru_params(d);
    GruJob gj = {ahead.first_eid, ahead.count, ahead.win, ahead.n_win};
    if (ahead.count > 0)
        size_gru(d, plan, ahead.count, a.wins_est, &g);
    g.clear = a.qs.n_u;
    DecodeParams p = no_closing(d);
    p.n_event_blocks = events ? (a.count + kGruWaves - 1) / kGruWaves : 0;  // (a training step decodes itself)
    const bool expand = wants_inspection(a);
    p.n_expand_blocks = expand ? (a.roles * a.count + kGruWaves - 1) / kGruWaves : 0;
    if (a.fin_count > 0) {
        p.n_fin_row_blocks = (2 * a.fin_count + kGruWaves - 1) / kGruWaves;
        if (p.n_fin_row_blocks > 128)
            p.n_fin_row_blocks = 128;
        p.n_fin_slot_blocks = (2 * a.fin_count + kGruThreads - 1) / kGruThreads;
    }
    int blocks = g.n_gru + p.n_event_blocks + p.n_expand_blocks + p.n_fin_row_blocks + p.n_fin_slot_blocks;
    blocks = blocks > 0 ? blocks : 1;  // (block 0 clears the counter whatever else there is to do)
    void *args[] = {&aa, &gj, &ww, &g, &p};
    return hipLaunchKernel(gru_kernel(d, a.upd, a.mean_msg != nullptr, false), dim3(blocks), dim3(kGruThreads), args, (size_t)gru_lds_bytes(d), s);
}

}  // namespace tig
