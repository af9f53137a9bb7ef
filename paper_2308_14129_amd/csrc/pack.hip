// Weight preparation (once, in tig_init): algebraic folding in fp64, zero padding to matrix-core
// tile sizes, and re-ordering so that every wavefront operand load is one contiguous 1 KiB read.
//
// Foldings (exact algebra on the attention embedding f and merge MLP of Sec. II-C):
//   * scores: <Q_h, W_K,h kv + b_K,h> / sqrt(d_h) = <q~_h, kv> + const, with
//       q~_h = (W_K,h^T W_Q[h, :M] / sqrt(d_h)) s_u + W_K,h^T (W_Q[h, M:] Phi(0) + b_Q,h) / sqrt(d_h);
//     the constant is the same for every neighbour slot and cancels in the softmax;
//   * values: sum_k a_k (W_V,h kv_k + b_V,h) = W_V,h (sum_k a_k kv_k) + b_V,h   (sum_k a_k = 1);
//   * out-projection and the first merge layer are linear in that sum, so
//       W_m1 [attn | s_u] + b_m1 = sum_h (W_m1a W_O[:, h] W_V,h) kvbar_h + W_m1m s_u
//                                  + b_m1 + W_m1a (W_O b_V + b_O);
//   * GRU: the hidden products of the r and z gates act on s_u, which is also the first M
//     entries of the message, so W_hr / W_hz are added onto those columns of W_ir / W_iz.
#include <hip/hip_runtime.h>

#include "tig_internal.h"

namespace tig {

namespace {

constexpr int kThreads = 256;

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *p) : base((char *)p) {}
    template <typename T>
    T *take(size_t count)
    {
        T *p = base ? (T *)(base + off) : nullptr;
        off += align_up(sizeof(T) * count);
        return p;
    }
};

// C[i*ldc + j] = c0[i] + C[..] (if add) + alpha * sum_k A[i*ars + k*acs] * B[k*brs + j*bcs]   (fp64 accumulate)
// A preparation is a dozen of such small products and as many copies: launched one by one they took 0.45 ms
// (launch after launch of 1 - 20 us each, five dozen in all); every stage of independent ones is one launch
// now (blockIdx.y names the product): 0.08 ms.
struct FoldJob {
    double *C;
    const void *A, *B;
    const float *c0;     // NULL, or added per row
    int ldc, ars, acs, brs, bcs, m, n, kdim;
    double alpha;
    bool a64, b64, add;  // operands in double; the previous value of C is added
    bool b_cos;          // B is taken as cos(B)
};
constexpr int kMaxFoldJobs = 25;  // of four heads
struct FoldJobs {
    FoldJob j[kMaxFoldJobs];
    int n;
};

template <typename TA, typename TB>
__device__ inline double fold_dot(const TA *A, int acs, const TB *B, int brs, int kdim, bool b_cos)
{
    // four partial sums: the loads of four steps are in flight together and the adds do not wait for each other
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int k = 0;
    if (b_cos) {
        for (; k < kdim; ++k)
            acc[k < (kdim & ~3) ? k & 3 : 0] += (double)A[(size_t)k * acs] * cos((double)B[(size_t)k * brs]);
        return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    }
    for (; k + 4 <= kdim; k += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            acc[u] += (double)A[(size_t)(k + u) * acs] * (double)B[(size_t)(k + u) * brs];
    }
    for (; k < kdim; ++k)
        acc[0] += (double)A[(size_t)k * acs] * (double)B[(size_t)k * brs];
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

__global__ void __launch_bounds__(kThreads) k_fold(FoldJobs jobs)
{
    const FoldJob &q = jobs.j[blockIdx.y];
    const int idx = blockIdx.x * kThreads + threadIdx.x;
    if (idx >= q.m * q.n)
        return;
    const int i = idx / q.n, j = idx % q.n;
    const size_t ao = (size_t)i * q.ars, bo = (size_t)j * q.bcs;
    double v;
    if (q.a64)
        v = q.b64 ? fold_dot((const double *)q.A + ao, q.acs, (const double *)q.B + bo, q.brs, q.kdim, false)
                  : fold_dot((const double *)q.A + ao, q.acs, (const float *)q.B + bo, q.brs, q.kdim, false);
    else
        v = q.b64 ? fold_dot((const float *)q.A + ao, q.acs, (const double *)q.B + bo, q.brs, q.kdim, false)
                  : fold_dot((const float *)q.A + ao, q.acs, (const float *)q.B + bo, q.brs, q.kdim, q.b_cos);
    double *c = q.C + (size_t)i * q.ldc + j;
    double base = q.add ? *c : 0.0;
    if (q.c0)
        base += (double)q.c0[i];
    *c = base + q.alpha * v;
}

hipError_t fold(hipStream_t s, const FoldJobs &jobs)
{
    int most = 1;
    for (int i = 0; i < jobs.n; ++i)
        most = jobs.j[i].m * jobs.j[i].n > most ? jobs.j[i].m * jobs.j[i].n : most;
    hipLaunchKernelGGL(k_fold, dim3((most + kThreads - 1) / kThreads, jobs.n), dim3(kThreads), 0, s, jobs);
    return hipGetLastError();
}

__global__ void k_to_revolutions(double *out, const float *in, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = (double)in[i] / 6.283185307179586476925286766559;
}

__device__ inline uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Lane-ordered layout read by the tile GEMMs: for output tile nt (16 rows of W), k-block kb,
// lane l: VL consecutive k's  W[nt*16 + l%16][kb*KB + VL*(l/16) + 0..VL-1], VL = KB/4.
// fp32: 4 floats per lane.  bf16: 8 values per lane, split as x = hi + lo with hi = bf16(x),
// lo = bf16(x - hi): 8 hi values (16 bytes) followed by the 8 lo values (16 bytes).
// Either way an element takes 4 bytes and one wavefront operand load is contiguous.
// Element idx of a prepared [rows_p x cols_p] matrix: value(r, c) of the source (0 in the padding).
template <bool BF16, typename F>
__device__ inline void pack_element(void *out, size_t idx, int rows, int cols, int cols_p, F value)
{
    constexpr int KB = BF16 ? 32 : 16;
    constexpr int VL = KB / 4;
    const int s = (int)(idx % VL);
    const int lane = (int)((idx / VL) % 64);
    const size_t blk = idx / (VL * 64);
    const int kbs = cols_p / KB;
    const int kb = (int)(blk % kbs);
    const int nt = (int)(blk / kbs);
    const int r = nt * 16 + (lane % 16);
    const int c = kb * KB + VL * (lane / 16) + s;
    float v = 0.0f;
    if (r < rows && c < cols)
        v = value(r, c);
    if (BF16) {
        uint16_t *o = (uint16_t *)out + (blk * 64 + lane) * 16 + s;
        const uint16_t hi = f32_to_bf16_rne(v);
        o[0] = hi;
        o[8] = f32_to_bf16_rne(v - __uint_as_float((uint32_t)hi << 16));
    } else {
        ((float *)out)[idx] = v;
    }
}

// What the embedding and closing launches read, out of the folded products: prepared matrices and padded
// vectors, one launch (blockIdx.y names the piece).
struct PackMat {
    void *out;
    const void *W, *W2;      // columns >= split come from W2 (both row-major, double or float)
    int ld, ld2, split;
    int rows, cols, rows_p, cols_p;
    int half, gap;           // rows >= half: taken `gap` rows earlier from W2h (a matrix of two stacked halves); 0: none
    const void *W2h;
    bool w64, w264;
};
struct PackVec {
    float *out;
    int n, n_pad;
    const double *a, *a2;    // terms, each may be NULL
    const float *b;
};
constexpr int kPackMats = 5, kPackVecs = 8;
struct PackJobs {
    PackMat m[kPackMats];
    PackVec v[kPackVecs];
};

__device__ inline float pack_value(const void *W, size_t i, bool w64)
{
    return w64 ? (float)((const double *)W)[i] : ((const float *)W)[i];
}

template <bool BF16>
__global__ void __launch_bounds__(kThreads) k_pack(PackJobs jobs)
{
    const size_t idx = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const int piece = blockIdx.y;
    if (piece < kPackMats) {
        const PackMat &q = jobs.m[piece];
        if (idx < (size_t)q.rows_p * q.cols_p)
            pack_element<BF16>(q.out, idx, q.rows, q.cols, q.cols_p, [&](int r, int c) {
                if (q.half > 0) {  // two stacked halves of half - gap rows each, zero rows between and after
                    const int h = r >= q.half ? 1 : 0, rr = h ? r - q.half : r;
                    return rr < q.half - q.gap ? pack_value(h ? q.W2h : q.W, (size_t)rr * q.ld + c, q.w64) : 0.0f;
                }
                return c < q.split ? pack_value(q.W, (size_t)r * q.ld + c, q.w64)
                                   : pack_value(q.W2, (size_t)r * q.ld2 + (c - q.split), q.w264);
            });
    } else {
        const PackVec &q = jobs.v[piece - kPackMats];
        if (idx < (size_t)q.n_pad) {
            double v = 0.0;
            if (idx < (size_t)q.n) {
                if (q.a)
                    v += q.a[idx];
                if (q.a2)
                    v += q.a2[idx];
                if (q.b)
                    v += (double)q.b[idx];
            }
            q.out[idx] = (float)v;
        }
    }
}

// Everything the state update's kernels read, prepared in one launch (a training step rebuilds it
// after every update of the masters): blockIdx.y names the piece -- 0, 1 the time encoding's
// parameters in revolutions; 2, 3 the r and z gates' matrices with the hidden weights folded onto the
// s_self columns (added in double precision); 4, 5 the n gate's input and hidden matrices; 6..9 the
// bias vectors (b_ir + b_hr, b_iz + b_hz, b_in, b_hn).
struct GruPackJob {
    double *time_w_rev, *time_b_rev;
    const float *time_w, *time_b, *W_i, *W_h, *b_i, *b_h;
    void *Wr, *Wz, *Win, *Whn;
    float *br, *bz, *bin, *bhn;
    int M, T, Dmsg, Ng, Kg, Khn;
    bool rnn;  // one gate only (pieces 0, 1, 2 and 6)
};

template <bool BF16>
__global__ void k_pack_gru(GruPackJob j)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int piece = blockIdx.y, M = j.M, D = j.Dmsg;
    if (j.rnn && piece > 2 && piece != 6)
        return;
    if (piece < 2) {
        if (idx < (size_t)j.T)
            (piece ? j.time_b_rev : j.time_w_rev)[idx] = (double)(piece ? j.time_b : j.time_w)[idx] / 6.283185307179586476925286766559;
    } else if (piece < 4) {
        const float *Wi = j.W_i + (size_t)(piece - 2) * M * D, *Wh = j.W_h + (size_t)(piece - 2) * M * M;
        if (idx < (size_t)j.Ng * j.Kg)
            pack_element<BF16>(piece == 2 ? j.Wr : j.Wz, idx, M, D, j.Kg, [&](int r, int c) {
                double v = (double)Wi[(size_t)r * D + c];
                if (c < M)
                    v += (double)Wh[(size_t)r * M + c];
                return (float)v;
            });
    } else if (piece == 4) {
        const float *W = j.W_i + (size_t)2 * M * D;
        if (idx < (size_t)j.Ng * j.Kg)
            pack_element<BF16>(j.Win, idx, M, D, j.Kg, [&](int r, int c) { return W[(size_t)r * D + c]; });
    } else if (piece == 5) {
        const float *W = j.W_h + (size_t)2 * M * M;
        if (idx < (size_t)j.Ng * j.Khn)
            pack_element<BF16>(j.Whn, idx, M, M, j.Khn, [&](int r, int c) { return W[(size_t)r * M + c]; });
    } else if (idx < (size_t)j.Ng) {
        const int i = (int)idx, g = piece - 6;  // 0: r, 1: z, 2: n (input side), 3: n (hidden side)
        double v = 0.0;
        if (i < M) {
            if (g < 2)
                v = (double)j.b_i[g * M + i] + (double)j.b_h[g * M + i];
            else
                v = (double)(g == 2 ? j.b_i : j.b_h)[2 * M + i];
        }
        (g == 0 ? j.br : g == 1 ? j.bz : g == 2 ? j.bin : j.bhn)[i] = (float)v;
    }
}

struct PackedLayout {
    double *time_w_rev, *time_b_rev;
    void *gru_Wr, *gru_Wz, *gru_Win, *gru_Whn;
    float *gru_br, *gru_bz, *gru_bin, *gru_bhn;
    void *emb_A1;
    float *emb_a1;
    void *emb_PR;
    float *emb_c, *emb_c0;
    void *emb_Wm2;
    float *emb_bm2;
    void *dec_W, *dec_WF;
    float *dec_b1, *dec_b1f, *dec_w2, *dec_b2;
    size_t bytes;
};

PackedLayout layout(const Dims &d, void *base)
{
    Carver c(base);
    PackedLayout L;
    const size_t e = (size_t)d.esz;
    L.time_w_rev = c.take<double>(d.T);
    L.time_b_rev = c.take<double>(d.T);
    L.gru_Wr = c.take<char>(e * d.Ng * d.Kg);
    L.gru_Wz = c.take<char>(e * d.Ng * d.Kg);
    L.gru_Win = c.take<char>(e * d.Ng * d.Kg);
    L.gru_Whn = c.take<char>(e * d.Ng * d.Khn);
    L.gru_br = c.take<float>(d.Ng);
    L.gru_bz = c.take<float>(d.Ng);
    L.gru_bin = c.take<float>(d.Ng);
    L.gru_bhn = c.take<float>(d.Ng);
    L.emb_A1 = c.take<char>(e * d.N1 * d.Mq);
    L.emb_a1 = c.take<float>(d.N1);
    L.emb_PR = c.take<char>(e * d.Ep * d.K2);
    L.emb_c = c.take<float>(d.Ep);
    L.emb_c0 = c.take<float>(d.Ep);
    L.emb_Wm2 = c.take<char>(e * d.Ep * d.Ek);
    L.emb_bm2 = c.take<float>(d.Ep);
    L.dec_W = c.take<char>(e * 2 * d.Ep * d.Ek);
    L.dec_b1 = c.take<float>(d.Ep);
    L.dec_WF = c.take<char>(e * 2 * d.Ep * d.Ek);
    L.dec_b1f = c.take<float>(d.Ep);
    L.dec_w2 = c.take<float>(d.Ep);
    L.dec_b2 = c.take<float>(1);
    L.bytes = c.off;
    return L;
}

struct ScratchLayout {
    double *cQ, *A1, *a1, *G, *P, *cvec, *cvec2, *decF, *bvec;
    size_t bytes;
};

ScratchLayout scratch_layout(const Dims &d, void *base)
{
    Carver c(base);
    ScratchLayout S;
    S.cQ = c.take<double>(d.da);
    S.A1 = c.take<double>((size_t)d.N1 * d.M);
    S.a1 = c.take<double>(d.N1);
    S.G = c.take<double>((size_t)d.E * d.da);
    S.P = c.take<double>((size_t)d.E * d.N1);
    S.cvec = c.take<double>(d.E);
    S.cvec2 = c.take<double>(d.E);
    S.decF = c.take<double>((size_t)2 * d.E * d.E);
    S.bvec = c.take<double>((size_t)2 * d.E);
    S.bytes = c.off;
    return S;
}

#define TIG_TRY(expr)              \
    do {                           \
        hipError_t e_ = (expr);    \
        if (e_ != hipSuccess)      \
            return e_;             \
    } while (0)

}  // namespace

size_t pack_scratch_bytes(const Dims &d) { return scratch_layout(d, nullptr).bytes; }
size_t packed_weights_bytes(const Dims &d) { return layout(d, nullptr).bytes; }

hipError_t pack_weights(const Dims &d, const tig_weights &w, void *dst, void *scratch,
                        PackedWeights *pw, hipStream_t s, int parts)
{
    const bool with_gru = (parts & kPackGru) != 0, with_embed = (parts & kPackEmbed) != 0;
    const bool with_dec = (parts & kPackDec) != 0;
    const PackedLayout L = layout(d, dst);
    const ScratchLayout S = scratch_layout(d, scratch);
    const int M = d.M, T = d.T, E = d.E, H = d.H, da = d.da, dh = d.dh, dkv = d.dkv;
    const int Dmsg = d.Dmsg;
    const dim3 blk(kThreads);
    auto grid = [](size_t n) { return dim3((unsigned)((n + kThreads - 1) / kThreads)); };

    // every prepared matrix and vector is written whole, padding included; the clears are for the gaps
    // between them and for the padded rows of the folding scratch
    if (parts == kPackAll)
        TIG_TRY(launch_fill_zero(dst, L.bytes, s));
    if (with_embed)
        TIG_TRY(launch_fill_zero(scratch, S.bytes, s));

    // time encoding parameters in revolutions: the kernels take cos(2 pi (w_rev x + b_rev))
    if (!with_gru) {
        hipLaunchKernelGGL(k_to_revolutions, grid(T), blk, 0, s, L.time_w_rev, w.time_w, T);
        hipLaunchKernelGGL(k_to_revolutions, grid(T), blk, 0, s, L.time_b_rev, w.time_b, T);
    }

    // ---- GRU: gates r, z with the hidden weights folded onto the s_self columns; one launch --
    if (with_gru) {
        GruPackJob j;
        j.time_w_rev = L.time_w_rev, j.time_b_rev = L.time_b_rev, j.time_w = w.time_w, j.time_b = w.time_b;
        j.W_i = w.W_i, j.W_h = w.W_h, j.b_i = w.b_i, j.b_h = w.b_h;
        j.Wr = L.gru_Wr, j.Wz = L.gru_Wz, j.Win = L.gru_Win, j.Whn = L.gru_Whn;
        j.br = L.gru_br, j.bz = L.gru_bz, j.bin = L.gru_bin, j.bhn = L.gru_bhn;
        j.rnn = (parts & kPackRnn) != 0;
        j.M = M, j.T = T, j.Dmsg = Dmsg, j.Ng = d.Ng, j.Kg = d.Kg, j.Khn = d.Khn;
        size_t most = (size_t)d.Ng * (d.Kg > d.Khn ? d.Kg : d.Khn);
        most = most > (size_t)T ? most : (size_t)T;
        const dim3 g2((unsigned)((most + kThreads - 1) / kThreads), 10);
        if (d.prec == TIG_BF16_MFMA)
            hipLaunchKernelGGL(k_pack_gru<true>, g2, blk, 0, s, j);
        else
            hipLaunchKernelGGL(k_pack_gru<false>, g2, blk, 0, s, j);
        TIG_TRY(hipGetLastError());
    }

    if (with_embed) {
        const double scale = 1.0 / sqrt((double)dh);
        // The embedding kernel holds a key/value row in the order [Phi (T) | s_v (M) | e (F)] (time
        // encoding first, so that its lanes are densely packed); the model's order is
        // [s_v | e | Phi].  seg[] maps each run of model columns to its place in the kernel's order.
        const int F = d.F;
        const int seg_src[3] = {M + F, 0, M};
        const int seg_dst[3] = {0, T, T + M};
        const int seg_len[3] = {T, M, F};
        const int ld_m1 = da + M;
        FoldJobs one = {}, two = {};
        auto add = [](FoldJobs &f, double *C, int ldc, const void *A, bool a64, int ars, int acs, const void *B, bool b64, int brs,
                      int bcs, int m, int n, int kdim, double alpha) -> FoldJob & {
            FoldJob &q = f.j[f.n++];
            q = FoldJob{C, A, B, nullptr, ldc, ars, acs, brs, bcs, m, n, kdim, alpha, a64, b64, false, false};
            return q;
        };
        // ---- products of the weights as given ---------------------------------------------
        {   // cQ = W_Q[:, M:] Phi(0) + b_Q
            FoldJob &q = add(one, S.cQ, 1, w.W_Q + M, false, da, 1, w.time_b, false, 1, 1, da, 1, T, 1.0);
            q.c0 = w.b_Q;
            q.b_cos = true;
        }
        for (int h = 0; h < H; ++h)  // A1_h[j][m] = scale * sum_r W_K[h*dh + r][j] * W_Q[h*dh + r][m]
            for (int g = 0; g < 3; ++g)
                add(one, S.A1 + ((size_t)h * d.dkvp + seg_dst[g]) * M, M, w.W_K + (size_t)h * dh * dkv + seg_src[g], false, 1, dkv,
                    w.W_Q + (size_t)h * dh * da, false, da, 1, seg_len[g], M, dh, scale);
        // G = W_m1[:, :da] W_O   [E x da]
        add(one, S.G, da, w.W_m1, false, ld_m1, 1, w.W_O, false, da, 1, E, da, da, 1.0);
        // c = b_m1 + W_m1a b_O + G b_V (first term here)
        add(one, S.cvec, 1, w.W_m1, false, ld_m1, 1, w.b_O, false, 1, 1, E, 1, da, 1.0);
        // The first decoder layer applied to h1 directly (merge layer 2 folded in), for launches whose row
        // tiles are whole roles: W_d1a W_m2, W_d1b W_m2 and b_d1 + (W_d1a + W_d1b) b_m2.
        for (int half = 0; half < 2; ++half) {
            add(one, S.decF + (size_t)half * E * E, E, w.W_d1 + half * E, false, 2 * E, 1, w.W_m2, false, E, 1, E, E, E, 1.0);
            add(one, S.bvec + (size_t)half * E, 1, w.W_d1 + half * E, false, 2 * E, 1, w.b_m2, false, 1, 1, E, 1, E, 1.0);
        }
        TIG_TRY(fold(s, one));
        // ---- products of those ------------------------------------------------------------
        for (int h = 0; h < H; ++h)
            for (int g = 0; g < 3; ++g) {
                // a1_h[j] = scale * sum_r W_K[h*dh + r][j] * cQ[h*dh + r]
                add(two, S.a1 + (size_t)h * d.dkvp + seg_dst[g], 1, w.W_K + (size_t)h * dh * dkv + seg_src[g], false, 1, dkv,
                    S.cQ + h * dh, true, 1, 1, seg_len[g], 1, dh, scale);
                // P_h = G[:, h*dh:(h+1)*dh] W_V[h*dh:(h+1)*dh, :]   [E x dkv]
                add(two, S.P + (size_t)h * d.dkvp + seg_dst[g], d.N1, S.G + h * dh, true, da, 1,
                    w.W_V + (size_t)h * dh * dkv + seg_src[g], false, dkv, 1, E, seg_len[g], dh, 1.0);
            }
        add(two, S.cvec2, 1, S.G, true, da, 1, w.b_V, false, 1, 1, E, 1, da, 1.0);
        TIG_TRY(fold(s, two));
        // ---- into the kernels' layouts ----------------------------------------------------
        PackJobs pj = {};
        pj.m[0] = PackMat{L.emb_A1, S.A1, nullptr, M, 0, M, d.N1, M, d.N1, d.Mq, 0, 0, nullptr, true, false};
        pj.m[1] = PackMat{L.emb_PR, S.P, w.W_m1 + da, d.N1, ld_m1, d.N1, E, d.N1 + M, d.Ep, d.K2, 0, 0, nullptr, true, false};
        pj.m[2] = PackMat{L.emb_Wm2, w.W_m2, nullptr, E, 0, E, E, E, d.Ep, d.Ek, 0, 0, nullptr, false, false};
        // decoder layer 1 split by operand: rows 0..E-1 <- W_d1[:, :E], rows Ep..Ep+E-1 <- W_d1[:, E:]
        pj.m[3] = PackMat{L.dec_W, w.W_d1, nullptr, 2 * E, 0, E, 2 * d.Ep, E, 2 * d.Ep, d.Ek, d.Ep, d.Ep - E, w.W_d1 + E, false, false};
        pj.m[4] = PackMat{L.dec_WF, S.decF, nullptr, E, 0, E, 2 * d.Ep, E, 2 * d.Ep, d.Ek, d.Ep, d.Ep - E, S.decF + (size_t)E * E, true, false};
        pj.v[0] = PackVec{L.emb_a1, d.N1, d.N1, S.a1, nullptr, nullptr};
        pj.v[1] = PackVec{L.emb_c, E, d.Ep, S.cvec, S.cvec2, w.b_m1};
        pj.v[2] = PackVec{L.emb_c0, E, d.Ep, nullptr, nullptr, w.b_m1};
        pj.v[3] = PackVec{L.emb_bm2, E, d.Ep, nullptr, nullptr, w.b_m2};
        pj.v[4] = PackVec{L.dec_b1, E, d.Ep, nullptr, nullptr, w.b_d1};
        pj.v[5] = PackVec{L.dec_b1f, E, d.Ep, S.bvec, S.bvec + E, w.b_d1};
        pj.v[6] = PackVec{L.dec_w2, E, d.Ep, nullptr, nullptr, w.w_d2};
        pj.v[7] = PackVec{L.dec_b2, 1, 1, nullptr, nullptr, w.b_d2};
        size_t most = d.N1;
        for (const PackMat &q : pj.m)
            most = (size_t)q.rows_p * q.cols_p > most ? (size_t)q.rows_p * q.cols_p : most;
        const dim3 g3((unsigned)((most + kThreads - 1) / kThreads), kPackMats + kPackVecs);
        if (d.prec == TIG_BF16_MFMA)
            hipLaunchKernelGGL(k_pack<true>, g3, blk, 0, s, pj);
        else
            hipLaunchKernelGGL(k_pack<false>, g3, blk, 0, s, pj);
        TIG_TRY(hipGetLastError());
    } else if (with_dec) {
        PackJobs pj = {};
        pj.m[3] = PackMat{L.dec_W, w.W_d1, nullptr, 2 * E, 0, E, 2 * d.Ep, E, 2 * d.Ep, d.Ek, d.Ep, d.Ep - E, w.W_d1 + E, false, false};
        pj.v[4] = PackVec{L.dec_b1, E, d.Ep, nullptr, nullptr, w.b_d1};
        pj.v[6] = PackVec{L.dec_w2, E, d.Ep, nullptr, nullptr, w.w_d2};
        pj.v[7] = PackVec{L.dec_b2, 1, 1, nullptr, nullptr, w.b_d2};
        const dim3 g3((unsigned)(((size_t)2 * d.Ep * d.Ek + kThreads - 1) / kThreads), kPackMats + kPackVecs);
        hipLaunchKernelGGL(d.prec == TIG_BF16_MFMA ? k_pack<true> : k_pack<false>, g3, blk, 0, s, pj);
        TIG_TRY(hipGetLastError());
    }

    pw->time_w_rev = L.time_w_rev;
    pw->time_b_rev = L.time_b_rev;
    pw->gru_Wr = L.gru_Wr;
    pw->gru_Wz = L.gru_Wz;
    pw->gru_Win = L.gru_Win;
    pw->gru_Whn = L.gru_Whn;
    pw->gru_br = L.gru_br;
    pw->gru_bz = L.gru_bz;
    pw->gru_bin = L.gru_bin;
    pw->gru_bhn = L.gru_bhn;
    pw->emb_A1 = L.emb_A1;
    pw->emb_a1 = L.emb_a1;
    pw->emb_PR = L.emb_PR;
    pw->emb_c = L.emb_c;
    pw->emb_c0 = L.emb_c0;
    pw->emb_Wm2 = L.emb_Wm2;
    pw->emb_bm2 = L.emb_bm2;
    pw->dec_W = L.dec_W;
    pw->dec_b1 = L.dec_b1;
    pw->dec_WF = L.dec_WF;
    pw->dec_b1f = L.dec_b1f;
    pw->dec_w2 = L.dec_w2;
    pw->dec_b2 = L.dec_b2;
    return hipSuccess;
}

}  // namespace tig
