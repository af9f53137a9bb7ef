// Launch of the embedding kernels (embed_tile.h; host side).
#include <hip/hip_runtime.h>

#include "embed_params.h"
#include "prepare.h"
#include "winners.h"

namespace tig {

namespace {

EmbedParams embed_params(const Dims &d, int most_mt)
{
    EmbedParams p;
    p.M = d.M;
    p.T = d.T;
    p.F = d.F;
    p.E = d.E;
    p.K = d.K;
    p.dkv = d.dkv;
    p.dkvp = d.dkvp;
    p.Mq = d.Mq;
    p.N1 = d.N1;
    p.K2 = d.K2;
    p.Ep = d.Ep;
    p.Ek = d.Ek;
    p.row_bytes = lds_row_bytes(d.N1 + d.Mq);
    p.ld1 = lds_row_bytes(d.Ek);
    p.most_mt = most_mt;
    p.n_tiles = p.spread = 0;
    p.n_commit = p.commit_beside = 0;
    p.phi_regs = p.mem_regs = p.feat_regs = 0;
    for (int n = 0; n * kWave < d.dkvp; ++n) {
        const int lo = n * kWave, hi = lo + kWave;
        if (lo < d.T)
            p.phi_regs |= 1 << n;
        if (hi > d.T && lo < d.T + d.M)
            p.mem_regs |= 1 << n;
        if (hi > d.T + d.M && lo < d.T + d.M + d.F)
            p.feat_regs |= 1 << n;
    }
    return p;
}

// (kernels of each precision are a translation unit of their own)
bool any_rows(const Dims &d, bool train) { return train || d.prec == TIG_FP32; }

const void *embed_kernel(const Dims &d, int rows, bool train)
{
    if (train)
        return embed_kernel_train(d);
    return any_rows(d, train) ? embed_kernel_fp32(d) : embed_kernel_bf16(d, rows);
}

int lds_of(const Dims &d, int rows)
{
    return rows * (lds_row_bytes(d.N1 + d.Mq) + lds_row_bytes(d.Ek) + 4 * 4 + 8) + d.T * 16 + 16;
}

hipError_t allow_lds(const Dims &d, const void *kernel, int rows)
{
    const int own = lds_of(d, rows);
    const int lds = embed_threads(d) == kScatterThreads && own < kOneLds ? kOneLds : own;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

int launch_lds(const Dims &d, const StepArgs &a, int rows)
{
    const int own = lds_of(d, rows);
    return a.sel.count > 0 && own < kOneLds ? kOneLds : (own < kPrepLds ? kPrepLds : own);
}

}  // namespace

int embed_lds_bytes(const Dims &d, int mt) { return lds_of(d, 16 * mt); }

// Most 16-row tiles per workgroup that LDS holds for one layer of a stack (0: none).
int layer_tiles(const Dims &d, int lds_limit)
{
    int mt = d.dkvp <= 512 ? 3 : 0;
    while (mt > 0 && embed_lds_bytes(d, mt) > lds_limit)
        --mt;
    return mt;
}

hipError_t prepare_embed_layer(const Dims &d, int most_mt) { return allow_lds(d, embed_kernel_layer(d), 16 * most_mt); }

hipError_t prepare_embed(const Dims &d, const LaunchPlan &plan, bool train)
{
    if (any_rows(d, train))
        return allow_lds(d, embed_kernel(d, 0, train), 16 * plan.emb_mt);
    hipError_t e = hipSuccess;
    for (int mt = 1; mt <= plan.emb_mt && e == hipSuccess; ++mt)
        e = allow_lds(d, embed_kernel(d, 16 * mt, train), 16 * mt);
    return e;
}

// Workgroups of the preparation of a batch of `count` events.  When it shares a launch, every
// workgroup occupies a compute unit (the launch's LDS size applies to all of its workgroups), so
// there are few, each wavefront with several entries; on its own, four entries per wavefront.
int prepare_workgroups(int count, bool shared)
{
    const int entries = 2 * count;
    int n = shared ? (entries + kPrepWaves - 1) / kPrepWaves : (entries + 4 * kPrepWaves - 1) / (4 * kPrepWaves);
    if (shared && n > 31)
        n = 31;
    const int least = (entries + kPrepThreads - 1) / kPrepThreads;  // one entry per thread at most
    return n < least ? least : n;
}

int embed_spare_workgroups(const Dims &d, const LaunchPlan &plan, int roles, int count)
{
    if (embed_threads(d) != kScatterThreads)
        return 0;
    // the selection workgroup and the preparation workgroups of a batch of the same size; the row
    // tiles keep at least three quarters of the compute units
    const int want = 1 + prepare_workgroups(count, true);
    return want <= plan.num_cus / 4 ? want : 0;
}

hipError_t launch_embed(const Dims &d, const LaunchPlan &plan, const PackedWeights &pw, const StepArgs &a,
                        hipStream_t s)
{
    StepArgs aa = a;
    PackedWeights ww = pw;
    const int threads = embed_threads(d);
    // memory overwrite, at the winner count recent steps had
    const bool train = a.tr.S != nullptr;  // (a training step overwrites the memory at its end)
    const bool commit = a.msg_count > 0 && !train;
    const int most_wins = 2 * a.msg_count, wins = a.wins_est > 0 && a.wins_est < most_wins ? a.wins_est : most_wins;
    const bool beside = commit && overwrite_beside(a.ded.count > 0 ? a.ded.n_wgs : 0, wins, threads / kWave);
    const int n_commit = commit && !beside ? overwrite_workgroups(wins, threads / kWave) : 0;
    const int extra = n_commit + (a.sel.count > 0 ? 1 : 0) + (a.ded.count > 0 ? a.ded.n_wgs : 0);
    const int cus = plan.num_cus > 0 ? plan.num_cus : 256;
    const int most = a.roles * a.count;
    const bool any = any_rows(d, train);
    // Compute units for the tiles.  Where the heights differ in the last bits, as many for every kind of call with that many
    // events: a call that prepares nothing leaves those free that another needs for it.
    int side = extra;
    if (any) {
        const int spare = winners_in_one_launch(a.count) ? embed_spare_workgroups(d, plan, a.roles, a.count) : 0;
        side = spare > 0 ? spare : overwrite_workgroups(2 * a.count, threads / kWave);
    }
    const int units = cus - side > 16 ? cus - side : 16;
    // (any height is correct: the grid covers the most rows the batch can have, and tiles beyond the actual count return)
    const int rows = !any && a.rows_est > 0 && a.rows_est < most ? a.rows_est : most;
    const int height = embed_height(any, a.roles == 3, plan.emb_mt, rows, units);
    EmbedParams p = embed_params(d, plan.emb_mt);
    p.spread = units;
    p.n_tiles = any ? any_workgroups(most, height, units) : step_workgroups(most, height, units);
    p.n_commit = n_commit;
    p.commit_beside = beside ? 1 : 0;
    void *args[] = {&aa, &ww, &p};
    return hipLaunchKernel(embed_kernel(d, height, train), dim3(p.n_tiles + extra), dim3(threads), args, (size_t)launch_lds(d, a, height), s);
}

// One attention layer over the rows of a.qs (d, pw: the layer's).  The grid fills the compute units once, but for `side` of
// them that other work of the launch may take; its workgroups take tile after tile.
hipError_t launch_embed_layer(const Dims &d, int most_mt, int num_cus, int side, const PackedWeights &pw, const StepArgs &a, hipStream_t s)
{
    StepArgs aa = a;
    PackedWeights ww = pw;
    const int extra = (a.sel.count > 0 ? 1 : 0) + (a.ded.count > 0 ? a.ded.n_wgs : 0);
    const int cus = num_cus > 0 ? num_cus : 256;
    const int units = cus - side > 16 ? cus - side : 16;
    const int most = a.roles * a.count;
    const int top = embed_height(true, a.roles == 3, most_mt, most, units);
    EmbedParams p = embed_params(d, most_mt);
    p.spread = units;
    p.n_tiles = layer_workgroups(most, top, units);
    void *args[] = {&aa, &ww, &p};
    return hipLaunchKernel(embed_kernel_layer(d), dim3(p.n_tiles + extra), dim3(embed_threads(d)), args, (size_t)launch_lds(d, a, top), s);
}

}  // namespace tig
