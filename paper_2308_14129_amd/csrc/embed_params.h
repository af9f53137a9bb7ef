// Launch parameters of the embedding kernels and the choice among their instances (host side).
#pragma once

#include "embed_rules.h"
#include "tig_internal.h"

namespace tig {

struct EmbedParams {
    int M, T, F, E, K;
    int dkv, dkvp, Mq, N1, K2, Ep, Ek;
    int row_bytes;  // LDS bytes per query row of the main buffer: [q~ / kvbar (N1) | s_u (Mq)]
    int ld1;        // row stride of the E-wide buffers, bytes
    int most_mt;    // sixteenths of the highest tile that LDS holds (embed_height)
    int n_tiles;    // workgroups that take row tiles
    int spread;     // tiles the rows are spread over if they are few (tiles_in_use)
    int n_commit;   // then: workgroups of the memory overwrite; the ones beyond prepare the next batch
    int commit_beside;  // the memory overwrite is done by those beyond, behind the query preparation
    // bit n set: register n of a key/value row (dims 64 n .. 64 n + 63 of [Phi | s_v | e]) holds
    // at least one dim of the time encoding / of the neighbour's memory / of the edge feature
    int phi_regs, mem_regs, feat_regs;
};

enum EmbedMode { kEmbedStep = 0, kEmbedTrain = 1, kEmbedLayer = 2 };

inline int npl_for(const Dims &d)
{
    const int need = (d.dkvp + 63) / 64;
    int npl = 1;
    while (npl < need)
        npl *= 2;
    return npl;
}

// must agree with EmbedShape (heads other than 1 and 2 run the 4-head kernels)
inline int embed_threads(const Dims &d) { return npl_for(d) >= 8 && d.H > 2 ? 512 : 1024; }

constexpr int kAnyRows = 0;  // a tile's rows: the kernel takes the height for the rows it finds

const void *embed_kernel_bf16(const Dims &d, int rows);
const void *embed_kernel_fp32(const Dims &d);
const void *embed_kernel_train(const Dims &d);
const void *embed_kernel_layer(const Dims &d);

}  // namespace tig
