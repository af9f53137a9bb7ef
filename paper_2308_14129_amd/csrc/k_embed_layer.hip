// The embedding kernels: one attention layer of a stack (embed_tile.h).
#include "embed_tile.h"

namespace tig {

const void *embed_kernel_layer(const Dims &d) { return pick<TIG_FP32, kEmbedLayer, kAnyRows>(d); }

}  // namespace tig
