// The embedding kernels: one attention layer of a stack (embed_tile.h).
#include "embed_tile.h"

namespace tig {

const void *embed_kernel_layer(const Dims &d, int mt) { return pick<TIG_FP32, kEmbedLayer>(d, mt); }

}  // namespace tig
