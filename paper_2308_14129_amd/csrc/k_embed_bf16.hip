// The embedding kernels: bf16 matrix cores (split operands) (embed_tile.h).
#include "embed_tile.h"

namespace tig {

#ifdef TIG_PHASE_CLOCKS
extern "C" __attribute__((visibility("default"))) int tig_debug_phase_clocks_bf16(unsigned long long *out, int n)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_clocks), sizeof(unsigned long long) * (size_t)n);
}
#endif

const void *embed_kernel_bf16(const Dims &d, int rows)
{
    return rows == 16   ? pick<TIG_BF16_MFMA, kEmbedStep, 16>(d)
           : rows == 32 ? pick<TIG_BF16_MFMA, kEmbedStep, 32>(d)
                        : pick<TIG_BF16_MFMA, kEmbedStep, 48>(d);
}

}  // namespace tig
