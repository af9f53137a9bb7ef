// The embedding kernels: fp32 matrix cores (embed_tile.h).
#include "embed_tile.h"

namespace tig {

#ifdef TIG_PHASE_CLOCKS
extern "C" __attribute__((visibility("default"))) int tig_debug_phase_clocks_fp32(unsigned long long *out, int n)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_clocks), sizeof(unsigned long long) * (size_t)n);
}
#endif

const void *embed_kernel_fp32(const Dims &d) { return pick<TIG_FP32, kEmbedStep, kAnyRows>(d); }

}  // namespace tig
