// Tile kernels of the 4- and 8-bit linears for launches of at most one 32x64 tile per CU: padding-free batches of a few sentences,
// poolers and classifiers of a batch.
//
// What bounds these launches is the instruction stream of one wave from its first copy to its last store, not memory and not the
// matrix cores: widening two operands for a single 32x32 product and the boundaries of the stages take a lone wave of the 64x64
// kernels 0.45-0.55 us per 128-byte stage, six times the products themselves.  So K is cut into as many parts as whole stages allow,
// each summed by a wave group of its own, and tiles are half as large, which takes twice as many CUs.  us of a launch, the best
// 64x64 kernel -> here: M = 440, N = 768 with a residual, K = 768 5.1 -> 4.4, K = 3072 7.6 -> 5.9; N = 1024, K = 4096 8.8 -> 6.7;
// M = 100, K = 1024, N = 4096 with GELU 5.6 -> 5.1; 8 bits, K = N = 768, M = 440 5.0 -> 4.6, K = 3072 7.6 -> 6.9.
#include "gemm_tile.h"

namespace mkq {

int run_gemm_i4_short(const GemmI4Params &p, int epi, int cfg, hipStream_t st)
{
    switch (cfg) {
    case 53: return launch_lines<GemmI4DmaCfg<32, 64, 1, 2, 128, 2>, 4, 4>(p, epi, st);
    case 54: return launch_lines<GemmI4DmaCfg<32, 64, 1, 2, 128, 2>, 4, 3>(p, epi, st);
    case 55: return launch_lines<GemmI4DmaCfg<32, 64, 1, 2, 128, 3>, 4, 2>(p, epi, st);
    default: return MKQ_ERR_UNSUPPORTED;
    }
}

int run_gemm_i8_short(const GemmI4Params &p, int epi, int cfg, hipStream_t st)
{
    if (cfg != 55) return MKQ_ERR_UNSUPPORTED;
    return launch_lines<GemmI4DmaCfg<32, 64, 1, 2, 128, 3>, 8, 2>(p, epi, st);
}

}  // namespace mkq
