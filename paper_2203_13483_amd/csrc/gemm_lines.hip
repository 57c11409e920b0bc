// Tile kernels of the 4- and 8-bit linears with stages of whole 128-byte lines per operand row.
//
// What bounds the tile kernels between the smallest and the largest sizes is the path from L2 to LDS.  L2 answers
// a CU with about 0.45 requests per cycle when all CUs ask, whether a request takes 64 or 128 bytes of its line:
// copies of 128-byte row pieces were measured at 56-58 bytes per cycle and CU, copies of 64-byte pieces at 30 (all
// 256 CUs, operands resident in L2), and a 128x128 tile needs 32 bytes per cycle to keep the matrix cores busy.
// A stage is therefore 256 4-bit (128 8-bit) codes of every row here: K % 256 == 0 (K % 128 == 0), half the stage
// boundaries, and twice the LDS per stage, so rings are two or three stages deep.
#include "gemm_tile.h"

namespace mkq {

template <class Cfg, int BITS, int KS = 1>
static int launch_lines(const GemmI4Params &p, int epi, hipStream_t st)
{
    if ((p.K % (1024 / BITS * KS)) != 0) return MKQ_ERR_UNSUPPORTED;
    switch (epi) {
    case EPI_F16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>, BITS, KS>(p, st);
    case EPI_BF16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_BF16, false, false>, BITS, KS>(p, st);
    case EPI_F32: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F32, false, false>, BITS, KS>(p, st);
    case EPI_F16_RES16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>, BITS, KS>(p, st);
    case EPI_I4_GELU:
        if constexpr (BITS == 4) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, true>, BITS, KS>(p, st);
        break;
    case EPI_I4:
        if constexpr (BITS == 4) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, false>, BITS, KS>(p, st);
        break;
    case EPI_I8_GELU:
        if constexpr (BITS == 8) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I8, false, true>, BITS, KS>(p, st);
        break;
    }
    return launch_gemm_i4_dma_generic<Cfg, BITS, KS>(p, st);
}

int run_gemm_i4_lines(const GemmI4Params &p, int epi, int cfg, hipStream_t st)
{
    switch (cfg) {
    case 43: return launch_lines<GemmI4DmaCfg<64, 64, 2, 2, 128, 2>, 4>(p, epi, st);
    case 44: return launch_lines<GemmI4DmaCfg<256, 128, 4, 2, 128, 3>, 4>(p, epi, st);
    case 45: return launch_lines<GemmI4DmaCfg<256, 256, 2, 4, 128, 2>, 4>(p, epi, st);
    case 46: return launch_lines<GemmI4DmaCfg<128, 128, 2, 2, 128, 2>, 4, 2>(p, epi, st);
    case 47: return launch_lines<GemmI4DmaCfg<64, 64, 2, 2, 128, 3>, 4, 2>(p, epi, st);
    case 48: return launch_lines<GemmI4DmaCfg<128, 64, 2, 2, 128, 2>, 4, 2>(p, epi, st);
    case 49: return launch_lines<GemmI4DmaCfg<128, 128, 4, 2, 128, 2>, 4>(p, epi, st);
    case 51: return launch_lines<GemmI4DmaCfg<128, 96, 4, 1, 128, 2>, 4, 2>(p, epi, st);
    default: return MKQ_ERR_UNSUPPORTED;
    }
}

int run_gemm_i8_lines(const GemmI4Params &p, int epi, int cfg, hipStream_t st)
{
    switch (cfg) {
    case 43: return launch_lines<GemmI4DmaCfg<64, 64, 2, 2, 128, 3>, 8>(p, epi, st);
    case 44: return launch_lines<GemmI4DmaCfg<256, 128, 4, 2, 128, 3>, 8>(p, epi, st);
    case 46: return launch_lines<GemmI4DmaCfg<128, 128, 2, 2, 128, 2>, 8>(p, epi, st);
    case 47: return launch_lines<GemmI4DmaCfg<64, 64, 2, 2, 128, 3>, 8, 2>(p, epi, st);
    case 51: return launch_lines<GemmI4DmaCfg<128, 96, 4, 1, 128, 4>, 8>(p, epi, st);
    case 52: return launch_lines<GemmI4DmaCfg<256, 192, 4, 2, 128, 2>, 8>(p, epi, st);
    default: return MKQ_ERR_UNSUPPORTED;
    }
}

}  // namespace mkq
