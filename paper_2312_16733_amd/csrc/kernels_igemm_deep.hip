// Tile variants of the implicit-GEMM kernel with deep rings, for launches of few tiles and for long reductions.
#include "igemm_kernel.h"

namespace sna {

#define SNA_DEEP_VARIANT(BM, BN, WM, WN, NS, FW, GATED_FN) \
  { BM, BN, 64 * (WM * WN + FW), IgemmCfg<BM, BN, WM, WN, NS, FW>::SMEM, NS, IgemmCfg<BM, BN, WM, WN, NS, FW>::STAGE_B, \
    IgemmCfg<BM, BN, WM, WN, NS, FW>::EPI_BYTES, igemm_kernel<BM, BN, WM, WN, NS, false, FW>, igemm_kernel<BM, BN, WM, WN, NS, true, FW>, GATED_FN, false, true, \
    deep_small(BM, BN, WM * WN, NS, FW), true }
const Variant kDeepVariants[kDeepVariantCount] = {
    SNA_DEEP_VARIANT(32, 32, 1, 1, 8, 4, (igemm_kernel<32, 32, 1, 1, 8, false, 4, true>)),
    SNA_DEEP_VARIANT(64, 64, 2, 2, 8, 4, (igemm_kernel<64, 64, 2, 2, 8, false, 4, true>)),
    SNA_DEEP_VARIANT(128, 96, 4, 1, 5, 4, nullptr),
};

}  // namespace sna
