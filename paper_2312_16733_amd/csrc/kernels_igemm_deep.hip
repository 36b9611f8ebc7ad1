// Tile variants of the implicit-GEMM kernel with deep rings, for launches of few tiles and for long reductions.
#include "igemm_kernel.h"

namespace sna {

#define SNA_DEEP_VARIANT(BM, BN, WM, WN, NS, FW, GATED_FN, PW, PW_CHUNKED, PW_GATED) \
  { BM, BN, 64 * (WM * WN + FW), IgemmCfg<BM, BN, WM, WN, NS, FW>::SMEM, NS, IgemmCfg<BM, BN, WM, WN, NS, FW>::STAGE_B, \
    IgemmCfg<BM, BN, WM, WN, NS, FW>::EPI_BYTES, igemm_kernel<BM, BN, WM, WN, NS, false, FW>, igemm_kernel<BM, BN, WM, WN, NS, true, FW>, GATED_FN, false, true, \
    deep_small(BM, BN, WM * WN, NS, FW), PW, PW_CHUNKED, PW_GATED, BM * BN < WM * WN * 32 * 32 ? 2 : 1 }
#define SNA_DEEP_SMALL(BM, BN, WM, WN, NS, FW) \
  SNA_DEEP_VARIANT(BM, BN, WM, WN, NS, FW, (igemm_kernel<BM, BN, WM, WN, NS, false, FW, true>), (igemm_pw_kernel<BM, BN, WM, WN, NS, false, FW, false>), \
                   (igemm_pw_kernel<BM, BN, WM, WN, NS, true, FW, false>), (igemm_pw_kernel<BM, BN, WM, WN, NS, false, FW, true>))
const Variant kDeepVariants[kDeepVariantCount] = {
    SNA_DEEP_SMALL(32, 32, 2, 1, 8, 4), SNA_DEEP_SMALL(64, 64, 2, 2, 8, 4),
    SNA_DEEP_VARIANT(128, 96, 4, 1, 5, 4, nullptr, nullptr, nullptr, nullptr),
};

}  // namespace sna
