// prefill_g64.hip -- prefill grouped GEMMs for quantization groups of 64 columns.
#include "prefill.hpp"

namespace mc {
template hipError_t launch_prefill_gemm<2>(const LayerArgs&, const int32_t*, const PrefillTables&,
                                           const PrefillGemm&, bool, int, hipStream_t);
}  // namespace mc
