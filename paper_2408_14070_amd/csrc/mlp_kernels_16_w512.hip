// 16-bit MLP kernels at padded width 512.
#include "mlp_16_decl.h"
#include "mlp_kernels_16.h"

namespace rid {

rid_status mlp_16_w512(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  return mlp16::run_width<512, true>(rt, e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
