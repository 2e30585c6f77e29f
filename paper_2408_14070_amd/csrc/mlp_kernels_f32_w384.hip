// FP32 MLP kernel at padded width 384: twelve waves of two 16-unit tiles.
#include "mlp_f32_decl.h"
#include "mlp_kernels_f32.h"

namespace rid {

rid_status mlp_f32_w384(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.resnet) {
    if (rt >= 2) return run_mlp_f32<384, 2, 12, 4, true>(e, x, B, A_out, g_out, t, st);
    return run_mlp_f32<384, 1, 12, 6, true>(e, x, B, A_out, g_out, t, st);
  }

  if (rt >= 2) return run_mlp_f32<384, 2, 12, 4, false>(e, x, B, A_out, g_out, t, st);
  return run_mlp_f32<384, 1, 12, 6, false>(e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
