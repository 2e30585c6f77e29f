// FP32 MLP kernel at padded width 128: a wave per 16-unit tile.
#include "mlp_f32_decl.h"
#include "mlp_kernels_f32.h"

namespace rid {

rid_status mlp_f32_w128(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.resnet) {
    if (rt >= 2) return run_mlp_f32<128, 2, 8, 4, true>(e, x, B, A_out, g_out, t, st);
    return run_mlp_f32<128, 1, 8, 6, true>(e, x, B, A_out, g_out, t, st);
  }
  if (rt >= 2) return run_mlp_f32<128, 2, 8, 4, false>(e, x, B, A_out, g_out, t, st);
  return run_mlp_f32<128, 1, 8, 6, false>(e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
