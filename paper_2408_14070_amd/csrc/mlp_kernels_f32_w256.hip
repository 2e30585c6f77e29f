// FP32 MLP kernel at padded width 256: a wave per 16-unit tile (two tiles at 64 rows,
// which halves the LDS reads of the activations).
#include "mlp_f32_decl.h"
#include "mlp_kernels_f32.h"

namespace rid {

rid_status mlp_f32_w256(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.resnet) {
    if (rt >= 2) return run_mlp_f32<256, 2, 16, 4, true>(e, x, B, A_out, g_out, t, st);
    return run_mlp_f32<256, 1, 16, 6, true>(e, x, B, A_out, g_out, t, st);
  }
  if (rt == 4) return run_mlp_f32<256, 4, 8, 4, false>(e, x, B, A_out, g_out, t, st);
  if (rt >= 2) return run_mlp_f32<256, 2, 16, 4, false>(e, x, B, A_out, g_out, t, st);
  return run_mlp_f32<256, 1, 16, 6, false>(e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
