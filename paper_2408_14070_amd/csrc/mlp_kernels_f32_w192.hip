// FP32 MLP kernel at padded width 192: a wave per 16-unit tile (two tiles at 64 rows).
#include "mlp_f32_decl.h"
#include "mlp_kernels_f32.h"

namespace rid {

rid_status mlp_f32_w192(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.resnet) {
    if (rt >= 2) return run_mlp_f32<192, 2, 12, 4, true>(e, x, B, A_out, g_out, t, st);
    return run_mlp_f32<192, 1, 12, 6, true>(e, x, B, A_out, g_out, t, st);
  }
  if (rt == 4) return run_mlp_f32<192, 4, 6, 4, false>(e, x, B, A_out, g_out, t, st);
  if (rt >= 2) return run_mlp_f32<192, 2, 12, 4, false>(e, x, B, A_out, g_out, t, st);
  return run_mlp_f32<192, 1, 12, 6, false>(e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
