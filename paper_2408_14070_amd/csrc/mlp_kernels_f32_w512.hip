// FP32 MLP kernel at padded width 512: 16 waves of two 16-unit tiles, at 32 rows and in the
// residual form 8 waves of four (256 registers a lane hold the accumulators,
// the tanh' stash and the residual).
#include "mlp_f32_decl.h"
#include "mlp_kernels_f32.h"

namespace rid {

rid_status mlp_f32_w512(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                      float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.resnet) return run_mlp_f32<512, 1, 8, 6, true>(e, x, B, A_out, g_out, t, st);
  if (rt >= 2) return run_mlp_f32<512, 2, 8, 4, false>(e, x, B, A_out, g_out, t, st);
  return run_mlp_f32<512, 1, 16, 6, false>(e, x, B, A_out, g_out, t, st);
}

}  // namespace rid
