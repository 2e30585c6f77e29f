// Fused training sweeps at padded width 256.
#include "train_f32_decl.h"
#include "train_sweep_f32.h"

namespace rid {

rid_status train_f32_w256(int rt, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<256, 1, 8, 4, true>(e, io, B, st);
  if (e.L > 4) return run_train_f32<256, 1, 8, 6, false>(e, io, B, st);
  if (rt == 2) return run_train_f32<256, 2, 8, 4, false>(e, io, B, st);
  return run_train_f32<256, 1, 8, 4, false>(e, io, B, st);
}

}  // namespace rid
