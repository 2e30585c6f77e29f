// Fused training sweeps at padded widths 320, 384.
#include "train_f32_decl.h"
#include "train_sweep_f32.h"

namespace rid {

rid_status train_f32_w320(int, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<320, 1, 10, 4, true>(e, io, B, st);
  return run_train_f32<320, 1, 10, 4, false>(e, io, B, st);
}

rid_status train_f32_w384(int, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<384, 1, 12, 4, true>(e, io, B, st);
  return run_train_f32<384, 1, 12, 4, false>(e, io, B, st);
}

}  // namespace rid
