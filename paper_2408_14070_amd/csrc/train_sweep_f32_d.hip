// Fused training sweeps at padded width 512.
#include "train_f32_decl.h"
#include "train_sweep_f32.h"

namespace rid {

rid_status train_f32_w512(int, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  return run_train_f32<512, 1, 8, 4, false>(e, io, B, st);
}

}  // namespace rid
