// Fused training sweeps at padded widths 64, 128, 192.
#include "train_f32_decl.h"
#include "train_sweep_f32.h"

namespace rid {

rid_status train_f32_w64(int rt, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<64, 1, 4, 4, true>(e, io, B, st);
  if (e.L > 4) return run_train_f32<64, 1, 4, 6, false>(e, io, B, st);
  if (rt == 2) return run_train_f32<64, 2, 4, 4, false>(e, io, B, st);
  return run_train_f32<64, 1, 4, 4, false>(e, io, B, st);
}

rid_status train_f32_w128(int rt, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<128, 1, 8, 4, true>(e, io, B, st);
  if (e.L > 4) return run_train_f32<128, 1, 8, 6, false>(e, io, B, st);
  if (rt == 2) return run_train_f32<128, 2, 8, 4, false>(e, io, B, st);
  return run_train_f32<128, 1, 8, 4, false>(e, io, B, st);
}

rid_status train_f32_w192(int rt, const rid_ensemble_impl& e, const TrainIo& io, int B,
                         hipStream_t st) {
  if (e.resnet) return run_train_f32<192, 1, 12, 4, true>(e, io, B, st);
  if (e.L > 4) return run_train_f32<192, 1, 6, 6, false>(e, io, B, st);
  if (rt == 2) return run_train_f32<192, 2, 12, 4, false>(e, io, B, st);
  return run_train_f32<192, 1, 12, 4, false>(e, io, B, st);
}

}  // namespace rid
