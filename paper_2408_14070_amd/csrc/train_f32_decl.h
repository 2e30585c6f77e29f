// Launchers of the fused training sweeps by padded width (several source
// files: they compile side by side).  rt: 16-sample tiles per workgroup.
#pragma once

#include "rid_internal.h"

namespace rid {
#define RID_TRAIN_F32(W)                                                                 \
  rid_status train_f32_w##W(int rt, const rid_ensemble_impl& e, const TrainIo& io, int B, \
                            hipStream_t st);
RID_TRAIN_F32(64) RID_TRAIN_F32(128) RID_TRAIN_F32(192) RID_TRAIN_F32(256)
RID_TRAIN_F32(320) RID_TRAIN_F32(384) RID_TRAIN_F32(512)
#undef RID_TRAIN_F32
}  // namespace rid
