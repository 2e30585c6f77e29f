// The FP32 MLP kernel's launchers by padded width, one source file each (they
// compile side by side).  rt: 16-row tiles per workgroup (1, 2 or 4).
#pragma once

#include "rid_internal.h"

namespace rid {
#define RID_MLP_F32(W)                                                                        \
  rid_status mlp_f32_w##W(int rt, const rid_ensemble_impl& e, const float* x, int B,          \
                          float* A_out, float* g_out, const TorsionInput* t, hipStream_t st);
RID_MLP_F32(64) RID_MLP_F32(128) RID_MLP_F32(192) RID_MLP_F32(256)
RID_MLP_F32(320) RID_MLP_F32(384) RID_MLP_F32(512)
#undef RID_MLP_F32
}  // namespace rid
