// The 16-bit MLP kernels' launchers by padded width, one source file each or
// two (they compile side by side).  rt: 16-walker tiles per workgroup.
#pragma once

#include "rid_internal.h"

namespace rid {
#define RID_MLP_16(W)                                                                        \
  rid_status mlp_16_w##W(int rt, const rid_ensemble_impl& e, const float* x, int B,          \
                         float* A_out, float* g_out, const TorsionInput* t, hipStream_t st);
RID_MLP_16(64) RID_MLP_16(128) RID_MLP_16(192) RID_MLP_16(256)
RID_MLP_16(320) RID_MLP_16(384) RID_MLP_16(512)
#undef RID_MLP_16
}  // namespace rid
