// Fused sweeps of the mean-force fitting step: the choice of the kernel's
// instantiation (kernel: train_sweep_f32.h).
#include "train_f32_decl.h"
#include "train_sweep_f32.h"

namespace rid {

namespace {

// hidden layers the registers hold: 6 to width 256, 4 above; 4 for residual
// networks, whose carries take the place of two layers' values (none past
// width 384)
int train_depth(int NP, bool res) {
  return res ? (NP <= 384 ? 4 : 0) : NP <= 256 ? kMaxHidden : 4;
}

bool train_fits(const rid_ensemble_impl& e, int R) {
  TrainF32Args a{};
  return train_f32_layout(e.split.NP, R, train_depth(e.split.NP, e.resnet), e.split.XP, e.n_cv, a) <=
         160 * 1024;
}

}  // namespace

bool train_fused_supported(const rid_ensemble_impl& e) {
  return e.prec == RID_FP32 && e.L <= train_depth(e.split.NP, e.resnet) && train_fits(e, 16);
}

rid_status launch_train_sweeps(const rid_ensemble_impl& e, const TrainIo& io, int B,
                               hipStream_t st) {
  if (!train_fused_supported(e))
    return fail(RID_EUNSUPPORTED, "no fused training kernel for this ensemble");
  const SplitDev& s = e.split;
  // 32 samples a workgroup halve the weight stream a sample costs; taken when
  // 16 would take more than one round of the 256 CUs
  const bool wide = s.NP <= 256 && e.L <= 4 && !e.resnet && train_fits(e, 32) &&
                    (long long)((B + 15) / 16) * e.K > 256;
  const int rt = wide ? 2 : 1;
  switch (s.NP) {
    case 64: return train_f32_w64(rt, e, io, B, st);
    case 128: return train_f32_w128(rt, e, io, B, st);
    case 192: return train_f32_w192(rt, e, io, B, st);
    case 256: return train_f32_w256(rt, e, io, B, st);
    case 320: return train_f32_w320(rt, e, io, B, st);
    case 384: return train_f32_w384(rt, e, io, B, st);
    case 512: return train_f32_w512(rt, e, io, B, st);
  }
  return fail(RID_EUNSUPPORTED, "no kernel for this padded width");
}

}  // namespace rid
