// Conservative switching's Hessian-vector products of FP32 ensembles: the
// kernel's instantiations (kernel: hvp_f32.h).
#include "hvp_f32.h"

namespace rid {
namespace {

// NW: waves; NWD: waves of the forms that hold more per unit (5 and 6 hidden
// layers, the residual carries), fewer so that each lane has more registers;
// 0: no such kernel.
template <int NP, int NW, int NWR, int NWD>
rid_status hvp_w(const rid_ensemble_impl& e, const float* x, const float* rho, const float* coef,
                 int B, float* T, hipStream_t st) {
  if constexpr (NWD > 0) {
    if (e.L > 4 && e.resnet) return run_hvp_f32<NP, 1, NWD, 6, true>(e, x, rho, coef, B, T, st);
    if (e.L > 4) return run_hvp_f32<NP, 1, NWD, 6, false>(e, x, rho, coef, B, T, st);
  }
  if constexpr (NWR > 0) {
    if (e.resnet) return run_hvp_f32<NP, 1, NWR, 4, true>(e, x, rho, coef, B, T, st);
  }
  return run_hvp_f32<NP, 1, NW, 4, false>(e, x, rho, coef, B, T, st);
}

int hvp_depth(int NP) { return NP <= 256 ? kMaxHidden : 4; }

}  // namespace

bool hvp_fused_supported(const rid_ensemble_impl& e) {
  // what the registers hold: 6 hidden layers to width 256, 4 above, no
  // residual form past 384
  if (e.prec != RID_FP32 || e.L > hvp_depth(e.split.NP) || (e.resnet && e.split.NP > 384))
    return false;
  HvpF32Args a{};
  return hvp_f32_layout(e.split.NP, 16, hvp_depth(e.split.NP), e.split.XP, a) <= 160 * 1024;
}

rid_status launch_hvp(const rid_ensemble_impl& e, const float* x, const float* rho,
                      const float* coef, int B, float* T, hipStream_t st) {
  if (e.prec == RID_FP32) {
    switch (e.split.NP) {
      case 64: return hvp_w<64, 4, 4, 4>(e, x, rho, coef, B, T, st);
      case 128: return hvp_w<128, 8, 8, 8>(e, x, rho, coef, B, T, st);
      case 192: return hvp_w<192, 12, 12, 6>(e, x, rho, coef, B, T, st);
      case 256: return hvp_w<256, 16, 16, 8>(e, x, rho, coef, B, T, st);
      case 320: return hvp_w<320, 10, 10, 0>(e, x, rho, coef, B, T, st);
      case 384: return hvp_w<384, 12, 12, 0>(e, x, rho, coef, B, T, st);
      case 512: return hvp_w<512, 8, 0, 0>(e, x, rho, coef, B, T, st);
    }
  }
  return fail(RID_EUNSUPPORTED, "no fused HVP kernel for this ensemble");
}

}  // namespace rid
