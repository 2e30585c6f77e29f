// Dispatch of the ensemble MLP kernels (forward + input gradient, mlp_kernels_f32.h
// for FP32 ensembles, mlp_kernels_16.h for 16-bit ones) and the weight packer
// of the 16-bit ones.
#include "device_common.h"
#include "mlp_16_decl.h"
#include "mlp_kernels_16.h"
#include "mlp_kernels_f32.h"

namespace rid {
namespace {

using namespace dev;
using mlp16::kTanhPrescale;

// ---------------------------------------------------------------------------
// weight packer: FP32 masters (packed layout) -> MFMA fragments, biases
// ---------------------------------------------------------------------------
struct PackLayer {
  unsigned w_off, b_off;  // float offsets inside one model's packed block
  int in, out;            // real widths
  int kin_pad;            // padded input width
  unsigned fwd_off, bwd_off;  // byte offsets inside one model's fragments
  int fmt_fwd, fmt_bwd;   // fragment formats (FragFmt)
};

// element format of a set of MFMA fragments
enum FragFmt { kFmtBF16 = 1, kFmtF16 = 2 };

struct VecArgs {
  unsigned b_off[kMaxHidden];
  int out[kMaxHidden];
  unsigned wo_off;
  int last_w;
  int vscale_on;          // reverse vectors in a 16-bit format: scale them
};

struct PackAll {
  PackLayer layer[kMaxHidden];
  VecArgs va;
  int L, K, NP;
};

// One launch packs a whole ensemble: block row y < 2L packs layer y/2 in
// direction y%2 (0: forward fragments, contraction = the layer input,
// pre-scaled by 2/ln 2; 1: backward, contraction = the layer output), each
// in its plan's format; row 2L packs the biases (pre-scaled), w_o and b_o,
// zero-padded to NP.  When the reverse sweep runs in FP16, w_o is stored
// times a per-member power of two that puts max |w_o| in [128, 256), so
// v_L = w_o tanh'_L and the vectors after it stay far inside FP16's range
// (and clear of its subnormals) through the sweep; the kernel undoes the
// scale, exactly, in A and g.  vscale[k] = (scale, 1 / scale).
__global__ void pack_kernel(const float* master, size_t per_model, PackAll pa,
                            unsigned char* frag, size_t frag_model_bytes, float* bias,
                            float* wo, float* bo, float* vscale) {
  const int NP = pa.NP;
  if ((int)blockIdx.y == 2 * pa.L) {
    __shared__ float red[256];
    const VecArgs& va = pa.va;
    for (int k = blockIdx.x; k < pa.K; k += gridDim.x) {
      const float* m = master + (size_t)k * per_model;
      for (int l = 0; l < pa.L; ++l)
        for (int j = threadIdx.x; j < NP; j += blockDim.x)
          bias[((size_t)k * pa.L + l) * NP + j] =
              j < va.out[l] ? kTanhPrescale * m[va.b_off[l] + j] : 0.f;
      float mx = 0.f;
      for (int j = threadIdx.x; j < va.last_w; j += blockDim.x) mx = fmaxf(mx, fabsf(m[va.wo_off + j]));
      red[threadIdx.x] = mx;
      __syncthreads();
      for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + h]);
        __syncthreads();
      }
      float sc = 1.f;
      if (va.vscale_on && red[0] > 0.f && red[0] < 3.0e38f) {
        int ex;
        (void)frexpf(red[0], &ex);            // red[0] = f 2^ex, f in [0.5, 1)
        sc = ldexpf(1.f, 8 - ex);             // red[0] sc in [128, 256)
      }
      for (int j = threadIdx.x; j < NP; j += blockDim.x)
        wo[(size_t)k * NP + j] = j < va.last_w ? m[va.wo_off + j] * sc : 0.f;
      if (threadIdx.x == 0) {
        bo[k] = m[va.wo_off + va.last_w];
        vscale[2 * k] = sc;
        vscale[2 * k + 1] = 1.f / sc;         // exact: sc is a power of two
      }
      __syncthreads();
    }
    return;
  }
  const PackLayer& pl = pa.layer[blockIdx.y >> 1];
  const int dir = blockIdx.y & 1;
  const int fmt = dir == 0 ? pl.fmt_fwd : pl.fmt_bwd;
  constexpr int KF = 32;
  constexpr int E = 8;                        // elements per lane (16 bytes)
  const int kc = dir == 0 ? pl.kin_pad : NP;
  const int nc = dir == 0 ? NP : pl.kin_pad;
  const int JT = nc / 16, KT = kc / KF;
  const size_t total = (size_t)pa.K * KT * JT * 64;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < total;
       t += (size_t)gridDim.x * blockDim.x) {
    const int lane = t % 64;
    size_t f = t / 64;
    const int jt = f % JT; f /= JT;
    const int kt = f % KT;
    const int k = __builtin_amdgcn_readfirstlane((int)(f / KT));   // (a wave's fragment)
    const __amdgpu_buffer_rsrc_t W = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(master + (size_t)k * per_model + pl.w_off), (short)0,
        4 * pl.in * pl.out, 0x00020000);
    const int col = jt * 16 + (lane & 15);
    float v[E];
    for (int e = 0; e < E; ++e) {
      const int kk = kt * KF + (KF / 4) * (lane >> 4) + e;
      // W is [out][in]; forward: (unit col = out, contraction kk = in);
      // backward: (unit col = in, contraction kk = out)
      const int o = dir == 0 ? col : kk;
      const int i = dir == 0 ? kk : col;
      // (outside: an offset past the resource, which reads as 0; a branch
      // around the load made the compiler wait on each)
      const int off = o < pl.out && i < pl.in ? 4 * (o * pl.in + i) : 0x7FFFFFF0;
      v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(W, off, 0, 0));
    }
    if (dir == 0)
      for (int e = 0; e < E; ++e) v[e] *= kTanhPrescale;
    unsigned short hv[E];
    for (int e = 0; e < E; ++e)
      hv[e] = fmt == kFmtBF16 ? __builtin_bit_cast(unsigned short, (__bf16)v[e])
                              : __builtin_bit_cast(unsigned short, (_Float16)v[e]);
    const uint4 out = make_uint4(hv[0] | (unsigned)hv[1] << 16, hv[2] | (unsigned)hv[3] << 16,
                                 hv[4] | (unsigned)hv[5] << 16, hv[6] | (unsigned)hv[7] << 16);
    unsigned char* dst = frag + (size_t)k * frag_model_bytes +
                         (dir == 0 ? pl.fwd_off : pl.bwd_off) +
                         (((size_t)kt * JT + jt) * 64 + lane) * 16;
    *reinterpret_cast<uint4*>(dst) = out;
  }
}

// 16-walker tiles per workgroup.  More tiles share a weight stream but leave
// CUs idle in small batches: measured (FP16, 38 CVs, 4 members, 4 hidden
// layers; us for 16 / 32 / 64 walkers a workgroup) a round of up to 256
// workgroups takes 12.8 / 14.0 / 19.5 at width 256, 17 / 19 / 25 at 320,
// 20 / 23 / 29 at 384, 29 / 33 / 42 at 512, each further round 7.3 / 9.8 / 18,
// 12 / 17 / 25, 15 / 21 / 31, 26 / 34 / 50: the cheapest number of rounds is
// taken.  Up to width 192 several workgroups share a CU and 64 walkers never
// paid (16384 walkers: 22.6 / 22.7 / 27.6 at 64, 44 / 35 / 37 at 128,
// 84 / 58 / 61 at 192); 32 do past a round (2001 walkers 10.5 / 10.3 and
// 14.0 / 13.3 at 128 and 192; 1000: 8.3 / 9.0 and 10.9 / 11.2), at 64 only
// where workgroups outnumber the CUs' places.  The tile must fit LDS.
int rows_16(const rid_ensemble_impl& e, int B) {
  const int NP = e.NP, NW = mlp16::waves(NP);
  auto wgs = [&](int rt) { return (long long)((B + 16 * rt - 1) / (16 * rt)) * e.K; };
  const double round[3] = {1.0, 1.35, NP > 256 ? 2.0 : 2.45};
  int best = 1;
  double least = 0.0;
  bool found = false;
  for (int i = 0, rt = 1; rt <= (NP >= 256 && e.L <= 4 ? 4 : 2); rt *= 2, ++i) {
    if (mlp16::lds_bytes(e, 16 * rt, NW) > 160 * 1024) continue;
    double c = round[i] * (double)((wgs(rt) + 255) / 256);
    if (NP <= 192) c = rt == (wgs(1) > (NP == 64 ? 2048 : 256) ? 2 : 1) ? 0.0 : 1.0;
    if (!found || c < least) {
      found = true;
      least = c;
      best = rt;
    }
  }
  return best;
}

// Whether the MLP kernel computes its walkers' torsions itself (a launch less)
// or the CVs are encoded first: in the kernel every member does it again, a
// wave at a time.  It pays where the call is one round of 16-walker workgroups
// whose atoms fit an activation buffer, and a wave has few torsions.  Measured, time
// encoding first over time in the kernel (4 members, 4 hidden layers, 1 to 1000
// walkers): 2 CVs 1.03 to 1.12 (1.20 for one walker at width 64, where 100 take
// 0.92); 18 CVs 1.00 to 1.08, but 0.87 to 0.96 at width 64 (72 CVs a wave);
// 38 CVs, FP32, 1.04 to 1.06 at widths 192 to 320 (38 or 76 a wave), 0.86 at 64
// (152), and, FP16, 0.93 to 1.00 at 128 to 320 (76); 120 CVs (atoms gathered in
// several passes) 0.35 to 1.00.  From 1500 walkers on 0.40 to 1.03.
bool gather_pays(const rid_ensemble_impl& e, const TorsionInput& t, int B) {
  if ((long long)((B + 15) / 16) * e.K > 256) return false;
  const bool f32 = e.prec == RID_FP32;
  const int NP = e.split.NP;
  const int waves = !f32 ? mlp16::waves(e.NP)
                    : NP <= 256 ? NP / 16 : NP == 512 && !e.resnet ? 16 : NP == 512 ? 8 : NP / 32;
  const int cvs = (16 + waves - 1) / waves * e.n_cv;   // torsions a wave computes
  if (f32) return mlp_f32_gathers(NP, 16, t.sys->n_uniq) && cvs <= 80;
  return mlp16::gathers(e, 16, t.sys->n_uniq) && cvs <= 64;
}

rid_status dispatch(const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                    float* g_out, const TorsionInput* t, hipStream_t st) {
  if (e.prec == RID_FP32) return dispatch_mlp_f32(e, x, B, A_out, g_out, t, st);
  if (e.resnet) return fail(RID_EUNSUPPORTED, "residual connections need an FP32 ensemble");
  const int rt = t ? 1 : rows_16(e, B);
  switch (e.NP) {
    case 64: return mlp_16_w64(rt, e, x, B, A_out, g_out, t, st);
    case 128: return mlp_16_w128(rt, e, x, B, A_out, g_out, t, st);
    case 192: return mlp_16_w192(rt, e, x, B, A_out, g_out, t, st);
    case 256: return mlp_16_w256(rt, e, x, B, A_out, g_out, t, st);
    case 320: return mlp_16_w320(rt, e, x, B, A_out, g_out, t, st);
    case 384: return mlp_16_w384(rt, e, x, B, A_out, g_out, t, st);
    case 512: return mlp_16_w512(rt, e, x, B, A_out, g_out, t, st);
  }
  return fail(RID_EUNSUPPORTED, "no kernel for this padded width");
}

}  // namespace

// g_out == nullptr: free energies only.
rid_status launch_mlp(const rid_ensemble_impl& e, const float* x, int B,
                      float* A_out, float* g_out, hipStream_t st) {
  return dispatch(e, x, B, A_out, g_out, nullptr, st);
}

rid_status launch_mlp_from_pos(const rid_ensemble_impl& e, const TorsionInput& tin,
                               int B, float* A_out, float* g_out, hipStream_t st) {
  // the in-kernel gather computes torsions only: systems with distance CVs
  // take the encoding from cv_eval_kernel, as calls do where that is cheaper
  if (tin.sys->has_dist || !gather_pays(e, tin, B)) return RID_EUNSUPPORTED;
  return dispatch(e, nullptr, B, A_out, g_out, &tin, st);
}

rid_status pack_ensemble_weights(rid_ensemble_impl& e, hipStream_t st) {
  ++e.master_gen;     // the masters may have changed: copies made from them are stale
  e.frag_dirty = true;               // until the packing is launched
  if (e.prec == RID_FP32) {
    const rid_status r = pack_split_weights(e, st);
    e.frag_dirty = r != RID_OK;
    return r;
  }
  const int L = e.L;
  PackAll pa{};
  pa.L = L;
  pa.K = e.K;
  pa.NP = e.NP;
  unsigned off = 0;
  int prev = 2 * e.n_cv;
  for (int l = 0; l < L; ++l) {
    PackLayer& pl = pa.layer[l];
    pl.w_off = off;
    pl.in = prev;
    pl.out = e.widths[l];
    off += (unsigned)(pl.out * pl.in);
    pl.b_off = off;
    pa.va.b_off[l] = off;
    pa.va.out[l] = pl.out;
    off += (unsigned)pl.out;
    pl.kin_pad = e.layers[l].kin_pad;
    pl.fwd_off = (unsigned)e.layers[l].fwd_off;
    pl.bwd_off = (unsigned)e.layers[l].bwd_off;
    // the plan's formats: first layer, hidden-layer forward, reverse sweep
    switch (e.prec) {
      case RID_BF16:
        pl.fmt_fwd = l == 0 ? kFmtF16 : kFmtBF16;
        pl.fmt_bwd = kFmtF16;
        break;
      case RID_FP16:
        pl.fmt_fwd = pl.fmt_bwd = kFmtF16;
        break;
      default:                         // RID_BF16_ALL
        pl.fmt_fwd = pl.fmt_bwd = kFmtBF16;
        break;
    }
    prev = pl.out;
  }
  pa.va.wo_off = off;
  pa.va.last_w = prev;
  pa.va.vscale_on = e.prec == RID_BF16 || e.prec == RID_FP16;
  const dim3 grid(256, 2 * L + 1), block(256);
  hipLaunchKernelGGL(pack_kernel, grid, block, 0, st, e.d_master, e.per_model, pa, e.d_frag,
                     e.frag_bytes_per_model, e.d_bias, e.d_wo, e.d_bo, e.d_vscale);
  RID_HIP(hipGetLastError());
  e.frag_dirty = false;
  return RID_OK;
}

}  // namespace rid
