// FP32 ensembles: packing of the split-FP16 weights and the choice of the MLP
// kernel's instantiation (kernel: mlp_kernels_f32.h; number format:
// mlp_split.h).
#include "mlp_kernels_f32.h"

#include "mlp_f32_decl.h"

namespace rid {
namespace {

using namespace dev;

struct SplitPackArgs {
  const float* master;
  unsigned long long per_model;
  unsigned w_off[kMaxHidden], b_off[kMaxHidden], fwd_off[kMaxHidden], bwd_off[kMaxHidden];
  int in[kMaxHidden], out[kMaxHidden], kin_pad[kMaxHidden];
  unsigned wo_off;
  int L, K, NP, RW;
  unsigned char* frag;
  unsigned long long frag_bytes;
  float *bias, *rs, *bound, *wo, *bo;
  const uint8_t* raw;              // [n] or null
  int n;
  float *raw_w, *raw_max;
};

// One block per (16-row tile, layer and direction, member): its waves hold
// the tile's whole contraction in registers (at most 16 k-chunks, 4 a wave),
// so the row maxima and absolute sums, the scales and the split fragments
// come from one read of the masters.  Block row 2L writes the biases and
// output weights, row 2L + 1 the raw CVs' FP32 weights (zero in layer 1's forward
// fragments, so that they set no row's scale).  Rows and contraction: forward,
// units x inputs (weights times 2/ln 2); backward, inputs x units.
__global__ __launch_bounds__(256) void pack_split_kernel(SplitPackArgs p) {
  const int k = blockIdx.z, y = blockIdx.y, jt = blockIdx.x;
  const float* m = p.master + (size_t)k * p.per_model;
  const int NP = p.NP;
  if (y == 2 * p.L) {
    for (int e = jt * 256 + threadIdx.x; e < (p.L + 1) * NP; e += gridDim.x * 256) {
      const int l = e / NP, j = e - l * NP;
      if (l < p.L)
        p.bias[((size_t)k * p.L + l) * NP + j] =
            j < p.out[l] ? kTanhPrescale * m[p.b_off[l] + j] : 0.f;
      else
        p.wo[(size_t)k * NP + j] = j < p.out[p.L - 1] ? m[p.wo_off + j] : 0.f;
    }
    if (jt == 0 && threadIdx.x == 0) p.bo[k] = m[p.wo_off + p.out[p.L - 1]];
    return;
  }
  if (y == 2 * p.L + 1) {              // a wave per CV, its lanes over the units
    const int nw = gridDim.x * 4, lane = threadIdx.x & 63, sets = (p.n + 15) / 16;
    for (int i = jt * 4 + (threadIdx.x >> 6); i < 16 * sets; i += nw) {
      const bool raw = i < p.n && p.raw[min(i, p.n - 1)];
      float mx = 0.f;
      for (int j = lane; j < NP; j += 64) {
        const float w = raw && j < p.out[0] ? m[p.w_off[0] + j * p.in[0] + i] : 0.f;
        p.raw_w[(((size_t)k * (NP / 16) + j / 16) * sets + i / 16) * 256 +
                (((i & 15) >> 2) * 16 + (j & 15)) * 4 + (i & 3)] = kTanhPrescale * w;
        mx = fmaxf(mx, fabsf(w));
      }
#pragma unroll
      for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s));
      if (lane == 0 && i < p.n) p.raw_max[(size_t)k * p.n + i] = mx;
    }
    return;
  }
  const int l = y >> 1, dir = y & 1;
  const int kc = dir == 0 ? p.kin_pad[l] : NP;      // contraction
  const int nr = dir == 0 ? NP : p.kin_pad[l];      // rows
  if (jt * 16 >= nr) return;
  const int in = p.in[l], outw = p.out[l];
  const float* W = m + p.w_off[l];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = jt * 16 + (lane & 15), g = lane >> 4;
  const int KT = kc / kSplitKF;
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(W), (short)0, 4 * in * outw, 0x00020000);
  float v[4][8];
  float mx = 0.f, sum = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int kt = wave + 4 * q;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = kt * kSplitKF + 8 * g + e;
      const int o = dir == 0 ? row : kk, i = dir == 0 ? kk : row;
      bool ok = kt < KT && o < outw && i < in;
      if (p.raw && y == 0) ok = ok && !p.raw[min(i < p.n ? i : i - p.n, p.n - 1)];
      // (outside: an offset past the resource, which reads as 0.  As a branch
      // around the load the compiler waited on each of the 32: 12.9 us a pack
      // of 4 x [300 x 4], 8.4 so, and 10.3 with the second set of fragments)
      const int off = ok ? 4 * (o * in + i) : 0x7FFFFFF0;
      v[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, off, 0, 0));
    }
  }
  const float pre = dir == 0 ? kTanhPrescale : 1.f, pre_lo = dir == 0 ? kTanhPrescaleLow : 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mx = fmaxf(mx, fabsf(v[q][e]));
      sum += fabsf(v[q][e]);
    }
  __shared__ float rm[4][16], rsum[4][16];
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  if (lane < 16) {
    rm[wave][lane] = mx;
    rsum[wave][lane] = sum;
  }
  __syncthreads();
  const int r = lane & 15;
  mx = pre * fmaxf(fmaxf(rm[0][r], rm[1][r]), fmaxf(rm[2][r], rm[3][r]));
  sum = pre * ((rsum[0][r] + rsum[1][r]) + (rsum[2][r] + rsum[3][r]));
  // the row's largest weight to [2^9, 2^10); rows of zeros, infinities or
  // NaNs keep a scale that stays a normal number
  const int ex = min(max(split_exp(__float_as_uint(mx)), -100), 126);
  const float sc = __uint_as_float((unsigned)(127 + 10 - ex) << 23);
  if (wave == 0) {
    if (lane < 16) {
      const float inv = __uint_as_float((unsigned)(127 - 10 + ex) << 23);
      p.rs[(((size_t)k * p.L + l) * 2 + dir) * p.RW + row] =
          dir == 0 && l > 0 ? inv * kActUnscale : inv;
    }
    // a hair above the true sum, so that its rounding cannot undercut it
    float b = sum * 1.0001f;
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1) b = fmaxf(b, __shfl_xor(b, s));
    if (lane == 0) p.bound[(((size_t)k * p.L + l) * 2 + dir) * 32 + jt] = b;
  }
  unsigned char* base = p.frag + (size_t)k * p.frag_bytes + (dir == 0 ? p.fwd_off[l] : p.bwd_off[l]);
  const int JT = nr / 16;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int kt = wave + 4 * q;
    if (kt >= KT) break;
    h8 hi, lo, lo2;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // lo takes what the product with the pre-scale rounds off, and the
      // pre-scale's own rounding: either is the same for every sample, so that
      // sums over a batch do not average it out.  (The value as the compiler has
      // not seen it: it rounded the product to hi in two ways, one for lo.)
      const float w = v[q][e] * sc;
      float x = w * pre;
      asm("" : "+v"(x));
      hi[e] = (_Float16)x;
      float r = (x - (float)hi[e]) + __builtin_fmaf(w, pre_lo, __builtin_fmaf(w, pre, -x));
      asm("" : "+v"(r));
      lo[e] = (_Float16)r;
      // lo's own rounding is the same for every sample too: the second set's lo
      // is off by as much the other way (exactly where r fits FP16 but for its
      // last bit, as all of a backward row's do), and half the tiles of a
      // training step read it
      lo2[e] = (_Float16)(r + (r - (float)lo[e]));
    }
    unsigned char* dst = base + ((size_t)kt * JT + jt) * kSplitFrag + lane * 16;
    unsigned char* dst2 = dst + (size_t)p.K * p.frag_bytes;
    *reinterpret_cast<uint4*>(dst) = __builtin_bit_cast(uint4, hi);
    *reinterpret_cast<uint4*>(dst + kFragBytes) = __builtin_bit_cast(uint4, lo);
    *reinterpret_cast<uint4*>(dst2) = __builtin_bit_cast(uint4, hi);
    *reinterpret_cast<uint4*>(dst2 + kFragBytes) = __builtin_bit_cast(uint4, lo2);
  }
}

// Row tiles (16 walkers each) per workgroup, at most `most`.  A workgroup
// streams all of its member's weights whatever its rows, so its time grows
// slowly with them; the call takes ceil(workgroups / 256 CUs) rounds, each
// slowed by up to 0.3 when every CU streams.  Measured (4 members, 38 CVs,
// 4 layers, us): width 256, 16 walkers 18.8 / 22.6 / 35.5 with 1 / 2 / 4
// tiles, 1024 walkers 24.2 / 25.5 / 38.8, 1300: 39.6 / 25.9 / 38.7, 4096:
// 90 / 59 / 48, 20000: 395 / 274 / 224; width 512, 600 walkers 66.8 / 70.3
// with 1 / 2 tiles, 1024: 77.9 / 71.8, 2000: 146 / 96.  The cheapest wins,
// the smaller tile on a tie.  Widths 64 and 128 keep several workgroups on a
// CU: there two tiles pay from 2048 workgroups (16384 walkers 44.7 / 36.9,
// 4096: 14.3 / 15.0) and past one workgroup a CU (2000: 15.9 / 14.4, 1024:
// 11.5 / 13.4); four never did (16384: 57 and 97 against 37 and 81).
int split_rows(int NP, int B, int K, int most) {
  auto wgs = [&](int rt) { return (long long)((B + 16 * rt - 1) / (16 * rt)) * K; };
  if (NP <= 128) return most > 1 && wgs(1) > (NP == 64 ? 2048 : 256) ? 2 : 1;
  const double t[3] = {1.0, NP > 384 ? 1.08 : 1.25, 2.0};
  int best = 1;
  double cost = 0.0;
  for (int i = 0, rt = 1; rt <= most; rt *= 2, ++i) {
    const long long w = wgs(rt);
    const double c = t[i] * (double)((w + 255) / 256) * (1.0 + 0.3 * std::min(1.0, w / 256.0));
    if (rt == 1 || c < cost) {
      cost = c;
      best = rt;
    }
  }
  return best;
}

}  // namespace

// Parts of the input-gradient contraction: more parts spread its few column
// tiles over the waves; the partials must fit the free activation buffer, a
// condition on the widths alone (rows cancel), so every row tile sums in the
// same order.
int split_u0_parts(int NP, int XP) {
  const int AW = NP > XP ? NP : XP;
  for (int q = 4; q > 1; q /= 2)
    if ((NP / kSplitKF) % q == 0 && q * (XP + 4) <= AW + 4 && (XP / 16) * (q / 2) < NP / 16)
      return q;
  return 1;
}

int split_width(int wmax) {
  for (int v : {64, 128, 192, 256, 320, 384})
    if (wmax <= v) return v;
  return 512;
}

void split_layout(rid_ensemble_impl& e) {
  SplitDev& s = e.split;
  int wmax = 0;
  for (int w : e.widths) wmax = std::max(wmax, w);
  s.NP = split_width(wmax);
  s.XP = round_up(2 * e.n_cv, kSplitKF);
  s.RW = std::max(s.NP, s.XP);
  s.layers.resize(e.L);
  size_t off = 0;
  for (int l = 0; l < e.L; ++l) {
    LayerDev& ld = s.layers[l];
    ld.kin_pad = l == 0 ? s.XP : s.NP;
    const size_t bytes = (size_t)(ld.kin_pad / kSplitKF) * (s.NP / 16) * kSplitFrag;
    ld.fwd_off = off;
    ld.bwd_off = off + bytes;
    off += 2 * bytes;
  }
  s.frag_bytes = off;
}

SplitView split_view(const rid_ensemble_impl& e) {
  const SplitDev& s = e.split;
  SplitView v{};
  v.frag = s.frag;
  v.frag_bytes = s.frag_bytes;
  for (int l = 0; l < e.L; ++l) {
    v.fwd_off[l] = (unsigned)s.layers[l].fwd_off;
    v.bwd_off[l] = (unsigned)s.layers[l].bwd_off;
  }
  v.bias = s.bias;
  v.rs = s.rs;
  v.bound = s.bound;
  v.wo = s.wo;
  v.bo = s.bo;
  v.RW = s.RW;
  v.raw_w = s.raw_w;
  v.raw_max = s.raw_max;
  v.raw_sets = s.raw_sets;
  return v;
}

rid_status pack_split_weights(rid_ensemble_impl& e, hipStream_t st) {
  SplitDev& s = e.split;
  SplitPackArgs p{};
  p.master = e.d_master;
  p.per_model = e.per_model;
  unsigned off = 0;
  int prev = 2 * e.n_cv;
  for (int l = 0; l < e.L; ++l) {
    p.in[l] = prev;
    p.out[l] = e.widths[l];
    p.w_off[l] = off;
    off += (unsigned)(prev * e.widths[l]);
    p.b_off[l] = off;
    off += (unsigned)e.widths[l];
    p.kin_pad[l] = s.layers[l].kin_pad;
    p.fwd_off[l] = (unsigned)s.layers[l].fwd_off;
    p.bwd_off[l] = (unsigned)s.layers[l].bwd_off;
    prev = e.widths[l];
  }
  p.wo_off = off;
  p.L = e.L; p.K = e.K; p.NP = s.NP; p.RW = s.RW;
  p.frag = s.frag; p.frag_bytes = s.frag_bytes;
  p.bias = s.bias; p.rs = s.rs; p.bound = s.bound; p.wo = s.wo; p.bo = s.bo;
  p.raw = e.d_raw; p.n = e.n_cv; p.raw_w = s.raw_w; p.raw_max = s.raw_max;
  hipLaunchKernelGGL(pack_split_kernel, dim3(s.RW / 16, 2 * e.L + (s.raw_sets ? 2 : 1), e.K),
                     dim3(256), 0, st, p);
  RID_HIP(hipGetLastError());
  return RID_OK;
}

rid_status dispatch_mlp_f32(const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                            float* g_out, const TorsionInput* t, hipStream_t st) {
  const SplitDev& s = e.split;
  // up to 64 rows at widths 192 and 256 (32 above: registers and LDS; 32
  // below: more never paid), 32 for residual networks (16 at the widest), 16
  // for more than 4 hidden layers (the tanh' stash)
  int most = e.L > 4 || (e.resnet && s.NP > 384) ? 1
             : e.resnet || s.NP < 192 || s.NP > 256 ? 2 : 4;
  for (; most > 1; most /= 2) {
    MlpF32Args a{};
    if (mlp_f32_layout(s.NP, 16 * most, 4, s.XP, e.n_cv, t != nullptr, a) <= 160 * 1024)
      break;
  }
  const int rt = t ? 1 : split_rows(s.NP, B, e.K, most);
  switch (s.NP) {
    case 64: return mlp_f32_w64(rt, e, x, B, A_out, g_out, t, st);
    case 128: return mlp_f32_w128(rt, e, x, B, A_out, g_out, t, st);
    case 192: return mlp_f32_w192(rt, e, x, B, A_out, g_out, t, st);
    case 256: return mlp_f32_w256(rt, e, x, B, A_out, g_out, t, st);
    case 320: return mlp_f32_w320(rt, e, x, B, A_out, g_out, t, st);
    case 384: return mlp_f32_w384(rt, e, x, B, A_out, g_out, t, st);
    case 512: return mlp_f32_w512(rt, e, x, B, A_out, g_out, t, st);
  }
  return fail(RID_EUNSUPPORTED, "no kernel for this padded width");
}

}  // namespace rid
