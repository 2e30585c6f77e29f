// Hessian-vector products for conservative switching, FP32 ensembles
// (template; instantiated by padded width in hvp_f32.hip).  For walker w and
// member k, with rho_x = (dx/ds) w_k (w_k the walker's deviation direction,
// zero outside the switching band):
//   u0  = dA_k/dx                          (reverse sweep)
//   u0d = H_x rho_x = d/dt u0(x + t rho_x)  (forward-over-reverse)
// and the member's term of d eps/ds, chained to the angles:
//   T_k[i] = -sin s_i u0d[i] + cos s_i u0d[n+i] - w_ki (cos s_i u0[i] + sin s_i u0[n+i])
// (a raw CV, encoded (s, 0), is linear: T_k[i] = u0d[i]).
// With t_l = tanh(z_l), d_l = 1 - t_l^2 and the terms in brackets for
// residual layers l >= 2:
//   zd_l = W_l hd_{l-1}, td_l = d_l zd_l, hd_l = td_l [+ hd_{l-1}],
//   dd_l = -2 t_l td_l (tangent of d_l),
//   u_L = w_o, ud_L = 0, v_l = u_l d_l, vd_l = ud_l d_l + u_l dd_l,
//   u_{l-1} = W_l^T v_l [+ u_l], ud_{l-1} = W_l^T vd_l [+ ud_l].
// One workgroup owns 16 RT walkers of one member: rows [0, R) of its
// activation tile are the walkers' primal vectors, rows [R, 2R) their
// tangents, so every weight fragment streamed from L2 (what bounds it) feeds
// both; d and dd stay in registers between the sweeps.  The products run as
// split FP16 (mlp_split.h), the rows' scales from bounds on their largest
// entries:  |hd_l| <= R_l max|hd_{l-1}|, |u_{l-1}| <= C_l max|u_l|,
// |ud_{l-1}| <= C_l (max|ud_l| + 2 max|td_l| max|u_l|), each plus the
// residual's own, |v| <= |u|, |vd_l| <= |ud_l| + 2 max|td_l| |u_l|
// (C, R: largest absolute column and row sums of the layer's weights).
// 500 walkers, 38 CVs, 4 x [256 x 4]: 55 us with FP32 MFMA, 25 us now.
#pragma once

#include <algorithm>
#include <type_traits>

#include "mlp_split.h"

namespace rid {

struct HvpF32Args {
  const float* x;      // [B][2n] encoding cos s | sin s (raw CVs (s, 0))
  const float* rho;    // [B][K][n] w_k
  const float* coef;   // [B] Abar sigma'(eps): a tile whose walkers are all 0 is skipped
  const uint8_t* raw;  // [n] 1: raw CV, or null
  float* T_out;        // [K][B][n]
  int B, n, K, L, XP, n_tiles, xcd_grp, u0_parts;
  SplitView w;
  unsigned off_wo, off_mx;   // LDS byte offsets
};

namespace dev {

// tracked row maxima (hd, td, u, ud per layer), the raw CVs' bounds on layer
// 1's tangents, the layer bounds
__host__ __device__ constexpr int hvp_track_words(int LM, int R) {
  return 4 * (LM + 1) * R + R + 2 * (kMaxHidden + 1);
}

template <int NP, int RT, int NW, int LM, bool RES>
__global__ __launch_bounds__(NW * 64) void hvp_f32_kernel(HvpF32Args p) {
  constexpr int CT = NP / (16 * NW);
  constexpr int R = 16 * RT;
  constexpr int JT = NP / 16;
  constexpr int NK = NP / kSplitKF;
  constexpr int PD = CT < 4 ? 2 : 1;
  constexpr int PDH = split_depth(NK, CT);
  constexpr bool EARLY = CT < (RES ? 2 : 4);   // epilogue operands before the product
  static_assert(CT >= 1 && CT * 16 * NW == NP, "width/wave split");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int k, tile;
  map_block(blockIdx.x, p.K, p.xcd_grp, k, tile);
  if (tile >= p.n_tiles) return;
  const int row0 = tile * R;
  // every wave takes the same vote, so a skipped tile leaves as a whole
  if (!__any(p.coef[min(row0 + (lane % R), p.B - 1)] != 0.f)) return;

  const int n = p.n, L = p.L, XP = p.XP, X2 = 2 * p.n;
  constexpr int AS = split_row_halfs(NP);
  constexpr int BUF = 2 * R * AS;              // primal rows, then tangent rows
  const int AX = split_row_halfs(XP);          // row stride of the input tile
  _Float16* const buf1 = reinterpret_cast<_Float16*>(smem);
  _Float16* const buf0 = buf1 + BUF;
  auto buf = [&](int i) { return i & 1 ? buf1 : buf0; };
  float* u0 = reinterpret_cast<float*>(buf0);  // partials of u0 | u0d
  const int US = XP + 4;
  float* wos = reinterpret_cast<float*>(smem + p.off_wo);   // [NP]
  unsigned* mx = reinterpret_cast<unsigned*>(smem + p.off_mx);
  unsigned* m_hd = mx;                                      // slot j: hd of layer j - 1
  unsigned* m_td = m_hd + (LM + 1) * R;
  unsigned* m_u = m_td + (LM + 1) * R;
  unsigned* m_ud = m_u + (LM + 1) * R;
  float* m_raw = reinterpret_cast<float*>(m_ud + (LM + 1) * R);   // [R]
  float* cb = m_raw + R;                       // C_l (slot 0: max |w_o|)
  float* rb = cb + kMaxHidden + 1;             // R_l

  const unsigned char* fbase = p.w.frag + (size_t)k * p.w.frag_bytes;
  const float* bias = p.w.bias + (size_t)k * L * NP;
  const float* rs = p.w.rs + (size_t)k * L * 2 * p.w.RW;
  const int jt0 = wave * CT;
  const int wl = lane & 15;
  const int uq = 4 * (lane >> 4);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(fbase), (short)0, (int)p.w.frag_bytes, 0x00020000);
  auto wsrc = [&](unsigned off) {
    return SplitSrc{rsrc, (int)off + jt0 * kSplitFrag, JT * kSplitFrag};
  };
  auto wfwd = [&](int j) { return wsrc(p.w.fwd_off[j]); };
  auto wbwd = [&](int j) { return wsrc(p.w.bwd_off[j]); };
  SplitRing<PD, CT> wr;
  SplitRing<PDH, CT> wh;
  split_preload<PD, CT>(wr, wfwd(0), XP / kSplitKF, lane);
  f4 bnext[CT], rnext[CT];
  const VecSrc vrs = vec_src(rs, L * 2 * p.w.RW), vbias = vec_src(bias, L * NP);
  auto load_rs = [&](int j, int dir) {
#pragma unroll
    for (int c = 0; c < CT; ++c) rnext[c] = vrs.ld4((j * 2 + dir) * p.w.RW + (jt0 + c) * 16, uq);
  };
  auto load_bias = [&](int j) {
#pragma unroll
    for (int c = 0; c < CT; ++c) bnext[c] = vbias.ld4(j * NP + (jt0 + c) * 16, uq);
  };
  load_rs(0, 0);
  load_bias(0);
  for (int i = threadIdx.x; i < NP; i += NW * 64) wos[i] = p.w.wo[(size_t)k * NP + i];
  for (int i = R + threadIdx.x; i < 4 * (LM + 1) * R; i += NW * 64) mx[i] = 0u;   // not slot 0 of hd
  for (int t = wave; t < 2 * L; t += NW) {
    const int l = t >> 1, dir = t & 1;
    float b = 0.f;
    if (dir == 1 && l == 0) {
      for (int i = lane; i < NP; i += 64) b = fmaxf(b, fabsf(p.w.wo[(size_t)k * NP + i]));
    } else if (lane < JT) {
      b = p.w.bound[(((size_t)k * L + l) * 2 + dir) * 32 + lane];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) b = fmaxf(b, __shfl_xor(b, m));
    if (lane == 0) {
      if (dir == 0) rb[l] = b * kTanhUnscale;
      else cb[l] = b;
    }
  }
  // input rows, a wave per walker: x (primal) and rho_x = (dx/ds) w (tangent),
  // columns [2n, XP) and the raw CVs' (added in FP32) zero; walkers past B are
  // zero rows
  constexpr int kCvq = 4;                      // n <= 256: CVs per lane
  for (int i = wave; i < R; i += NW) {
    const int row = row0 + i;
    float x0[kCvq], x1[kCvq], r0[kCvq], r1[kCvq], mraw = 0.f, mr = 0.f;
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      x0[q] = x1[q] = r0[q] = r1[q] = 0.f;
      if (c < n && row < p.B) {
        x0[q] = p.x[(size_t)row * X2 + c];
        x1[q] = p.x[(size_t)row * X2 + n + c];
        const float w = p.rho[((size_t)row * p.K + k) * n + c];
        if (p.raw && p.raw[c]) {
          x0[q] = x1[q] = 0.f;
          mraw += p.w.raw_max[(size_t)k * n + c] * fabsf(w);
        } else {
          r0[q] = -x1[q] * w;
          r1[q] = x0[q] * w;
        }
        mr = fmaxf(mr, fmaxf(fabsf(r0[q]), fabsf(r1[q])));
      }
    }
#pragma unroll
    for (int q = 32; q >= 1; q >>= 1) {
      mraw += __shfl_xor(mraw, q);
      mr = fmaxf(mr, __shfl_xor(mr, q));
    }
    const float sr = split_scale(split_clamp_exp(split_exp(__float_as_uint(mr))));
    if (lane == 0) {
      m_raw[i] = 1.0001f * mraw;       // (the sum's rounding cannot undercut it)
      m_hd[i] = __float_as_uint(mr);
    }
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      if (c < n) {
        split_store1(buf0 + i * AX + c, XP, x0[q] * kActScale);
        split_store1(buf0 + i * AX + n + c, XP, x1[q] * kActScale);
        split_store1(buf0 + (R + i) * AX + c, XP, r0[q] * sr);
        split_store1(buf0 + (R + i) * AX + n + c, XP, r1[q] * sr);
      }
    }
    for (int c = X2 + lane; c < XP; c += 64) {
      split_store1(buf0 + i * AX + c, XP, 0.f);
      split_store1(buf0 + (R + i) * AX + c, XP, 0.f);
    }
  }
  __syncthreads();

  f4 sd[LM - 1][RT][CT], sdd[LM - 1][RT][CT];   // d and dd of hidden layers 1..L-1
  f4 ca[RT][CT], cd[RT][CT];                    // residual carries (h, hd), then (u, ud)
  float iv[RT], ivd[RT];                        // inverse scales of the operand rows
  auto zero = [&](f4 (&a)[2 * RT][CT]) {
#pragma unroll
    for (int rt = 0; rt < 2 * RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) a[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
  };
  auto lds4 = [&](_Float16* buf, int r, int c, const f4& v) {
    split_store4(buf + r * AS + (jt0 + c) * 16 + uq, NP, v);
  };
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    iv[rt] = kActUnscale;
    ivd[rt] = split_unscale(split_clamp_exp(split_exp(m_hd[rt * 16 + wl])));
  }
  // forward epilogue of layer j (0-based): h and hd to the next buffer, or
  // v_L and vd_L at the top
  auto fwd_epi = [&](int j, const f4 (&acc)[2 * RT][CT], _Float16* out) __attribute__((always_inline)) {
    const float un = j == 0 ? kTanhUnscale : kTanhUnscale * kActScale;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int r = rt * 16 + wl;
      const float mh = __uint_as_float(m_hd[j * R + r]);
      const float tb = rb[j] * mh + (j == 0 ? m_raw[r] : 0.f);   // >= |td_j|
      const bool top = j == L - 1;
      const int e0 = split_clamp_exp(split_exp(__float_as_uint(cb[0])));
      const int e1 = split_clamp_exp(split_exp(
          __float_as_uint(top ? 2.f * tb * cb[0] : RES && j >= 1 ? tb + mh : tb)));
      const float sc0 = split_scale(e0), sc1 = split_scale(e1);
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        f4 t, d;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float dq;
          t[q] = tanh_and_grad(__builtin_fmaf(acc[rt][c][q] * iv[rt], rnext[c][q], bnext[c][q]), dq);
          d[q] = dq;
        }
        const f4 td = d * (acc[RT + rt][c] * ivd[rt] * (rnext[c] * un));
        const f4 dd = -2.f * t * td;
        split_track(m_td + j * R + r, td);
        // (registers are written in straight-line code: a store in each arm of
        // a branch becomes one store through a selected address, in scratch)
        f4 h = t, hd = td;
        if constexpr (RES) {
          if (j >= 1) {
            h += ca[rt][c];
            hd += cd[rt][c];
          }
        }
        if (j < LM - 1) {
          sd[j < LM - 1 ? j : 0][rt][c] = d;
          sdd[j < LM - 1 ? j : 0][rt][c] = dd;
        }
        const f4 w4 = *reinterpret_cast<const f4*>(wos + (jt0 + c) * 16 + uq);
        if constexpr (RES) {
          ca[rt][c] = top ? w4 : h;
          cd[rt][c] = top ? f4{0.f, 0.f, 0.f, 0.f} : hd;
        }
        lds4(out, r, c, top ? w4 * d * sc0 : h * kActScale);
        lds4(out, R + r, c, (top ? w4 * dd : hd) * sc1);
        if (!top) split_track(m_hd + (j + 1) * R + r, hd);
      }
      // (a forward layer's row scales already hold 2^-10)
      iv[rt] = top ? split_unscale(e0) : 1.f;
      ivd[rt] = split_unscale(e1);
    }
  };
  {
    f4 acc[2 * RT][CT];
    zero(acc);
    split_gemm_run<2 * RT, CT, PD>(acc, wr, buf0, AX, XP, wfwd(0), XP / kSplitKF, lane);
    if (p.raw) {            // acc becomes the pre-activation and its tangent, raw CVs on top
#pragma unroll
      for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          acc[rt][c] = acc[rt][c] * iv[rt] * rnext[c] + bnext[c];
          acc[RT + rt][c] *= ivd[rt] * rnext[c];
        }
        rnext[c] = f4{1.f, 1.f, 1.f, 1.f};
        bnext[c] = f4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) iv[rt] = ivd[rt] = 1.f;
      const int rows = min(R, p.B - row0), ks = p.K * n;
      const __amdgpu_buffer_rsrc_t xr = row_src(p.x + (size_t)row0 * X2, rows, X2),
                                   rr = row_src(p.rho + (size_t)row0 * ks, rows, ks);
      raw_gemm<2 * RT, CT>(acc, raw_src(p.w, k, NP, n), jt0, lane, [&](int rt, int i) {
        return rt < RT ? raw_value(row_ld(xr, (rt * 16 + wl) * X2 + i))
                       : row_ld(rr, ((rt - RT) * 16 + wl) * ks + k * n + i);
      });
    }
    if (L > 1) split_preload<PDH, CT>(wh, wfwd(1), NK, lane);
    fwd_epi(0, acc, buf1);
    __syncthreads();
  }
  layers_up<1, LM>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      f4 acc[2 * RT][CT];
      zero(acc);
      if constexpr (EARLY) {
        load_rs(j, 0);
        load_bias(j);
      }
      split_gemm_hidden<2 * RT, CT, PDH, NK, false>(acc, wh, buf(j), AS, NP, wfwd(j), true,
                                                    j + 1 < L ? wfwd(j + 1) : wbwd(L - 1), lane);
      if constexpr (!EARLY) {
        load_rs(j, 0);
        load_bias(j);
      }
      fwd_epi(j, acc, buf(j + 1));
      __syncthreads();
    }
  });
  // reverse: v_{l-1} = u d, vd_{l-1} = ud d + u dd
  layers_down<LM - 1, 1>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      _Float16* out = buf(j);
      f4 acc[2 * RT][CT];
      zero(acc);
      if constexpr (EARLY) load_rs(j, 1);
      split_gemm_hidden<2 * RT, CT, PDH, NK, false>(acc, wh, buf(j + 1), AS, NP, wbwd(j),
                                                    j >= 2, wbwd(j >= 2 ? j - 1 : j), lane);
      if constexpr (!EARLY) load_rs(j, 1);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int r = rt * 16 + wl;
        const float mu = j == L - 1 ? cb[0] : __uint_as_float(m_u[j * R + r]);
        const float mud = j == L - 1 ? 0.f : __uint_as_float(m_ud[j * R + r]);
        const float bu = (cb[j] + (RES ? 1.f : 0.f)) * mu;
        const float bud = cb[j] * (mud + 2.f * __uint_as_float(m_td[j * R + r]) * mu) +
                          (RES ? mud : 0.f);
        const int e0 = split_clamp_exp(split_exp(__float_as_uint(bu)));
        const int e1 = split_clamp_exp(split_exp(
            __float_as_uint(bud + 2.f * __uint_as_float(m_td[(j - 1) * R + r]) * bu)));
        const float sc0 = split_scale(e0), sc1 = split_scale(e1);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          f4 u = acc[rt][c] * iv[rt] * rnext[c];
          f4 ud = acc[RT + rt][c] * ivd[rt] * rnext[c];
          if constexpr (RES) {
            u += ca[rt][c];
            ca[rt][c] = u;
            ud += cd[rt][c];
            cd[rt][c] = ud;
          }
          if (j >= 2) {
            split_track(m_u + (j - 1) * R + r, u);
            split_track(m_ud + (j - 1) * R + r, ud);
          }
          lds4(out, r, c, u * sd[j - 1][rt][c] * sc0);
          lds4(out, R + r, c, (ud * sd[j - 1][rt][c] + u * sdd[j - 1][rt][c]) * sc1);
        }
        iv[rt] = split_unscale(e0);
        ivd[rt] = split_unscale(e1);
      }
      __syncthreads();
    }
  });
  // u0 | u0d = W_1^T [v_1 | vd_1], contraction split as in the MLP kernel (vectors in
  // buffer 1, partials in buffer 0)
  auto u0_stage = [&](auto parts_c) {
    constexpr int PARTS = decltype(parts_c)::value;
    constexpr int KQ = NK / PARTS;
    const _Float16* in = buf1;
    const int JT0 = XP / 16;
    for (int it = wave; it < JT0 * PARTS; it += NW) {
      const int t = it / PARTS, q = it - t * PARTS;
      const SplitSrc src{rsrc,
                         (int)p.w.bwd_off[0] + t * kSplitFrag + q * KQ * JT0 * kSplitFrag,
                         JT0 * kSplitFrag};
      const f4 r4 = vrs.ld4(p.w.RW + t * 16, uq);   // backward row scales of layer 1
      constexpr int PU = KQ < 4 ? KQ : 4;
      SplitRing<PU, 1> w0;
      split_preload<PU, 1>(w0, src, KQ, lane);
      f4 a1[2 * RT][1];
#pragma unroll
      for (int rt = 0; rt < 2 * RT; ++rt) a1[rt][0] = f4{0.f, 0.f, 0.f, 0.f};
      split_gemm_run<2 * RT, 1, PU>(a1, w0, in + q * KQ * kSplitKF, AS, NP, src, KQ, lane);
      float* uq0 = u0 + q * 2 * R * US;
#pragma unroll
      for (int rt = 0; rt < 2 * RT; ++rt)
        *reinterpret_cast<f4*>(uq0 + (rt * 16 + wl) * US + t * 16 + uq) =
            a1[rt][0] * (rt < RT ? iv[rt % RT] : ivd[rt % RT]) * r4;
    }
  };
  const int parts = p.u0_parts;
  if (NK % 4 == 0 && parts == 4) u0_stage(std::integral_constant<int, NK % 4 == 0 ? 4 : 1>{});
  else if (parts == 2) u0_stage(std::integral_constant<int, 2>{});
  else u0_stage(std::integral_constant<int, 1>{});
  __syncthreads();
  auto u0_at = [&](int i, int c) {
    float v = u0[i * US + c];
    for (int q = 1; q < parts; ++q) v += u0[q * 2 * R * US + i * US + c];
    return v;
  };
  for (int e = threadIdx.x; e < R * n; e += NW * 64) {
    const int i = e / n, c = e - i * n;
    const int row = row0 + i;
    if (row < p.B) {
      float T;
      if (p.raw && p.raw[c]) {
        T = u0_at(R + i, c);
      } else {
        const float cs = p.x[(size_t)row * X2 + c], sn = p.x[(size_t)row * X2 + n + c];
        const float w = p.rho[((size_t)row * p.K + k) * n + c];
        T = -sn * u0_at(R + i, c) + cs * u0_at(R + i, n + c) -
            w * (cs * u0_at(i, c) + sn * u0_at(i, n + c));
      }
      p.T_out[((size_t)k * p.B + row) * n + c] = T;
    }
  }
}

}  // namespace dev

SplitView split_view(const rid_ensemble_impl& e);
int split_u0_parts(int NP, int XP);

inline size_t hvp_f32_layout(int NP, int R, int LM, int XP, HvpF32Args& a) {
  auto al = [](size_t v) { return (unsigned)((v + 15) / 16 * 16); };
  const size_t buf = (size_t)2 * R * dev::split_row_halfs(NP) * 2;
  // buffer 0 also holds the input rows and the partials of u0 (XP > NP: one part)
  a.off_wo = al(buf + std::max(buf, (size_t)2 * R * dev::split_row_halfs(XP) * 2));
  a.off_mx = al(a.off_wo + (size_t)NP * 4);
  return a.off_mx + (size_t)dev::hvp_track_words(LM, R) * 4;
}

template <int NP, int RT, int NW, int LM, bool RES>
rid_status run_hvp_f32(const rid_ensemble_impl& e, const float* x, const float* rho,
                       const float* coef, int B, float* T, hipStream_t st) {
  static size_t attr = 0;
  constexpr int R = 16 * RT;
  const SplitDev& s = e.split;
  HvpF32Args a{};
  const size_t lds = hvp_f32_layout(NP, R, LM, s.XP, a);
  if (lds > 160 * 1024) return fail(RID_EUNSUPPORTED, "shape too large for the HVP kernel");
  auto kern = dev::hvp_f32_kernel<NP, RT, NW, LM, RES>;
  if (lds > 64 * 1024 && lds > attr) {
    RID_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
    attr = lds;
  }
  a.x = x; a.rho = rho; a.coef = coef; a.raw = e.d_raw; a.T_out = T;
  a.B = B; a.n = e.n_cv; a.K = e.K; a.L = e.L; a.XP = s.XP;
  a.n_tiles = (B + R - 1) / R;
  a.xcd_grp = (8 % e.K == 0) ? 8 / e.K : 0;
  a.u0_parts = split_u0_parts(NP, s.XP);
  a.w = split_view(e);
  const int grid = a.xcd_grp > 0 ? 8 * ((a.n_tiles + a.xcd_grp - 1) / a.xcd_grp)
                                  : a.n_tiles * e.K;
  launch_timed(kProfHvp, kern, dim3(grid), dim3(NW * 64), (uint32_t)lds, st, a);
  RID_HIP(hipGetLastError());
  return RID_OK;
}

}  // namespace rid
