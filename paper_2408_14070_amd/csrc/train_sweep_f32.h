// The sweeps of one mean-force fitting step, fused (template; instantiated by
// padded width in train_sweep_f32_*.hip).  One workgroup takes 16 RT samples
// of one member.  Loss L = (1/B) sum_b |g(s_b) - F_b|^2 with g = dA/ds.  Its
// parameter gradient is the gradient of J = sum_b rho_b . g(s_b), with
// rho = 2 (g - F) / B held fixed (or an upstream rho given by the caller),
// and J is the tangent of A along rho_x = (dx/ds) rho.  With t_l = tanh(z_l),
// dropout factors S_l (1 without dropout), d_l = S_l (1 - t_l^2), and the
// terms in brackets for residual layers l >= 2, the kernel runs from LDS and
// registers:
//   primal forward   h_l = S_l t_l [+ h_{l-1}]
//   primal reverse   u_L = w_o, v_l = u_l d_l, u_{l-1} = W_l^T v_l [+ u_l];
//                    at the input g, the residual and rho_x
//   tangent forward  zd_l = W_l hd_{l-1}, hd_l = d_l zd_l [+ hd_{l-1}]
//   adjoint of J     lam_zd = d lam_hd, lam_z = d (lam_h - 2 t zd lam_hd),
//                    [lam_h ; lam_hd]_{l-1} = W_l^T [lam_z ; lam_zd]_l
//                    [+ [lam_h ; lam_hd]_l], top: lam_hd = w_o, lam_h = 0
// and writes what the batch-reduced weight gradients need: [h ; hd] of every
// layer input (x ; rho_x first) and [lam_z ; lam_zd] of every layer, each as
// [K][2B][width], plus the samples' squared residuals.  Raw CVs enter as
// (s, 0): their g is dA/dx_i and rho reaches the input as (rho_i, 0).
// Dropout: hidden unit j of layer l of sample b is kept with probability
// 1 - p: word j mod 4 of the Philox4x32-10 block with counter
// (b, step, 16 member + l, j div 4), kept when its uniform is >= p.
//
// The products run as split FP16 (mlp_split.h).  What bounds it: the weight
// stream (4 L - 1 layer products a tile, each streaming its matrix once), so
// large batches take 32 samples a workgroup; the adjoint's two rows share
// every fragment.  38 CVs, 4 x [256 x 4], 4096 samples: 330 us with FP32 MFMA
// (16 samples a workgroup), 172 us now; 18 CVs, residual 4 x [300 x 4] with
// dropout, 128 samples (the separate GEMM sweeps before, 29 launches): about
// 150 us, 72 us now, 32 workgroups each streaming its member once a sweep.  t
// and zd of the lane's units stay in VGPRs in FP32; the slabs are written from
// the FP32 values.  Row scales of the vectors with no
// fixed range come from bounds on the largest row entries (tracked in LDS):
//   |u_{l-1}|  <= C_l S max|u_l| [+ max|u_l|]           C: column sums of |W|
//   |hd_l|     <= S R_l max|hd_{l-1}| [+ max|hd_{l-1}|]  R: row sums of |W|
//   |lam_hd_{l-1}| <= C_l S max|lam_hd_l| [+ max|lam_hd_l|]
//   |lam_h_{l-1}|  <= C_l S (max|lam_h_l| + 2 max|zd_l| max|lam_hd_l|)
//                     [+ max|lam_h_l|]
#pragma once

#include <algorithm>
#include <type_traits>

#include "mlp_split.h"

namespace rid {

struct TrainF32Args {
  const float* s;      // [B][n]
  const float* F;      // [B][n] labels (null when rho is given)
  const float* rho;    // [B][K][n] upstream gradient of g, or null
  const uint8_t* raw;  // [n] 1: raw CV (null: every CV angular)
  float* hh[kMaxHidden + 1];   // [K][2B][wd[j]]
  float* sl[kMaxHidden];       // [K][2B][wd[j+1]]
  float* loss_rows;    // row b of member k at loss_rows[k * loss_ld + b], or null
  long long loss_ld;
  int row_base;        // batch index of row 0 (dropout counters)
  int B_norm;          // the whole batch's size (rho scale)
  int B, n, K, L, XP, n_tiles, xcd_grp, u0_parts;
  int wd[kMaxHidden + 1];      // 2n, then the hidden widths
  SplitView w;
  unsigned off_tin, off_xs, off_wo, off_mx;   // LDS byte offsets
  float drop_p, drop_inv;       // rate and 1/(1 - rate); 0 and 1 without dropout
  unsigned long long drop_seed;
  uint32_t step;
};

namespace dev {

typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// The value as the compiler has not seen it: d = S (1 - t^2) is formed again
// in each sweep instead of living in registers from the first one.
__device__ inline f4 reread(f4 v) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float x = v[q];
    asm("" : "+v"(x));
    v[q] = x;
  }
  return v;
}

// Four consecutive floats of an LDS array of `count` (none past its end).
__device__ inline f4 lds_ld4(const float* p, int i, int count) {
  f4 v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = p[min(i + q, count - 1)];
  return v;
}

// rows of tracked maxima: u, hd, zd, lam_h, lam_hd per layer, then the raw
// CVs' bounds on layer 1's tangents and the layer bounds
__host__ __device__ constexpr int train_track_words(int LM, int R) {
  return 5 * (LM + 1) * R + R + 2 * (kMaxHidden + 1);
}

template <int NP, int RT, int NW, int LM, bool RES>
__global__ __launch_bounds__(NW * 64) void train_f32_kernel(TrainF32Args p) {
  constexpr int CT = NP / (16 * NW);
  constexpr int R = 16 * RT;
  constexpr int JT = NP / 16;
  constexpr int NK = NP / kSplitKF;
  constexpr int PD = CT == 1 || (CT == 2 && NW <= 8) ? 2 : 1;
  constexpr int PDH = NK % 4 == 0 && (CT == 1 || (RT * CT == 2 && NW <= 8)) ? 3 : 1;
  // epilogue operands loaded before the product, where the registers allow it
  constexpr bool EARLY = CT == 1 || (CT == 2 && NW <= 8);
  constexpr bool ADB = RT * CT == 1;           // activations a k-step ahead
  static_assert(CT >= 1 && CT * 16 * NW == NP, "width/wave split");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int k, tile;
  map_block(blockIdx.x, p.K, p.xcd_grp, k, tile);
  if (tile >= p.n_tiles) return;
  const int row0 = tile * R;
  const int n = p.n, L = p.L, XP = p.XP, X2 = 2 * p.n, B = p.B;
  constexpr int AS = split_row_halfs(NP);
  constexpr int BUF = 2 * R * AS;              // primal rows, then tangent rows
  const int AX = split_row_halfs(XP);          // row stride of the input tiles
  _Float16* const buf1 = reinterpret_cast<_Float16*>(smem);
  _Float16* const buf0 = buf1 + BUF;
  float* u0 = reinterpret_cast<float*>(buf0);  // partials of u0
  // rho_x: the tangent rows of buffer 1, or a region of its own where the
  // input is wider than the layers
  _Float16* tin = XP <= NP ? buf1 + R * AS : reinterpret_cast<_Float16*>(smem + p.off_tin);
  const int US = XP + 4;
  float* xs = reinterpret_cast<float*>(smem + p.off_xs);    // [R][2n] dx/ds pairs' cos|sin
  float* wos = reinterpret_cast<float*>(smem + p.off_wo);   // [NP]
  unsigned* mx = reinterpret_cast<unsigned*>(smem + p.off_mx);
  unsigned* m_u = mx;                          // [LM + 1][R] each
  unsigned* m_hd = m_u + (LM + 1) * R;         // slot j: hd of layer j - 1 (0: rho_x)
  unsigned* m_zd = m_hd + (LM + 1) * R;
  unsigned* m_lh = m_zd + (LM + 1) * R;
  unsigned* m_lhd = m_lh + (LM + 1) * R;
  float* m_raw = reinterpret_cast<float*>(m_lhd + (LM + 1) * R);   // [R]
  float* cb = m_raw + R;                       // [kMaxHidden + 1] S C_l (slot 0: max |w_o|)
  float* rb = cb + kMaxHidden + 1;             // [kMaxHidden + 1] S R_l

  // odd tiles read the second set of fragments (the weights' rounding errors,
  // the same for every sample, then cancel in the sums over the batch)
  const unsigned char* fbase = p.w.frag + (size_t)((tile & 1) * p.K + k) * p.w.frag_bytes;
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
  const float S = p.drop_inv;
  // forward activations reach S (residual sums 6 S): their scale drops by
  // the power of two above S
  const int eS = p.drop_p > 0.f ? split_exp(__float_as_uint(S)) : 0;
  const float asc = __uint_as_float((unsigned)(127 + 10 - eS) << 23);
  const float aiv = __uint_as_float((unsigned)(127 + eS) << 23);   // asc * aiv = 2^10

  for (int i = threadIdx.x; i < NP; i += NW * 64) wos[i] = p.w.wo[(size_t)k * NP + i];
  for (int i = threadIdx.x; i < 5 * (LM + 1) * R; i += NW * 64) mx[i] = 0u;
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
      if (dir == 0) rb[l] = b * (kTanhUnscale * S);
      else cb[l] = l == 0 ? b : b * S;
    }
  }
  // dropout keep bits of this lane's units, 4 per hidden layer
  unsigned mbits[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) mbits[rt][c] = 0xFFFFFFFFu;
  if (p.drop_p > 0.f) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        unsigned mb = 0u;
        for (int j = 0; j < L; ++j) {
          uint32_t q4[4] = {(uint32_t)(p.row_base + row0 + rt * 16 + wl), p.step,
                            (uint32_t)(16 * k + j + 1), (uint32_t)(((jt0 + c) * 16 + uq) >> 2)};
          philox4x32_10(q4, (uint32_t)(p.drop_seed & 0xFFFFFFFFull),
                        (uint32_t)(p.drop_seed >> 32));
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (philox_uniform(q4[q]) >= p.drop_p) mb |= 1u << (4 * j + q);
        }
        mbits[rt][c] = mb;
      }
  }
  auto dsc = [&](int rt, int c, int j) {   // dropout factors of hidden layer j (0-based)
    f4 r;
    unsigned mb = mbits[rt][c];
    asm("" : "+v"(mb));                    // formed again where it is used
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = ((mb >> (4 * j + q)) & 1u) ? S : 0.f;
    return r;
  };
  // 4 units of tile c in row r (0 .. B-1, tangent rows: tang = 1) of a
  // [K][2B][w] array; units past w are padding and stay unwritten.  Buffer
  // stores: the member's slab (below 2^31 bytes) as a scalar resource and a
  // 32-bit lane offset, so that no address pairs live across the sweeps.
  auto put4 = [&](float* base, int w, int r, int tang, int c, const f4& v) {
    const int u = (jt0 + c) * 16 + uq;
    const __amdgpu_buffer_rsrc_t o = __builtin_amdgcn_make_buffer_rsrc(
        base + (size_t)k * 2 * B * w, (short)0, (int)(8u * (unsigned)B * (unsigned)w), 0x00020000);
    const int vo = 4 * (r * w + u), so = tang ? 4 * B * w : 0;
    if ((w & 3) == 0) {
      if (u < w)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, v), o, vo, so, 0);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (u + q < w)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[q]), o, vo + 4 * q, so, 0);
    }
  };
  // 4 (scaled) units of tile c into LDS row r of a buffer
  auto lds4 = [&](_Float16* buf, int r, int c, const f4& v) {
    split_store4(buf + r * AS + (jt0 + c) * 16 + uq, NP, v);
  };
  constexpr int kCvq = 4;                  // n <= 256: CVs per lane
  // input tile, a wave per sample: x into the primal rows (and hh[0]),
  // zeros past 2n and past B.  xs keeps cos s | sin s, for a raw CV (zero in
  // the tile: its part is added in FP32) its value and later its rho.
  for (int i = wave; i < R; i += NW) {
    const int row = row0 + i;
    float x0[kCvq], x1[kCvq];
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      x0[q] = x1[q] = 0.f;
      if (c < n) {
        const bool is_raw = p.raw && p.raw[c];
        float sv = 0.f, sn = 0.f, cs = 0.f;
        if (row < B) {
          sv = p.s[(size_t)row * n + c];
          sincosf(sv, &sn, &cs);
          if (is_raw) cs = sn = 0.f;
          float* h0 = p.hh[0] + ((size_t)k * 2 * B + row) * X2;
          h0[c] = is_raw ? sv : cs;
          h0[n + c] = sn;
        }
        x0[q] = cs;
        x1[q] = sn;
        xs[i * X2 + c] = is_raw ? raw_value(sv) : cs;
        xs[i * X2 + n + c] = sn;
      }
    }
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      if (c < n) {
        split_store1(buf0 + i * AX + c, XP, x0[q] * kActScale);
        split_store1(buf0 + i * AX + n + c, XP, x1[q] * kActScale);
      }
    }
    for (int c = X2 + lane; c < XP; c += 64) split_store1(buf0 + i * AX + c, XP, 0.f);
  }
  __syncthreads();

  f4 ts[LM][RT][CT];        // t of layers 0..L-1
  f4 zs[LM - 1][RT][CT];    // zd of layers 0..L-2
  f4 ca[RT][CT];            // residual carry (h, u, hd in turn)
  auto buf = [&](int i) { return i & 1 ? buf1 : buf0; };
  auto zero1 = [&](f4 (&a)[RT][CT]) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) a[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
  };

  // ---------------- primal forward ----------------
  // h to the next buffer (and HBM), or v_L = w_o d_L at the top
  float iv0 = kActUnscale;  // layer 1's (1 where raw CVs made acc the pre-activation)
  auto fwd_epi = [&](int j, const f4 (&acc)[RT][CT], _Float16* out) __attribute__((always_inline)) {
    const float vsc = split_scale(split_clamp_exp(split_exp(__float_as_uint(cb[0])) + eS));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float iv = j == 0 ? iv0 : aiv;
      const int brow = row0 + rt * 16 + wl;
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        f4 t, d;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float dq;
          t[q] = tanh_and_grad<true>(__builtin_fmaf(acc[rt][c][q] * iv, rnext[c][q], bnext[c][q]),
                                     dq);
          d[q] = dq;
        }
        ts[j][rt][c] = t;
        const f4 sc = dsc(rt, c, j);
        const bool top = j == L - 1;
        f4 h = t * sc;
        if constexpr (RES) {
          if (j >= 1) h += ca[rt][c];
        }
        const f4 w4 = *reinterpret_cast<const f4*>(wos + (jt0 + c) * 16 + uq);
        // (the carry is written in straight-line code: a store in each arm of
        // a branch becomes one through a selected address, in scratch)
        if constexpr (RES) ca[rt][c] = top ? w4 : h;    // h, then u_L
        lds4(out, rt * 16 + wl, c, top ? w4 * d * sc * vsc : h * asc);
        if (!top && brow < B) put4(p.hh[j + 1], p.wd[j + 1], brow, 0, c, h);
      }
    }
  };
  {
    f4 acc[RT][CT];
    zero1(acc);
    load_rs(0, 0);
    load_bias(0);
    split_gemm_run<RT, CT, PD>(acc, wr, buf0, AX, XP, wfwd(0), XP / kSplitKF, lane);
    if (p.raw) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc[rt][c][q] = __builtin_fmaf(acc[rt][c][q] * iv0, rnext[c][q], bnext[c][q]);
        rnext[c] = f4{1.f, 1.f, 1.f, 1.f};
        bnext[c] = f4{0.f, 0.f, 0.f, 0.f};
      }
      iv0 = 1.f;
      raw_gemm<RT, CT>(acc, raw_src(p.w, k, NP, n), jt0, lane,
                       [&](int rt, int i) { return lds_ld4(xs, (rt * 16 + wl) * X2 + i, R * X2); });
    }
    if (L > 1) split_preload<PDH, CT>(wh, wfwd(1), NK, lane);
    fwd_epi(0, acc, buf1);
    __syncthreads();
  }
  layers_up<1, LM>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      f4 acc[RT][CT];
      zero1(acc);
      if constexpr (EARLY) {
        load_rs(j, 0);
        load_bias(j);
      }
      split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, buf(j), AS, NP, wfwd(j), true,
                                              j + 1 < L ? wfwd(j + 1) : wbwd(L - 1), lane);
      if constexpr (!EARLY) {
        load_rs(j, 0);
        load_bias(j);
      }
      fwd_epi(j, acc, buf(j + 1));
      __syncthreads();
    }
  });
  // ---------------- primal reverse to u0 ----------------
  float iv[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    iv[rt] = split_unscale(split_clamp_exp(split_exp(__float_as_uint(cb[0])) + eS));
  layers_down<LM - 1, 1>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      _Float16* out = buf(j);
      f4 acc[RT][CT];
      zero1(acc);
      if constexpr (EARLY) load_rs(j, 1);
      split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, buf(j + 1), AS, NP, wbwd(j), j >= 2,
                                              wbwd(j >= 2 ? j - 1 : j), lane);
      if constexpr (!EARLY) load_rs(j, 1);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float mu = j == L - 1 ? cb[0] : __uint_as_float(m_u[j * R + rt * 16 + wl]);
        const int e = split_clamp_exp(
            split_exp(__float_as_uint((cb[j] + (RES ? 1.f : 0.f)) * mu)) + eS);
        const float sc = split_scale(e);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          f4 u = acc[rt][c] * iv[rt] * rnext[c];
          if constexpr (RES) {
            u += ca[rt][c];
            ca[rt][c] = u;
          }
          if (j >= 2) split_track(m_u + (j - 1) * R + rt * 16 + wl, u);
          const f4 t = reread(ts[j - 1][rt][c]);
          lds4(out, rt * 16 + wl, c, u * ((1.f - t * t) * dsc(rt, c, j - 1)) * sc);
        }
        iv[rt] = split_unscale(e);
      }
      __syncthreads();
    }
  });
  // u0 = W_1^T v_1 (v_1 in buffer 1, the partials in buffer 0)
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
      constexpr int PU = KQ < 2 ? KQ : 2;
      SplitRing<PU, 1> w0;
      split_preload<PU, 1>(w0, src, KQ, lane);
      f4 a1[RT][1];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a1[rt][0] = f4{0.f, 0.f, 0.f, 0.f};
      split_gemm_run<RT, 1, PU>(a1, w0, in + q * KQ * kSplitKF, AS, NP, src, KQ, lane);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        *reinterpret_cast<f4*>(u0 + q * R * US + (rt * 16 + wl) * US + t * 16 + uq) =
            a1[rt][0] * iv[rt] * r4;
    }
  };
  const int parts = p.u0_parts;
  if (NK % 4 == 0 && parts == 4) u0_stage(std::integral_constant<int, NK % 4 == 0 ? 4 : 1>{});
  else if (parts == 2) u0_stage(std::integral_constant<int, 2>{});
  else u0_stage(std::integral_constant<int, 1>{});
  split_preload<PD, CT>(wr, wfwd(0), XP / kSplitKF, lane);   // tangent layer 1
  __syncthreads();
  auto u0_at = [&](int i, int c) {
    float v = u0[i * US + c];
    for (int q = 1; q < parts; ++q) v += u0[q * R * US + i * US + c];
    return v;
  };
  // ---------------- residual and rho_x (a wave per sample) ----------------
  // rho_x goes to tin, scaled by the row's largest entry, and to the tangent
  // half of hh[0]; a raw CV's (rho, 0) to xs instead of tin, with its bound on
  // layer 1's tangents
  for (int i = wave; i < R; i += NW) {
    const int row = row0 + i;
    float acc = 0.f, m = 0.f, mr = 0.f, rx0[kCvq], rx1[kCvq];
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      rx0[q] = rx1[q] = 0.f;
      if (c < n && row < B) {
        const bool is_raw = p.raw && p.raw[c];
        float cs = xs[i * X2 + c], sn = xs[i * X2 + n + c], rho;
        if (is_raw) {                  // dx/ds = (1, 0)
          cs = 0.f;
          sn = -1.f;
        }
        if (p.rho) {
          rho = p.rho[((size_t)row * p.K + k) * n + c];
        } else {
          const float gi = -sn * u0_at(i, c) + cs * u0_at(i, n + c);
          const float ri = gi - p.F[(size_t)row * n + c];
          acc += ri * ri;
          rho = 2.f * ri / (float)p.B_norm;
        }
        rx0[q] = -sn * rho;
        rx1[q] = cs * rho;
        float* h0 = p.hh[0] + ((size_t)k * 2 * B + B + row) * X2;
        h0[c] = rx0[q];
        h0[n + c] = rx1[q];
        if (is_raw) {
          xs[i * X2 + n + c] = rho;
          mr += p.w.raw_max[(size_t)k * n + c] * fabsf(rho);
          rx0[q] = rx1[q] = 0.f;
        }
        m = fmaxf(m, fmaxf(fabsf(rx0[q]), fabsf(rx1[q])));
      }
    }
    if (p.raw) {
#pragma unroll
      for (int q = 32; q >= 1; q >>= 1) mr += __shfl_xor(mr, q);
      if (lane == 0) m_raw[i] = S * 1.0001f * mr;   // (the sum's rounding cannot undercut it)
    }
#pragma unroll
    for (int q = 32; q >= 1; q >>= 1) {
      m = fmaxf(m, __shfl_xor(m, q));
      acc += __shfl_xor(acc, q);
    }
    const float sc = split_scale(split_clamp_exp(split_exp(__float_as_uint(m))));
    if (lane == 0) m_hd[i] = __float_as_uint(m);
#pragma unroll
    for (int q = 0; q < kCvq; ++q) {
      const int c = lane + 64 * q;
      if (c < n) {
        split_store1(tin + i * AX + c, XP, rx0[q] * sc);
        split_store1(tin + i * AX + n + c, XP, rx1[q] * sc);
      }
    }
    for (int c = X2 + lane; c < XP; c += 64) split_store1(tin + i * AX + c, XP, 0.f);
    if (p.loss_rows && row < B && lane == 0) p.loss_rows[(size_t)k * p.loss_ld + row] = acc;
  }
  __syncthreads();
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    iv[rt] = split_unscale(split_clamp_exp(split_exp(m_hd[rt * 16 + wl])));

  // ---------------- tangent forward, then the adjoint's top ----------------
  // (the forward row scales hold 2^-10 for the layers after the first)
  float iv2[RT];            // adjoint: inverse scale of the lam_zd rows (iv: lam_z)
  auto tan_epi = [&](int j, const f4 (&acc)[RT][CT], _Float16* out) __attribute__((always_inline)) {
    const float un = j == 0 ? kTanhUnscale : kTanhUnscale * kActScale;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int r = rt * 16 + wl;
      const int brow = row0 + r;
      const float mh = __uint_as_float(m_hd[j * R + r]);
      float zb = rb[j] * mh;                   // >= S |zd_j|
      if (j == 0 && p.raw) zb += m_raw[r];
      int e0, e1;
      if (j < L - 1) {
        e0 = e1 = split_clamp_exp(split_exp(__float_as_uint(RES && j >= 1 ? zb + mh : zb)));
      } else {
        e0 = split_clamp_exp(split_exp(__float_as_uint(2.f * zb * cb[0])));
        e1 = split_clamp_exp(split_exp(__float_as_uint(S * cb[0])));
      }
      const float sc0 = split_scale(e0), sc1 = split_scale(e1);
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const f4 zd = acc[rt][c] * iv[rt] * (rnext[c] * un);
        const f4 t = reread(ts[j][rt][c]);
        const f4 d = (1.f - t * t) * dsc(rt, c, j);
        f4 hd = d * zd;
        if constexpr (RES) {
          if (j >= 1) hd += ca[rt][c];
          ca[rt][c] = hd;
        }
        if (brow < B) put4(p.hh[j + 1], p.wd[j + 1], brow, 1, c, hd);
        if (j < L - 1) {
          lds4(out, R + r, c, hd * sc0);
          split_track(m_hd + (j + 1) * R + r, hd);
          split_track(m_zd + j * R + r, zd);
          if (j < LM - 1) zs[j < LM - 1 ? j : 0][rt][c] = zd;
        } else {
          const f4 w4 = *reinterpret_cast<const f4*>(wos + (jt0 + c) * 16 + uq);
          const f4 lzd = d * w4;
          const f4 lz = d * (-2.f * t * zd * w4);
          lds4(out, r, c, lz * sc0);
          lds4(out, R + r, c, lzd * sc1);
          if (brow < B) {
            put4(p.sl[j], p.wd[j + 1], brow, 0, c, lz);
            put4(p.sl[j], p.wd[j + 1], brow, 1, c, lzd);
          }
          split_track(m_zd + j * R + r, zd);
        }
      }
      iv[rt] = split_unscale(e0);
      iv2[rt] = split_unscale(e1);
    }
  };
  {
    f4 acc[RT][CT];
    zero1(acc);
    if constexpr (EARLY) load_rs(0, 0);
    split_gemm_run<RT, CT, PD>(acc, wr, tin, AX, XP, wfwd(0), XP / kSplitKF, lane);
    if constexpr (!EARLY) load_rs(0, 0);
    if (p.raw) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][c] *= iv[rt] * rnext[c];
        rnext[c] = f4{1.f, 1.f, 1.f, 1.f};
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) iv[rt] = 1.f;
      raw_gemm<RT, CT>(acc, raw_src(p.w, k, NP, n), jt0, lane,
                       [&](int rt, int i) { return lds_ld4(xs, (rt * 16 + wl) * X2 + n + i, R * X2); });
    }
    if (L > 1) split_preload<PDH, CT>(wh, wfwd(1), NK, lane);
    tan_epi(0, acc, buf0);
    __syncthreads();
  }
  layers_up<1, LM>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      f4 acc[RT][CT];
      zero1(acc);
      if constexpr (EARLY) load_rs(j, 0);
      split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, buf(j + 1) + R * AS, AS, NP, wfwd(j),
                                              true, j + 1 < L ? wfwd(j + 1) : wbwd(L - 1), lane);
      if constexpr (!EARLY) load_rs(j, 0);
      tan_epi(j, acc, buf(j));
      __syncthreads();
    }
  });
  // ---------------- adjoint reverse (primal and tangent rows together) ----------------
  f4 ch[RT][CT];            // residual carry of lam_h (ca: of lam_hd)
  if constexpr (RES) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        ch[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
        ca[rt][c] = *reinterpret_cast<const f4*>(wos + (jt0 + c) * 16 + uq);
      }
  }
  layers_down<LM - 1, 1>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j < L) {
      _Float16* out = buf(j + 1);
      f4 acc[2 * RT][CT];
#pragma unroll
      for (int rt = 0; rt < 2 * RT; ++rt)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
      if constexpr (EARLY) load_rs(j, 1);
      split_gemm_hidden<2 * RT, CT, PDH, NK, false>(acc, wh, buf(j), AS, NP, wbwd(j),
                                                  j >= 2, wbwd(j >= 2 ? j - 1 : j), lane);
      if constexpr (!EARLY) load_rs(j, 1);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int r = rt * 16 + wl;
        const int brow = row0 + r;
        // bounds of lam_hd and lam_h at the layer below, then of its lam_z rows
        const float mh = j == L - 1 ? 0.f : __uint_as_float(m_lh[j * R + r]);
        const float mhd = j == L - 1 ? cb[0] : __uint_as_float(m_lhd[j * R + r]);
        const float mz = __uint_as_float(m_zd[j * R + r]);
        const float mzp = __uint_as_float(m_zd[(j - 1) * R + r]);
        const float bhd = (cb[j] + (RES ? 1.f : 0.f)) * mhd;
        const float bh = cb[j] * (mh + 2.f * mz * mhd) + (RES ? mh : 0.f);
        const int e0 = split_clamp_exp(split_exp(__float_as_uint(S * (bh + 2.f * mzp * bhd))));
        const int e1 = split_clamp_exp(split_exp(__float_as_uint(S * bhd)));
        const float sc0 = split_scale(e0), sc1 = split_scale(e1);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          f4 lh = acc[rt][c] * iv[rt] * rnext[c];
          f4 lhd = acc[RT + rt][c] * iv2[rt] * rnext[c];
          if constexpr (RES) {
            lh += ch[rt][c];
            ch[rt][c] = lh;
            lhd += ca[rt][c];
            ca[rt][c] = lhd;
          }
          const f4 t = reread(ts[j - 1][rt][c]), zd = zs[j - 1][rt][c];
          const f4 d = (1.f - t * t) * dsc(rt, c, j - 1);
          const f4 lzd = d * lhd;
          const f4 lz = d * (lh - 2.f * t * zd * lhd);
          if (j >= 2) {
            lds4(out, r, c, lz * sc0);
            lds4(out, R + r, c, lzd * sc1);
            split_track(m_lh + (j - 1) * R + r, lh);
            split_track(m_lhd + (j - 1) * R + r, lhd);
          }
          if (brow < B) {
            put4(p.sl[j - 1], p.wd[j], brow, 0, c, lz);
            put4(p.sl[j - 1], p.wd[j], brow, 1, c, lzd);
          }
        }
        iv[rt] = split_unscale(e0);
        iv2[rt] = split_unscale(e1);
      }
      __syncthreads();
    }
  });
}

}  // namespace dev

SplitView split_view(const rid_ensemble_impl& e);
int split_u0_parts(int NP, int XP);

// LDS layout of one instantiation; returns the total bytes.
inline size_t train_f32_layout(int NP, int R, int LM, int XP, int n, TrainF32Args& a) {
  auto al = [](size_t v) { return (unsigned)((v + 15) / 16 * 16); };
  const size_t buf = (size_t)2 * R * dev::split_row_halfs(NP) * 2;
  // buffer 0 also holds the input rows and the partials of u0 (XP > NP: one part)
  const size_t in = (size_t)R * dev::split_row_halfs(XP) * 2;
  size_t off = buf + std::max(buf, in);
  a.off_tin = al(off);
  if (XP > NP) off = a.off_tin + in;
  a.off_xs = al(off);
  off = a.off_xs + (size_t)R * 2 * n * 4;
  a.off_wo = al(off);
  off = a.off_wo + (size_t)NP * 4;
  a.off_mx = al(off);
  return a.off_mx + (size_t)dev::train_track_words(LM, R) * 4;
}

template <int NP, int RT, int NW, int LM, bool RES>
rid_status run_train_f32(const rid_ensemble_impl& e, const TrainIo& io, int B, hipStream_t st) {
  static size_t attr = 0;
  constexpr int R = 16 * RT;
  const SplitDev& s = e.split;
  TrainF32Args a{};
  const size_t lds = train_f32_layout(NP, R, LM, s.XP, e.n_cv, a);
  if (lds > 160 * 1024) return fail(RID_EUNSUPPORTED, "shape too large for the training kernel");
  auto kern = dev::train_f32_kernel<NP, RT, NW, LM, RES>;
  if (lds > 64 * 1024 && lds > attr) {
    RID_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
    attr = lds;
  }
  a.s = io.s; a.F = io.F; a.rho = io.rho; a.raw = e.d_raw;
  a.loss_rows = io.loss_rows; a.loss_ld = io.loss_ld;
  a.row_base = io.row_base; a.B_norm = io.B_norm;
  for (int j = 0; j <= e.L; ++j) a.hh[j] = io.hh[j];
  for (int j = 0; j < e.L; ++j) a.sl[j] = io.sl[j];
  a.B = B; a.n = e.n_cv; a.K = e.K; a.L = e.L; a.XP = s.XP;
  a.n_tiles = (B + R - 1) / R;
  a.xcd_grp = (8 % e.K == 0) ? 8 / e.K : 0;
  a.u0_parts = split_u0_parts(NP, s.XP);
  a.wd[0] = 2 * e.n_cv;
  for (int j = 0; j < e.L; ++j) a.wd[j + 1] = e.widths[j];
  a.w = split_view(e);
  a.drop_p = io.drop_p;
  a.drop_inv = io.drop_p > 0.f ? 1.f / (1.f - io.drop_p) : 1.f;
  a.drop_seed = io.drop_seed;
  a.step = io.step;
  const int grid = a.xcd_grp > 0 ? 8 * ((a.n_tiles + a.xcd_grp - 1) / a.xcd_grp)
                                  : a.n_tiles * e.K;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), (uint32_t)lds, st, a);
  RID_HIP(hipGetLastError());
  return RID_OK;
}

}  // namespace rid
