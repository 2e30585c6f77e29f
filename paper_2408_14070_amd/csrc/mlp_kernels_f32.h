// The FP32 ensembles' fused forward + input-gradient kernel (template; the
// mlp_kernels_f32_*.hip files instantiate it by padded width).
//
// The method is that of mlp_kernels.hip (tanh layers, one reverse sweep for
// g = dA/ds, activations in LDS, tanh' in VGPRs, nothing in HBM between
// layers); the products run as split FP16 (mlp_split.h).  What bounds it:
// the weights.  Every workgroup streams its member's fragments (4 bytes a
// weight, both directions) from L2 into VGPRs, at most 64 bytes a clock per
// CU (57 measured when all CUs stream), while the three FP16 products of 16
// rows take a third of that time; so a workgroup takes as many 16-walker row
// tiles (RT) as the LDS and the registers hold without idling CUs
// (split_rows()).  Against the FP32 MFMA form it replaced (kernel time):
// 1024 walkers, 38 CVs, 4 x [256 x 4]: 33.1 -> 22.5 us; 20 000: 598 -> 224;
// 333 walkers, 120 CVs, 4 x [512 x 4]: 120.6 -> 71; 12 walkers, 18 CVs,
// residual 4 x [300 x 4] (padded to 320 instead of 512): 98.7 -> 38; energies
// of 2000 MCMC walkers 32.5 -> 15 us; force error against FP64 7.1e-7 -> 5.2e-7.
//
// Every walker's result is the same bits whatever the tile it lands in: the
// contraction order, the partial sums of A (per 16-unit tile, in tile order)
// and the parts of the input-gradient product depend on the widths only.
#pragma once

#include <algorithm>
#include <type_traits>

#include "mlp_split.h"

namespace rid {

struct MlpF32Args {
  const float* x;      // [B][2n] input encoding (plain kernel)
  int B, n, K, L, XP, n_tiles, xcd_grp;
  SplitView w;
  float* A_out;        // [K][B]
  float* g_out;        // [K][B][n]
  unsigned off_red, off_mx, off_xs, off_wo;   // LDS byte offsets
  int u0_parts;        // parts of the input-gradient contraction (1, 2 or 4)
  dev::SysView sv;          // torsion input (bias path)
  const float* pos;    // [B][n_atoms][3]
  const uint8_t* raw;  // raw[i] = 1: CV i is non-angular, encoded (s_i, 0)
};

namespace dev {

// GRAD = false: the free energies only (no tanh' stash, no reverse sweep).
// RES: residual layers, h_l = h_{l-1} + tanh(z_l) for l >= 2.
template <int NP, int RT, int NW, int LM, bool FROM_POS, bool GRAD, bool RES>
__global__ __launch_bounds__(NW * 64) void mlp_f32_kernel(MlpF32Args p) {
  constexpr int CT = NP / (16 * NW);
  constexpr int R = 16 * RT;
  constexpr int JT = NP / 16;
  constexpr int NK = NP / kSplitKF;
  constexpr int PD = 2;                        // first layer's weight pipeline depth
  constexpr int PDH = split_depth(NK, CT);
  // activation fragments a k-step ahead, and the epilogue's bias and row
  // scales loaded before the product, where the registers allow it
  constexpr bool ADB = RT * CT == 1 || (RT * CT <= 4 && NW <= 12 && !RES);
  constexpr bool EARLY = CT < 4;
  static_assert(CT >= 1 && CT * 16 * NW == NP, "width/wave split");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int k, tile;
  map_block(blockIdx.x, p.K, p.xcd_grp, k, tile);
  if (tile >= p.n_tiles) return;
  const int row0 = tile * R;
  const int n = p.n, L = p.L, XP = p.XP, X2 = 2 * p.n;
  constexpr int AS = split_row_halfs(NP);      // row stride (halfs)
  constexpr int BUF = R * AS;                  // halfs per ping-pong buffer
  const int AX = split_row_halfs(XP);          // row stride of the input tile
  _Float16* const buf1 = reinterpret_cast<_Float16*>(smem);
  _Float16* const buf0 = buf1 + BUF;
  auto buf = [&](int i) { return i & 1 ? buf1 : buf0; };
  float* u0 = reinterpret_cast<float*>(buf0);                // partials of u0
  const int US = XP + 4;
  float* red = reinterpret_cast<float*>(smem + p.off_red);   // [JT][R]
  unsigned* mx = reinterpret_cast<unsigned*>(smem + p.off_mx);   // [LM][R] row maxima
  int* ec = reinterpret_cast<int*>(mx + LM * R);             // [kMaxHidden + 1] bounds (exponents)
  float* xs = reinterpret_cast<float*>(smem + p.off_xs);     // [R][2n] cos|sin (FROM_POS)
  float* wos = reinterpret_cast<float*>(smem + p.off_wo);    // [NP] output weights

  const unsigned char* fbase = p.w.frag + (size_t)k * p.w.frag_bytes;
  const float* bias = p.w.bias + (size_t)k * L * NP;
  const float* rs = p.w.rs + (size_t)k * L * 2 * p.w.RW;     // [L][2][RW]
  const int jt0 = wave * CT;
  const int wl = lane & 15;                    // walker within a 16-row tile
  const int uq = 4 * (lane >> 4);              // first of the lane's 4 units in a tile
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(fbase), (short)0, (int)p.w.frag_bytes, 0x00020000);
  auto wsrc = [&](unsigned off) {
    return SplitSrc{rsrc, (int)off + jt0 * kSplitFrag, JT * kSplitFrag};
  };
  // plain input: the first column batch of the tile's encoding is loaded
  // before anything else (rows to the waves in turn, lanes over float2
  // columns)
  constexpr int RW_ = FROM_POS ? 1 : (R + NW - 1) / NW;      // rows per wave
  float2 xv[RW_];
  auto load_x = [&](int cb) {
    const int col = cb + lane;
#pragma unroll
    for (int j = 0; j < RW_; ++j) {
      const int i = wave + j * NW;
      const int row = row0 + i;
      xv[j] = (i < R && col < n && row < p.B)
                  ? *reinterpret_cast<const float2*>(p.x + (size_t)row * X2 + 2 * col)
                  : make_float2(0.f, 0.f);
    }
  };
  if constexpr (!FROM_POS) load_x(0);
  SplitRing<PD, CT> wr;              // first layer
  SplitRing<PDH, CT> wh;             // hidden layers
  split_preload<PD, CT>(wr, wsrc(p.w.fwd_off[0]), XP / kSplitKF, lane);
  f4 bnext[CT], rnext[CT];           // bias and row scales of the coming epilogue
  const VecSrc vrs = vec_src(rs, L * 2 * p.w.RW), vbias = vec_src(bias, L * NP);
  auto load_fwd = [&](int l) {
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      bnext[c] = vbias.ld4(l * NP + (jt0 + c) * 16, uq);
      rnext[c] = vrs.ld4(l * 2 * p.w.RW + (jt0 + c) * 16, uq);
    }
  };
  auto load_bwd = [&](int l) {
#pragma unroll
    for (int c = 0; c < CT; ++c) rnext[c] = vrs.ld4((l * 2 + 1) * p.w.RW + (jt0 + c) * 16, uq);
  };
  load_fwd(0);
  for (int i = threadIdx.x; i < NP; i += NW * 64) wos[i] = p.w.wo[(size_t)k * NP + i];
  if constexpr (GRAD) {
    for (int i = threadIdx.x; i < LM * R; i += NW * 64) mx[i] = 0u;
    // exponents of the backward layers' row-sum bounds (slot l), and of the
    // largest |w_o| (slot 0: layer 0's bound is never needed)
    for (int l = wave; l < L; l += NW) {
      float b = 0.f;
      if (l > 0) {
        if (lane < JT) b = p.w.bound[(((size_t)k * L + l) * 2 + 1) * 32 + lane];
      } else {
        for (int i = lane; i < NP; i += 64) b = fmaxf(b, fabsf(p.w.wo[(size_t)k * NP + i]));
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) b = fmaxf(b, __shfl_xor(b, m));
      if (RES && l > 0) b += 1.f;    // the skip adds the layer's own dA/dh
      if (lane == 0) ec[l] = split_exp(__float_as_uint(b));
    }
  }

  // ---------------- input tile: x = [cos s | sin s] -> buffer 0 ----------------
  if constexpr (FROM_POS) {
    // torsions of the tile's walkers (the gather scratch, buffer 1, holds them
    // all: gather_pays).  Gather: a lane owns coordinates j = lane + 64m of the
    // unique-atom list and copies them for the walkers of its wave (walkers to
    // the waves in turn); then a lane per torsion.  Coordinates go in chunks of
    // kGatherBatch per lane: the chunk's index loads, then its coordinate loads
    // for the wave's walkers, then the stores.  Slots past the end are clamped to
    // the last coordinate or walker (they store that slot's own value again), so
    // no load sits behind a branch; walkers past B get zeros.
    float* sp = reinterpret_cast<float*>(buf1);   // [R][U][3]
    const int U3 = 3 * p.sv.U;
    constexpr int WPW = (R + NW - 1) / NW;    // walkers per wave, at most
    constexpr int QB = WPW < 4 ? WPW : 4;     // walkers per batch of loads
    const size_t wstride = (size_t)p.sv.n_atoms * 3;
    for (int j0 = lane; j0 < U3; j0 += kGatherBatch * 64) {
      int jc[kGatherBatch], a[kGatherBatch];
#pragma unroll
      for (int m = 0; m < kGatherBatch; ++m) {
        jc[m] = min(j0 + m * 64, U3 - 1);
        const int u = jc[m] / 3;
        a[m] = 3 * p.sv.uniq[u] + (jc[m] - 3 * u);
      }
#pragma unroll 1
      for (int q0 = 0; wave + q0 * NW < R; q0 += QB) {
        float v[QB][kGatherBatch];
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const int row = min(row0 + min(wave + (q0 + q) * NW, R - 1), p.B - 1);
#pragma unroll
          for (int m = 0; m < kGatherBatch; ++m) v[q][m] = p.pos[row * wstride + a[m]];
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const int i = min(wave + (q0 + q) * NW, R - 1);
#pragma unroll
          for (int m = 0; m < kGatherBatch; ++m)
            sp[i * U3 + jc[m]] = row0 + i < p.B ? v[q][m] : 0.f;
        }
      }
    }
    __syncthreads();
    for (int i = wave; i < R; i += NW) {
      for (int c = lane; c < n; c += 64) {
        float cs = 0.f, sn = 0.f;
        if (row0 + i < p.B) {
          const Torsion t = torsion(sp + i * U3, p.sv.lq + 4 * c);
          torsion_cos_sin(t, cs, sn);
        }
        xs[i * X2 + c] = cs;
        xs[i * X2 + n + c] = sn;
        split_store1(buf0 + i * AX + c, XP, cs * kActScale);
        split_store1(buf0 + i * AX + n + c, XP, sn * kActScale);
      }
    }
    for (int i = wave; i < R; i += NW)
      for (int c = X2 + lane; c < XP; c += 64) split_store1(buf0 + i * AX + c, XP, 0.f);
  } else {
    // the column batches of the tile (the first one is already in xv);
    // padding columns [X2, XP) get zeros (X2 is even), and so do the raw CVs'
    // (their part of layer 1 is added in FP32)
    const int hp = XP / 2;
    for (int cb = 0; cb < hp; cb += 64) {
      const int col = cb + lane;               // float2 column
      if (cb > 0) load_x(cb);
      if (col < hp) {
        bool zx = false, zy = false;
        if (p.raw) {
          zx = 2 * col < n && p.raw[min(2 * col, n - 1)];
          zy = 2 * col + 1 < n && p.raw[min(2 * col + 1, n - 1)];
        }
#pragma unroll
        for (int j = 0; j < RW_; ++j) {
          const int i = wave + j * NW;
          const float vx = zx ? 0.f : xv[j].x * kActScale, vy = zy ? 0.f : xv[j].y * kActScale;
          if (i < R) split_store2(buf0 + i * AX + 2 * col, XP, vx, vy);
        }
      }
    }
  }
  __syncthreads();

  f4 st[LM - 1][RT][CT];             // tanh' of hidden layers 1..L-1
  f4 ares[RT][CT];                   // RES: the layer's input h, then dA/dh (FP32)
  float apart[RT][CT];               // the lane's part of A = w_o . h_L, per unit tile

  // ---------------- forward: h_l = tanh(W_l h_{l-1} + b_l) ----------------
  // tile epilogues: y = acc * rs + b, tanh and its derivative; a layer
  // before the last stores h_l into the other buffer and keeps tanh'; the
  // last layer stores v_L = w_o * tanh' (scaled) and its part of A.
  // h scaled by kActScale, d = tanh'
  auto act_tile = [&](const f4& z, const f4& b, const f4& r, float iv, f4& h, f4& d) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float dq;
      const float t = tanh_and_grad(__builtin_fmaf(z[q] * iv, r[q], b[q]), dq);
      h[q] = t * kActScale;
      d[q] = dq;
    }
  };
  auto mid_tile = [&](int l, int rt, int c, const f4& z, float iv, _Float16* out) {
    f4 h, d;
    act_tile(z, bnext[c], rnext[c], iv, h, d);
    if constexpr (RES) {
      if (l >= 1) h += ares[rt][c];  // the lane's own units of h_{l-1}
      ares[rt][c] = h;
    }
    split_store4(out + (rt * 16 + wl) * AS + (jt0 + c) * 16 + uq, NP, h);
    if constexpr (GRAD) st[l][rt][c] = d;
  };
  auto last_tile = [&](int rt, int c, const f4& z, float iv, bool skip, _Float16* out) {
    const int u = (jt0 + c) * 16 + uq;
    const f4 w4 = *reinterpret_cast<const f4*>(wos + u);
    f4 h, d;
    act_tile(z, bnext[c], rnext[c], iv, h, d);
    if constexpr (RES) {
      if (skip) h += ares[rt][c];
      ares[rt][c] = w4;              // dA/dh_L = w_o
    }
    apart[rt][c] = w4[0] * h[0] + w4[1] * h[1] + w4[2] * h[2] + w4[3] * h[3];
    if constexpr (GRAD) {
      const f4 v = w4 * d;
      if constexpr (!RES)
        split_track(mx + (L - 1) * R + rt * 16 + wl, v);
      split_store4(out + (rt * 16 + wl) * AS + u, NP, v * split_scale(split_clamp_exp(ec[0])));
    }
  };
  // the product after forward layer l: forward layer l+1, or the first backward
  auto next_after_fwd = [&](int l) {
    return wsrc(l + 1 < L ? p.w.fwd_off[l + 1] : p.w.bwd_off[L > 1 ? L - 1 : 0]);
  };
  auto zero = [&](f4 (&acc)[RT][CT]) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
  };

  {  // layer 1 (input width XP)
    _Float16* out = buf1;
    f4 acc[RT][CT];
    zero(acc);
    split_gemm_run<RT, CT, PD>(acc, wr, buf0, AX, XP, wsrc(p.w.fwd_off[0]), XP / kSplitKF, lane);
    float iv = kActUnscale;
    if constexpr (!FROM_POS) {
      if (p.raw) {                     // acc becomes y, the raw CVs' part on top
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              acc[rt][c][q] = __builtin_fmaf(acc[rt][c][q] * iv, rnext[c][q], bnext[c][q]);
          rnext[c] = f4{1.f, 1.f, 1.f, 1.f};
          bnext[c] = f4{0.f, 0.f, 0.f, 0.f};
        }
        iv = 1.f;
        const __amdgpu_buffer_rsrc_t xr =
            row_src(p.x + (size_t)row0 * X2, min(R, p.B - row0), X2);
        raw_gemm<RT, CT>(acc, raw_src(p.w, k, NP, n), jt0, lane, [&](int rt, int i) {
          return raw_value(row_ld(xr, (rt * 16 + wl) * X2 + i));
        });
      }
    }
    if (L > 1) split_preload<PDH, CT>(wh, next_after_fwd(0), NK, lane);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        if (L > 1) mid_tile(0, rt, c, acc[rt][c], iv, out);
        else last_tile(rt, c, acc[rt][c], iv, false, out);
      }
    __syncthreads();
  }
  // hidden layers before the last
  layers_up<1, LM - 1>([&](auto lc) __attribute__((always_inline)) {
    constexpr int l = decltype(lc)::value;
    if (l < L - 1) {
      const _Float16* in = buf(l);
      _Float16* out = buf(l + 1);
      f4 acc[RT][CT];
      zero(acc);
      if constexpr (EARLY) load_fwd(l);
      split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, in, AS, NP, wsrc(p.w.fwd_off[l]), true,
                                              next_after_fwd(l), lane);
      if constexpr (!EARLY) load_fwd(l);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int c = 0; c < CT; ++c) mid_tile(l, rt, c, acc[rt][c], 1.f, out);
      __syncthreads();
    }
  });
  if (L > 1) {  // the last hidden layer (index L-1)
    const _Float16* in = buf(L - 1);
    _Float16* out = buf(L);
    f4 acc[RT][CT];
    zero(acc);
    if constexpr (EARLY) load_fwd(L - 1);
    split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, in, AS, NP, wsrc(p.w.fwd_off[L - 1]), GRAD,
                                            wsrc(p.w.bwd_off[L - 1]), lane);
    if constexpr (!EARLY) load_fwd(L - 1);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CT; ++c) last_tile(rt, c, acc[rt][c], 1.f, true, out);
    __syncthreads();
  }
  // A = w_o . h_L + b_o: the lanes' partials over the 4 unit groups, then
  // (after the next barrier) over the unit tiles in order
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      float v = apart[rt][c];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) red[(jt0 + c) * R + rt * 16 + wl] = v;
    }
  auto store_A = [&]() {
    for (int i = threadIdx.x; i < R; i += NW * 64) {
      float a = 0.f;
#pragma unroll
      for (int j = 0; j < JT; ++j) a += red[j * R + i];
      if (row0 + i < p.B)
        p.A_out[(size_t)k * p.B + row0 + i] = __builtin_fmaf(a, kActUnscale, p.w.bo[k]);
    }
  };
  if constexpr (!GRAD) {
    __syncthreads();
    store_A();
    return;
  }

  // ------------- reverse sweep: v_{l-1} = (W_l^T v_l) * tanh'_{l-1} -------------
  // The row scale of v_{l-1} comes from the row's largest entry of v_l (RES:
  // of dA/dh_l) times the layer's bound; iv undoes the scale of the operand.
  float iv[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) iv[rt] = split_unscale(split_clamp_exp(ec[0]));
  layers_down<LM - 1, 1>([&](auto lc) __attribute__((always_inline)) {
    constexpr int l = decltype(lc)::value;
    if (l < L) {
      const _Float16* in = buf(l + 1);
      _Float16* out = buf(l);
      f4 acc[RT][CT];
      zero(acc);
      if constexpr (EARLY) load_bwd(l);
      split_gemm_hidden<RT, CT, PDH, NK, ADB>(acc, wh, in, AS, NP, wsrc(p.w.bwd_off[l]), l >= 2,
                                              wsrc(p.w.bwd_off[l >= 2 ? l - 1 : l]), lane);
      if constexpr (!EARLY) load_bwd(l);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        // RES: dA/dh_L = w_o for every row, bounded by slot 0
        const int em = RES && l == L - 1 ? ec[0] : split_exp(mx[l * R + rt * 16 + wl]);
        const int e = split_clamp_exp(ec[l] + em);
        const float sc = split_scale(e);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          f4 y = acc[rt][c] * iv[rt] * rnext[c];
          if constexpr (RES) {
            ares[rt][c] += y;
            y = ares[rt][c];
          }
          const f4 v = y * st[l - 1][rt][c];
          if (l >= 2) split_track(mx + (l - 1) * R + rt * 16 + wl, RES ? y : v);
          split_store4(out + (rt * 16 + wl) * AS + (jt0 + c) * 16 + uq, NP, v * sc);
        }
        iv[rt] = split_unscale(e);
      }
      __syncthreads();
    }
  });
  // ------------- layer 1 backward: u0 = W_1^T v_1 -------------
  // XP/16 column tiles, each tile's contraction cut into parts so that they
  // spread over the waves; partial sums to LDS (part q at u0 + q * R * US),
  // added in part order when u0 is read.  v_1 sits in buffer 1, the partials
  // in buffer 0.
  auto u0_stage = [&](auto parts_c) {
    constexpr int PARTS = decltype(parts_c)::value;
    constexpr int KQ = NK / PARTS;             // k-steps per part
    const _Float16* in = buf1;
    const int JT0 = XP / 16;
    for (int it = wave; it < JT0 * PARTS; it += NW) {
      const int t = it / PARTS, q = it - t * PARTS;
      const SplitSrc src{rsrc,
                         (int)p.w.bwd_off[0] + t * kSplitFrag + q * KQ * JT0 * kSplitFrag,
                         JT0 * kSplitFrag};
      const f4 r4 = vrs.ld4(p.w.RW + t * 16, uq);   // backward row scales of layer 1
      constexpr int PU = KQ < 4 ? KQ : 4;      // loads in flight
      SplitRing<PU, 1> w0;
      split_preload<PU, 1>(w0, src, KQ, lane);
      f4 a1[RT][1];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a1[rt][0] = f4{0.f, 0.f, 0.f, 0.f};
      split_gemm_run<RT, 1, PU>(a1, w0, in + q * KQ * kSplitKF, AS, NP, src, KQ, lane);
      float* uq0 = u0 + q * R * US;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        *reinterpret_cast<f4*>(uq0 + (rt * 16 + wl) * US + t * 16 + uq) =
            a1[rt][0] * iv[rt] * r4;
    }
  };
  // chain to the angles: g_i = -sin s_i u0[i] + cos s_i u0[n+i]
  auto chain = [&](auto parts_c) {
    constexpr int PARTS = decltype(parts_c)::value;
    auto u0_at = [&](int i, int c) {
      float v = u0[i * US + c];
#pragma unroll
      for (int q = 1; q < PARTS; ++q) v += u0[q * R * US + i * US + c];
      return v;
    };
    for (int e = threadIdx.x; e < R * n; e += NW * 64) {
      const int i = e / n, c = e - i * n;
      const int row = row0 + i;
      if (row < p.B) {
        const float* xr = FROM_POS ? xs + i * X2 : p.x + (size_t)row * X2;
        const float cs = xr[c];
        const float sn = xr[n + c];
        float gv = -sn * u0_at(i, c) + cs * u0_at(i, n + c);
        if constexpr (!FROM_POS) {
          if (p.raw && p.raw[c]) gv = u0_at(i, c);
        }
        p.g_out[((size_t)k * p.B + row) * n + c] = gv;
      }
    }
  };
  auto finish = [&](auto parts_c) {
    u0_stage(parts_c);
    __syncthreads();
    store_A();
    chain(parts_c);
  };
  if (NK % 4 == 0 && p.u0_parts == 4) finish(std::integral_constant<int, NK % 4 == 0 ? 4 : 1>{});
  else if (p.u0_parts == 2) finish(std::integral_constant<int, 2>{});
  else finish(std::integral_constant<int, 1>{});
}

}  // namespace dev

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
SplitView split_view(const rid_ensemble_impl& e);
inline unsigned align16(size_t v) { return (unsigned)((v + 15) / 16 * 16); }

int split_u0_parts(int NP, int XP);

// LDS layout of one instantiation; returns the total bytes.
inline size_t mlp_f32_layout(int NP, int R, int LM, int XP, int n, bool from_pos,
                             MlpF32Args& a) {
  const size_t buf = (size_t)R * dev::split_row_halfs(NP) * 2;
  // buffer 0 also holds the input rows and the partials of u0 (XP > NP: one part)
  size_t off = buf + std::max(buf, (size_t)R * dev::split_row_halfs(XP) * 2);
  a.off_red = align16(off);
  off = a.off_red + (size_t)(NP / 16) * R * 4;
  a.off_mx = align16(off);
  off = a.off_mx + (size_t)LM * R * 4 + (kMaxHidden + 1) * 4;
  a.off_xs = align16(off);
  off = a.off_xs + (from_pos ? (size_t)R * 2 * n * 4 : 0);
  a.off_wo = align16(off);
  return a.off_wo + (size_t)NP * 4;
}
// Whether buffer 1 (free before layer 1) holds a tile's torsion atoms.
inline bool mlp_f32_gathers(int NP, int R, int U) {
  return (size_t)R * dev::split_row_halfs(NP) * 2 >= (size_t)R * U * 12;
}

// One instantiation.  RID_EUNSUPPORTED (without a message of its own where
// the caller has another form to take) when the LDS does not hold it.
template <int NP, int RT, int NW, int LM, bool RES>
rid_status run_mlp_f32(const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                       float* g_out, const TorsionInput* tin, hipStream_t st) {
  static size_t attr_bytes[3] = {0, 0, 0};   // dynamic-LDS limit set per kernel
  constexpr int R = 16 * RT;
  const bool from_pos = tin != nullptr, grad = g_out != nullptr;
  const SplitDev& s = e.split;
  MlpF32Args a{};
  const size_t lds = mlp_f32_layout(NP, R, LM, s.XP, e.n_cv, from_pos, a);
  if (lds > 160 * 1024) return fail(RID_EUNSUPPORTED, "shape too large for the MLP kernel's LDS");
  if (from_pos && (RT > 1 || !grad || !mlp_f32_gathers(NP, R, tin->sys->n_uniq)))
    return fail(RID_EUNSUPPORTED, "in-kernel torsions: not this form (gather_pays)");
  auto kern = grad ? dev::mlp_f32_kernel<NP, RT, NW, LM, false, true, RES>
                   : dev::mlp_f32_kernel<NP, RT, NW, LM, false, false, RES>;
  if constexpr (RT == 1) {
    if (from_pos) kern = dev::mlp_f32_kernel<NP, RT, NW, LM, true, true, RES>;
  }
  const int ki = grad ? (from_pos ? 1 : 0) : 2;
  if (lds > 64 * 1024 && lds > attr_bytes[ki]) {
    RID_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
    attr_bytes[ki] = lds;
  }
  a.x = x; a.B = B; a.n = e.n_cv; a.K = e.K; a.L = e.L; a.XP = s.XP;
  a.n_tiles = (B + R - 1) / R;
  a.xcd_grp = (8 % e.K == 0) ? 8 / e.K : 0;
  a.w = split_view(e);
  a.u0_parts = split_u0_parts(NP, s.XP);
  a.A_out = A_out; a.g_out = g_out;
  a.raw = e.d_raw;
  if (from_pos) {
    const rid_system_impl& sy = *tin->sys;
    a.sv = dev::SysView{sy.n_atoms, sy.n_uniq, sy.n_cv, sy.d_uniq, sy.d_lquads, sy.d_csr_ptr,
                   sy.d_csr_ent, sy.d_atom_local};
    a.pos = tin->pos;
  }
  const int grid = a.xcd_grp > 0 ? 8 * ((a.n_tiles + a.xcd_grp - 1) / a.xcd_grp)
                                  : a.n_tiles * e.K;
  launch_timed(kProfMlp, kern, dim3(grid), dim3(NW * 64), (uint32_t)lds, st, a);
  RID_HIP(hipGetLastError());
  return RID_OK;
}
}  // namespace rid
