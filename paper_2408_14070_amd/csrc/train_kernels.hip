// Mean-force fitting step ("Training phase"): the models' CV gradients are
// fitted to mean-force labels, so the loss gradient in the weights needs the
// derivative of dA/ds -- a double backward.
//
// With rho_b = 2 (g_b - F_b) / B mapped to the input x (rho_x), the weight
// gradient of L = (1/B) sum_b |g_b - F_b|^2 equals the gradient of
// J = sum_b rho_x,b . dA/dx with rho_x held fixed:
//   primal   h_l = tanh(W_l h_{l-1} + b_l)                 (h_0 = x)
//   backward v_L = w_o (1-h_L^2), u_{l-1} = W_l^T v_l, v_l = u_l (1-h_l^2)
//   tangent  zd_l = W_l hd_{l-1}, hd_l = (1-h_l^2) zd_l     (hd_0 = rho_x)
//   adjoint  lam_hd_L = w_o, lam_h_L = 0; for l = L..1:
//            lam_zd = (1-h_l^2) lam_hd, lam_h -= 2 h_l zd_l lam_hd,
//            lam_z = (1-h_l^2) lam_h,
//            dW_l = lam_z^T h_{l-1} + lam_zd^T hd_{l-1}, db_l = sum lam_z,
//            [lam_h ; lam_hd]_{l-1} = [lam_z ; lam_zd] W_l
//   dw_o = sum hd_L, db_o = 0.
// Then one Adam step on the FP32 masters.
//
// The sweeps run fused (train_sweep_f32.h); 16-bit ensembles, and the few FP32
// forms the fused kernel does not hold (train_fused_supported), take them as
// separate GEMMs here, in the same general form.  With t_l =
// tanh(z_l), dropout factors S_l (1 without dropout) and d_l = S_l (1 - t_l^2):
//   primal   h_l = S_l t_l (+ h_{l-1} for a residual layer l >= 2)
//   backward u_L = w_o, v_l = u_l d_l, u_{l-1} = W_l^T v_l (+ u_l, residual)
//   tangent  hd_l = d_l zd_l (+ hd_{l-1}, residual)
//   adjoint  lam_zd = d_l lam_hd, lam_z = d_l (lam_h - 2 t_l zd_l lam_hd),
//            [lam_h ; lam_hd]_{l-1} = [lam_z ; lam_zd] W_l (+ [lam_h ; lam_hd]_l,
//            residual)
// Raw CVs (angular mask 0) enter as (s, 0): their mean force is dA/dx_i and
// rho reaches the input as (rho_i, 0).
//
// Layout: batched over the K members; "stacked" tensors hold the primal
// quantity in rows [0, B) and the tangent one in rows [B, 2B) of each
// member's slab, so one GEMM moves both halves, and the weight gradient is a
// single contraction over 2B rows.  The general sweeps' GEMMs are one
// hand-written FP32-MFMA kernel (LDS double buffering, arbitrary strides, fused
// epilogues); the weight gradients of both forms are wgrad_kernel's, split along
// the batch with a fixed-order reduction, so the whole step is deterministic.
#include "device_common.h"

namespace rid {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int BK = 16;              // contraction block
constexpr int kThreads = 256;

enum Epi {
  EPI_STORE = 0,      // C = acc
  EPI_BIAS_TANH = 1,  // C = tanh(acc + bias[n])
  EPI_GEN = 2         // r = acc + add; C = r (if C); C2 = r * mul + add2 (if C2)
};

struct GemmArgs {
  const float* A;
  long long sAb, sAm, sAk;
  const float* Bm;
  long long sBb, sBk, sBn;
  float* C;
  long long sCb, sCm, sCn;
  float* C2;                      // second output (EPI_GEN): C's row and
  long long sC2b;                 // column strides, own batch stride
  const float* bias;
  long long sBiasb;
  // EPI_GEN operands (each null or indexed like C, with its own batch stride)
  const float* add;
  long long sAddb;
  const float* mul;
  long long sMulb;
  const float* add2;
  long long sAdd2b;
  int M, N, Kc, batch, mode;
  int modeA, modeB;               // operand load modes (TileLoad), set by gemm()
};

// One operand tile of TR rows x BK contraction into LDS [row][k].  Element
// (r, k) of the operand is at X[r * sR + k * sK].  Modes: 0 scalar loads,
// k fastest; 1 scalar, rows fastest; 2 float4 along k (sK == 1); 3 float4
// along rows (sR == 1).  The float4 modes need 16-byte alignment and an
// extent along the vector that is a multiple of 4 (gemm() checks).
template <int TR, int BKT = BK>
struct TileLoad {
  static constexpr int NS = TR * BKT / kThreads;   // elements per thread
  float v[NS];
  // Branch-free loads (the mode is uniform; the two mappings are selected,
  // an element outside the operand reads its first one), so every load of a
  // tile is in flight before anything waits on one.  The outside elements
  // are zeroed when the tile is stored to LDS, after the block's MFMAs.
  // VEC: the float4 modes (chosen at compile time, so that no branch joins
  // the two load paths: a join makes the compiler wait on the loads there).
  unsigned long long in_mask;
  template <bool VEC>
  __device__ inline void load(const float* X, long long sR, long long sK, int mode, int r0,
                              int R, int kb, int k_end, int tid) {
    static_assert(NS <= 64, "one mask bit per element");
    in_mask = 0ull;
    if constexpr (VEC && NS >= 4) {
      const bool kv = mode == 2;
#pragma unroll
      for (int j = 0; j < NS / 4; ++j) {
        const int idx = tid + kThreads * j;
        const int r = kv ? idx / (BKT / 4) : (idx % (TR / 4)) * 4;
        const int k = kv ? (idx % (BKT / 4)) * 4 : idx / (TR / 4);
        const int gr = r0 + r, gk = kb + k;
        const bool in = gr < R && gk < k_end;
        in_mask |= (unsigned long long)in << j;
        const f4 x = *reinterpret_cast<const f4*>(X + (in ? gr * sR + gk * sK : 0));
        v[4 * j] = x[0];
        v[4 * j + 1] = x[1];
        v[4 * j + 2] = x[2];
        v[4 * j + 3] = x[3];
      }
    } else {
      const bool kf = (mode & 1) == 0;     // modes 0 and 2: k fastest
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const int idx = tid + kThreads * j;
        const int k = kf ? idx % BKT : idx / TR;
        const int r = kf ? idx / BKT : idx % TR;
        const int gr = r0 + r, gk = kb + k;
        const bool in = gr < R && gk < k_end;
        in_mask |= (unsigned long long)in << j;
        v[j] = X[in ? gr * sR + gk * sK : 0];
      }
    }
  }
  template <bool VEC>
  __device__ inline void store(float (*S)[BKT + 4], int mode, int tid) const {
    if constexpr (VEC && NS >= 4) {
#pragma unroll
      for (int j = 0; j < NS / 4; ++j) {
        const int idx = tid + kThreads * j;
        const bool in = (in_mask >> j) & 1ull;
        const f4 x = in ? f4{v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]}
                        : f4{0.f, 0.f, 0.f, 0.f};
        if (mode == 2) {
          const int r = idx / (BKT / 4), k = (idx % (BKT / 4)) * 4;
          *reinterpret_cast<f4*>(&S[r][k]) = x;
        } else {
          const int k = idx / (TR / 4), r = (idx % (TR / 4)) * 4;
#pragma unroll
          for (int e = 0; e < 4; ++e) S[r + e][k] = x[e];
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const int idx = tid + kThreads * j;
        int r, k;
        if ((mode & 1) == 0) { k = idx % BKT; r = idx / BKT; } else { r = idx % TR; k = idx / TR; }
        S[r][k] = ((in_mask >> j) & 1ull) ? v[j] : 0.f;
      }
    }
  }
};

__device__ inline float tanh_fast(float z) {
  const float e = __expf(2.f * z);
  return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + e);
}

// C[b] = A[b] (M x Kc) * B[b] (Kc x N) on FP32 MFMA, tiles of TM x TN with
// 4 waves of (TM/2) x (TN/2); operands staged through double-buffered LDS
// in contraction blocks of BKT.  128 x 128 tiles (16 accumulator tiles per
// wave) reuse each LDS operand fragment four times; 64 x 64 tiles serve
// narrow shapes.  Grids too small to fill the chip (small batches) take
// 64-deep blocks: each block costs about one memory latency, so a deeper
// block divides the latency-bound time of such a GEMM by four.
template <int TM, int TN, int BKT, bool VA, bool VB>
__global__ __launch_bounds__(kThreads) void gemm_f32_kernel(GemmArgs g) {
  constexpr int WM = TM / 2, WN = TN / 2;           // wave tile
  constexpr int TI = WM / 16, TJ = WN / 16;         // 16 x 16 MFMA tiles per wave
  static_assert(BKT % 16 == 0, "contraction blocks of whole 16-deep MFMA sets");
  __shared__ __attribute__((aligned(16))) float As[2][TM][BKT + 4];
  __shared__ __attribute__((aligned(16))) float Bs[2][TN][BKT + 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.z;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
  const float* A = g.A + b * g.sAb;
  const float* Bp = g.Bm + b * g.sBb;
  TileLoad<TM, BKT> ta;
  TileLoad<TN, BKT> tb;
  auto load = [&](int kb) {
    ta.template load<VA>(A, g.sAm, g.sAk, g.modeA, m0, g.M, kb, g.Kc, tid);
    tb.template load<VB>(Bp, g.sBn, g.sBk, g.modeB, n0, g.N, kb, g.Kc, tid);
  };
  auto store = [&](int buf) {
    ta.template store<VA>(As[buf], g.modeA, tid);
    tb.template store<VB>(Bs[buf], g.modeB, tid);
  };

  const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;
  const int r = lane & 15, gq = lane >> 4;
  f4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  int buf = 0;
  load(0);
  store(0);
  __syncthreads();
  for (int kb = 0; kb < g.Kc; kb += BKT) {
    const bool more = kb + BKT < g.Kc;
    if (more) load(kb + BKT);
#pragma unroll
    for (int sb = 0; sb < BKT / 16; ++sb) {
      f4 a[TI], bb[TJ];
#pragma unroll
      for (int i = 0; i < TI; ++i)
        a[i] = *reinterpret_cast<const f4*>(&As[buf][wm + i * 16 + r][16 * sb + 4 * gq]);
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        bb[j] = *reinterpret_cast<const f4*>(&Bs[buf][wn + j * 16 + r][16 * sb + 4 * gq]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
            acc[i][j] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], bb[j][e], acc[i][j], 0, 0, 0);
    }
    if (more) {
      store(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
  }

  // Epilogue, one row of 16 x 16 tiles at a time: the operands it reads
  // (bias, add, mul, add2) are loaded for all of the row's elements before
  // any is used (an element outside C reads element 0 and is not stored),
  // so their loads are in flight together.
  float* C = g.C ? g.C + b * g.sCb : nullptr;
  constexpr int E = TJ * 4;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    long long ci[E];
    bool in[E];
    float bi[TJ], ad[E], mu[E], a2[E];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int n = n0 + wn + j * 16 + r;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm + i * 16 + 4 * gq + q;
        in[4 * j + q] = n < g.N && m < g.M;
        ci[4 * j + q] = in[4 * j + q] ? m * g.sCm + n * g.sCn : 0;
      }
      bi[j] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) ad[e] = mu[e] = a2[e] = 0.f;
    if (g.mode == EPI_BIAS_TANH) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) bi[j] = g.bias[b * g.sBiasb + min(n0 + wn + j * 16 + r, g.N - 1)];
    } else if (g.mode == EPI_GEN) {
      if (g.add)
#pragma unroll
        for (int e = 0; e < E; ++e) ad[e] = g.add[b * g.sAddb + ci[e]];
      if (g.C2) {
#pragma unroll
        for (int e = 0; e < E; ++e) mu[e] = g.mul[b * g.sMulb + ci[e]];
        if (g.add2)
#pragma unroll
          for (int e = 0; e < E; ++e) a2[e] = g.add2[b * g.sAdd2b + ci[e]];
      }
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = 4 * j + q;
        if (!in[e]) continue;
        const float v = acc[i][j][q];
        if (g.mode == EPI_STORE) {
          C[ci[e]] = v;
        } else if (g.mode == EPI_BIAS_TANH) {
          C[ci[e]] = tanh_fast(v + bi[j]);
        } else {
          const float rr = g.add ? v + ad[e] : v;
          if (C) C[ci[e]] = rr;
          if (g.C2) {
            float o = rr * mu[e];
            if (g.add2) o += a2[e];
            g.C2[b * g.sC2b + ci[e]] = o;
          }
        }
      }
  }
}

// x = [cos s | sin s] into the primal half of every member's stacked slab
// (raw CVs, raw[i] = 1: (s_i, 0))
__global__ void train_embed_kernel(const float* s, int B, int n, int K, const uint8_t* raw,
                                   float* HH0, long long slab) {
  const long long total = (long long)K * B * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e / ((long long)B * n));
    const long long r = e - (long long)k * B * n;
    const int b = (int)(r / n), i = (int)(r - (long long)b * n);
    const float si = s[(long long)b * n + i];
    float sn, cs;
    sincosf(si, &sn, &cs);
    const bool is_raw = raw && raw[i];
    float* row = HH0 + k * slab + (long long)b * 2 * n;
    row[i] = is_raw ? si : cs;
    row[n + i] = is_raw ? 0.f : sn;
  }
}

// Activation stage of hidden layer l (1-based) from its tanh branch
// T = tanh(z_l) [K][B][w]: h_l = S t (+ h_{l-1} when residual) into the
// primal half of the stacked slab, and d_l = S (1 - t^2) into D.  S is the
// dropout factor: unit j of sample b of member k is kept when the uniform of
// word j mod 4 of the Philox4x32-10 block with counter (b, step, 16 k + l,
// j div 4) and key (seed) is >= p, scaled by 1/(1 - p); 1 without dropout.
// b is the sample's index in the whole batch: row r of a chunk is sample
// row_base + r.  A thread handles the 4 units of one block.
__global__ void act_kernel(const float* T, int l, int w, int B, int K, int row_base,
                           float drop_p, float drop_inv, unsigned long long seed,
                           uint32_t step, const float* Hprev, long long slab_prev, float* H,
                           long long slab, float* D) {
  const int nq = (w + 3) / 4;
  const long long total = (long long)K * B * nq;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e / ((long long)B * nq));
    const long long rq = e - (long long)k * B * nq;
    const int b = (int)(rq / nq), q = (int)(rq - (long long)b * nq);
    // the four units' loads first (units past w re-read the last one, and a
    // missing Hprev re-reads T; neither is used), the mask bits meanwhile
    const long long ob = ((long long)k * B + b) * w;               // [K][B][w]
    const float* hsrc = Hprev ? Hprev + (long long)k * slab_prev + (long long)b * w : T + ob;
    float tv[4], hv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = min(4 * q + u, w - 1);
      tv[u] = T[ob + j];
      hv[u] = hsrc[j];
    }
    uint32_t c[4] = {(uint32_t)(row_base + b), step, (uint32_t)(16 * k + l), (uint32_t)q};
    if (drop_p > 0.f)
      dev::philox4x32_10(c, (uint32_t)(seed & 0xFFFFFFFFull), (uint32_t)(seed >> 32));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = 4 * q + u;
      if (j >= w) break;
      const float sc = drop_p > 0.f ? (dev::philox_uniform(c[u]) >= drop_p ? drop_inv : 0.f)
                                    : 1.f;
      const float t = tv[u];
      float h = sc * t;
      if (Hprev) h += hv[u];
      H[(long long)k * slab + (long long)b * w + j] = h;
      D[ob + j] = sc * (1.f - t * t);
    }
  }
}

// The layer weights of every member into the aligned copy: block row
// y = k L + l copies layer l's matrix (row-major [out][in], cnt floats) of
// member k from master + k*pm + src[l] to wpad + k*pmp + dst[l], its blocks
// striding over the matrix (contiguous, coalesced, no index arithmetic).
struct WpadCopy {
  long long src[kMaxHidden], dst[kMaxHidden], cnt[kMaxHidden];
  int L;
};
__global__ void wpad_copy_kernel(const float* master, long long pm, float* wpad, long long pmp,
                                 WpadCopy c) {
  const int k = blockIdx.y / c.L, l = blockIdx.y - k * c.L;
  const float* src = master + k * pm + c.src[l];
  float* dst = wpad + k * pmp + c.dst[l];
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < c.cnt[l];
       e += (long long)gridDim.x * blockDim.x)
    dst[e] = src[e];
}

// out[k][b][j] = w_o[k][j] (the top of the reverse sweeps: u_L, lam_hd_L),
// into rows [r0, r0 + B) of a [K][rows][w] slab (the other rows, if any, 0)
__global__ void top_kernel(const float* master, long long per_model, int wo_off, int w, int B,
                           int K, int rows, int r0, float* out) {
  const long long total = (long long)K * rows * w;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e / ((long long)rows * w));
    const long long r = e - (long long)k * rows * w;
    const int row = (int)(r / w), j = (int)(r - (long long)row * w);
    out[e] = (row >= r0 && row < r0 + B) ? master[k * per_model + wo_off + j] : 0.f;
  }
}

// v_L = w_o d_L
__global__ void vlast_kernel(const float* DL, const float* master, long long per_model,
                             int wo_off, int w, int B, int K, float* V) {
  const long long total = (long long)K * B * w;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e / ((long long)B * w));
    const long long r = e - (long long)k * B * w;
    const int j = (int)(r % w);
    V[e] = master[k * per_model + wo_off + j] * DL[e];
  }
}

// g = chain(u0, s); residual; per-row squared residual; rho_x into the
// tangent half of the stacked input slab.  With an upstream gradient
// rho [B][K][n] given instead of labels, rho_x is built from it directly.
// One wave per (member, sample) row, lanes over the CVs; the row's squared
// residual is a fixed-order shuffle sum over the lanes.  B rows of a batch
// of B_norm samples (rho = 2 (g - F) / B_norm); row b of member k's squared
// residual goes to loss_rows[k * loss_ld + b].
constexpr int kResWaves = 4;
__global__ __launch_bounds__(kResWaves * 64) void residual_kernel(
    const float* s, const float* F, const float* rho_in, const float* U0, int B, int B_norm,
    int n, int K, const uint8_t* raw, float* HH0, long long slab, float* loss_rows,
    long long loss_ld) {
  const long long e = (long long)blockIdx.x * kResWaves + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (e >= (long long)K * B) return;
  const int k = (int)(e / B), b = (int)(e - (long long)k * B);
  const float* u = U0 + e * 2 * n;
  float* rx = HH0 + k * slab + ((long long)B + b) * 2 * n;
  float acc = 0.f;
  // (every load of a CV first, without branches: a null raw table reads the
  // CV bytes of s instead, unused; F or rho_in, whichever is given)
  const uint8_t* rawp = raw ? raw : reinterpret_cast<const uint8_t*>(s);
  for (int i = lane; i < n; i += 64) {
    const float sv = s[(long long)b * n + i];
    const uint8_t rv = rawp[i];
    const float ua = u[i], ub = u[n + i];
    const float fv = rho_in ? rho_in[((long long)b * K + k) * n + i] : F[(long long)b * n + i];
    float sn, cs;
    sincosf(sv, &sn, &cs);
    if (raw && rv) {                  // raw CV: x_i = s_i, dx/ds = (1, 0)
      sn = -1.f;
      cs = 0.f;
    }
    float rho;
    if (rho_in) {
      rho = fv;
    } else {
      const float gi = -sn * ua + cs * ub;
      const float ri = gi - fv;
      acc += ri * ri;
      rho = 2.f * ri / (float)B_norm;
    }
    rx[i] = -sn * rho;
    rx[n + i] = cs * rho;
  }
  if (loss_rows) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
    if (lane == 0) loss_rows[(long long)k * loss_ld + b] = acc;
  }
}

// Adjoint stage of layer l: given t_l, d_l, zd_l (each [K][B][w]) and the
// stacked (lam_h ; lam_hd) of layer l, produce the stacked (lam_z ; lam_zd).
__global__ void adjoint_kernel(const float* Tl, const float* Dl, const float* Zd,
                               const float* LAM, long long slab_lam, int w, int B, int K,
                               float* S, long long slab_s) {
  const long long total = (long long)K * B * w;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(e / ((long long)B * w));
    const long long r = e - (long long)k * B * w;   // row-major offset inside the primal half
    const float t = Tl[e], d = Dl[e], zd = Zd[e];
    const float lh = LAM[k * slab_lam + r];
    const float lhd = LAM[k * slab_lam + (long long)B * w + r];
    S[k * slab_s + r] = d * (lh - 2.f * t * zd * lhd);   // lam_z
    S[k * slab_s + (long long)B * w + r] = d * lhd;       // lam_zd
  }
}

// The loss of one member: the mean of its per-row losses r[0:B] (each thread
// adds its rows in row order, eight loads in flight, then a fixed pairwise
// tree over red[256]).  One block of 256 threads.
__device__ inline void member_loss(const float* r, int B, float* loss, float* red) {
  float acc = 0.f;
  int b = threadIdx.x;
  for (; b + 7 * 256 < B; b += 8 * 256) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = r[b + j * 256];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += v[j];
  }
  for (; b < B; b += 256) acc += r[b];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = red[0] / (float)B;
}

// Adam's update of parameter e by gradient gi (old: the parameter and its
// moments, loaded ahead of what delivers gi).
struct AdamOld {
  float theta, m, v;
};
__device__ inline AdamOld adam_load(const AdamStep& a, long long e) {
  return AdamOld{a.theta[e], a.m[e], a.v[e]};
}
__device__ inline void adam_update(const AdamStep& a, const AdamOld& old, long long e, float gi) {
  const float mi = 0.9f * old.m + 0.1f * gi;
  const float vi = 0.999f * old.v + 0.001f * gi * gi;
  a.m[e] = mi;
  a.v[e] = vi;
  a.theta[e] = old.theta - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + 1e-8f);
}
__global__ void adam_kernel(AdamStep a, const float* g, long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    adam_update(a, adam_load(a, e), e, g[e]);
}

// Weight gradients of all layers of one pass over a batch, in one launch.
// Layer l, member b, split s: C = sum over the rows k of chunk s of
// A[b][k][m] B[b][k][n]; A holds [lam_z ; lam_zd], B [h ; hd] (2R rows each,
// primal then tangent: the contraction runs over their rows).  A workgroup
// owns a 64 x 64 tile of one chunk; its four waves take every fourth step of
// 16 rows and their partial tiles are added through LDS in a fixed order
// ((w0 + w2) + (w1 + w3)), so the result does not depend on timing.
// Workgroups of the first column tile also sum A over the primal rows (the
// bias gradient).
//
// The products run on the BF16 matrix units at 16 times the FP32 rate, the
// operands split in registers, x = x1 + x2 + x3, six products (the others are
// below 2^-26).  BF16 has FP32's range and the three parts hold all 24 bits, so
// every entry of the gradient is as precise as its own terms, however small
// beside the rest of its layer (Adam normalises each entry by itself).  FP16
// pairs, three products, need a scale per slab: 99 instead of 120 us at 4096
// samples below, but a unit whose lam is 2^-12 of the layer's largest lost 4
// bits, and one at 2^-26 its whole gradient.  A lane holds 8 consecutive rows
// of one column (the 32x32x16 MFMA's layout), loaded straight from the
// row-major slabs (128-byte row segments, two steps ahead, no LDS, no barriers
// in the loop).  A step's six products go into a cleared accumulator that is then
// added to the running one: products far smaller than an MFMA's accumulator
// are rounded toward minus infinity, and the gradient sums thousands of them
// (4096 samples: error 1.9e-7 of the gradient, 1.05e-7 so, with FP32 MFMA
// 0.82e-7; 2.4 % of a step).  For the same reason the sums of rows and of partials
// add eight values in a tree before they meet the running sum.
//
// What bounds it: the slabs, 235 MB at 4096 samples of 4 x [256 x 4], read at
// 2 TB/s (293 MB with the L2's misses), and the splits and products beside
// them (matrix units 0.42 busy).  Measured per pass there: 205 us with FP32
// MFMA and a launch per layer (and 38 us of column sums, partial sums and
// losses in seven more), 125 us now; 128 samples of residual 4 x [300 x 4]: 41 (and 14) us before, 19 us now.
// With FP16 pairs, 8-byte loads of column pairs took 103 instead of 99 us;
// 128 x 128 tiles split once through LDS 90 us at 4096 samples and 5 % off a
// step of 16384, but 15 % longer below 500 samples.
// The launch also covers what else the batch reductions need: the column sums
// of hd_L (the output weights' gradient, per chunk of kColRows rows) and, on
// the last pass, the members' losses.
struct WgradLayer {
  const float* A;
  const float* B;
  long long sAb, sBb;
  int lda, ldb, M, N, tn, tile0;   // tn: column tiles; tile0: first tile of the layer
  float* C;           // tile of split s, member b: C + s*sCs + b*sCb, [M][N]
  long long sCs, sCb;
  float* csum;        // bias sums: csum + s*csum_ss + b*csum_sb, [M]
  long long csum_ss, csum_sb;
};
constexpr int kColRows = 128;      // rows of a partial column sum
struct WgradArgs {
  WgradLayer l[kMaxHidden];
  int nl, tiles;                   // layers, tiles of all layers
  int R, batch, ksplit, kchunk, xcd;   // rows of a half; chunks, whole steps of each
  int main_blocks;                 // workgroups of the products
  // column sums of X [batch][.][w] (member stride sXb) over its R rows, part c of
  // member b at out + c*s_part + b*s_mem; null: none
  const float* X;
  long long sXb;
  int w, col_parts;
  float* col_out;
  long long col_part, col_mem;
  // losses from rows [batch][B] (null: none), and the zero of the output bias
  const float* rows;
  int B;
  float* loss;
  float* zero;                     // one entry per member, stride s_zero (null: none)
  long long s_zero;
};

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float fl2 __attribute__((ext_vector_type(2)));
constexpr int kWgLdsStride = 65;   // padded row of a partial tile in LDS
constexpr int kWgTile = 64;        // tile edge of a workgroup
constexpr int kWgStep = 16;        // contraction rows of a step

__device__ inline float tree8(const float (&v)[8]) {
  return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// The three BF16 parts of eight values.
struct Split8 {
  uint4 p[3];
  __device__ inline void set(const float (&x)[8]) {
    unsigned q[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector((fl2{a, b}), bf2));
        q[t][i] = u;
        if (t < 2) {
          a -= __uint_as_float(u << 16);
          b -= __uint_as_float(u & 0xFFFF0000u);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) p[t] = make_uint4(q[t][0], q[t][1], q[t][2], q[t][3]);
  }
};

__device__ inline void wg_mfma(f16v& c, const uint4& a, const uint4& b) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a),
                                              __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// The workgroups past the products: column sums, then losses (red: 256 floats).
__device__ inline void wgrad_extra(const WgradArgs& g, int blk, float* red) {
  const int ct = (g.w + 63) / 64, n_col = g.X ? ct * g.col_parts * g.batch : 0;
  if (blk >= n_col) {
    const int b = blk - n_col;
    if (threadIdx.x == 0 && g.zero) g.zero[b * g.s_zero] = 0.f;
    if (g.rows && g.loss) member_loss(g.rows + (long long)b * g.B, g.B, g.loss + b, red);
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blk / (ct * g.col_parts), r = blk - b * ct * g.col_parts;
  const int c = r / ct, j = (r - c * ct) * 64 + lane;
  const int r0 = c * kColRows, r1 = min(g.R, r0 + kColRows);
  const float* x = g.X + b * g.sXb + min(j, g.w - 1);
  float acc = 0.f;
  int k = r0 + wave;
  for (; k + 28 < r1; k += 32) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = x[(long long)(k + 4 * q) * g.w];
    acc += tree8(v);
  }
  for (; k < r1; k += 4) acc += x[(long long)k * g.w];
  red[64 * wave + lane] = acc;
  __syncthreads();
  if (wave == 0 && j < g.w)
    g.col_out[c * g.col_part + b * g.col_mem + j] =
        ((red[lane] + red[64 + lane]) + red[128 + lane]) + red[192 + lane];
}

// The tile of a workgroup: its layer, member, split and tile in the layer.
struct WgradTile {
  int li, b, s, m0, n0;
};
__device__ inline bool wgrad_tile(const WgradArgs& g, int blk, WgradTile& w) {
  int chunk, tile;
  if (g.xcd) {                     // all tiles of a chunk on one XCD
    const int q = blk >> 3;
    tile = q % g.tiles;
    chunk = (q / g.tiles) * 8 + (blk & 7);
  } else {
    tile = blk % g.tiles;
    chunk = blk / g.tiles;
  }
  if (chunk >= g.batch * g.ksplit) return false;
  w.b = chunk / g.ksplit;
  w.s = chunk - w.b * g.ksplit;
  w.li = 0;
#pragma unroll
  for (int i = 1; i < kMaxHidden; ++i)
    if (i < g.nl && tile >= g.l[i].tile0) w.li = i;
  const int t2 = tile - g.l[w.li].tile0, tn = g.l[w.li].tn;
  w.m0 = (t2 / tn) * kWgTile;
  w.n0 = (t2 % tn) * kWgTile;
  return true;
}

// (two workgroups a CU: without the bound the compiler took registers for one)
__global__ __launch_bounds__(256, 2) void wgrad_kernel(WgradArgs g) {
  __shared__ float red[2][64][kWgLdsStride];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x >= g.main_blocks) {
    wgrad_extra(g, blockIdx.x - g.main_blocks, &red[0][0][0]);
    return;
  }
  WgradTile wt;
  if (!wgrad_tile(g, blockIdx.x, wt)) return;
  const int b = wt.b, s = wt.s, m0 = wt.m0, n0 = wt.n0;
  const WgradLayer& L = g.l[wt.li];
  const int lo = lane & 31, hi = lane >> 5;
  // The whole 16-row steps of the primal half, then of the tangent half, are
  // numbered through; this wave takes every fourth of the chunk's.  The rows
  // left over in each half (R mod 16) fall to waves 0 and 1 of the last chunk.
  const int R = g.R, half = R / kWgStep, rest = R - half * kWgStep;
  const int c_begin = min(2 * half, s * g.kchunk), c_end = min(2 * half, c_begin + g.kchunk);
  const int n_st = (max(c_end - c_begin - wave, 0) + 3) / 4;
  auto step = [&](int i) { return c_begin + wave + 4 * min(i, n_st - 1); };
  // A lane's column is clamped into the operand: one outside only feeds
  // accumulator rows or columns that are never stored.  Buffer loads: the
  // lane's byte offset in the vector offset, the row's in the scalar offset.
  const int lda = L.lda, ldb = L.ldb;
  const int ca[2] = {min(m0 + lo, L.M - 1), min(m0 + 32 + lo, L.M - 1)};
  const int cb[2] = {min(n0 + lo, L.N - 1), min(n0 + 32 + lo, L.N - 1)};
  const int oa[2] = {4 * (8 * hi * lda + ca[0]), 4 * (8 * hi * lda + ca[1])};
  const int ob[2] = {4 * (8 * hi * ldb + cb[0]), 4 * (8 * hi * ldb + cb[1])};
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(L.A + b * L.sAb), (short)0, 0x7FFFFFF0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(L.B + b * L.sBb), (short)0, 0x7FFFFFF0, 0x00020000);
  const bool csum_wg = L.csum && n0 == 0;

  f16v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f16v{};
  float cs[2] = {0.f, 0.f};
  auto ldf = [](const __amdgpu_buffer_rsrc_t& r, int vo, int so) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
  };
  // loaded steps: [slot][a0, a1, b0, b1][row]
  float ring[3][4][8];
  auto issue = [&](float (&v)[4][8], int t) {
    const int k = kWgStep * t + (t >= half ? rest : 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int sa = 4 * (k + e) * lda, sb = 4 * (k + e) * ldb;
      v[0][e] = ldf(ra, oa[0], sa);
      v[1][e] = ldf(ra, oa[1], sa);
      v[2][e] = ldf(rb, ob[0], sb);
      v[3][e] = ldf(rb, ob[1], sb);
    }
  };
  auto consume = [&](const float (&v)[4][8], bool tangent) {
    if (csum_wg && !tangent) {
      cs[0] += tree8(v[0]);
      cs[1] += tree8(v[1]);
    }
    Split8 fb[2];
    fb[0].set(v[2]);
    fb[1].set(v[3]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      Split8 fa;
      fa.set(v[i]);
      constexpr int pa[6] = {0, 2, 1, 0, 1, 0};   // small products first
      constexpr int pb[6] = {2, 0, 1, 1, 0, 0};
      f16v sum[2] = {f16v{}, f16v{}};
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) wg_mfma(sum[j], fa.p[pa[t]], fb[j].p[pb[t]]);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] += sum[j];
    }
  };
  // (a step past the last one re-reads the last, never consumed)
  if (n_st > 0) {
    issue(ring[0], step(0));
    issue(ring[1], step(1));
  }
  for (int i = 0; i < n_st; i += 3) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
      if (i + p < n_st) {
        issue(ring[(p + 2) % 3], step(i + p + 2));
        __builtin_amdgcn_sched_barrier(0);
        consume(ring[p], step(i + p) >= half);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  if (rest > 0 && s == g.ksplit - 1 && wave < 2) {   // the rest of a half; zeros past it
    const int k0 = wave * R + half * kWgStep, k1 = (wave + 1) * R;
    float v[4][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = k0 + 8 * hi + e, kc = min(k, k1 - 1);
      const bool in = k < k1;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float x = ldf(ra, 4 * (kc * lda + ca[i]), 0);
        const float y = ldf(rb, 4 * (kc * ldb + cb[i]), 0);
        v[i][e] = in ? x : 0.f;
        v[2 + i][e] = in ? y : 0.f;
      }
    }
    consume(v, wave == 1);
  }
  // accumulator element v of a 32 x 32 tile: row 8 (v / 4) + 4 hi + v % 4,
  // column lo.  Waves 2, 3 park their tiles; waves 0, 1 add them; wave 1
  // parks the sum; wave 0 adds it and writes the slab.
  // (one accumulator tile at a time: the scheduling barriers keep the
  // compiler from reading all four tiles into registers at once)
  auto park = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          red[slot][32 * i + 8 * (v / 4) + 4 * hi + (v % 4)][32 * j + lo] = acc[i][j][v];
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto take = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          acc[i][j][v] += red[slot][32 * i + 8 * (v / 4) + 4 * hi + (v % 4)][32 * j + lo];
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  // the bias sums: combine the two row halves of a lane pair, then the
  // waves in the same fixed order through LDS
  __shared__ float cred[4][64];
  if (csum_wg) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      cs[i] += __shfl_xor(cs[i], 32);
      if (hi == 0) cred[wave][32 * i + lo] = cs[i];
    }
  }
  if (wave >= 2) park(wave - 2);
  __syncthreads();
  if (wave < 2) take(wave);
  __syncthreads();
  if (wave == 1) park(0);
  __syncthreads();
  if (wave == 0) {
    take(0);
    park(1);
  }
  __syncthreads();
  // the summed tile, stored by all waves: a row per wave and store, one
  // column per lane (256-byte row segments)
  float* Ct = L.C + s * L.sCs + b * L.sCb + (long long)m0 * L.N + n0;
  for (int r = wave; r < 64 && m0 + r < L.M; r += 4)
    if (n0 + lane < L.N)
      Ct[(long long)r * L.N + lane] = red[1][r][lane];
  if (csum_wg && wave == 0) {
    const int m = m0 + lane;
    const float v = (cred[0][lane] + cred[2][lane]) + (cred[1][lane] + cred[3][lane]);
    if (m < L.M) L.csum[s * L.csum_ss + b * L.csum_sb + m] = v;
  }
}

// The gradient from the partials of one pass: dW_l and db_l over the split
// slabs, dw_o over the column sums' parts, each in part order (added to what
// the gradient holds when accumulate is set); on the last pass the output
// bias's zero and the losses.  Block row y < nl: layer y; y == nl: the rest.
struct ReduceLayer {
  const float* part;               // [ks][K][M][N]
  const float* bpart;              // [ks][K][M]
  int M, N;
  long long w_off, b_off;
};
struct ReduceArgs {
  ReduceLayer l[kMaxHidden];
  int nl, ks, K, accumulate;
  float* grad;
  long long pm;
  const float* cpart;              // [cparts][K][w], null: none
  int cparts, w;
  long long wo_off;
  const float* rows;               // [K][B]: losses (last pass), or null
  int B;
  float* loss;
  int last;                        // zero the output bias's gradient
  AdamStep adam;
};
__device__ inline float sum_parts(const float* src, long long stride, int n) {
  // parts in order, eight loads in flight and added in a tree
  float acc = 0.f;
  int s = 0;
  for (; s + 8 <= n; s += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[(s + j) * stride];
    acc += tree8(v);
  }
  for (; s < n; ++s) acc += src[s * stride];
  return acc;
}
// An entry's gradient: stored, or (adam.theta set) taken into the update.
__device__ inline void put_grad(const ReduceArgs& g, const AdamOld& old, long long o, float v) {
  if (g.accumulate) v = g.grad[o] + v;
  if (g.adam.theta) adam_update(g.adam, old, o, v);
  else g.grad[o] = v;
}
__global__ __launch_bounds__(256) void grad_reduce_kernel(ReduceArgs g) {
  auto load = [&](long long o) { return g.adam.theta ? adam_load(g.adam, o) : AdamOld{0.f, 0.f, 0.f}; };
  __shared__ float red[256];
  const long long step = (long long)gridDim.x * 256, first = blockIdx.x * 256LL + threadIdx.x;
  if ((int)blockIdx.y < g.nl) {
    const ReduceLayer& L = g.l[blockIdx.y];
    const long long mn = (long long)L.M * L.N, total = g.K * mn, all = total + (long long)g.K * L.M;
    for (long long e = first; e < all; e += step) {
      const bool wt = e < total;
      const long long x = wt ? e : e - total, per = wt ? mn : L.M;
      const int k = (int)(x / per);
      const long long o = k * g.pm + (wt ? L.w_off : L.b_off) + (x - k * per);
      const AdamOld old = load(o);
      const float v = sum_parts((wt ? L.part : L.bpart) + x, wt ? total : (long long)g.K * L.M, g.ks);
      put_grad(g, old, o, v);
    }
    return;
  }
  if (g.cpart) {
    const long long all = (long long)g.K * g.w;
    for (long long e = first; e < all; e += step) {
      const int k = (int)(e / g.w);
      const long long o = k * g.pm + g.wo_off + (e - (long long)k * g.w);
      const AdamOld old = load(o);
      const float v = sum_parts(g.cpart + e, all, g.cparts);
      put_grad(g, old, o, v);
    }
  }
  if (!g.last) return;
  for (int k = blockIdx.x; k < g.K; k += gridDim.x) {
    if (threadIdx.x == 0) {
      const long long o = k * g.pm + g.wo_off + g.w;
      if (g.adam.theta) adam_update(g.adam, adam_load(g.adam, o), o, 0.f);
      else g.grad[o] = 0.f;
    }
    if (g.rows && g.loss) member_loss(g.rows + (long long)k * g.B, g.B, g.loss + k, red);
    __syncthreads();
  }
}

inline int grid1d(long long total) {
  return (int)std::min<long long>((total + 255) / 256, 4096);
}

// Load mode of one operand (see TileLoad): float4 along the unit-stride
// dimension when alignment and extents allow, else scalar.
int load_mode(const float* X, long long sR, long long sK, long long sBatch, int R, int Kc) {
  const bool al = (reinterpret_cast<uintptr_t>(X) % 16 == 0) && sBatch % 4 == 0;
  if (sK == 1) return (al && sR % 4 == 0 && Kc % 4 == 0) ? 2 : 0;
  if (sR == 1) return (al && sK % 4 == 0 && R % 4 == 0) ? 3 : 1;
  return 0;
}

// One tile shape, with the float4 load modes of the two operands as
// compile-time choices.
template <int TM, int TN, int BKT>
void launch_gemm_tile(dim3 grid, const GemmArgs& g, hipStream_t st) {
  const bool va = g.modeA >= 2, vb = g.modeB >= 2;
  if (va && vb)
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, BKT, true, true>), grid, dim3(kThreads), 0, st, g);
  else if (va)
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, BKT, true, false>), grid, dim3(kThreads), 0, st, g);
  else if (vb)
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, BKT, false, true>), grid, dim3(kThreads), 0, st, g);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, BKT, false, false>), grid, dim3(kThreads), 0, st, g);
}

#ifndef RID_GEMM_DEEP_WGS
#define RID_GEMM_DEEP_WGS 256
#endif
rid_status gemm(const GemmArgs& g0, hipStream_t st) {
  GemmArgs g = g0;
  g.modeA = load_mode(g.A, g.sAm, g.sAk, g.sAb, g.M, g.Kc);
  g.modeB = load_mode(g.Bm, g.sBn, g.sBk, g.sBb, g.N, g.Kc);
  // 128 x 128 tiles only when they still give every CU several workgroups
  // (one 4-wave workgroup per CU leaves one wave per SIMD to hide latency);
  // 32 x 64 tiles when 64 x 64 would leave CUs with fewer than two
  const long long tiles128 =
      (long long)((g.N + 127) / 128) * ((g.M + 127) / 128) * g.batch;
  const long long tiles64 =
      (long long)((g.N + 63) / 64) * ((g.M + 63) / 64) * g.batch;
  if (g.M >= 128 && g.N >= 128 && tiles128 >= 1024) {
    dim3 grid((g.N + 127) / 128, (g.M + 127) / 128, g.batch);
    launch_gemm_tile<128, 128, BK>(grid, g, st);
  } else if (g.M > 32 && tiles64 < 512) {
    dim3 grid((g.N + 63) / 64, (g.M + 31) / 32, g.batch);
    // fewer workgroups than CUs: latency-bound, 64-deep contraction blocks
    const long long wgs = (long long)grid.x * grid.y * grid.z;
    if (wgs < RID_GEMM_DEEP_WGS && g.Kc > 48)
      launch_gemm_tile<32, 64, 64>(grid, g, st);
    else
      launch_gemm_tile<32, 64, BK>(grid, g, st);
  } else {
    dim3 grid((g.N + 63) / 64, (g.M + 63) / 64, g.batch);
    launch_gemm_tile<64, 64, BK>(grid, g, st);
  }
  RID_HIP(hipGetLastError());
  return RID_OK;
}

// The batch reductions of one pass of R rows (contraction over 2R stacked
// rows): the layers' products, and what g says of column sums and losses.
// Where one split, one column part and no earlier pass make the partials the
// result, the kernel writes the gradient itself; else it writes partials
// (region part, bias partials bpart, column parts cpart) and a second launch
// adds them up, and takes Adam's step with them (a launch and a pass over the
// gradient less: 2048 samples of 4 x [256 x 4] 150 -> 144 us a step, 1024 of
// [300 x 4] 146 -> 142; in the first launch's epilogue, where that writes the
// gradient, the same cost 5 us of a 37 us step).  Layers: operands, shapes and offsets in the packed layout.
struct GradLayer {
  const float* A;                  // lam slab [K][2R][M]
  const float* B;                  // activation slab [K][2R][N]
  int M, N;
  long long w_off, b_off;
};
struct GradPass {
  GradLayer l[kMaxHidden];
  int nl, K, R, ks, kchunk;
  float *part, *bpart, *cpart;
  float* grad;
  long long pm;
  bool accumulate, last;
  const float* X;                  // hd_L rows (member stride sXb), or null
  long long sXb, wo_off;
  int w;
  const float* rows;               // last pass: [K][B] row losses, or null
  int B;
  float* loss;
  AdamStep adam;                   // the last of all layers' passes: take the step (theta null: none)
};
int col_parts(int R) { return (R + kColRows - 1) / kColRows; }

rid_status grad_pass(const GradPass& g, hipStream_t st) {
  WgradArgs a{};
  ReduceArgs r{};
  const int Kc = 2 * g.R;
  if (g.kchunk < 1 || g.nl < 1 || g.R < 1)
    return fail(RID_EINVAL, "weight-gradient pass: bad shape");
  const bool direct = g.ks == 1 && !g.accumulate && (!g.X || col_parts(g.R) == 1);
  a.nl = r.nl = g.nl;
  a.R = g.R; a.batch = g.K; a.ksplit = g.ks; a.kchunk = g.kchunk;
  long long off = 0, boff = 0;
  for (int i = 0; i < g.nl; ++i) {
    const GradLayer& s = g.l[i];
    WgradLayer& d = a.l[i];
    const long long mn = (long long)s.M * s.N;
    // row byte offsets are 32-bit scalar offsets (passes are sized to fit)
    if ((long long)Kc * std::max(s.M, s.N) * 4 > 0x7FFFFFFFLL)
      return fail(RID_EUNSUPPORTED, "weight-gradient pass: slab too large for 32-bit offsets");
    d.A = s.A; d.lda = s.M; d.sAb = (long long)Kc * s.M;
    d.B = s.B; d.ldb = s.N; d.sBb = (long long)Kc * s.N;
    d.M = s.M; d.N = s.N;
    d.tn = (s.N + kWgTile - 1) / kWgTile;
    d.tile0 = a.tiles;
    a.tiles += d.tn * ((s.M + kWgTile - 1) / kWgTile);
    if (direct) {
      d.C = g.grad + s.w_off; d.sCb = g.pm;
      d.csum = g.grad + s.b_off; d.csum_sb = g.pm;
    } else {
      d.C = g.part + off * g.ks; d.sCs = g.K * mn; d.sCb = mn;
      d.csum = g.bpart + boff * g.ks; d.csum_ss = (long long)g.K * s.M; d.csum_sb = s.M;
      r.l[i] = ReduceLayer{d.C, d.csum, s.M, s.N, s.w_off, s.b_off};
    }
    off += g.K * mn;
    boff += (long long)g.K * s.M;
  }
  const int chunks = g.K * g.ks;
  a.xcd = chunks >= 8;
  a.main_blocks = a.xcd ? 8 * a.tiles * ((chunks + 7) / 8) : a.tiles * chunks;
  int extra = 0;
  if (g.X) {
    a.X = g.X; a.sXb = g.sXb; a.w = g.w; a.col_parts = col_parts(g.R);
    if (direct) {
      a.col_out = g.grad + g.wo_off; a.col_mem = g.pm;
    } else {
      a.col_out = g.cpart; a.col_part = (long long)g.K * g.w; a.col_mem = g.w;
      r.cpart = g.cpart; r.cparts = a.col_parts;
    }
    extra += ((g.w + 63) / 64) * a.col_parts * g.K;
  }
  if (direct && g.last) {
    a.rows = g.rows; a.B = g.B; a.loss = g.loss;
    a.zero = g.grad + g.wo_off + g.w; a.s_zero = g.pm;
    extra += g.K;
  }
  hipLaunchKernelGGL(wgrad_kernel, dim3(a.main_blocks + extra), dim3(256), 0, st, a);
  RID_HIP(hipGetLastError());
  if (direct) {
    if (g.adam.theta) {
      hipLaunchKernelGGL(adam_kernel, dim3(grid1d(g.K * g.pm)), dim3(256), 0, st, g.adam, g.grad,
                         g.K * g.pm);
      RID_HIP(hipGetLastError());
    }
    return RID_OK;
  }
  r.ks = g.ks; r.K = g.K; r.accumulate = g.accumulate ? 1 : 0;
  r.grad = g.grad; r.pm = g.pm; r.w = g.w; r.wo_off = g.wo_off;
  r.adam = g.adam;
  r.last = g.last ? 1 : 0; r.rows = g.rows; r.B = g.B; r.loss = g.loss;
  long long most = 1;
  for (int i = 0; i < g.nl; ++i)
    most = std::max(most, (long long)g.K * g.l[i].M * (g.l[i].N + 1));
  hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)std::min<long long>((most + 255) / 256, 1024),
                                              g.nl + 1), dim3(256), 0, st, r);
  RID_HIP(hipGetLastError());
  return RID_OK;
}

// Rows per pass over the batch: all B when the pass's stored activations
// (floats_per_row floats a row) fit the budget, else equal chunks, each a
// multiple of 64 rows and at least 64, that do.  A pass also stays below
// the rows whose 2R-row slabs of width wmax the weight-gradient kernel can
// address with 32-bit byte offsets (about 500 k rows at width 512).
int chunk_rows(long long floats_per_row, int B, size_t budget, int wmax) {
  const long long cap = ((1LL << 31) - 1) / (8LL * std::max(wmax, 1));
  const long long fit =
      std::min(cap, (long long)(budget / (sizeof(float) * (size_t)floats_per_row)));
  if (fit >= B) return B;
  const long long step = std::max<long long>(64, fit / 64 * 64);
  const long long chunks = (B + step - 1) / step;
  return (int)std::min<long long>(step, (B + chunks - 1) / chunks + 63) / 64 * 64;
}

// Split of the 2R-row contraction of a pass of R rows over nl layers'
// products: the number of equal chunks (a power of two, at least 256 rows
// each) that costs least.  A CU works through `per_cu` tiles of rows + 160
// (a workgroup's start and its tile's way through LDS cost what 160 rows do);
// one tile alone on a CU runs at 0.8 of the rate two reach together, and a
// chunk's partial gradient costs 1 row per 5.7 kB written and read back.
// Measured per training step (us, 4 members of [256 x 4] unless noted; chunks
// 1 / 2 / 4): 1024 samples 116 / 110 / 118, 4096 samples 338 / 300 / 308,
// 16384 samples 1370 / 1233 / 1245, 4096 samples of [300 x 4] 622 / 486 / 474,
// one member and 4096 samples, chunks 4 / 8 / 16: 104 / 100 / 107.
struct WgradSplit {
  int ks, kchunk;
};
WgradSplit wgrad_split(int K, const int* M, const int* N, int nl, int R) {
  long long tiles = 0, params = 0;
  for (int i = 0; i < nl; ++i) {
    tiles += (long long)((M[i] + kWgTile - 1) / kWgTile) * ((N[i] + kWgTile - 1) / kWgTile);
    params += (long long)M[i] * N[i];
  }
  WgradSplit best{1, 0};
  double least = 0;
  for (int ks = 1; ks <= 64 && (ks == 1 || 2LL * R >= 256LL * ks); ks *= 2) {
    const long long chunks = (long long)K * ks;
    const double per_cu = chunks >= 8 ? std::ceil(tiles * ((chunks + 7) / 8) / 32.0)
                                      : std::ceil(tiles * chunks / 256.0);
    const double cost = per_cu * (2.0 * R / ks + 160) * (per_cu == 1 ? 1.25 : 1.0) +
                        (ks > 1 ? K * params * 8.0 * ks / 46e3 : 0.0);
    if (ks == 1 || cost < least) {
      least = cost;
      best.ks = ks;
    }
  }
  best.kchunk = std::max(1, (2 * (R / kWgStep) + best.ks - 1) / best.ks);
  return best;
}

// The training step with the sweeps fused into one kernel (train_sweep_f32.h):
// it writes [h ; hd] of every layer input and [lam_z ; lam_zd] of every
// layer, then the batch reductions run as before: dW_l = S_l^T [h ; hd]_{l-1}
// (split over the 2R rows), db_l = column sums of lam_z, dw_o = column sums
// of hd_L.  A batch larger than the training budget allows runs in chunks of
// Bc rows, in row order: each chunk's reductions are added to the gradient
// in chunk order, so the step stays deterministic, and only one chunk's
// activations are ever held.  Workspace regions are 256-byte aligned (the
// kernel stores float4).
rid_status mf_grad_fused(rid_ensemble_impl& e, const float* s, const float* F,
                         const float* rho, int B, float* loss, float* grad_out,
                         hipStream_t st, const std::vector<int>& w,
                         const std::vector<long long>& w_off,
                         const std::vector<long long>& b_off, long long wo_off,
                         const AdamStep& adam) {
  const int K = e.K, L = e.L, n = e.n_cv;
  int wmax = 0;
  for (int v : w) wmax = std::max(wmax, v);
  long long per_row = 0;
  for (int l = 0; l <= L; ++l) per_row += (long long)K * 2 * w[l] * (l > 0 ? 2 : 1);
  const int Bc = chunk_rows(per_row, B, e.train_budget, wmax);
  std::vector<int> wm(w.begin() + 1, w.end());   // rows of dW_l; w: its columns
  const int ks_max = wgrad_split(K, wm.data(), w.data(), L, Bc).ks;
  auto al = [](long long v) { return (v + 63) / 64 * 64; };
  std::vector<long long> hh(L + 1), sl(L);
  long long tot = 0;
  for (int l = 0; l <= L; ++l) {
    hh[l] = tot;
    tot = al(tot + (long long)K * 2 * Bc * w[l]);
  }
  for (int l = 1; l <= L; ++l) {
    sl[l - 1] = tot;
    tot = al(tot + (long long)K * 2 * Bc * w[l]);
  }
  long long parts = 0, bparts = 0;
  for (int l = 0; l < L; ++l) {
    parts += (long long)K * w[l + 1] * w[l];
    bparts += (long long)K * w[l + 1];
  }
  const long long part = tot; tot = al(tot + parts * ks_max);
  const long long grad = tot; tot = al(tot + (long long)e.n_params);
  const long long lrows = tot; tot = al(tot + (long long)K * B);
  const long long cpart = tot; tot = al(tot + (long long)col_parts(Bc) * K * w[L]);
  const long long bpart = tot; tot = al(tot + bparts * ks_max);
  rid_status rs = e.ws_train.ensure(sizeof(float) * tot);
  if (rs != RID_OK) return rs;
  float* W = e.ws_train.as<float>();
  const long long pm = (long long)e.per_model;
  float* G = grad_out ? grad_out : W + grad;
  ProfScope ps(kProfTrain, st);
  if ((rs = ensure_packed(e, st)) != RID_OK) return rs;
  TrainIo io{};
  io.loss_ld = B;
  io.B_norm = B;
  io.drop_p = e.drop_p;
  io.drop_seed = e.drop_seed;
  io.step = (uint32_t)((unsigned long long)e.step & 0xFFFFFFFFull);
  for (int l = 0; l <= L; ++l) io.hh[l] = W + hh[l];
  for (int l = 0; l < L; ++l) io.sl[l] = W + sl[l];
  for (int r0 = 0; r0 < B; r0 += Bc) {
    const int R = std::min(Bc, B - r0);
    const bool acc = r0 > 0;
    const WgradSplit sp = wgrad_split(K, wm.data(), w.data(), L, R);
    io.s = s + (size_t)r0 * n;
    io.F = rho ? nullptr : F + (size_t)r0 * n;
    io.rho = rho ? rho + (size_t)r0 * K * n : nullptr;
    io.loss_rows = rho ? nullptr : W + lrows + r0;
    io.row_base = r0;
    if ((rs = launch_train_sweeps(e, io, R, st)) != RID_OK) return rs;
    GradPass g{};
    g.nl = L; g.K = K; g.R = R; g.ks = sp.ks; g.kchunk = sp.kchunk;
    for (int l = 0; l < L; ++l)      // dW_l = S^T [h ; hd]_{l-1}, db_l = sum of lam_z
      g.l[l] = GradLayer{W + sl[l], W + hh[l], w[l + 1], w[l], w_off[l], b_off[l]};
    g.part = W + part; g.bpart = W + bpart; g.cpart = W + cpart;
    g.grad = G; g.pm = pm;
    g.accumulate = acc; g.last = r0 + R >= B;
    g.X = W + hh[L] + (long long)R * w[L]; g.sXb = 2LL * R * w[L]; g.w = w[L]; g.wo_off = wo_off;
    g.rows = rho ? nullptr : W + lrows; g.B = B; g.loss = loss;
    if (g.last) g.adam = adam;
    if ((rs = grad_pass(g, st)) != RID_OK) return rs;
  }
  return RID_OK;
}

}  // namespace

// Gradient in the packed parameter layout of
//   F given:   L = sum_k (1/B) sum_b |g_k(s_b) - F_b|^2      (loss[k] written)
//   rho given: J = sum_k sum_b rho[b][k] . g_k(s_b)
// into grad_out (or the workspace's gradient slot when grad_out is null).
// With adam.theta set the parameters are updated instead and no gradient is
// kept.  Both forms hold at most
// the ensemble's training budget of activations: a larger batch is taken in
// chunks of rows whose weight-gradient contributions are added in chunk order.
// The aligned weight copy of the general sweeps, allocated on first use and
// refreshed when the masters have changed since it was made.
rid_status ensure_wpad(rid_ensemble_impl& e, const std::vector<int>& w,
                       const std::vector<long long>& w_off, hipStream_t st) {
  const int L = e.L;
  e.wpad_off.assign(L, 0);
  long long off = 0;
  for (int l = 0; l < L; ++l) {
    e.wpad_off[l] = off;
    off += ((long long)w[l + 1] * w[l] + 3) / 4 * 4;
  }
  e.wpad_pm = off;
  const void* before = e.wpad.ptr;
  rid_status rs = e.wpad.ensure(sizeof(float) * (size_t)e.K * e.wpad_pm);
  if (rs != RID_OK) return rs;
  if (e.wpad.ptr != before) e.wpad_gen = 0;    // a new buffer holds nothing yet
  if (e.wpad_gen == e.master_gen) return RID_OK;
  WpadCopy c{};
  c.L = L;
  long long cmax = 1;
  for (int l = 0; l < L; ++l) {
    c.src[l] = w_off[l];
    c.dst[l] = e.wpad_off[l];
    c.cnt[l] = (long long)w[l + 1] * w[l];
    cmax = std::max(cmax, c.cnt[l]);
  }
  const unsigned bx = (unsigned)std::min<long long>((cmax + 255) / 256, 256);
  hipLaunchKernelGGL(wpad_copy_kernel, dim3(bx, e.K * L), dim3(256), 0, st, e.d_master,
                     (long long)e.per_model, e.wpad.as<float>(), e.wpad_pm, c);
  RID_HIP(hipGetLastError());
  e.wpad_gen = e.master_gen;
  return RID_OK;
}

rid_status launch_mf_grad(rid_ensemble_impl& e, const float* s, const float* F,
                          const float* rho, int B, float* loss, float* grad_out,
                          hipStream_t st, InputHvp* hvp, const AdamStep& adam) {
  // input mode (hvp != null, rho given): the same primal, tangent and
  // adjoint sweeps, but the adjoint runs down to the input instead of
  // forming weight gradients
  const bool input_mode = hvp != nullptr;
  if (input_mode && !rho) return fail(RID_EINVAL, "input mode needs an upstream gradient");
  const int K = e.K, L = e.L, n = e.n_cv, X = 2 * n;
  std::vector<int> w(L + 1);
  w[0] = X;
  for (int l = 0; l < L; ++l) w[l + 1] = e.widths[l];
  int wmax = X;
  for (int v : w) wmax = std::max(wmax, v);
  // packed offsets inside one model's block
  std::vector<long long> w_off(L), b_off(L);
  long long off = 0;
  for (int l = 0; l < L; ++l) {
    w_off[l] = off;
    off += (long long)w[l + 1] * w[l];
    b_off[l] = off;
    off += w[l + 1];
  }
  const long long wo_off = off;
  const long long pm = (long long)e.per_model;
  if (!input_mode && train_fused_supported(e))
    return mf_grad_fused(e, s, F, rho, B, loss, grad_out, st, w, w_off, b_off, wo_off, adam);

  // the general form: residual layers, dropout (training only), raw CVs
  const bool res = e.resnet;
  const float drop_p = input_mode ? 0.f : e.drop_p;
  const float drop_inv = drop_p > 0.f ? 1.f / (1.f - drop_p) : 1.f;
  const uint8_t* raw = e.raw.empty() ? nullptr : e.d_raw;
  auto skip = [&](int l) { return res && l >= 2; };   // layer l (1-based) adds its input

  // rows per pass (input mode hands per-row results back: one pass)
  long long per_row = (long long)K * (8 + (res ? 2 : 0)) * wmax;
  for (int l = 0; l <= L; ++l) per_row += (long long)K * w[l] * (l > 0 ? 5 : 2);
  const int Bc = input_mode ? B : chunk_rows(per_row, B, e.train_budget, wmax);
  int ks_max = 1;
  for (int l = 0; l < L; ++l) ks_max = std::max(ks_max, wgrad_split(K, &w[l + 1], &w[l], 1, Bc).ks);

  // workspace (floats), sized for Bc rows; a pass of R <= Bc rows uses the
  // same regions with R-row strides
  std::vector<long long> hh(L + 1), zd(L + 1), tt(L + 1), dd(L + 1);
  long long tot = 0;
  for (int l = 0; l <= L; ++l) {
    hh[l] = tot;
    tot += (long long)K * 2 * Bc * w[l];
  }
  for (int l = 1; l <= L; ++l) {
    zd[l] = tot; tot += (long long)K * Bc * w[l];
    tt[l] = tot; tot += (long long)K * Bc * w[l];
    dd[l] = tot; tot += (long long)K * Bc * w[l];
  }
  const long long vA = tot; tot += (long long)K * Bc * wmax;
  const long long vB = tot; tot += (long long)K * Bc * wmax;
  const long long uA = tot; tot += res ? (long long)K * Bc * wmax : 0;
  const long long uB = tot; tot += res ? (long long)K * Bc * wmax : 0;
  const long long lamA = tot; tot += (long long)K * 2 * Bc * wmax;
  const long long lamB = tot; tot += (long long)K * 2 * Bc * wmax;
  const long long sbuf = tot; tot += (long long)K * 2 * Bc * wmax;
  long long part_slab = 0;
  for (int l = 0; l < L; ++l) part_slab = std::max(part_slab, (long long)K * w[l + 1] * w[l]);
  const long long part = tot; tot += part_slab * ks_max;
  const long long grad = tot; tot += (long long)e.n_params;
  const long long lrows = tot; tot += (long long)K * B;
  const long long cpart = tot; tot += (long long)col_parts(Bc) * K * wmax;
  const long long bpart = tot; tot += (long long)ks_max * K * wmax;
  rid_status rs = e.ws_train.ensure(sizeof(float) * tot);
  if (rs != RID_OK) return rs;
  float* W = e.ws_train.as<float>();
  float* P = e.d_master;
  float* G = grad_out ? grad_out : W + grad;
  ProfScope ps(kProfTrain, st);
  const uint32_t step32 = (uint32_t)((unsigned long long)e.step & 0xFFFFFFFFull);
  // the weight operands come from the aligned copy (float4 loads)
  if ((rs = ensure_wpad(e, w, w_off, st)) != RID_OK) return rs;
  const float* WP = e.wpad.as<float>();
  const long long pmp = e.wpad_pm;
  const std::vector<long long>& wq = e.wpad_off;

  for (int r0 = 0; r0 < B; r0 += Bc) {
    const int R = std::min(Bc, B - r0);
    const bool acc = r0 > 0;
    const float* sR = s + (size_t)r0 * n;
    const float* FR = rho ? nullptr : F + (size_t)r0 * n;
    const float* rhoR = rho ? rho + (size_t)r0 * K * n : nullptr;
    auto slab = [&](int l) { return 2LL * R * w[l]; };
    // ---- primal forward: t_l = tanh(W_l h_{l-1} + b_l), then h_l and d_l ----
    hipLaunchKernelGGL(train_embed_kernel, dim3(grid1d((long long)K * R * n)), dim3(256), 0,
                       st, sR, R, n, K, raw, W + hh[0], slab(0));
    RID_HIP(hipGetLastError());
    for (int l = 1; l <= L; ++l) {
      GemmArgs g{};
      g.A = W + hh[l - 1]; g.sAb = slab(l - 1); g.sAm = w[l - 1]; g.sAk = 1;
      g.Bm = WP + wq[l - 1]; g.sBb = pmp; g.sBk = 1; g.sBn = w[l - 1];
      g.C = W + tt[l]; g.sCb = (long long)R * w[l]; g.sCm = w[l]; g.sCn = 1;
      g.bias = P + b_off[l - 1]; g.sBiasb = pm;
      g.M = R; g.N = w[l]; g.Kc = w[l - 1]; g.batch = K; g.mode = EPI_BIAS_TANH;
      if ((rs = gemm(g, st)) != RID_OK) return rs;
      hipLaunchKernelGGL(act_kernel, dim3(grid1d((long long)K * R * ((w[l] + 3) / 4))),
                         dim3(256), 0, st, W + tt[l], l, w[l], R, K, r0, drop_p, drop_inv,
                         e.drop_seed, step32, skip(l) ? W + hh[l - 1] : nullptr, slab(l - 1),
                         W + hh[l], slab(l), W + dd[l]);
      RID_HIP(hipGetLastError());
    }
    // ---- primal backward to u0: v_l = u_l d_l, u_{l-1} = W_l^T v_l (+ u_l) ----
    hipLaunchKernelGGL(vlast_kernel, dim3(grid1d((long long)K * R * w[L])), dim3(256), 0, st,
                       W + dd[L], P, pm, (int)wo_off, w[L], R, K, W + vA);
    RID_HIP(hipGetLastError());
    long long uin = uA, uout = uB;
    if (res) {   // u_L = w_o
      hipLaunchKernelGGL(top_kernel, dim3(grid1d((long long)K * R * w[L])), dim3(256), 0, st,
                         P, pm, (int)wo_off, w[L], R, K, R, 0, W + uin);
      RID_HIP(hipGetLastError());
    }
    long long vin = vA, vout = vB;
    for (int l = L; l >= 1; --l) {
      GemmArgs g{};
      g.A = W + vin; g.sAb = (long long)R * w[l]; g.sAm = w[l]; g.sAk = 1;
      g.Bm = WP + wq[l - 1]; g.sBb = pmp; g.sBk = w[l - 1]; g.sBn = 1;
      g.sCb = (long long)R * w[l - 1]; g.sCm = w[l - 1]; g.sCn = 1;
      g.M = R; g.N = w[l - 1]; g.Kc = w[l]; g.batch = K;
      if (l > 1) {
        // v_{l-1} = (W_l^T v_l (+ u_l)) d_{l-1}; with a skip u_{l-1} is kept
        g.mode = EPI_GEN;
        g.C = skip(l) ? W + uout : nullptr;
        g.add = skip(l) ? W + uin : nullptr; g.sAddb = (long long)R * w[l];
        g.C2 = W + vout; g.sC2b = (long long)R * w[l - 1];
        g.mul = W + dd[l - 1]; g.sMulb = (long long)R * w[l - 1];
      } else {
        g.mode = EPI_STORE;
        g.C = W + vout;
      }
      if ((rs = gemm(g, st)) != RID_OK) return rs;
      std::swap(vin, vout);
      if (skip(l)) std::swap(uin, uout);
    }
    // vin now holds u0 [K][R][2n]
    hipLaunchKernelGGL(residual_kernel,
                       dim3((unsigned)(((long long)K * R + kResWaves - 1) / kResWaves)),
                       dim3(kResWaves * 64), 0, st,
                       sR, FR, rhoR, W + vin, R, B, n, K, raw, W + hh[0], slab(0),
                       rho ? nullptr : W + lrows + r0, (long long)B);
    RID_HIP(hipGetLastError());
    // ---- tangent forward: zd_l = W_l hd_{l-1}, hd_l = d_l zd_l (+ hd_{l-1}) ----
    for (int l = 1; l <= L; ++l) {
      GemmArgs g{};
      g.A = W + hh[l - 1] + (long long)R * w[l - 1]; g.sAb = slab(l - 1); g.sAm = w[l - 1];
      g.sAk = 1;
      g.Bm = WP + wq[l - 1]; g.sBb = pmp; g.sBk = 1; g.sBn = w[l - 1];
      g.C = W + zd[l]; g.sCb = (long long)R * w[l]; g.sCm = w[l]; g.sCn = 1;
      g.C2 = W + hh[l] + (long long)R * w[l]; g.sC2b = slab(l);
      g.mul = W + dd[l]; g.sMulb = (long long)R * w[l];
      if (skip(l)) {
        g.add2 = W + hh[l - 1] + (long long)R * w[l - 1];
        g.sAdd2b = slab(l - 1);
      }
      g.M = R; g.N = w[l]; g.Kc = w[l - 1]; g.batch = K; g.mode = EPI_GEN;
      if ((rs = gemm(g, st)) != RID_OK) return rs;
    }
    // ---- adjoint sweep with weight gradients (or down to the input) ----
    long long lin = lamA, lout = lamB;
    // top: lam_h_L = 0, lam_hd_L = w_o (stacked rows [0, R) and [R, 2R))
    hipLaunchKernelGGL(top_kernel, dim3(grid1d((long long)K * 2 * R * w[L])), dim3(256), 0, st,
                       P, pm, (int)wo_off, w[L], R, K, 2 * R, R, W + lin);
    RID_HIP(hipGetLastError());
    for (int l = L; l >= 1; --l) {
      hipLaunchKernelGGL(adjoint_kernel, dim3(grid1d((long long)K * R * w[l])), dim3(256), 0,
                         st, W + tt[l], W + dd[l], W + zd[l], W + lin, 2LL * R * w[l], w[l], R,
                         K, W + sbuf, 2LL * R * w[l]);
      RID_HIP(hipGetLastError());
      // dW_l = S^T [h_{l-1}; hd_{l-1}]  (contraction over 2R rows, split),
      // db_l = sum of lam_z; with layer 1, dw_o = sum_b hd_L and, on the last
      // pass, the losses
      if (!input_mode) {
        GradPass g{};
        const WgradSplit sp = wgrad_split(K, &w[l], &w[l - 1], 1, R);
        g.nl = 1; g.K = K; g.R = R; g.ks = sp.ks; g.kchunk = sp.kchunk;
        g.l[0] = GradLayer{W + sbuf, W + hh[l - 1], w[l], w[l - 1], w_off[l - 1], b_off[l - 1]};
        g.part = W + part; g.bpart = W + bpart; g.cpart = W + cpart;
        g.grad = G; g.pm = pm;
        g.accumulate = acc; g.wo_off = wo_off; g.w = w[L];
        if (l == 1) {
          g.last = r0 + R >= B;
          g.X = W + hh[L] + (long long)R * w[L]; g.sXb = slab(L);
          g.rows = rho ? nullptr : W + lrows; g.B = B; g.loss = loss;
        }
        if ((rs = grad_pass(g, st)) != RID_OK) return rs;
      }
      if (l > 1 || input_mode) {
        // [lam_h ; lam_hd]_{l-1} = [lam_z ; lam_zd] W_l (+ [lam_h ; lam_hd]_l)
        GemmArgs g{};
        g.A = W + sbuf; g.sAb = 2LL * R * w[l]; g.sAm = w[l]; g.sAk = 1;
        g.Bm = WP + wq[l - 1]; g.sBb = pmp; g.sBk = w[l - 1]; g.sBn = 1;
        g.C = W + lout; g.sCb = 2LL * R * w[l - 1]; g.sCm = w[l - 1]; g.sCn = 1;
        g.M = 2 * R; g.N = w[l - 1]; g.Kc = w[l]; g.batch = K;
        if (skip(l)) {
          g.mode = EPI_GEN;
          g.add = W + lin; g.sAddb = 2LL * R * w[l];
        } else {
          g.mode = EPI_STORE;
        }
        if ((rs = gemm(g, st)) != RID_OK) return rs;
        std::swap(lin, lout);
      }
    }
    if (input_mode) {
      // lin: [lam_h0 ; lam_hd0] per member (rows [0, B): d J / dx); vin: u0
      hvp->lam_x = W + lin;
      hvp->u0 = W + vin;
      hvp->slab_lam = 2LL * B * X;
      return RID_OK;
    }
  }
  if (adam.theta) {
    hipLaunchKernelGGL(adam_kernel, dim3(grid1d(K * pm)), dim3(256), 0, st, adam, G, K * pm);
    RID_HIP(hipGetLastError());
  }
  return RID_OK;
}

rid_status launch_train_step(rid_ensemble_impl& e, const float* s, const float* F,
                             int B, float lr, float* loss, hipStream_t st) {
  const int t = (int)(e.step + 1);
  const AdamStep adam{e.d_master, e.d_m, e.d_v, lr, 1.f - std::pow(0.9f, (float)t),
                      1.f - std::pow(0.999f, (float)t)};
  rid_status rs = launch_mf_grad(e, s, F, nullptr, B, loss, nullptr, st, nullptr, adam);
  if (rs != RID_OK) return rs;
  e.step += 1;
  e.frag_dirty = true;
  ++e.master_gen;
  return RID_OK;
}

}  // namespace rid
