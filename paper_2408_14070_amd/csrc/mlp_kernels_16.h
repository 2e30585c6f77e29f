// 16-bit ensembles of MLP free-energy models: the fused forward + input-gradient
// kernel (fed from atom positions on the bias path where that is cheaper).
// FP32 ensembles: mlp_kernels_f32.h.
//
// What bounds it: at width 512 and 16384 walkers of 8 members (393 us, 1.10
// PFLOP/s) the matrix units, 0.56 busy at 2.0 GHz, beside the weight stream
// from L2 (64 walkers a workgroup, all that LDS and registers hold); in small
// calls the latency of the layers, one after the other (rows_16, waves).
//
// Method ("Training phase"): each ensemble member is an MLP with tanh hidden
// layers and a scalar output A(x); the bias needs the mean force
// g = dA/ds (Box 2), obtained by one reverse sweep through the same layers.
// x = [cos s | sin s].
//
// Kernel design (gfx950):
//  * One workgroup owns R = 16*RT walkers of ONE member.  Its waves split the
//    hidden units; each wave streams its units' weight fragments straight
//    from L2 into VGPRs (no weight reuse inside a workgroup, so no LDS hop)
//    with buffer loads whose k-chunk offset sits in a scalar register.  The
//    loads run a few k-steps ahead of the MFMAs through a register ring that
//    scheduling barriers keep in order, and continue across layers (weights
//    do not depend on activations).  The weights are the MFMA A operand and
//    the activations the B operand, so each lane ends up holding 4
//    consecutive units of one walker: one packed LDS store per 4 outputs,
//    and the bias enters as the accumulator's initial value.
//  * The activation tile (shared by all waves) lives in LDS, ping-ponged
//    between two buffers so each layer needs one barrier; it holds x, then
//    h_1 .. h_L, then the reverse-sweep vectors v_l.
//  * tanh'(z_l) = 1 - h_l^2 is computed in FP32 and kept in VGPRs for the
//    reverse sweep, in FP16 (BF16 in the all-BF16 plan; 64-walker tiles would
//    not fit an FP32 copy): nothing goes to HBM between layers.
//  * 16-bit arithmetic plans (Plan below) choose the operand format of the
//    first layer, of the hidden-layer forward GEMMs and of the reverse sweep
//    separately.  The precision form runs the hidden-layer forward GEMMs in
//    BF16 and the first layer and the reverse sweep in FP16 (same MFMA rate):
//    the mean force is linear in the reverse sweep's roundings but sees the
//    forward sweep's only through tanh', so the reverse sweep's operand
//    format sets most of the force error.  The reverse vectors carry a
//    per-member power-of-two scale (exact) that keeps them inside FP16's
//    range.
//  * Forward weights and biases are stored pre-multiplied by 2/ln 2, so the
//    epilogue evaluates tanh from exp2 of the GEMM output and one reciprocal.
//  * Blocks are mapped XCD-aware: when K divides 8, member k runs on XCDs
//    {k*8/K, ...}, so each XCD's L2 holds only its members' weights.
//  * On the bias path each workgroup can compute the torsions of its walkers
//    itself from the positions (gather_pays; elsewhere the CVs are encoded
//    first).  The
//    FP64 deviation, switch and chain rule run in a second kernel: handing
//    the members' results to one workgroup inside this launch needs
//    device-scope fences, which on gfx950 write back and invalidate the
//    whole per-XCD L2 and so evict the weights the other workgroups stream.
#pragma once

#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace rid {
namespace mlp16 {

using namespace dev;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

struct BF16 {
  using T = __bf16;
  static constexpr int KF = 32;
  __device__ static inline void mma(const uint4& a, const uint4& b, f4& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a),
                                                __builtin_bit_cast(bf8, b), c,
                                                0, 0, 0);
  }
  __device__ static inline T from_float(float v) { return (__bf16)v; }
};

struct F16 {
  using T = _Float16;
  static constexpr int KF = 32;
  __device__ static inline void mma(const uint4& a, const uint4& b, f4& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a),
                                               __builtin_bit_cast(h8, b), c,
                                               0, 0, 0);
  }
  __device__ static inline T from_float(float v) { return (_Float16)v; }
};

// Arithmetic plan of the MLP kernel: MFMA operand format of the first layer
// (P1), of the hidden-layer forward GEMMs (PH) and of the reverse sweep (PB),
// and the storage type of tanh' between the sweeps (S).  The formats of one
// plan share an element size, so the activation tile's layout is the same
// for every layer.
template <class P1_, class PH_, class PB_, class S_>
struct Plan {
  using P1 = P1_;
  using PH = PH_;
  using PB = PB_;
  using S = S_;
};
using PlanBF16 = Plan<F16, BF16, F16, _Float16>;      // the BF16 precision form
using PlanF16 = Plan<F16, F16, F16, _Float16>;
using PlanBF16All = Plan<BF16, BF16, BF16, __bf16>;   // every operand BF16

// Four consecutive elements of type T as one register group.
template <class T> struct Pack4;
template <class H> struct Pack16 {
  typedef H h2 __attribute__((ext_vector_type(2)));
  typedef float fl2 __attribute__((ext_vector_type(2)));
  uint2 v;
  // two packed round-to-nearest-even conversions (v_cvt_pk_*_f32)
  __device__ inline void set(const f4& x) {
    v.x = __builtin_bit_cast(uint32_t, __builtin_convertvector((fl2{x[0], x[1]}), h2));
    v.y = __builtin_bit_cast(uint32_t, __builtin_convertvector((fl2{x[2], x[3]}), h2));
  }
  __device__ inline f4 get() const {
    f4 r;
    r[0] = (float)__builtin_bit_cast(H, (unsigned short)(v.x & 0xffffu));
    r[1] = (float)__builtin_bit_cast(H, (unsigned short)(v.x >> 16));
    r[2] = (float)__builtin_bit_cast(H, (unsigned short)(v.y & 0xffffu));
    r[3] = (float)__builtin_bit_cast(H, (unsigned short)(v.y >> 16));
    return r;
  }
  __device__ inline void store(H* dst) const { *reinterpret_cast<uint2*>(dst) = v; }
};
template <> struct Pack4<__bf16> : Pack16<__bf16> {};

// two consecutive elements of type T (one 4- or 8-byte LDS store)
template <class T> struct Pack2 {
  typedef T t2 __attribute__((ext_vector_type(2)));
  typedef float fl2 __attribute__((ext_vector_type(2)));
  __device__ static inline void store(T* dst, float a, float b) {
    *reinterpret_cast<t2*>(dst) = __builtin_convertvector((fl2{a, b}), t2);
  }
};
template <> struct Pack4<_Float16> : Pack16<_Float16> {};

// Forward weights and biases are stored multiplied by 2/ln 2, so a forward
// GEMM yields y = 2 z / ln 2 and exp(2z) = 2^y takes no multiply.
constexpr float kTanhPrescale = 2.8853900817779268f;

// tanh and its derivative from one exponential and one reciprocal, given the
// pre-scaled pre-activation y: with r = 1 / (1 + 2^y):  tanh z = 1 - 2r,
// 1 - tanh^2 z = (1 - h)(1 + h).  Saturates cleanly (2^y -> inf gives r = 0;
// 2^y -> 0 gives r = 1).  Absolute error of a few 1e-7, below the FP32
// rounding of the GEMM that feeds it.
__device__ inline float tanh_and_grad(float y, float& d) {
  const float e = __builtin_amdgcn_exp2f(y);
  const float r = __builtin_amdgcn_rcpf(1.f + e);
  const float h = __builtin_fmaf(-2.f, r, 1.f);
  d = __builtin_fmaf(-h, h, 1.f);
  return h;
}

struct MlpArgs {
  const float* x;      // [B][2n] input encoding (plain kernel)
  int B, n, K, L, XP, n_tiles, xcd_grp;
  const unsigned char* frag;
  unsigned long long frag_model_bytes;
  unsigned fwd_off[kMaxHidden];
  unsigned bwd_off[kMaxHidden];
  const float* bias;   // [K][L][NP]
  const float* wo;     // [K][NP]
  const float* bo;     // [K]
  const float* vscale; // [K][2] power-of-two scale folded into wo and its inverse
  float* A_out;        // [K][B]
  float* g_out;        // [K][B][n]
  // LDS layout (byte offsets; activation buffer 0 starts at 0)
  unsigned off_u0, off_red, off_xs, off_ph0, off_wo;
  // torsion input (bias path)
  SysView sv;
  const float* pos;    // [B][n_atoms][3]
  // encoding input: CVs with raw[i] = 1 are non-angular, encoded (s_i, 0),
  // so dA/ds_i = dA/dx_i (null: every CV angular)
  const uint8_t* raw;
};

__device__ inline void map_block(int b, int K, int grp, int& k, int& tile) {
  if (grp > 0) {
    int x = b & 7;
    k = x / grp;
    tile = (b >> 3) * grp + (x % grp);
  } else {
    k = b % K;
    tile = b / K;
  }
}

// acc[rt][c] += W(units of tile jt0 + c, 0:KL) * act(walkers of rt, 0:KL)^T
// (output tile: 16 units x 16 walkers; lane holds units 4(lane/16)+q of
// walker lane%16)
// Software pipeline: weight fragments (from L2/HBM) are loaded PD k-steps
// ahead through a ring of PD+1 register slots; activation fragments (LDS)
// either one k-step ahead through two slots (ADB) or next to their use.
// Scheduling barriers pin "issue next loads -> MFMAs of this step", so the
// compiler cannot sink a global load next to its first use and expose the
// memory latency; without ADB they let LDS reads and ALU work move freely.
#ifndef RID_PD_16
#define RID_PD_16 1
#endif
#ifndef RID_ADB_16
#define RID_ADB_16 1
#endif
#ifndef RID_SCHED
#define RID_SCHED 1
#endif
template <bool ALL>
__device__ inline void sched_fence() {
#if RID_SCHED
  // mask: instruction classes allowed to cross (ALU, VALU, SALU, MFMA, DS,
  // transcendental) -- everything except vector-memory loads and stores
  __builtin_amdgcn_sched_barrier(ALL ? 0 : 0x078F);
#endif
}

// Activation rows are padded by this many bytes (bank spread of the
// row-strided LDS accesses).
#ifndef RID_ACT_PAD_BYTES
#define RID_ACT_PAD_BYTES 16
#endif

// Hidden-layer GEMMs: passes over the contraction and weight pipeline depth
// (PD+1 must divide passes * k-steps: 1 or 3).
#ifndef RID_NPASS_16
#define RID_NPASS_16 1
#endif
#ifndef RID_PDH_16
#define RID_PDH_16 1
#endif

// Where a wave's weight fragments come from: a buffer resource over one
// member's fragments (range-checked by the hardware), the byte offset of
// k-chunk 0 of the wave's first unit tile, and the bytes per k-chunk.  A
// load is one buffer_load_dwordx4 with the lane's 16 bytes as the only
// vector offset; the k-chunk goes into the scalar offset and the tile into
// the instruction's immediate, so no vector registers hold addresses.
struct WSrc {
  __amdgpu_buffer_rsrc_t r;
  int soff, kstride;
  __device__ inline uint4 ld(int kk, int c, int lane) const {
    return __builtin_bit_cast(
        uint4, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + c * kFragBytes,
                                                     soff + kk * kstride, 0));
  }
};

// Weight ring: slot kt % (PD+1) holds the fragments of k-step kt.
template <int PD, int CT>
struct WRing {
  uint4 w[PD + 1][CT];
};

// Issue the loads of k-steps 0..PD-1 of a layer into the ring.
template <int PD, int CT>
__device__ inline void ring_preload(WRing<PD, CT>& wr, const WSrc& src, int n_kt, int lane) {
#pragma unroll
  for (int s = 0; s < PD; ++s)
    if (s < n_kt)
#pragma unroll
      for (int c = 0; c < CT; ++c) wr.w[s][c] = src.ld(s, c, lane);
}

// The k-loop of a GEMM with a run-time contraction length (first layer,
// input-gradient GEMM).  On entry the ring holds the first PD k-steps; the
// following ones are issued PD steps ahead.
template <class P, int RT, int CT, int PD>
__device__ inline void gemm_run(f4 (&acc)[RT][CT], WRing<PD, CT>& wr,
                                const typename P::T* act, int as, const WSrc& src, int n_kt,
                                int lane) {
  constexpr int KF = P::KF;
  constexpr bool ADB = RID_ADB_16;
  constexpr int S = PD + 1;
  constexpr int U = (S % 2) ? 2 * S : S;      // unroll: static ring indices
  const int r = lane & 15, g = lane >> 4;
  const typename P::T* arow = act + r * as + g * (KF / 4);
  uint4 a[ADB ? 2 : 1][RT];
  if (ADB && n_kt > 0)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      a[0][rt] = *reinterpret_cast<const uint4*>(arow + rt * 16 * as);
  for (int kb = 0; kb < n_kt; kb += U) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int kt = kb + i;
      if (kt < n_kt) {
        const int kp = kt + PD;
        if (kp < n_kt)
#pragma unroll
          for (int c = 0; c < CT; ++c)
            wr.w[(i + PD) % S][c] = src.ld(kp, c, lane);
        if (ADB && kt + 1 < n_kt)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            a[(i + 1) % 2][rt] =
                *reinterpret_cast<const uint4*>(arow + rt * 16 * as + (kt + 1) * KF);
        sched_fence<ADB>();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const uint4 av = ADB ? a[i % 2][rt]
                               : *reinterpret_cast<const uint4*>(arow + rt * 16 * as + kt * KF);
#pragma unroll
          for (int c = 0; c < CT; ++c) P::mma(wr.w[i % S][c], av, acc[rt][c]);
        }
        sched_fence<ADB>();
      }
    }
  }
}

template <class P, int RT, int CT, int PD>
__device__ inline void gemm_tiles(f4 (&acc)[RT][CT], const typename P::T* act, int as,
                                  const WSrc& src, int n_kt, int lane) {
  WRing<PD, CT> wr;
  ring_preload<PD, CT>(wr, src, n_kt, lane);
  gemm_run<P, RT, CT, PD>(acc, wr, act, as, src, n_kt, lane);
}

// Hidden-layer GEMM (contraction length NK k-steps, known at compile time),
// in NPASS passes over the contraction, each computing CT/NPASS of the
// wave's unit tiles (two passes halve the weight registers per k-step at
// the price of reading the activations from LDS once per pass).  The
// weight ring streams all passes as one sequence of NPASS*NK steps, and
// after the last MFMA it already issues the next layer's first PD steps
// (weights do not depend on activations), so a layer starts with its
// weights in flight through the previous epilogue and barrier.  Slot
// numbering stays step % S across layers because S divides NPASS*NK.
template <class P, int RT, int CT, int NPASS, int PD, int NK>
__device__ inline void gemm_hidden(f4 (&acc)[RT][CT], WRing<PD, CT / NPASS>& wr,
                                   const typename P::T* act, int as, const WSrc& src,
                                   bool has_next, const WSrc& next, int lane) {
  constexpr int KF = P::KF;
  constexpr int S = PD + 1;
  constexpr int CH = CT / NPASS;
  constexpr int NV = NPASS * NK;
  static_assert(CH * NPASS == CT && NV % S == 0, "ring slots must line up across layers");
  const int r = lane & 15, g = lane >> 4;
  const typename P::T* arow = act + r * as + g * (KF / 4);
  uint4 a[2][RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) a[0][rt] = *reinterpret_cast<const uint4*>(arow + rt * 16 * as);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int vp = v + PD;                     // weight step issued now
    if (vp < NV) {
#pragma unroll
      for (int c = 0; c < CH; ++c) wr.w[vp % S][c] = src.ld(vp % NK, (vp / NK) * CH + c, lane);
    } else if (has_next) {
#pragma unroll
      for (int c = 0; c < CH; ++c) wr.w[vp % S][c] = next.ld(vp - NV, c, lane);
    }
    if (v + 1 < NV) {
      const int kn = (v + 1) % NK;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        a[(v + 1) % 2][rt] = *reinterpret_cast<const uint4*>(arow + rt * 16 * as + kn * KF);
    }
    sched_fence<true>();
    const int cb = (v / NK) * CH;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int c = 0; c < CH; ++c) P::mma(wr.w[v % S][c], a[v % 2][rt], acc[rt][cb + c]);
    sched_fence<true>();
  }
}

// GRAD = false: the free energies only (the forward sweep, no tanh' stash,
// no reverse sweep, no g output).
template <class PL, int NP, int RT, int NW, int LM, bool FROM_POS, bool GRAD>
__global__ __launch_bounds__(NW * 64) void mlp_kernel(MlpArgs p) {
  using P = typename PL::PH;         // hidden-layer forward GEMMs
  using P1 = typename PL::P1;        // first layer
  using PB = typename PL::PB;        // reverse sweep
  using T = typename P::T;
  using T1 = typename P1::T;
  using TB = typename PB::T;
  static_assert(sizeof(T1) == sizeof(T) && sizeof(TB) == sizeof(T) && P1::KF == P::KF &&
                    PB::KF == P::KF, "one element size per plan");
  using SP = Pack4<T>;               // hidden activations
  using SB = Pack4<TB>;              // reverse vectors
  using SS = Pack4<typename PL::S>;  // tanh' between the sweeps
  constexpr int KF = P::KF;
  constexpr int CT = NP / (16 * NW);
  constexpr int R = 16 * RT;
  constexpr int JT = NP / 16;
  static_assert((CT == 1 || CT == 2 || CT == 4) && CT * 16 * NW == NP, "width/wave split");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int k, tile;
  map_block(blockIdx.x, p.K, p.xcd_grp, k, tile);
  if (tile >= p.n_tiles) return;
  const int row0 = tile * R;
  const int n = p.n, L = p.L, XP = p.XP, X2 = 2 * p.n;
  const int AW = NP > XP ? NP : XP;           // activation tile width
  const int AS = AW + RID_ACT_PAD_BYTES / (int)sizeof(T);    // row stride (+16 bytes)
  const int BUF = R * AS;                     // elements per ping-pong buffer
  T* act = reinterpret_cast<T*>(smem);
  T1* act1 = reinterpret_cast<T1*>(smem);      // the input tile (first layer's format)
  float* u0 = reinterpret_cast<float*>(smem + p.off_u0);
  const int US = XP + 4;
  float* red = reinterpret_cast<float*>(smem + p.off_red);   // [NW][R]
  float* xs = reinterpret_cast<float*>(smem + p.off_xs);     // [R][2n] FP32 cos|sin
  float* wos = reinterpret_cast<float*>(smem + p.off_wo);    // [NP] output weights

  const unsigned char* fbase = p.frag + (size_t)k * p.frag_model_bytes;
  const float* bias = p.bias + (size_t)k * L * NP;
  const float* wo = p.wo + (size_t)k * NP;

  // first forward layer's weights and biases go in flight before the input
  // tile is built
  constexpr int PD = RID_PD_16;
  constexpr int NPASS = RID_NPASS_16;
  constexpr int CH = CT / NPASS;     // unit tiles per pass of a hidden-layer GEMM
  constexpr int NK = NP / KF;        // k-steps of a hidden-layer GEMM
  constexpr int PDW = RID_PDH_16;
  constexpr int PDH = (NPASS * NK) % (PDW + 1) == 0 ? PDW : 1;   // its weight pipeline depth
  const int jt0 = wave * CT;
  const int uq = 4 * (lane >> 4);    // first of this lane's 4 units in a tile
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(fbase), (short)0, (int)p.frag_model_bytes, 0x00020000);
  // fragments of one layer (byte offset off) for this wave's unit tiles
  auto wsrc = [&](unsigned off) {
    return WSrc{rsrc, (int)off + jt0 * kFragBytes, JT * kFragBytes};
  };
  // plain input: the first column batch of the tile's encoding is loaded
  // before anything else, so its loads return ahead of the weight and bias
  // loads queued behind them (rows of the tile go to the waves in turn; a
  // wave's lanes cover a row in float2 columns)
  constexpr int RW = FROM_POS ? 1 : (R + NW - 1) / NW;   // rows per wave, at most
  float2 xv[RW];
  auto load_x = [&](int cb) {
    const int col = cb + lane;                // float2 column
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const int i = wave * RW + j, row = row0 + i;
      xv[j] = (col < p.n && (R % NW == 0 || i < R) && row < p.B)
                  ? *reinterpret_cast<const float2*>(p.x + (size_t)row * X2 + 2 * col)
                  : make_float2(0.f, 0.f);
    }
  };
  if constexpr (!FROM_POS) load_x(0);
  WRing<PD, CT> wr;                  // first layer
  WRing<PDH, CH> wh;                 // hidden layers (passes of CH tiles)
  ring_preload<PD, CT>(wr, wsrc(p.fwd_off[0]), XP / KF, lane);
  f4 bnext[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
    bnext[c] = *reinterpret_cast<const f4*>(bias + (jt0 + c) * 16 + uq);

  for (int i = threadIdx.x; i < NP; i += NW * 64) wos[i] = wo[i];   // published below

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
    float* sp = reinterpret_cast<float*>(smem + p.off_ph0);   // [R][U][3]
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
        act1[i * AS + c] = P1::from_float(cs);
        act1[i * AS + n + c] = P1::from_float(sn);
      }
    }
    for (int i = wave; i < R; i += NW)
      for (int c = X2 + lane; c < XP; c += 64) act1[i * AS + c] = P1::from_float(0.f);
  } else {
    // the column batches of the tile (the first one is already in xv);
    // padding columns [X2, XP) get zeros (X2 is even)
    const int h2 = X2 / 2, hp = XP / 2;
    for (int cb = 0; cb < hp; cb += 64) {
      const int col = cb + lane;              // float2 column
      if (cb > 0) load_x(cb);
      if (col < hp) {
#pragma unroll
        for (int j = 0; j < RW; ++j) {
          const int i = wave * RW + j;
          if (R % NW != 0 && i >= R) break;
          Pack2<T1>::store(act1 + i * AS + 2 * col, xv[j].x, xv[j].y);
          if (col < h2) *reinterpret_cast<float2*>(xs + i * X2 + 2 * col) = xv[j];
        }
      }
    }
  }
  __syncthreads();

  const int wl = lane & 15;          // walker within a 16-walker tile
  SS st[LM - 1][RT][CT];             // tanh' of hidden layers 1..L-1
  // the packed w_o carries a per-member power-of-two scale (exact), so the
  // reverse vectors start scaled; the scale is undone where A and g are
  // written (uniform loads of its inverse there)
  auto a_total = [&](int i) {
    float a = 0.f;
    for (int w = 0; w < NW; ++w) a += red[w * R + i];
    return __builtin_fmaf(a, p.vscale[2 * k + 1], p.bo[k]);
  };
  int cur = 0;

  // ---------------- forward: h_l = tanh(W_l h_{l-1} + b_l) ----------------
  // tile epilogues: tanh and its derivative; a layer before the last stores
  // h_l into the other buffer and stashes tanh'; the last layer stores
  // v_L = w_o * tanh' and accumulates the lane's part of A = w_o . h_L.
  float apart[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) apart[rt] = 0.f;
  auto mid_tile = [&](int l, int rt, int c, const f4& z, T* out) {
    f4 h, d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float dq;
      h[q] = tanh_and_grad(z[q], dq);
      d[q] = dq;
    }
    SP o;
    o.set(h);
    o.store(out + (rt * 16 + wl) * AS + (jt0 + c) * 16 + uq);
    if constexpr (GRAD) st[l][rt][c].set(d);
  };
  auto last_tile = [&](int rt, int c, const f4& z, T* out) {
    const int u = (jt0 + c) * 16 + uq;
    const f4 w4 = *reinterpret_cast<const f4*>(wos + u);
    f4 h, d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float dq;
      h[q] = tanh_and_grad(z[q], dq);
      d[q] = dq;
    }
    apart[rt] += w4[0] * h[0] + w4[1] * h[1] + w4[2] * h[2] + w4[3] * h[3];
    if constexpr (GRAD) {
      SB o;
      o.set(w4 * d);
      o.store(reinterpret_cast<TB*>(out) + (rt * 16 + wl) * AS + u);
    }
  };
  // the GEMM after forward layer l: forward layer l+1, or the first backward
  auto next_after_fwd = [&](int l) {
    return wsrc(l + 1 < L ? p.fwd_off[l + 1] : p.bwd_off[L > 1 ? L - 1 : 0]);
  };
  auto load_bias = [&](int l) {
#pragma unroll
    for (int c = 0; c < CT; ++c)
      bnext[c] = *reinterpret_cast<const f4*>(bias + l * NP + (jt0 + c) * 16 + uq);
  };

  {  // layer 1 (input width XP): one pass over all CT tiles
    T* out = act + BUF;
    f4 acc[RT][CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt][c] = bnext[c];
    gemm_run<P1, RT, CT, PD>(acc, wr, act1, AS, wsrc(p.fwd_off[0]), XP / KF, lane);
    if (L > 1) {
      ring_preload<PDH, CH>(wh, next_after_fwd(0), NK, lane);
      load_bias(1);
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) mid_tile(0, rt, c, acc[rt][c], out);
    } else {
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) last_tile(rt, c, acc[rt][c], out);
    }
    cur = 1;
    __syncthreads();
  }
  // hidden layers before the last
#pragma unroll
  for (int l = 1; l < LM - 1; ++l) {
    if (l < L - 1) {
      const T* in = act + cur * BUF;
      T* out = act + (cur ^ 1) * BUF;
      f4 acc[RT][CT];
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][c] = bnext[c];
      gemm_hidden<P, RT, CT, NPASS, PDH, NK>(acc, wh, in, AS, wsrc(p.fwd_off[l]), true,
                                             next_after_fwd(l), lane);
      load_bias(l + 1);
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) mid_tile(l, rt, c, acc[rt][c], out);
      cur ^= 1;
      __syncthreads();
    }
  }
  if (L > 1) {  // the last hidden layer (index L-1)
    const T* in = act + cur * BUF;
    T* out = act + (cur ^ 1) * BUF;
    f4 acc[RT][CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt][c] = bnext[c];
    gemm_hidden<P, RT, CT, NPASS, PDH, NK>(acc, wh, in, AS, wsrc(p.fwd_off[L - 1]), GRAD,
                                           wsrc(p.bwd_off[L - 1]), lane);
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) last_tile(rt, c, acc[rt][c], out);
    cur ^= 1;
    __syncthreads();
  }
  // A = w_o . h_L + b_o: the lanes' partials reduced over the 4 unit groups,
  // then (after the last barrier) over the waves
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float v = apart[rt];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lane < 16) red[wave * R + rt * 16 + wl] = v;
  }
  if constexpr (!GRAD) {
    __syncthreads();
    for (int i = threadIdx.x; i < R; i += NW * 64) {
      const float a = a_total(i);
      if (row0 + i < p.B) p.A_out[(size_t)k * p.B + row0 + i] = a;
    }
    return;
  }

  // ------------- reverse sweep: v_{l-1} = (W_l^T v_l) * tanh'_{l-1} -------------
  auto bwd_tile = [&](int l, int rt, int c, const f4& y, T* out) {
    SB o;
    o.set(y * st[l - 1][rt][c].get());
    o.store(reinterpret_cast<TB*>(out) + (rt * 16 + wl) * AS + (jt0 + c) * 16 + uq);
  };
#pragma unroll
  for (int l = LM - 1; l >= 1; --l) {
    if (l < L) {
      const T* in = act + cur * BUF;
      T* out = act + (cur ^ 1) * BUF;
      f4 acc[RT][CT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[rt][c] = f4{0.f, 0.f, 0.f, 0.f};
      gemm_hidden<PB, RT, CT, NPASS, PDH, NK>(acc, wh, reinterpret_cast<const TB*>(in), AS,
                                              wsrc(p.bwd_off[l]), l >= 2,
                                              wsrc(p.bwd_off[l >= 2 ? l - 1 : l]), lane);
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) bwd_tile(l, rt, c, acc[rt][c], out);
      cur ^= 1;
      __syncthreads();
    }
  }
  // layer 1 backward: u0 = W_1^T v_1.  v_1 sits in buffer 1 (2L-1 buffer
  // flips), so u0 may alias buffer 0.
  {
    const T* in = act + cur * BUF;
    const int JT0 = XP / 16;
    for (int t = wave; t < JT0; t += NW) {
      f4 a1[RT][1];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a1[rt][0] = f4{0.f, 0.f, 0.f, 0.f};
      gemm_tiles<PB, RT, 1, 7>(
          a1, reinterpret_cast<const TB*>(in), AS,
          WSrc{rsrc, (int)p.bwd_off[0] + t * kFragBytes, JT0 * kFragBytes}, NK, lane);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        *reinterpret_cast<f4*>(u0 + (rt * 16 + wl) * US + t * 16 + uq) = a1[rt][0];
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R; i += NW * 64) {
    const float a = a_total(i);
    if (row0 + i < p.B) p.A_out[(size_t)k * p.B + row0 + i] = a;
  }
  // chain to the angles: g_i = -sin s_i u0[i] + cos s_i u0[n+i]
  const float ivs = p.vscale[2 * k + 1];
  for (int e = threadIdx.x; e < R * n; e += NW * 64) {
    const int i = e / n, c = e - i * n;
    const int row = row0 + i;
    if (row < p.B) {
      const float cs = xs[i * X2 + c];
      const float sn = xs[i * X2 + n + c];
      float gv = -sn * u0[i * US + c] + cs * u0[i * US + n + c];
      if constexpr (!FROM_POS) {
        if (p.raw && p.raw[c]) gv = u0[i * US + c];
      }
      p.g_out[((size_t)k * p.B + row) * n + c] = gv * ivs;
    }
  }
}

// Waves of a workgroup: one unit tile each up to 192 units, two to 384, four
// at 512: with four unit tiles a wave everywhere a SIMD held one wave, or none,
// and nothing hid its loads and epilogues (2001 walkers of 4 members, FP16, 64
// walkers a workgroup: 29 / 12 us at width 64, 23 / 13 at 128, 24 / 20 at 256;
// at 512 16 waves spill).  One number for all row tiles: the order A is summed
// in follows the waves, and a walker's A does not depend on its row tile.
__host__ __device__ constexpr int waves(int NP) {
  return NP <= 192 ? NP / 16 : NP <= 384 ? NP / 32 : NP / 64;
}

inline unsigned align16(size_t v) { return (unsigned)((v + 15) / 16 * 16); }

// LDS layout of one instantiation; returns the total bytes.
inline size_t mlp_layout(int R, int NW, int AS, size_t tsize, int XP, int n, int NPw, MlpArgs& a) {
  const size_t buf = (size_t)R * AS * tsize;
  size_t off = 2 * buf;
  const size_t u0_bytes = (size_t)R * (XP + 4) * 4;
  if (u0_bytes <= buf) {
    a.off_u0 = 0;                       // buffer 0 is free in the last GEMM
  } else {
    a.off_u0 = align16(off);
    off = a.off_u0 + u0_bytes;
  }
  a.off_red = align16(off);
  off = a.off_red + (size_t)NW * R * 4;
  a.off_xs = align16(off);
  off = a.off_xs + (size_t)R * 2 * n * 4;
  a.off_wo = align16(off);              // output weights w_o [NP]
  a.off_ph0 = (unsigned)buf;            // gather scratch: buffer 1, free before layer 1
  return a.off_wo + (size_t)NPw * 4;
}

inline int row_stride(const rid_ensemble_impl& e) {   // elements of an activation row
  return (e.NP > e.XP ? e.NP : e.XP) + RID_ACT_PAD_BYTES / 2;
}
// Bytes of LDS of one shape (NW: waves; R: walkers).
inline size_t lds_bytes(const rid_ensemble_impl& e, int R, int NW) {
  MlpArgs a{};
  return mlp_layout(R, NW, row_stride(e), 2, e.XP, e.n_cv, e.NP, a);
}
// Whether buffer 1 (free before layer 1) holds a tile's torsion atoms.
inline bool gathers(const rid_ensemble_impl& e, int R, int U) {
  return (size_t)R * row_stride(e) * 2 >= (size_t)R * U * 12;
}

template <class PL, int NP, int RT, int NW, int LM>
rid_status run_mlp(const rid_ensemble_impl& e, const float* x, int B,
                   float* A_out, float* g_out, const TorsionInput* tin,
                   hipStream_t st) {
  static size_t attr_bytes[3] = {0, 0, 0};   // dynamic-LDS limit set per kernel
  constexpr int R = 16 * RT;
  using P = typename PL::PH;
  using T = typename P::T;
  const bool from_pos = tin != nullptr;
  static_assert(sizeof(T) == 2, "16-bit activations");
  MlpArgs a{};
  const size_t lds = mlp_layout(R, NW, row_stride(e), sizeof(T), e.XP, e.n_cv, NP, a);
  if (lds > 160 * 1024)
    return fail(RID_EUNSUPPORTED, "shape too large for the MLP kernel's LDS");
  // without g_out only the free energies are computed (plain input only)
  const bool grad = g_out != nullptr;
  if (from_pos && (RT > 1 || !grad || !gathers(e, R, tin->sys->n_uniq)))
    return fail(RID_EUNSUPPORTED, "in-kernel torsions: not this form (gather_pays)");
  auto kern = grad ? mlp_kernel<PL, NP, RT, NW, LM, false, true>
                   : mlp_kernel<PL, NP, RT, NW, LM, false, false>;
  if constexpr (RT == 1) {
    if (from_pos) kern = mlp_kernel<PL, NP, RT, NW, LM, true, true>;
  }
  const int ki = grad ? (from_pos ? 1 : 0) : 2;
  if (lds > 64 * 1024 && lds > attr_bytes[ki]) {
    RID_HIP(hipFuncSetAttribute((const void*)kern,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_bytes[ki] = lds;
  }
  a.x = x; a.B = B; a.n = e.n_cv; a.K = e.K; a.L = e.L; a.XP = e.XP;
  a.n_tiles = (B + R - 1) / R;
  a.xcd_grp = (8 % e.K == 0) ? 8 / e.K : 0;
  a.frag = e.d_frag; a.frag_model_bytes = e.frag_bytes_per_model;
  for (int l = 0; l < e.L; ++l) {
    a.fwd_off[l] = (unsigned)e.layers[l].fwd_off;
    a.bwd_off[l] = (unsigned)e.layers[l].bwd_off;
  }
  a.bias = e.d_bias; a.wo = e.d_wo; a.bo = e.d_bo; a.vscale = e.d_vscale;
  a.A_out = A_out; a.g_out = g_out;
  a.raw = e.d_raw;
  if (from_pos) {
    const rid_system_impl& s = *tin->sys;
    a.sv = SysView{s.n_atoms, s.n_uniq, s.n_cv, s.d_uniq, s.d_lquads, s.d_csr_ptr,
                   s.d_csr_ent, s.d_atom_local};
    a.pos = tin->pos;
  }
  int grid;
  if (a.xcd_grp > 0)
    grid = 8 * ((a.n_tiles + a.xcd_grp - 1) / a.xcd_grp);
  else
    grid = a.n_tiles * e.K;
  launch_timed(kProfMlp, kern, dim3(grid), dim3(NW * 64), (uint32_t)lds, st, a);
  RID_HIP(hipGetLastError());
  return RID_OK;
}

// One padded width: the plan of the ensemble's precision, rt 16-walker tiles
// a workgroup (1, 2 or, up to 4 hidden layers and where W4, 4).
template <class PL, int NP, bool W4>
rid_status run_plan(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                    float* g_out, const TorsionInput* t, hipStream_t st) {
  constexpr int NW = waves(NP);
  if (rt == 1) return run_mlp<PL, NP, 1, NW, 6>(e, x, B, A_out, g_out, t, st);
  if (e.L > 4) return run_mlp<PL, NP, 2, NW, 6>(e, x, B, A_out, g_out, t, st);
  if constexpr (W4) {
    if (rt == 4) return run_mlp<PL, NP, 4, NW, 4>(e, x, B, A_out, g_out, t, st);
  }
  return run_mlp<PL, NP, 2, NW, 4>(e, x, B, A_out, g_out, t, st);
}
template <int NP, bool W4>
rid_status run_width(int rt, const rid_ensemble_impl& e, const float* x, int B, float* A_out,
                     float* g_out, const TorsionInput* t, hipStream_t st) {
  switch (e.prec) {
    case RID_BF16:     return run_plan<PlanBF16, NP, W4>(rt, e, x, B, A_out, g_out, t, st);
    case RID_FP16:     return run_plan<PlanF16, NP, W4>(rt, e, x, B, A_out, g_out, t, st);
    case RID_BF16_ALL: return run_plan<PlanBF16All, NP, W4>(rt, e, x, B, A_out, g_out, t, st);
    default: break;
  }
  return fail(RID_EUNSUPPORTED, "unknown precision");
}

}  // namespace mlp16
}  // namespace rid
