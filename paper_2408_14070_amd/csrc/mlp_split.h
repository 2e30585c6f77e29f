// FP32 matrix products on the FP16 matrix units: every operand is split into
// two FP16 values, x = hi + lo with hi = fp16(x), lo = fp16(x - hi), and a
// product is three MFMAs into one FP32 accumulator, w_lo h_hi + w_hi h_lo +
// w_hi h_hi (the dropped w_lo h_lo is below 2^-23 of the product).
//
// Why: FP32 MFMA runs at 1/16 of the FP16 rate, so three FP16 products take
// 3/16 of its matrix time, and hi and lo together are the four bytes an FP32
// weight takes.  On 256-long dot products of tanh activations and Xavier
// weights the error against FP64 is 1.8e-7 rms of the result, that of the
// FP32 MFMA chain 2.9e-7: the split keeps 22-23 bits of each operand, and
// 24 accumulator roundings (one per 32 products) replace 256.
//
// Range: FP16 spans 2^-24 .. 2^16, so every operand row is scaled by a power
// of two (exact) before it is split, and the result is scaled back:
//  * weights: one scale per row of the product (an output unit), from the
//    row's largest weight, which lands in [2^9, 2^10); lo's resolution is
//    then 2^-34 of the row's maximum.  The rounding of lo is the same for every
//    sample, so sums over a batch keep it; the packer makes a second set of
//    fragments whose lo errs the other way, and odd tiles of a training step
//    read that one (gradient of 4096 samples, 38 CVs, 4 x [256 x 4]: 1.04e-7 of
//    its norm with one set, 0.80e-7 with two, 0.82e-7 with FP32 MFMA; time of
//    two steps 854 -> 859 us, of eight of 128 samples 942 -> 952 us);
//  * activations h of the forward sweep: |h| <= 6 (tanh, up to 6 residual
//    layers), scaled by 2^10, and so the cosines and sines of the input;
//  * raw CVs have no range at all (their weights neither, nor their entries
//    of the tangents' input): layer 1 adds their part in FP32 (raw_gemm), and
//    the split products get zeros in their columns;
//  * vectors with no fixed range (reverse, tangent, adjoint sweeps): one
//    scale per row (a walker's vector), from a bound that cannot overflow:
//    the largest entry of the previous layer's vector (tracked in LDS) times
//    the largest absolute row sum of the layer's weights (from the packer).
//    The bound is typically 2^4 to 2^6 above the true maximum.  lo's smallest
//    step is 2^-24 and values stay below 2^14, so a pair keeps 22 bits down to
//    2^-16 of the bound and one less per power of two below (11 at 2^-28).
#pragma once

#include <type_traits>

#include "device_common.h"

namespace rid {
namespace dev {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// f(integral_constant i) for i = I .. N-1, or I down to N: layer loops whose
// index must be a compile-time constant (the per-layer register arrays) however
// large the body is; an unroll pragma gives up on the larger ones.
template <int I, int N, class F>
__device__ __attribute__((always_inline)) inline void layers_up(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    layers_up<I + 1, N>(f);
  }
}
template <int I, int N, class F>
__device__ __attribute__((always_inline)) inline void layers_down(F&& f) {
  if constexpr (I >= N) {
    f(std::integral_constant<int, I>{});
    layers_down<I - 1, N>(f);
  }
}

constexpr int kSplitKF = 32;             // contraction indices per MFMA
constexpr int kSplitFrag = 2 * kFragBytes;   // hi block, then lo block
constexpr float kActScale = 1024.f;      // scale of forward activations
constexpr float kActUnscale = 1.f / 1024.f;
constexpr int kTargetExp = 14;           // scaled vectors stay below 2^14

// Activation rows in LDS: [hi: AW halfs][lo: AW halfs][pad 16 bytes]; AW a
// multiple of 32, so row starts are spread over the banks like 16-byte
// padded rows of 4 AW bytes.  Hidden vectors take AW = NP, the input tile its
// own XP.  The two ping-pong buffers lie [buffer 1][buffer 0, input tile,
// partials of u0], so that every hidden address is a constant offset; layer
// j reads buffer j & 1.
__host__ __device__ constexpr int split_row_halfs(int AW) { return 2 * AW + 8; }

// Where a wave's weight fragments come from: a buffer resource over one
// member's fragments (range-checked by the hardware), the byte offset of
// k-chunk 0 of the wave's first unit tile, and the bytes per k-chunk.  A
// load is one buffer_load_dwordx4 with the lane's 16 bytes as the only
// vector offset, the k-chunk in the scalar offset, tile and half in the
// instruction's immediate.
struct SplitSrc {
  __amdgpu_buffer_rsrc_t r;
  int soff, kstride;
  __device__ inline uint4 ld(int kk, int c, int half, int lane) const {
    return __builtin_bit_cast(
        uint4, __builtin_amdgcn_raw_buffer_load_b128(
                   r, lane * 16 + c * kSplitFrag + half * kFragBytes, soff + kk * kstride, 0));
  }
};

// Weight ring: slot kt % (PD+1) holds the fragments (hi, lo) of k-step kt.
template <int PD, int CT>
struct SplitRing {
  uint4 w[PD + 1][CT][2];
};

template <int PD, int CT>
__device__ inline void split_ring_load(SplitRing<PD, CT>& wr, int slot, const SplitSrc& src,
                                       int kk, int lane) {
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int h = 0; h < 2; ++h) wr.w[slot][c][h] = src.ld(kk, c, h, lane);
}

// Issue the loads of k-steps 0..PD-1 of a layer into the ring.
template <int PD, int CT>
__device__ inline void split_preload(SplitRing<PD, CT>& wr, const SplitSrc& src, int n_kt,
                                     int lane) {
#pragma unroll
  for (int s = 0; s < PD; ++s)
    if (s < n_kt) split_ring_load(wr, s, src, s, lane);
}

__device__ inline void split_mfma(f4& c, const uint4& a, const uint4& b) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b),
                                             c, 0, 0, 0);
}

// Fragments of the activation rows (hi, lo) of k-step kt.
template <int RT>
__device__ inline void split_act(uint4 (&a)[RT][2], const _Float16* arow, int as, int lo_off,
                                 int kt) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      a[rt][h] = *reinterpret_cast<const uint4*>(arow + rt * 16 * as + h * lo_off +
                                                 kt * kSplitKF);
}

// The three products of one k-step, small ones first.
template <int RT, int CT>
__device__ inline void split_step(f4 (&acc)[RT][CT], const uint4 (&w)[CT][2],
                                  const uint4 (&a)[RT][2]) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) split_mfma(acc[rt][c], w[c][1], a[rt][0]);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) split_mfma(acc[rt][c], w[c][0], a[rt][1]);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) split_mfma(acc[rt][c], w[c][0], a[rt][0]);
}

// Four consecutive floats of a uniform array (row scales, biases): the
// array as a scalar resource, the element as a scalar offset plus the lane's.
struct VecSrc {
  __amdgpu_buffer_rsrc_t r;
  __device__ inline f4 ld4(int uniform, int lane_off) const {
    return __builtin_bit_cast(
        f4, __builtin_amdgcn_raw_buffer_load_b128(r, 4 * lane_off, 4 * uniform, 0));
  }
};
__device__ inline VecSrc vec_src(const float* p, int count) {
  return VecSrc{__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, 4 * count,
                                                  0x00020000)};
}

// The scheduling barrier that pins "issue next loads -> MFMAs of this step":
// without it the compiler sinks a load next to its first use.
__device__ inline void split_fence() { __builtin_amdgcn_sched_barrier(0); }

// acc[rt][c] += W(tile c of src) act(rows of rt)^T, run-time contraction
// (first layer, input-gradient product).  On entry the ring holds the first
// PD k-steps.
template <int RT, int CT, int PD>
__device__ inline void split_gemm_run(f4 (&acc)[RT][CT], SplitRing<PD, CT>& wr,
                                      const _Float16* act, int as, int lo_off,
                                      const SplitSrc& src, int n_kt, int lane) {
  constexpr int S = PD + 1;
  const _Float16* arow = act + (lane & 15) * as + (lane >> 4) * 8;
  for (int kb = 0; kb < n_kt; kb += S) {
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int kt = kb + i;
      if (kt < n_kt) {
        if (kt + PD < n_kt) split_ring_load(wr, (i + PD) % S, src, kt + PD, lane);
        uint4 a[RT][2];
        split_act<RT>(a, arow, as, lo_off, kt);
        split_fence();
        split_step<RT, CT>(acc, wr.w[i], a);
        split_fence();
      }
    }
  }
}

// The same with a compile-time contraction of NK k-steps (hidden layers):
// the activation fragments are read one k-step ahead (ADB) or with their
// use, and after the last MFMA the next layer's first PD weight steps are
// already issued, so a layer starts with its weights in flight through the
// previous epilogue and barrier.  Ring slots line up across layers because
// PD + 1 divides NK.
template <int RT, int CT, int PD, int NK, bool ADB>
__device__ inline void split_gemm_hidden(f4 (&acc)[RT][CT], SplitRing<PD, CT>& wr,
                                         const _Float16* act, int as, int lo_off,
                                         const SplitSrc& src, bool has_next,
                                         const SplitSrc& next, int lane) {
  constexpr int S = PD + 1;
  static_assert(NK % S == 0, "ring slots must line up across layers");
  const _Float16* arow = act + (lane & 15) * as + (lane >> 4) * 8;
  uint4 a[ADB ? 2 : 1][RT][2];
  if constexpr (ADB) split_act<RT>(a[0], arow, as, lo_off, 0);
#pragma unroll
  for (int v = 0; v < NK; ++v) {
    if (v + PD < NK) {
      split_ring_load(wr, (v + PD) % S, src, v + PD, lane);
    } else if (has_next) {
      split_ring_load(wr, (v + PD) % S, next, v + PD - NK, lane);
    }
    if constexpr (ADB) {
      if (v + 1 < NK) split_act<RT>(a[(v + 1) % 2], arow, as, lo_off, v + 1);
    } else {
      split_act<RT>(a[0], arow, as, lo_off, v);
    }
    split_fence();
    split_step<RT, CT>(acc, wr.w[v % S], a[ADB ? v % 2 : 0]);
    split_fence();
  }
}

// Weight pipeline depth of the hidden-layer products: deep enough to keep
// the L2 stream in flight, a divisor constraint (PD + 1 | NK) and registers.
__host__ __device__ constexpr int split_depth(int NK, int CT) {
  return CT == 1 && NK % 4 == 0 ? 3 : 1;
}

// Four scaled values into an activation row: hi and lo, 8 bytes each.
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float fl2 __attribute__((ext_vector_type(2)));
__device__ inline void split_store4(_Float16* dst, int lo_off, const f4& x) {
  const h2 a = __builtin_convertvector((fl2{x[0], x[1]}), h2);
  const h2 b = __builtin_convertvector((fl2{x[2], x[3]}), h2);
  const h2 c = __builtin_convertvector((fl2{x[0] - (float)a[0], x[1] - (float)a[1]}), h2);
  const h2 d = __builtin_convertvector((fl2{x[2] - (float)b[0], x[3] - (float)b[1]}), h2);
  *reinterpret_cast<uint2*>(dst) =
      make_uint2(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b));
  *reinterpret_cast<uint2*>(dst + lo_off) =
      make_uint2(__builtin_bit_cast(unsigned, c), __builtin_bit_cast(unsigned, d));
}
__device__ inline void split_store2(_Float16* dst, int lo_off, float x, float y) {
  const h2 a = __builtin_convertvector((fl2{x, y}), h2);
  const h2 c = __builtin_convertvector((fl2{x - (float)a[0], y - (float)a[1]}), h2);
  *reinterpret_cast<h2*>(dst) = a;
  *reinterpret_cast<h2*>(dst + lo_off) = c;
}
__device__ inline void split_store1(_Float16* dst, int lo_off, float x) {
  const _Float16 a = (_Float16)x;
  dst[0] = a;
  dst[lo_off] = (_Float16)(x - (float)a);
}

// The exponent e with x < 2^e for finite x >= 0 given as float bits (129 for
// an infinity or a NaN, -126 for 0).
__device__ inline int split_exp(unsigned bits) { return (int)((bits >> 23) & 255u) - 126; }
// Power-of-two scale that takes values below 2^e to below 2^kTargetExp, and
// its inverse; e is held inside a range where both are normal numbers.
__device__ inline int split_clamp_exp(int e) { return min(max(e, -100), 126); }
__device__ inline float split_scale(int e) {
  return __uint_as_float((unsigned)(127 + kTargetExp - e) << 23);
}
__device__ inline float split_unscale(int e) {
  return __uint_as_float((unsigned)(127 - kTargetExp + e) << 23);
}
// Largest |v| of a row, gathered by every wave of the workgroup.
__device__ inline void split_track(unsigned* m, const f4& v) {
  const float a = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
  atomicMax(m, __float_as_uint(a));
}

// Forward weights and biases are stored multiplied by 2/ln 2, so a forward
// product yields y = 2 z / ln 2 and exp(2z) = 2^y takes no multiply.
constexpr float kTanhPrescale = 2.8853900817779268f;
constexpr float kTanhPrescaleLow = 3.8519260e-8f;   // 2/ln 2 less that float

// ln 2 / 2: undoes the forward pre-scale where no bias is added (tangents)
constexpr float kTanhUnscale = 0.34657359027997264f;

// tanh and its derivative from one exponential and one reciprocal, given the
// pre-scaled pre-activation y: with e = 2^-|y| <= 1, r = 1 / (1 + e) and
// s = e r, |tanh z| = r - s and tanh' = 4 s (1 - s).  s keeps its relative
// precision as the unit saturates, and so does tanh'; 1 - tanh^2 carries tanh's
// rounding.  TANH_ONLY (the training sweeps, which form tanh' from tanh again):
// |tanh z| = 1 - 2 s from |z| = 0.55 on (e = 1/3), which leaves the reciprocal's
// rounding out; below it r - s is the more precise.  y of any size and either
// infinity saturate, a NaN stays one.  |z| from 6 to 14, largest errors: tanh'
// 1e-11, in the training sweeps 6e-8 (3e-7 as 1 - h^2 with
// h = (e^2z - 1) / (e^2z + 1)).
template <bool TANH_ONLY = false>
__device__ inline float tanh_and_grad(float y, float& d) {
  const float e = __builtin_amdgcn_exp2f(-__builtin_fabsf(y));
  const float r = __builtin_amdgcn_rcpf(1.f + e);
  const float s = e * r;
  float h = __builtin_fmaf(-e, r, r);
  if constexpr (TANH_ONLY) {
    h = e > 1.f / 3.f ? h : __builtin_fmaf(-2.f, s, 1.f);
    d = __builtin_fmaf(-h, h, 1.f);
  } else {
    const float s4 = 4.f * s;
    d = __builtin_fmaf(-s4, s, s4);
  }
  return __builtin_copysignf(h, y);
}

// The raw CVs' part of layer 1 on FP32 MFMA, acc += W x over the CVs in sets of
// 16 (those that hold a raw one): weights in FP32 fragments, lane l holding unit
// l % 16 and CVs 4 (l / 16) .. + 3 of the set, zero for angular CVs; x(rt, i) is
// the lane's walker's values of CVs i .. i + 3 in row tile rt (whatever stands
// past the last CV is not used).  What bounds it is the loads of x: every wave
// reads the tile's 16 rows, 16 bytes a lane (as four loads a lane 38 raw CVs cost
// 3.0 us instead of 1.3).  1000 walkers of 4 x [256 x 4]: 27.0 us without, 27.8
// with 12 of 38 CVs raw, 28.3 with all (36.2 when every product ran on FP32
// MFMA); 300 walkers, 200 raw CVs, 4 x [512 x 4]: 91 and 101 (135).
struct RawSrc {
  __amdgpu_buffer_rsrc_t r;   // one member's fragments
  unsigned sets;              // bit t: set t holds a raw CV
  int n_sets, n;
};
template <int RT, int CT, class X>
__device__ inline void raw_gemm(f4 (&acc)[RT][CT], const RawSrc& s, int jt0, int lane, X&& x) {
  for (unsigned m = s.sets; m; m &= m - 1) {
    const int t = __builtin_ctz(m), i = 16 * t + 4 * (lane >> 4);
    f4 w[CT], v[RT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
      w[c] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(
                                        s.r, lane * 16, ((jt0 + c) * s.n_sets + t) * 1024, 0));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) v[rt] = x(rt, i);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float ve = i + e < s.n ? v[rt][e] : 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c)
          acc[rt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][e], ve, acc[rt][c], 0, 0, 0);
      }
  }
}
// A raw CV's value; an infinity becomes a number large enough to saturate
// (padded units have zero weights, and 0 inf is a NaN).
__device__ inline float raw_value(float s) {
  return __builtin_isinf(s) ? __builtin_copysignf(1e30f, s) : s;
}
__device__ inline f4 raw_value(f4 s) {
  return f4{raw_value(s[0]), raw_value(s[1]), raw_value(s[2]), raw_value(s[3])};
}

// Block -> (member, tile), XCD-aware: when K divides 8 (grp = 8 / K), member
// k runs on XCDs {k grp, ...}, so each XCD's L2 holds only its members'
// weights.
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

}  // namespace dev

// Kernel-side view of an ensemble's split weights (rid_split in the handle).
struct SplitView {
  const unsigned char* frag;          // [2][K][frag_bytes]: the weights rounded two ways
  unsigned long long frag_bytes;
  unsigned fwd_off[kMaxHidden], bwd_off[kMaxHidden];
  const float* bias;                  // [K][L][NP], times 2/ln 2
  const float* rs;                    // [K][L][2][RW] inverse row scales, forward | backward
  const float* bound;                 // [K][L][2][32] largest absolute row sum per unit tile
  const float* wo;                    // [K][NP]
  const float* bo;                    // [K]
  int RW;                             // row stride of rs: max(NP, XP)
  const float* raw_w;                 // raw CVs' FP32 fragments (RawSrc)
  const float* raw_max;               // [K][n] largest |weight| of a raw CV
  unsigned raw_sets;
};

namespace dev {
__device__ inline RawSrc raw_src(const SplitView& w, int k, int NP, int n) {
  const int sets = (n + 15) / 16, floats = NP * 16 * sets;
  return RawSrc{__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w.raw_w + (size_t)k * floats),
                                                  (short)0, 4 * floats, 0x00020000),
                w.raw_sets, sets, n};
}
// Rows [0, rows) of a row-major array as a buffer (range-checked: rows past the
// end read as 0), for the raw CVs' values.
__device__ inline __amdgpu_buffer_rsrc_t row_src(const float* p, int rows, int stride) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, 4 * rows * stride,
                                           0x00020000);
}
__device__ inline f4 row_ld(const __amdgpu_buffer_rsrc_t& r, int offset) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, 4 * offset, 0, 0));
}
}  // namespace dev

}  // namespace rid
