// Selection phase ("Selection"; "SelectorConfig": cluster_threshold,
// numb_cluster_lower / numb_cluster_upper, max_selection): the CV frames
// whose model deviation reaches the lower trust level are clustered with a
// distance threshold, the threshold is adapted until the cluster count lies
// in the window, and one representative per cluster is selected.
//
// Clustering (the paper names a threshold, not the algorithm): frames in
// order; a frame joins the first cluster, in founding order, whose leader is
// within the threshold, otherwise it founds a cluster and leads it.  The
// distance is periodic in every angular CV (differences wrapped to
// (-pi, pi]; raw CVs unwrapped), each square optionally weighted by the CV's
// clustering weight (the CV settings' "weights"), and the decision
// d^2 <= t^2 is taken in FP32 with the squares summed in CV order,
// contraction off, so the labels do not depend on the launch shape.
//
// GPU form of the sequential rule, exact, in rounds over the frames that no
// leader has matched yet (a bit each):
//  * sel_walk_kernel, one workgroup: the first G unmatched frames (a thread
//    and an LDS row each) are walked in order.  The first still unmatched one
//    founds a cluster and all later ones are compared with it at once; then
//    the next one founds, until none is left.
//  * sel_match_kernel, all CUs: every other unmatched frame (all of them come
//    later than the window) is compared with the round's new leaders in
//    founding order, up to the first within the threshold.
// A frame therefore meets all leaders founded before it, in founding order,
// and founds exactly when none is within the threshold.  Frames of known
// clusters leave the mask after one round, so the windows hold mostly frames
// of new ones, and a call takes a few rounds whatever its length.  A founding
// costs one barrier and one distance (about 1 us), a round about 25 us beside
// its foundings; the rounds, not the distances, bound the call.  With
// threshold adjustment, one pass clusters up to kSlots thresholds side by
// side (blockIdx.y = slot, each with its own workspace); select_core.h takes
// the rule's steps over their counts.  20 000 frames of 38 CVs, 24 thresholds, cap 51: a pass took
// 1.67 ms when windows were runs of consecutive frames, 64 to 8192 long,
// matched by the walking workgroup itself, and takes 0.36 ms now (six rounds,
// walks 26-43 us, matches 5-37 us; with two LDS reads per CV and leader and
// without the limit on a round's foundings 0.66 ms).
#include <climits>

#include "device_common.h"
#include "select_core.h"

namespace rid {
namespace {

using namespace dev;

constexpr int kFiltered = -2;      // eps below eps0
constexpr int kOverCap = -1;       // would found a cluster past the cap
constexpr int kWalkThreads = 1024; // frames of a window, at most
constexpr int kWalkWaves = kWalkThreads / kWave;
constexpr size_t kTileBytes = 144 * 1024;   // LDS for the frames' CVs
constexpr int kMatchWaves = 4;     // 64-frame words per workgroup, at most
constexpr int kLeadRows = 16;      // leaders staged in LDS at a time
constexpr int kSlots = 24;         // thresholds clustered side by side in one pass
static_assert(kSlots <= selcore::kMaxSlots, "slot count");

struct ClusterArgs {
  const float* s;        // [B][n] frames
  const float* eps;      // [B] or null (no filter)
  float eps0, t2;
  int B, n, cap, words;
  float* LR;             // [cap][n] leaders' CVs
  int* leader;           // [cap] frame index of each leader
  int* state;            // kState* below
  int* labels;           // [B]
  unsigned long long* pend;   // [ceil(B/64)] bit f%64 of word f/64: frame f unmatched
  const uint8_t* raw;    // [n] or null: CVs with raw[i] = 1 are not periodic
  const float* w;        // [n] or null: per-CV weights of the squared differences
};
enum {
  kLeaders = 0,          // leaders so far
  kDone = 1,             // 1: every frame is labelled once this round ends
  kOver = 2,             // some frame would have founded past the cap
  kNew = 3,              // first leader of the current round
  kWord = 4,             // mask words before this one are empty
  kStateInts = 8         // ints of state per slot
};
constexpr int kAbandoned = 2;      // kDone: more leaders than the window allows

// Thresholds clustered in one pass: slot k (blockIdx.y) clusters at t2[k]
// into its own workspace, the pointers above advanced by k strides.
struct ClusterSlots {
  float t2[kSlots];
  long long sLR, sLabels;   // floats of LR, ints of labels per slot (labels: 0 with one slot)
  int sLeader, sPend;       // ints of leader, words of pend per slot
};

__device__ inline ClusterArgs slot_args(const ClusterArgs& a0, const ClusterSlots& sl) {
  const int k = blockIdx.y;
  ClusterArgs a = a0;
  a.t2 = sl.t2[k];
  a.LR += k * sl.sLR;
  a.labels += k * sl.sLabels;
  a.leader += k * sl.sLeader;
  a.pend += (size_t)k * sl.sPend;
  a.state += k * kStateInts;
  return a;
}

// Whether a leader lies within t2 of the lane's frame: FP32, differences
// wrapped to (-pi, pi] unless raw[i], squares weighted by w[i] where w is
// given, summed in CV order, no fused multiply-add.  The wrapped difference
// enters as its magnitude, min(|d|, ||d| - 2 pi|): the same value as
// subtracting or adding 2 pi outside (-pi, pi] (2 pi is twice the FP32 pi, so
// the two meet exactly at |d| = pi), in three operations instead of seven.
// The sum only grows, so a wave stops once no active lane is within t2 (a
// NaN never is).
constexpr float kTwoPi = 6.28318530717959f;
__device__ inline float add_square(float acc, float lead, float x) {
#pragma clang fp contract(off)
  const float d = lead - x;
  const float m = __builtin_fminf(__builtin_fabsf(d), __builtin_fabsf(__builtin_fabsf(d) - kTwoPi));
  const float sq = m * m;
  return acc + sq;
}

// Any CV count and metric, both rows in memory (lead the same for every lane).
__device__ inline bool within_rows(const float* lead, const float* x, const ClusterArgs& a) {
#pragma clang fp contract(off)
  const int n = a.n;
  float acc = 0.f;
  auto add = [&](int i) {
    if (!a.raw && !a.w) {
      acc = add_square(acc, lead[i], x[i]);
      return;
    }
    float d = __builtin_fabsf(lead[i] - x[i]);
    if (!a.raw || !a.raw[i]) d = __builtin_fminf(d, __builtin_fabsf(d - kTwoPi));
    float sq = d * d;
    if (a.w) sq = sq * a.w[i];
    acc = acc + sq;
  };
  int i = 0;
  for (; i + 8 <= n; i += 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) add(i + j);
    if (!__any(acc <= a.t2)) return false;
  }
  for (; i < n; ++i) add(i);
  return acc <= a.t2;
}

// The lane's frame as the comparisons take it.  NV > 0: up to 8 NV CVs of the
// plain metric in registers, zero past the last CV (zero differences add
// nothing), the leader's row read 16 bytes at a time (one LDS access for the
// wave): the row form's two LDS reads a CV bound both kernels.  NV = 0: rows.
typedef float f4 __attribute__((ext_vector_type(4)));
template <int NV>
struct FrameCv {
  float x[8 * NV];
  __device__ inline void load(const float* row) {
#pragma unroll
    for (int i = 0; i < 2 * NV; ++i) {
      const f4 v = *reinterpret_cast<const f4*>(row + 4 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * i + j] = v[j];
    }
  }
  __device__ inline bool within(const float* lead, const ClusterArgs& a) const {
    float acc = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const f4 l0 = *reinterpret_cast<const f4*>(lead + 8 * v);
      const f4 l1 = *reinterpret_cast<const f4*>(lead + 8 * v + 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = add_square(acc, l0[j], x[8 * v + j]);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = add_square(acc, l1[j], x[8 * v + 4 + j]);
      if (v + 1 < NV && !__any(acc <= a.t2)) return false;
    }
    return acc <= a.t2;
  }
};
template <>
struct FrameCv<0> {
  const float* row;
  __device__ inline void load(const float* r) { row = r; }
  __device__ inline bool within(const float* lead, const ClusterArgs& a) const {
    return within_rows(lead, row, a);
  }
};
// Row stride (floats) of a frame in LDS.  NV = 0: odd, so that lanes on
// consecutive rows fall into different banks.
__host__ __device__ inline int frame_stride(int n, int NV) { return NV ? 8 * NV : n | 1; }

// The mask of the kept frames, the labels of the others, the state.
__global__ __launch_bounds__(256) void sel_init_kernel(ClusterArgs a0, ClusterSlots sl) {
  const ClusterArgs a = slot_args(a0, sl);
  const int lane = threadIdx.x % kWave;
  const int w = blockIdx.x * 4 + threadIdx.x / kWave;
  if (blockIdx.x == 0 && threadIdx.x < kStateInts) a.state[threadIdx.x] = 0;
  if (w >= a.words) return;
  const int f = w * 64 + lane;
  const bool in = f < a.B;
  const bool keep = in && (!a.eps || a.eps[f] >= a.eps0);
  const unsigned long long m = __ballot(keep);
  if (lane == 0) a.pend[w] = m;
  if (in && !keep) a.labels[f] = kFiltered;
}

// One round's walk (see the head of the file), at most max_new foundings:
// the frames still unmatched then go back into the mask.  A slot with more
// than `enough` leaders is abandoned (done, its labels incomplete).  LDS: the
// window's frames [G][stride], their indices [G].
template <int NV>
__global__ __launch_bounds__(kWalkThreads) void sel_walk_kernel(ClusterArgs a0, ClusterSlots sl,
                                                                int G, int max_new, int enough) {
  const ClusterArgs a = slot_args(a0, sl);
  extern __shared__ __attribute__((aligned(16))) float tile[];
  __shared__ int wsum[kWalkWaves], firsts[2][kWalkWaves];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int n = a.n, st = frame_stride(n, NV);
  int* list = reinterpret_cast<int*>(tile + (size_t)G * st);
  const int n_start = a.state[kLeaders];
  if (a.state[kDone]) {
    if (tid == 0) a.state[kNew] = n_start;
    return;
  }
  // the first G unmatched frames: a thread per mask word, ranks by a prefix
  // sum; words are cleared of the bits taken
  int g = 0, w0 = a.state[kWord];
  bool rest = false;                        // unmatched frames beyond the window
  for (; w0 < a.words && !rest; w0 += kWalkThreads) {
    const int w = w0 + tid;
    unsigned long long m = w < a.words ? a.pend[w] : 0ull;
    const int cnt = __popcll(m);
    int scan = cnt;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int v = __shfl_up(scan, o);
      if (lane >= o) scan += v;
    }
    if (lane == kWave - 1) wsum[wave] = scan;
    __syncthreads();
    int base = g, tot = 0;
    for (int q = 0; q < kWalkWaves; ++q) {
      if (q < wave) base += wsum[q];
      tot += wsum[q];
    }
    int rank = base + scan - cnt;
    const unsigned long long m0 = m;
    for (; m && rank < G; ++rank) {
      const int b = __ffsll((long long)m) - 1;
      m &= m - 1;
      list[rank] = w * 64 + b;
    }
    if (m != m0) a.pend[w] = m;
    g = min(G, g + tot);
    // everything up to here is taken unless the window is full
    rest = __syncthreads_or(m != 0ull);
  }
  // (the last batch may hold words with bits left: the next round starts there)
  const int w_next = rest ? w0 - kWalkThreads : a.words;
  // a full window may leave whole words unread behind it
  const bool last = !rest && w0 >= a.words;
  // the window's CVs, kBatch loads in flight per thread (element e = q n + i
  // stepped by the thread count without divisions; past the end, q is clamped
  // to the last frame and the value is not stored)
  constexpr int kBatch = 16;
  const int tot = g * n, dq = kWalkThreads / n, di = kWalkThreads % n;
  for (int e0 = 0; e0 < tot; e0 += kBatch * kWalkThreads) {
    int q = (e0 + tid) / n, i = (e0 + tid) - q * n;
    float v[kBatch];
    int o[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      v[j] = a.s[(size_t)list[min(q, g - 1)] * n + i];
      o[j] = q < g ? q * st + i : -1;
      q += dq;
      i += di;
      if (i >= n) {
        i -= n;
        ++q;
      }
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (o[j] >= 0) tile[o[j]] = v[j];
  }
  if (NV > 0)
    for (int e = tid; e < g * (st - n); e += kWalkThreads)
      tile[(size_t)(e / (st - n)) * st + n + e % (st - n)] = 0.f;
  __syncthreads();
  // the ordered walk
  FrameCv<NV> fr;
  fr.load(tile + (size_t)min(tid, max(g - 1, 0)) * st);
  int label = tid < g ? -2 : 0;             // -2: not matched yet
  int n_new = 0, over = 0;
  for (int it = 0;; ++it) {
    const unsigned long long m = __ballot(label == -2);
    if (lane == 0)
      firsts[it & 1][wave] = m ? wave * kWave + __ffsll((long long)m) - 1 : kWalkThreads;
    __syncthreads();
    int first = kWalkThreads;
#pragma unroll
    for (int q = 0; q < kWalkWaves; ++q) first = min(first, firsts[it & 1][q]);
    if (first == kWalkThreads) break;
    const int out = n_start + n_new;
    if (out >= a.cap) {                     // no room: what is left is over the cap
      if (label == -2) label = kOverCap;
      over = 1;
      break;
    }
    const float* xl = tile + (size_t)first * st;
    for (int i = tid; i < n; i += kWalkThreads) a.LR[(size_t)out * n + i] = xl[i];
    if (tid == first) {
      label = out;
      a.leader[out] = list[first];
    }
    if (label == -2 && fr.within(xl, a)) label = out;
    if (++n_new == max_new) break;
  }
  // (the mask words of the window were stored before the barriers above)
  const bool back = tid < g && label == -2;
  if (back) atomicOr(&a.pend[list[tid] >> 6], 1ull << (list[tid] & 63));
  else if (tid < g) a.labels[list[tid]] = label;
  const bool all = !__syncthreads_or(back);
  if (tid == 0) {
    a.state[kLeaders] = n_start + n_new;
    a.state[kNew] = n_start;
    a.state[kWord] = all ? w_next : list[0] >> 6;
    if (over) a.state[kOver] = 1;
    // a full cap: the match kernel of this round labels every frame left
    const int now = n_start + n_new;
    a.state[kDone] = now > enough ? kAbandoned : (last && all) || now >= a.cap;
  }
}

// One round's matching: a wave per mask word, a lane per frame, the round's
// leaders staged in LDS kLeadRows at a time.  LDS: leaders
// [kLeadRows][stride], then each wave's frames [64][stride].
template <int NV>
__global__ __launch_bounds__(kMatchWaves * kWave) void sel_match_kernel(ClusterArgs a0,
                                                                        ClusterSlots sl) {
  const ClusterArgs a = slot_args(a0, sl);
  extern __shared__ __attribute__((aligned(16))) float tile[];
  const int nt = blockDim.x, tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = a.n, st = frame_stride(n, NV);
  const int w = blockIdx.x * (nt / kWave) + wave;
  const int l0 = a.state[kNew], l1 = a.state[kLeaders];
  if (a.state[kDone] == kAbandoned) return;
  const bool full = l1 >= a.cap;
  const unsigned long long m0 = w < a.words ? a.pend[w] : 0ull;
  if (!__syncthreads_or(m0 != 0ull && (l1 > l0 || full))) return;
  float* lead = tile;
  float* fr = tile + (size_t)(kLeadRows + wave * kWave) * st;
  // the word's frames: all 64 rows are one stretch of memory (rows past B are
  // not read), eight loads in flight per lane
  if (m0 && l1 > l0) {
    const int rows = min(64, a.B - w * 64), tot = rows * n;
    const float* src = a.s + (size_t)w * 64 * n;
    const int dq = kWave / n, di = kWave % n;
    for (int e0 = 0; e0 < tot; e0 += 8 * kWave) {
      int q = (e0 + lane) / n, i = (e0 + lane) - q * n;
      float v[8];
      int o[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int e = e0 + j * kWave + lane;
        v[j] = src[min(e, tot - 1)];
        o[j] = e < tot ? q * st + i : -1;
        q += dq;
        i += di;
        if (i >= n) {
          i -= n;
          ++q;
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (o[j] >= 0) fr[o[j]] = v[j];
    }
  }
  if (NV > 0 && m0 && l1 > l0)
    for (int e = lane; e < kWave * (st - n); e += kWave)
      fr[(e / (st - n)) * st + n + e % (st - n)] = 0.f;
  bool open = (m0 >> lane) & 1ull;
  int label = kOverCap;
  FrameCv<NV> x;
  for (int j0 = l0; j0 < l1; j0 += kLeadRows) {
    const int rows = min(kLeadRows, l1 - j0);
    __syncthreads();                         // the frames, and the last leaders' readers
    for (int e = tid; e < rows * st; e += nt) {
      const int r = e / st, i = e - r * st;
      lead[e] = i < n ? a.LR[(size_t)(j0 + r) * n + i] : 0.f;
    }
    if (j0 == l0) x.load(fr + lane * st);
    __syncthreads();
    for (int j = 0; j < rows; ++j)
      if (open && x.within(lead + j * st, a)) {
        label = j0 + j;
        open = false;
      }
  }
  const unsigned long long left = __ballot(open);
  const int f = w * 64 + lane;
  if (((m0 >> lane) & 1ull) && (!open || full)) a.labels[f] = label;
  if (lane == 0 && m0) {
    a.pend[w] = full ? 0ull : left;
    if (full && left) a.state[kOver] = 1;
  }
}

// Frames of a walk's window.
int walk_frames(int n, int NV) {
  const int g = (int)(kTileBytes / (sizeof(float) * frame_stride(n, NV) + sizeof(int)));
  return std::min(kWalkThreads, g / kWave * kWave);
}
size_t walk_lds(int n, int NV, int G) {
  return (size_t)G * (sizeof(float) * frame_stride(n, NV) + sizeof(int));
}
size_t match_lds(int n, int NV, int waves) {
  return sizeof(float) * (size_t)(kLeadRows + waves * kWave) * frame_stride(n, NV);
}

// Device memory of one clustering call (one allocation): `slots` copies of
// the per-pass buffers (labels only with more than one slot; one slot
// writes the caller's).
struct ClusterWs {
  void* buf = nullptr;
  ~ClusterWs() {
    if (buf) (void)hipFree(buf);
  }
};

// One clustering pass at thresholds t[0..T) side by side (slot k at t[k]);
// synchronises the stream.  On return st_h[k * kStateInts ...] is the state of
// slot k.  enough: slots with more leaders are abandoned.  Rounds are launched
// kRounds at a time: the first ones take most calls to the end, and a look at
// the state costs more than two idle rounds.
constexpr int kRounds = 8;
template <int NV>
rid_status cluster_pass_nv(const ClusterArgs& a, const ClusterSlots& sl, int T, int enough,
                           hipStream_t st, int* st_h) {
  const int G = walk_frames(a.n, NV);
  const size_t wlds = walk_lds(a.n, NV, G);
  int mw = kMatchWaves;
  while (match_lds(a.n, NV, mw) > 150 * 1024) --mw;
  const size_t mlds = match_lds(a.n, NV, mw);
  static size_t attr[2] = {0, 0};
  if (wlds > 64 * 1024 && wlds > attr[0]) {
    RID_HIP(hipFuncSetAttribute((const void*)sel_walk_kernel<NV>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)wlds));
    attr[0] = wlds;
  }
  if (mlds > 64 * 1024 && mlds > attr[1]) {
    RID_HIP(hipFuncSetAttribute((const void*)sel_match_kernel<NV>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)mlds));
    attr[1] = mlds;
  }
  // side by side, a round lasts as long as its slot with the most foundings:
  // a quarter of the cap each (the slots with few need several rounds anyway)
  const int max_new = T > 1 ? std::max(16, (a.cap + 3) / 4) : kWalkThreads;
  // a round labels a whole window or founds max_new clusters
  const long long most = (a.B + G - 1) / G + a.cap / max_new + 1;
  for (long long r = 0; r < most;) {
    for (int i = 0; i < kRounds && r < most; ++i, ++r) {
      hipLaunchKernelGGL(sel_walk_kernel<NV>, dim3(1, T), dim3(kWalkThreads), (uint32_t)wlds, st, a,
                         sl, G, max_new, enough);
      RID_HIP(hipGetLastError());
      hipLaunchKernelGGL(sel_match_kernel<NV>, dim3((a.words + mw - 1) / mw, T), dim3(mw * kWave),
                         (uint32_t)mlds, st, a, sl);
      RID_HIP(hipGetLastError());
    }
    RID_HIP(hipMemcpyAsync(st_h, a.state, sizeof(int) * kStateInts * T, hipMemcpyDeviceToHost, st));
    RID_HIP(hipStreamSynchronize(st));
    bool done = true;
    for (int k = 0; k < T; ++k) done = done && st_h[k * kStateInts + kDone];
    if (done) break;
  }
  return RID_OK;
}

rid_status cluster_pass(const ClusterArgs& a, ClusterSlots sl, const float* t, int T, int enough,
                        hipStream_t st, int* st_h) {
  for (int k = 0; k < T; ++k) sl.t2[k] = t[k] * t[k];
  hipLaunchKernelGGL(sel_init_kernel, dim3((a.words + 3) / 4, T), dim3(256), 0, st, a, sl);
  RID_HIP(hipGetLastError());
  // registers hold up to 64 CVs of the plain metric
  if (a.raw || a.w || a.n > 64) return cluster_pass_nv<0>(a, sl, T, enough, st, st_h);
  if (a.n <= 16) return cluster_pass_nv<2>(a, sl, T, enough, st, st_h);
  if (a.n <= 40) return cluster_pass_nv<5>(a, sl, T, enough, st, st_h);
  return cluster_pass_nv<8>(a, sl, T, enough, st, st_h);
}

}  // namespace

rid_status launch_cluster(const float* s, int B, int n, const uint8_t* raw, const float* w,
                          const float* eps,
                          float eps0, float threshold, int lower, int upper, int adapt, int cap,
                          int* labels, int* leaders, int leaders_out, int* n_leaders,
                          int* n_clusters, float* t_used, hipStream_t st) {
  const int words = (B + 63) / 64;
  // slots: one without adaptation; with it as many as fit in 256 MiB, at most kSlots
  const size_t per_slot = sizeof(float) * (size_t)n * cap + sizeof(int) * (size_t)cap +
                          sizeof(int) * (size_t)B + sizeof(unsigned long long) * words +
                          sizeof(int) * 4;
  const int T = adapt ? (int)std::max<size_t>(1, std::min<size_t>(kSlots, (256u << 20) / per_slot))
                      : 1;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t b_lr = al(sizeof(float) * (size_t)n * cap * T), b_ld = al(sizeof(int) * (size_t)cap * T),
               b_st = al(sizeof(int) * kStateInts * T),
               b_pd = al(sizeof(unsigned long long) * (size_t)words * T),
               b_lb = T > 1 ? al(sizeof(int) * (size_t)B * T) : 0;
  ClusterWs ws;
  RID_HIP(hipMalloc(&ws.buf, b_lr + b_ld + b_st + b_pd + b_lb));
  unsigned char* wp = static_cast<unsigned char*>(ws.buf);
  float* ws_LR = reinterpret_cast<float*>(wp);
  int* ws_leader = reinterpret_cast<int*>(wp + b_lr);
  int* ws_state = reinterpret_cast<int*>(wp + b_lr + b_ld);
  unsigned long long* ws_pend = reinterpret_cast<unsigned long long*>(wp + b_lr + b_ld + b_st);
  int* ws_labels = T > 1 ? reinterpret_cast<int*>(wp + b_lr + b_ld + b_st + b_pd) : nullptr;
  ClusterArgs a{};
  a.s = s;
  a.raw = raw;
  a.w = w;
  a.eps = eps;
  a.eps0 = eps0;
  a.B = B;
  a.n = n;
  a.cap = cap;
  a.words = words;
  a.LR = ws_LR;
  a.leader = ws_leader;
  a.state = ws_state;
  a.labels = T > 1 ? ws_labels : labels;
  a.pend = ws_pend;
  ClusterSlots sl{};
  sl.sLR = (long long)n * cap;
  sl.sLabels = T > 1 ? B : 0;
  sl.sLeader = cap;
  sl.sPend = words;
  // threshold adjustment (first iteration of the workflow), T thresholds
  // per pass (select_core.h)
  std::vector<int> st_h((size_t)kStateInts * T);
  auto pass = [&](const float* ts, int nts, int* counts) -> int {
    // a slot past the window needs its count no further: the rule goes on
    const int enough = nts > 1 ? upper : INT_MAX;
    const rid_status r = cluster_pass(a, sl, ts, nts, enough, st, st_h.data());
    if (r != RID_OK) return r;
    for (int j = 0; j < nts; ++j) {
      const int* sj = st_h.data() + (size_t)j * kStateInts;
      counts[j] = !sj[kDone] ? -1 : sj[kLeaders] + (sj[kOver] ? 1 : 0);
    }
    return 0;
  };
  selcore::Outcome res;
  const int rr = selcore::adjust_threshold(threshold, lower, upper, adapt != 0, T, pass, res);
  if (rr == selcore::kIncomplete)
    return fail(RID_EDEVICE, "clustering did not reach the last frame");
  if (rr != 0) return (rid_status)rr;
  int k = res.slot, count = res.count;
  const float t = res.t;
  if (st_h[(size_t)k * kStateInts + kDone] == kAbandoned) {
    // the rule ran out of adjustments on a slot past the window: cluster its
    // threshold alone, to the end
    k = 0;
    const rid_status r = cluster_pass(a, sl, &t, 1, INT_MAX, st, st_h.data());
    if (r != RID_OK) return r;
    if (!st_h[kDone]) return fail(RID_EDEVICE, "clustering did not reach the last frame");
    count = st_h[kLeaders] + (st_h[kOver] ? 1 : 0);
  }
  const int* sk = st_h.data() + (size_t)k * kStateInts;
  if (T > 1)
    RID_HIP(hipMemcpyAsync(labels, ws_labels + (size_t)k * B, sizeof(int) * (size_t)B,
                           hipMemcpyDeviceToDevice, st));
  const int nl = std::min(sk[kLeaders], leaders_out);
  if (leaders && nl > 0)
    RID_HIP(hipMemcpyAsync(leaders, ws_leader + (size_t)k * cap, sizeof(int) * (size_t)nl,
                           hipMemcpyDeviceToDevice, st));
  RID_HIP(hipStreamSynchronize(st));
  if (n_leaders) *n_leaders = nl;
  *n_clusters = count;
  if (t_used) *t_used = t;
  return RID_OK;
}

}  // namespace rid
