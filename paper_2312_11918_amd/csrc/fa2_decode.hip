// Attention of ONE query per sequence (a decoding step), gfx950.
//
// With a single query row the work is reading K and V once: 4 d bytes and 4 d FLOP per key.  The 128-row tile kernel
// spends a workgroup's LDS staging, barriers and MFMAs on one live row, and its grid is B*H workgroups, which leaves
// most of the chip idle for a small batch.  Here nothing is staged: a group of d/8 lanes owns a key, every lane loads
// 16 bytes of its row straight into registers (a wavefront instruction reads 1 KiB), dots them with its piece of q in
// fp32, and the group's lanes add up with DPP.  The same lanes then hold 8 columns of O and load V in the same way.
// P stays in fp32.  About 22 vector instructions per 2 KiB of K and V, a third of what the vector pipes could issue
// while HBM delivers them: the bound is HBM, so what counts is bytes in flight and all CUs reading.  B16 H16 Nk2048
// d128: 57 us in the tile kernel, 41 here (6.5 TB/s); B1 H32 Nk16001 d64: 181 and 27 (4.9 TB/s).
//
//  * every lane group keeps its own running maximum, row sum and piece of O over the keys it sees; they are merged
//    once at the end, within the wavefront by lane exchanges, between wavefronts through LDS;
//  * K of the next step is requested as soon as this step's dot products have consumed K, V of the next once this step's
//    sums have consumed V; a step of the loop ends with both landed (the compiler waits for all loads before it moves them
//    into the registers of the next step), so what hides their latency is the CU's other wavefronts;
//  * the keys of a head are split over `splits` workgroups when B*H workgroups do not fill the CUs.  Partial
//    (O, maximum, sum) then go to the caller's workspace in fp32 and a second kernel merges them.
#include "fa2_internal.h"

namespace fa2 {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr float kLn2 = 0.69314718055994530942f;
constexpr float kNoKey = -3.402823466e38f;   // reference point of a part that has seen no key: the lowest finite number
constexpr int kMaxWaves = 8;   // wavefronts per workgroup
constexpr int kFewSplits = 16;       // most splits that the merge adds up with one thread per column
constexpr int kMergeThreads = 256;   // threads of a workgroup of the merge, with more splits
constexpr int kUnroll = 4;     // keys per lane group and step (8: 1...7 % slower, 2: 0...5 % slower)

// element i of eight 16-bit elements as fp32
template <int DT> __device__ __forceinline__ float elem(u32x4 x, int i) {
  if constexpr (DT == FA2_FP16) {
    return (float)__builtin_bit_cast(f16x8, x)[i];
  } else {
    return __builtin_bit_cast(float, (i & 1) ? (x[i / 2] & 0xffff0000u) : (x[i / 2] << 16));
  }
}

template <int DT> __device__ __forceinline__ uint16_t round16(float x) {
  if constexpr (DT == FA2_FP16) return __builtin_bit_cast(uint16_t, (_Float16)x);
  else return __builtin_bit_cast(uint16_t, (__bf16)x);
}

template <int kCtrl> __device__ __forceinline__ float dpp(float x) {
  const int u = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(u, u, kCtrl, 0xf, 0xf, true));
}

// Sum over the G lanes (8, 16 or 32, aligned) that share a key, in every one of them.
template <int G> __device__ __forceinline__ float group_sum(float x) {
  x += dpp<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);    // quad_perm [2,3,0,1]
  x += dpp<0x141>(x);   // row_half_mirror: the other quad of eight lanes
  if constexpr (G >= 16) x += dpp<0x140>(x);   // row_mirror: the other eight lanes of sixteen
  if constexpr (G >= 32) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // the other sixteen of 32 lanes
    x = __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
  }
  return x;
}

// exp2(a - b) for two reference points, b the larger: exactly 1 where they are equal, so the difference must not be
// contracted with the product that one of them came from (see the reference points in the kernel).  A part that saw no key has
// kNoKey: its weight is 0 beside any other.
__device__ __forceinline__ float weight(float a, float b) {
#pragma clang fp contract(off)
  return __builtin_amdgcn_exp2f(a - b);
}

// Workgroup (b, split, h), the head running fastest so that workgroups started together read neighbouring addresses.
// Its keys [split * chunk, min(Nk, (split + 1) * chunk)) are dealt to the wavefronts kUnroll * 64 / G at a time.
// Reference points and exponents are in units of log2 (scaled logits times log2 e).
template <int DT, int D, bool kSplit>
__global__ __launch_bounds__(kMaxWaves * 64) void fa2_decode_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ LSE, float* __restrict__ part_o, float* __restrict__ part_ml, int H,
    int Nk, float scale_log2e, int splits, int chunk) {
  constexpr int G = D / 8;             // lanes per key
  constexpr int kKeys = 64 / G;        // keys per wavefront load
  constexpr int kStep = kKeys * kUnroll;   // keys per wavefront and step
  __shared__ float o_lds[kMaxWaves][D];
  __shared__ float m_lds[kMaxWaves], l_lds[kMaxWaves];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
  const int h = blockIdx.x % H, bs = blockIdx.x / H;
  const int split = kSplit ? bs % splits : 0, b = kSplit ? bs / splits : bs;
  const int first = split * chunk, last = min(Nk, first + chunk) - 1;   // every split holds a key
  const int group = lane / G, piece = lane % G;

  const size_t head = (size_t)h * D;
  const uint16_t* kp = K + (size_t)b * Nk * H * D + head;   // one batch entry spans less than 4 GiB
  const uint16_t* vp = V + (size_t)b * Nk * H * D + head;
  const uint32_t row_bytes = (uint32_t)H * D * 2u;
  // 16 bytes of row `key` (clamped into the split: rows past it are loaded as copies and masked).  K and V are read once:
  // as non-temporal loads they are 7...13 % faster than as plain ones (47.3 against 52.0 us at B8 H16 Nk4096 d128,
  // 27.8 against 31.2 at B1 H32 Nk16001 d64).
  auto row = [&](const uint16_t* base, int key) __attribute__((always_inline)) {
    const uint32_t off = (uint32_t)min(key, last) * row_bytes + 16u * (uint32_t)piece;
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + off));
  };

  float q[8];
  {
    const u32x4 x = *reinterpret_cast<const u32x4*>(Q + ((size_t)b * H + h) * D + 8 * piece);
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = elem<DT>(x, i);
  }
  // m is the maximum of the unscaled logits, mc the reference point of the exponentials: m times the scale, rounded to fp32.
  // Everything is held relative to the ROUNDED product: its rounding error cancels between P, O and l, and a step that
  // does not raise the maximum rescales by exactly 1.  (Rescaled against the unrounded product, O and l picked up the
  // same factor 2^(rounding error) on every step: LSE off by 8e-4 after 256 steps at logits around 1000.)
  float o[8], m = -INFINITY, mc = kNoKey, l = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = 0.f;

  u32x4 kx[kUnroll], vx[kUnroll];
  int key0 = first + wave * kStep + group;   // this group's first key of the step
  const int stride = waves * kStep;
  if (key0 - group <= last) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) kx[u] = row(kp, key0 + u * kKeys);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) vx[u] = row(vp, key0 + u * kKeys);
  }
  for (; key0 - group <= last; key0 += stride) {
    const bool more = key0 - group + stride <= last;   // the same in all lanes (but held per lane)
    float s[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      s[u] = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) s[u] = __builtin_fmaf(elem<DT>(kx[u], i), q[i], s[u]);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) kx[u] = row(kp, key0 + stride + u * kKeys);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      s[u] = group_sum<G>(s[u]);
      if (key0 + u * kKeys > last) s[u] = -INFINITY;
    }
    float m_new = m;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) m_new = fmaxf(m_new, s[u]);
    // A group that has seen no key yet keeps m = -inf and kNoKey: the exponentials of its masked keys are 0 against it.  So
    // are those of logits that overflow once scaled (keys masked by the caller with the lowest value of the type).
    const float mc_new = fmaxf(m_new * scale_log2e, kNoKey);
    const float alpha = weight(mc, mc_new);
    m = m_new;
    mc = mc_new;
    l *= alpha;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] *= alpha;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u], scale_log2e, -mc));
      l += p;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = __builtin_fmaf(elem<DT>(vx[u], i), p, o[i]);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) vx[u] = row(vp, key0 + stride + u * kKeys);
    }
  }

  // merge the lane groups of the wavefront
  float m_all = mc;
#pragma unroll
  for (int x = G; x < 64; x *= 2) m_all = fmaxf(m_all, __shfl_xor(m_all, x));
  const float w = weight(mc, m_all);
  l *= w;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] *= w;
#pragma unroll
  for (int x = G; x < 64; x *= 2) {
    l += __shfl_xor(l, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] += __shfl_xor(o[i], x);
  }
  if (lane < G) {
#pragma unroll
    for (int i = 0; i < 8; ++i) o_lds[wave][8 * piece + i] = o[i];
    if (lane == 0) {
      m_lds[wave] = m_all;
      l_lds[wave] = l;
    }
  }
  __syncthreads();
  // merge the wavefronts, thread t column t (+ the thread count: a single wavefront covers d = 128 in two turns)
  float m_wg = -INFINITY, l_wg = 0.f;
  for (int i = 0; i < waves; ++i) m_wg = fmaxf(m_wg, m_lds[i]);
  for (int i = 0; i < waves; ++i) l_wg += weight(m_lds[i], m_wg) * l_lds[i];
  const size_t bh = (size_t)b * H + h;
  for (int c = tid; c < D; c += blockDim.x) {
    float sum = 0.f;
    for (int i = 0; i < waves; ++i) sum += weight(m_lds[i], m_wg) * o_lds[i][c];
    if constexpr (kSplit) part_o[(bh * splits + split) * D + c] = sum;
    else O[bh * D + c] = round16<DT>(sum / l_wg);
  }
  if (tid == 0) {
    if constexpr (kSplit) {
      part_ml[2 * (bh * splits + split)] = m_wg;
      part_ml[2 * (bh * splits + split) + 1] = l_wg;
    } else if (LSE != nullptr) {
      LSE[bh] = m_wg * kLn2 + __builtin_logf(l_wg);
    }
  }
}

// Merge of the splits of one (b, h).  Latency-bound (a few KiB per head).
//  * Up to kFewSplits: thread t is column t, and the loads of a loop over the splits are independent of each other.
//  * More: 16 columns per wavefront, lane t the columns 4 (t % 4) ... + 3 of the splits t / 4, t / 4 + 16, ..., which it merges
//    four at a time, all their loads under way at once; the sixteen lanes of a column are merged at the end.  Up to 16 splits
//    this is the slower one (8 / 10 / 16 splits, d = 64 / 128 / 128: 28.0 / 12.05 / 9.82 us a call, 27.2 / 11.75 / 9.44 by columns).
// Per call, by columns / by lane groups: B1 H2 Nk32768 d128 (128 splits) 18.9 / 11.6 us, B1 H6 Nk3000 d256 (42) 11.8 / 9.2, B1 H6
// Nk32768 d64 (42) 16.4 / 14.1, B3 H2 Nk20000 d256 (42) 27.9 / 25.2, B1 H12 Nk3000 d128 (21) 10.3 / 9.2.
template <int DT, int D>
__global__ __launch_bounds__(kMergeThreads) void fa2_decode_merge_kernel(const float* __restrict__ part_o,
                                                                         const float* __restrict__ part_ml,
                                                                         uint16_t* __restrict__ O, float* __restrict__ LSE,
                                                                         int splits) {
  constexpr int kWavesPerHead = D / 16, kAhead = 4;
  if (splits <= kFewSplits) {
    const size_t bh = blockIdx.x;
    const float* ml = part_ml + 2 * bh * splits;
    const float* po = part_o + bh * splits * D + threadIdx.x;
    float m = -INFINITY;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) m = fmaxf(m, ml[2 * s]);
    float l = 0.f, sum = 0.f;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) {
      const float w = __builtin_amdgcn_exp2f(ml[2 * s] - m);   // reference points are finite (kNoKey at least)
      l += w * ml[2 * s + 1];
      sum += w * po[(size_t)s * D];
    }
    O[bh * D + threadIdx.x] = round16<DT>(sum / l);
    if (LSE != nullptr && threadIdx.x == 0) LSE[bh] = m * kLn2 + __builtin_logf(l);
    return;
  }
  const int lane = threadIdx.x & 63, group = lane >> 2;
  const unsigned wave = blockIdx.x * (kMergeThreads / 64) + (threadIdx.x >> 6);
  const size_t bh = wave / kWavesPerHead;
  const int column = 16 * (wave % kWavesPerHead) + 4 * (lane & 3);
  const float* po = part_o + bh * splits * D + column;
  const f32x2* ml = reinterpret_cast<const f32x2*>(part_ml) + bh * splits;
  float m = kNoKey, l = 0.f;   // reference points are finite (kNoKey at least)
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int s = group; s < splits; s += 16 * kAhead) {
    f32x2 y[kAhead];
    f32x4 x[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int at = min(s + 16 * i, splits - 1);
      y[i] = ml[at];
      x[i] = *reinterpret_cast<const f32x4*>(po + (size_t)at * D);
    }
    float m_new = m;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) m_new = fmaxf(m_new, y[i][0]);
    const float alpha = weight(m, m_new);
    m = m_new;
    l *= alpha;
    o *= alpha;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const float w = s + 16 * i < splits ? weight(y[i][0], m) : 0.f;
      l = __builtin_fmaf(w, y[i][1], l);
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(w, x[i][c], o[c]);
    }
  }
  float m_all = m;
#pragma unroll
  for (int i = 4; i < 64; i *= 2) m_all = fmaxf(m_all, __shfl_xor(m_all, i));
  const float w = weight(m, m_all);
  l *= w;
  o *= w;
#pragma unroll
  for (int i = 4; i < 64; i *= 2) {
    l += __shfl_xor(l, i);
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] += __shfl_xor(o[c], i);
  }
  if (group == 0) {
    uint16_t* out = O + bh * D + column;
    const uint32_t lo = round16<DT>(o[0] / l) | (uint32_t)round16<DT>(o[1] / l) << 16;
    const uint32_t hi = round16<DT>(o[2] / l) | (uint32_t)round16<DT>(o[3] / l) << 16;
    *reinterpret_cast<u32x2*>(out) = u32x2{lo, hi};
    if (LSE != nullptr && column == 0) LSE[bh] = m_all * kLn2 + __builtin_logf(l);
  }
}

struct Plan {
  int waves, splits, chunk;   // wavefronts per workgroup, splits of a head's keys, keys per split
};

// Measured (bf16, K and V from HBM, us): B1 H32 Nk16001 d64 runs in 116 unsplit, 30.3 / 26.6 / 35.4 / 27.9 with 6 / 8 /
// 10 / 16 splits; B3 H12 Nk30000 d64 in 179, 48.1 with 7 splits (252 workgroups) and 65.6 with 8 (288); B16 H16 Nk2048
// d128 in 44.4 unsplit, 47.1 with 2; B12 H24 Nk1500 d128 (288 heads) in 49.7 unsplit, 43.4 / 41.5 / 40.0 with 2 / 3 / 4.
// So: one round of the CUs, as full as the head count allows; if that leaves more than a quarter of the CUs idle, the
// count of up to five rounds whose last one is fullest.  More wavefronts than 8 per workgroup were never faster.
Plan plan_of(int B, int H, int Nk, int d, bool may_split) {
  const int step = kUnroll * 64 / (d / 8);   // keys per wavefront and step
  const long long heads = (long long)B * H;
  Plan p{kMaxWaves, 1, Nk};
  // A head of fewer keys is done (in 14 us at 1024 keys, d = 128) before a second launch pays: the merge costs 4 us on
  // the GPU and as much again on the host.
  if (may_split && heads < 2 * kCUs && (long long)Nk * d >= 128 * 1024) {
    auto rounds = [&](long long s) { return (heads * s + kCUs - 1) / kCUs; };
    long long best = heads < kCUs ? kCUs / heads : 1;
    if (4 * heads * best < 3 * rounds(best) * kCUs) {
      for (long long s = best + 1; heads * s <= 5 * kCUs; ++s)
        if (s * rounds(best) > best * rounds(s)) best = s;   // fuller: s / rounds(s) is larger
    }
    const long long most = Nk / (kMaxWaves * step);   // a step of keys for every wavefront
    if (best > most) best = most;
    if (best > 1) {
      p.chunk = (int)((Nk + best - 1) / best);
      p.splits = (Nk + p.chunk - 1) / p.chunk;
    }
  }
  // At least half of the wavefronts hold a key; the others (130 keys at d = 64: three of eight) merge with weight 0.
  while (p.waves > 1 && (p.waves / 2) * step >= p.chunk) p.waves /= 2;
  // Unsplit heads that fill the CUs read faster as fewer streams: 41.1 against 44.4 us at B16 H16 Nk2048 d128, 33.3
  // against 35.0 at 320 heads of 1000 keys; level (39.9 / 38.7) at 576 heads.  From 2048 heads on four wavefronts
  // also keep the launch's thread count within 32 bits for every problem the tile kernels take.
  const bool few_streams = (heads >= kCUs && heads < 2 * kCUs) || heads >= 8 * kCUs;
  if (few_streams && p.splits == 1 && p.waves > 4) p.waves = 4;
  return p;
}

template <int DT, int D> int launch(const Problem& p, void* workspace, size_t workspace_bytes) {
  const bool room = workspace != nullptr && workspace_bytes >= decode_workspace(p.B, p.H, p.Nk, D);
  const Plan plan = plan_of(p.B, p.H, p.Nk, D, room);
  const uint16_t *q = static_cast<const uint16_t*>(p.Q), *k = static_cast<const uint16_t*>(p.K),
                 *v = static_cast<const uint16_t*>(p.V);
  uint16_t* o = static_cast<uint16_t*>(p.O);
  const int heads = p.B * p.H;
  if (plan.splits == 1)
    return enqueue(fa2_decode_kernel<DT, D, false>, heads, plan.waves * 64, p.stream, q, k, v, o, p.LSE, nullptr, nullptr,
                   p.H, p.Nk, p.scale_log2e, 1, p.Nk);
  float* part_o = static_cast<float*>(workspace);
  float* part_ml = part_o + (size_t)heads * plan.splits * D;
  const int rc = enqueue(fa2_decode_kernel<DT, D, true>, heads * plan.splits, plan.waves * 64, p.stream, q, k, v, o, p.LSE,
                         part_o, part_ml, p.H, p.Nk, p.scale_log2e, plan.splits, plan.chunk);
  if (rc != FA2_OK) return rc;
  const bool few = plan.splits <= kFewSplits;
  return enqueue(fa2_decode_merge_kernel<DT, D>, few ? heads : heads * (D / 16) / (kMergeThreads / 64), few ? D : kMergeThreads,
                 p.stream, part_o, part_ml, o, p.LSE, plan.splits);
}

}  // namespace

bool decode_accepts(int B, int H, int Nq) { return Nq == 1 && (long long)B * H <= 0x7fffffffLL; }

size_t decode_workspace(int B, int H, int Nk, int d) {
  const Plan p = plan_of(B, H, Nk, d, true);
  return p.splits == 1 ? 0 : (size_t)B * H * p.splits * (d + 2) * sizeof(float);
}

int decode(const Problem& p, void* workspace, size_t workspace_bytes) {
  if (p.dtype == FA2_FP16) {
    return p.d == 64    ? launch<FA2_FP16, 64>(p, workspace, workspace_bytes)
           : p.d == 128 ? launch<FA2_FP16, 128>(p, workspace, workspace_bytes)
                        : launch<FA2_FP16, 256>(p, workspace, workspace_bytes);
  }
  return p.d == 64    ? launch<FA2_BF16, 64>(p, workspace, workspace_bytes)
         : p.d == 128 ? launch<FA2_BF16, 128>(p, workspace, workspace_bytes)
                      : launch<FA2_BF16, 256>(p, workspace, workspace_bytes);
}

}  // namespace fa2
