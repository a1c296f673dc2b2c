// Attention whose Q tiles are too few to fill the chip: the keys are split over workgroups as well.
//
// The 128-row tile kernel runs one workgroup per Q tile; a chunk of 512 queries in 16 heads is 64 of them, on 256 CUs that
// hold two each, and a lone workgroup, with one wavefront per SIMD, runs its softmax and its MFMAs one after the other
// (1.0 us per K/V tile at d = 128).  Here the keys of a Q tile are cut into halves inside a workgroup of eight wavefronts
// (d <= 128; 1.3 us per PAIR of tiles), and, where the caller gives a workspace, into slices over workgroups whose partial
// results a second kernel on the same stream merges.  The price is that kernel (5 us) and the partial O in fp32, written
// and read once (64 KiB per workgroup at d = 128).  B1 H16 Nq512 Nk8192 d128: 129 us whole, 41 here; B1 H12 N3088 d128
// causal, in one launch: 64 and 45.  (Fewer query rows than that are fa2_short.hip's: tiles of 32.)
#include "fa2_split_plan.h"
#include "fa2_tile_kernel.h"

namespace fa2 {
namespace {

constexpr float kLn2 = 0.69314718055994530942f;
static_assert(kPlanRows == kBr && 64 == kBc && kSplitMinKeys == FA2_SPLIT_MIN_KEYS, "the tiles and limits that the plan counts in");

// Merge of the slices of one Q tile's 32 rows (those of one wavefront): thread t holds row t % 32 and columns
// 8 (t / 32) ... + 7.  The partial O is read as the tile kernel held it: 32 lanes read 512 consecutive bytes.
template <int DT, int D, bool kCausal>
__global__ __launch_bounds__(4 * D) void fa2_split_merge_kernel(SplitArgs split, uint16_t* __restrict__ O,
                                                                float* __restrict__ LSE, int H, int Nq, int n_qtiles) {
  using E = Elem<DT>;
  const int wave = blockIdx.x % kWaves, tile = blockIdx.x / kWaves;   // wavefront of the Q tile, Q tile over all heads
  const int bh = tile / n_qtiles, qt = tile - bh * n_qtiles;
  // slices that hold keys of this Q tile
  const int n = kCausal ? ((qt + 1) * 2 + split.chunk - 1) / split.chunk : split.slices;
  const int r = threadIdx.x & 31, piece = threadIdx.x >> 5;
  const int row = qt * kBr + wave * 32 + r;
  if (n == 1 || row >= Nq) return;   // (one slice: stored by the tile kernel)
  const size_t slot = (size_t)tile * split.slices;
  const float* ml = split.part_ml + 2 * (slot * kBr + wave * 32 + r);
  const float* po = split.part_o + ((slot * kWaves + wave) * (D / 8) + piece) * 256 + r * 4;
  float m = -INFINITY;
#pragma unroll 4
  for (int s = 0; s < n; ++s) m = fmaxf(m, ml[(size_t)s * 2 * kBr]);
  float l = 0.f;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
  for (int s = 0; s < n; ++s) {
    const f32x2 x = *reinterpret_cast<const f32x2*>(ml + (size_t)s * 2 * kBr);
    const float* p = po + (size_t)s * kBr * D;
    const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 128);
    const float w = __builtin_amdgcn_exp2f(x[0] - m);   // reference points are finite (kLowest at least)
    l += w * x[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = __builtin_fmaf(w, a[i], lo[i]);
      hi[i] = __builtin_fmaf(w, b[i], hi[i]);
    }
  }
  const float inv_l = 1.0f / l;
  const u32x4 out = {E::pack2(lo[0] * inv_l, lo[1] * inv_l), E::pack2(lo[2] * inv_l, lo[3] * inv_l),
                     E::pack2(hi[0] * inv_l, hi[1] * inv_l), E::pack2(hi[2] * inv_l, hi[3] * inv_l)};
  const int b = bh / H, h = bh - b * H;
  *reinterpret_cast<u32x4*>(O + (((size_t)b * Nq + row) * H + h) * D + 8 * piece) = out;
  if (LSE != nullptr && piece == 0) LSE[(size_t)bh * Nq + row] = m * kLn2 + __builtin_logf(l);
}

size_t bytes_of(int slices, long long q_tiles, int d) {
  return slices == 1 ? 0 : (size_t)q_tiles * slices * kBr * (d + 2) * sizeof(float);
}

// The plan that a call with so many bytes of workspace runs: slices only if they fit, otherwise the best plan without any, as
// for a call with no workspace (a smaller number of slices that fits is not taken: what a call does depends on whether it
// has the workspace that split_workspace() names, not on how much it has).
SplitPlan plan_with(int B, int H, int Nq, int Nk, int d, bool causal, size_t workspace) {
  const SplitPlan p = split_plan(B, H, Nq, Nk, d, causal, workspace != 0);
  if (p.slices == 1 || workspace >= bytes_of(p.slices, (long long)B * H * ((Nq + kBr - 1) / kBr), d)) return p;
  return split_plan(B, H, Nq, Nk, d, causal, false);
}

SplitArgs args_of(const SplitPlan& plan, void* workspace, long long q_tiles, int d) {
  SplitArgs a;
  a.part_o = static_cast<float*>(workspace);
  a.part_ml = a.part_o + (size_t)q_tiles * plan.slices * kBr * d;
  a.chunk = plan.chunk;
  a.slices = plan.slices;
  a.items = plan.items;
  return a;
}

template <int DT, int D, bool kCausal> int launch(const Problem& p, const SplitPlan& plan, void* workspace) {
  const int n_q = (p.Nq + kBr - 1) / kBr;
  const SplitArgs split = args_of(plan, workspace, (long long)p.B * p.H * n_q, D);
  const int total = p.B * p.H * plan.items;
  uint16_t* o = static_cast<uint16_t*>(p.O);
  constexpr int kWv = D <= 128 ? 2 * kWaves : kWaves;   // eight wavefronts: the keys in two halves within the workgroup
  const int rc = enqueue(fa2_fwd_kernel<DT, D, kWv, 2, kCausal, true, true>, total, kWv * 64, p.stream,
                         static_cast<const uint16_t*>(p.Q), static_cast<const uint16_t*>(p.K),
                         static_cast<const uint16_t*>(p.V), o, p.LSE, p.H, p.Nq, p.Nk, p.scale_log2e, n_q, total, 1, split);
  if (rc != FA2_OK || plan.slices == 1) return rc;
  return enqueue(fa2_split_merge_kernel<DT, D, kCausal>, p.B * p.H * n_q * kWaves, 4 * D, p.stream, split, o, p.LSE, p.H,
                 p.Nq, n_q);
}

template <int DT, int D> int launch(const Problem& p, const SplitPlan& plan, void* workspace) {
  return p.causal ? launch<DT, D, true>(p, plan, workspace) : launch<DT, D, false>(p, plan, workspace);
}

}  // namespace

size_t split_workspace(int B, int H, int Nq, int Nk, int d, bool causal) {
  const SplitPlan p = split_plan(B, H, Nq, Nk, d, causal, true);
  return p.use ? bytes_of(p.slices, (long long)B * H * ((Nq + kBr - 1) / kBr), d) : 0;
}

bool split_tiles(const Problem& p, void* workspace, size_t workspace_bytes, int* rc) {
  const SplitPlan plan = plan_with(p.B, p.H, p.Nq, p.Nk, p.d, p.causal, workspace == nullptr ? 0 : workspace_bytes);
  if (!plan.use) return false;
  if (p.dtype == FA2_FP16) {
    *rc = p.d == 64    ? launch<FA2_FP16, 64>(p, plan, workspace)
          : p.d == 128 ? launch<FA2_FP16, 128>(p, plan, workspace)
                       : launch<FA2_FP16, 256>(p, plan, workspace);
  } else {
    *rc = p.d == 64    ? launch<FA2_BF16, 64>(p, plan, workspace)
          : p.d == 128 ? launch<FA2_BF16, 128>(p, plan, workspace)
                       : launch<FA2_BF16, 256>(p, plan, workspace);
  }
  return true;
}

}  // namespace fa2
