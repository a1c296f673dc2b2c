// Attention whose Q tiles are too few to fill the chip: the keys are split over workgroups as well.
//
// The 128-row tile kernel runs one workgroup per Q tile; a chunk of 512 queries in 16 heads is 64 of them, on 256 CUs that
// hold two each, and a lone workgroup, with one wavefront per SIMD, runs its softmax and its MFMAs one after the other
// (1.0 us per K/V tile at d = 128).  Here the keys of a Q tile are cut into halves inside a workgroup of eight wavefronts
// (d <= 128; 1.3 us per PAIR of tiles), and, where the caller gives a workspace, into slices over workgroups whose partial
// results a second kernel on the same stream merges.  The price is that kernel (5 us) and the partial O in fp32, written
// and read once (64 KiB per workgroup at d = 128).  B1 H16 Nq512 Nk8192 d128: 129 us whole, 41 here; B1 H16 N1111 d128
// causal, in one launch: 29 and 19.
#include "fa2_tile_kernel.h"

namespace fa2 {
namespace {

constexpr float kLn2 = 0.69314718055994530942f;

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

struct Plan {
  int chunk, slices, items;   // K/V tiles per slice, slices of the longest Q tile, workgroups per head
  bool use;                   // false: the tile kernel's whole launch is the better one
};

size_t bytes_of(int slices, long long q_tiles, int d) {
  return slices == 1 ? 0 : (size_t)q_tiles * slices * kBr * (d + 2) * sizeof(float);
}

// The plan for a problem by estimated time, with or without a workspace for slices.
//
// The estimates (us) are fits to about thirty shapes, bf16 N(0,1), K and V from HBM, and hold to about 15 %.  A whole
// launch costs a start plus a time per K/V tile of its longest workgroup.  Halved workgroups pay more to start and
// merge and less than 2x per pair of tiles, more of it the more CUs are busy (the clock drops); slices add the second
// kernel and the partial O.  Measured, whole / halves / best slices: B1 H16 Nq512 Nk8192 d128 136.7 / 92.1 / 43.5 (4
// slices); B1 H16 N1111 d128 causal 31.0 / 21.2 / 23.5; B2 H8 N2048 d128 44.3 / 36.7 / 53.7; B1 H6 N3000 d128 causal 58.5 /
// 36.9 / 30.0; B2 H32 Nq300 Nk3000 d64 39.7 / 29.4 / 38.0; B1 H16 N512 d128 12.1 / 12.8 / 17.3.  With more Q tiles than CUs
// and no mask the whole launch was always ahead (B2 H12 N1500 d128, 288 Q tiles: 39.4 / 48.8 / 58.9).  Under the causal
// mask it runs one workgroup per PAIR of Q tiles, and single ones, longest first, fill the CUs better up to about 1000 Q
// tiles: B1 H12 N3088 d128 (300) 63.7 / 44.5, B5 H2 N6401 d64 (510) 103.5 / 70.1, B5 H24 N620 d256 (600) 78.6 / 61.3 (d = 256:
// unpaired, not halved); level from there (B3 H12 N3245 d128, 936 Q tiles: 107.8 / 106.8).
Plan plan_of(int B, int H, int Nq, int Nk, int d, bool causal, bool may_slice) {
  const long long heads = (long long)B * H;
  const int n_q = (Nq + kBr - 1) / kBr, n_k = 2 * ((Nk + kBr - 1) / kBr);
  Plan best{n_k, 1, n_q, false};
  const long long q_tiles = heads * n_q;
  if (n_k <= 4 || q_tiles > (causal ? 4 : 1) * kCUs) return best;
  struct Fit {
    float start, tile, tile_shared;         // whole launch: start, per tile with one workgroup on a CU, with more
    float start_split, step, step_crowd;    // split launch: start, per step (a tile of either half), more of it at 256 CUs
    float merge;                            // second kernel
  };
  const Fit fit = d == 64    ? Fit{4.5f, 0.65f, 0.95f, 6.0f, 0.78f, 0.22f, 5.5f}
                  : d == 128 ? Fit{5.5f, 1.0f, 1.45f, 7.2f, 1.3f, 0.5f, 5.5f}
                             : Fit{7.0f, 2.0f, 2.0f, 9.0f, 2.05f, 0.0f, 8.0f};   // d = 256: slices only, a step is one tile
  // causal: pairs of Q tiles, whose tile counts add up to n_k + 2, with an epilogue each
  const bool pairs = causal && n_q > 1;
  const float busy = (float)(heads * (pairs ? (n_q + 1) / 2 : n_q)) / kCUs;
  const float tile = busy <= 1.0f ? fit.tile * (1.0f + 0.2f * busy * busy) : fit.tile_shared;
  float least = fit.start + tile * (pairs ? n_k + 2 : n_k) + (pairs ? 3.0f : 0.0f);
  if (d == 256 && busy > 1.0f) least *= busy <= 2.0f ? 2.0f : busy;   // one workgroup per CU: whole rounds
  least *= q_tiles > kCUs ? 0.92f : 0.97f;   // in doubt the whole launch
  const float kv_mb = (float)(heads * Nk) * d * 4e-6f;
  const int rows = n_q > 1 ? kBr : (Nq + 31) / 32 * 32;   // of a workgroup that wavefronts work on
  int last = 0;
  for (int s = 1; s <= n_k / 4; ++s) {
    const int chunk = ((n_k + s - 1) / s + 3) / 4 * 4;
    if (chunk == last) continue;
    last = chunk;
    const int slices = (n_k + chunk - 1) / chunk;
    const long long items = causal ? (long long)slices * n_q - (long long)(chunk / 2) * slices * (slices - 1) / 2
                                   : (long long)slices * n_q;
    const long long groups = heads * items;
    if (slices > 1 && (!may_slice || groups > 2 * kCUs || Nk < FA2_SPLIT_MIN_KEYS)) break;
    const int rounds = (int)((groups + kCUs - 1) / kCUs);
    const int steps = d == 256 ? (chunk < n_k ? chunk : n_k) : chunk / 2;
    const float fill = groups < kCUs ? (float)groups / kCUs : 1.0f;
    // causal: workgroups of all lengths, the longest first, so the CUs end together
    const float work = (float)heads * n_q * (n_q + 2) * (d == 256 ? 1.0f : 0.5f) / kCUs;
    const float length = !causal ? (float)steps * rounds : work > steps ? work : (float)steps;
    float loop = (fit.step + fit.step_crowd * fill * rows / kBr) * length;
    const float memory = kv_mb / 4.5f;   // K and V at 4.5 TB/s: MB per us
    if (loop < memory) loop = memory;
    const float turns = !causal ? (float)rounds : groups > kCUs ? 0.3f + 0.7f * groups / kCUs : 1.0f;
    const float time = fit.start_split * turns + loop +
                       (slices > 1 ? fit.merge + (float)groups * rows * d * 8e-6f / 5.0f : 0.0f);
    if (time < least) {
      least = time;
      best = Plan{chunk, slices, (int)items, true};
    }
  }
  return best;
}

// The plan that a call with so many bytes of workspace runs: slices only if they fit, otherwise the best plan without any, as
// for a call with no workspace (a smaller number of slices that fits is not taken: what a call does depends on whether it
// has the workspace that split_workspace() names, not on how much it has).
Plan plan_with(int B, int H, int Nq, int Nk, int d, bool causal, size_t workspace) {
  const Plan p = plan_of(B, H, Nq, Nk, d, causal, workspace != 0);
  if (p.slices == 1 || workspace >= bytes_of(p.slices, (long long)B * H * ((Nq + kBr - 1) / kBr), d)) return p;
  return plan_of(B, H, Nq, Nk, d, causal, false);
}

SplitArgs args_of(const Plan& plan, void* workspace, long long q_tiles, int d) {
  SplitArgs a;
  a.part_o = static_cast<float*>(workspace);
  a.part_ml = a.part_o + (size_t)q_tiles * plan.slices * kBr * d;
  a.chunk = plan.chunk;
  a.slices = plan.slices;
  a.items = plan.items;
  return a;
}

template <int DT, int D, bool kCausal> int launch(const Problem& p, void* workspace, size_t workspace_bytes) {
  const Plan plan = plan_with(p.B, p.H, p.Nq, p.Nk, D, kCausal, workspace_bytes);
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

template <int DT, int D> int launch(const Problem& p, void* workspace, size_t workspace_bytes) {
  return p.causal ? launch<DT, D, true>(p, workspace, workspace_bytes) : launch<DT, D, false>(p, workspace, workspace_bytes);
}

}  // namespace

bool split_accepts(int B, int H, int Nq, int Nk, int d, bool causal, size_t workspace) {
  return plan_with(B, H, Nq, Nk, d, causal, workspace).use;
}

size_t split_workspace(int B, int H, int Nq, int Nk, int d, bool causal) {
  const Plan p = plan_of(B, H, Nq, Nk, d, causal, true);
  return p.use ? bytes_of(p.slices, (long long)B * H * ((Nq + kBr - 1) / kBr), d) : 0;
}

int split_tiles(const Problem& p, void* workspace, size_t workspace_bytes) {
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
