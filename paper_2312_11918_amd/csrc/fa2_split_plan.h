// Which launch a problem of few query tiles gets (host only, no HIP): whole, or with its keys cut.  See fa2_split.hip.
#ifndef FA2_SPLIT_PLAN_H_
#define FA2_SPLIT_PLAN_H_

namespace fa2 {

constexpr int kCUs = 256;           // compute units of the whole chip (choice of tile shapes and of key splits)
constexpr int kPlanRows = 128;      // query rows per Q tile; a K/V tile holds 64 keys
constexpr int kSplitMinKeys = 512;  // fewest keys that are cut into slices

struct SplitPlan {
  int chunk, slices, items;   // K/V tiles per slice, slices of the longest Q tile, workgroups per head
  bool use;                   // false: the tile kernel's whole launch is the better one
};

// The plan for a problem by estimated time, with or without a workspace for slices.
//
// The estimates (us) are fits to about 480 shapes, N(0,1), of 8 to 1024 Q tiles; most hold to about 15 %, those of slices are
// up to 25 % too high.  A whole launch costs a start plus a time per K/V tile of its longest workgroup.  Halved workgroups pay
// more to start and merge and less than 2x per pair of tiles, more of it the more CUs are busy (the clock drops); slices
// add the second kernel and the partial O.  Measured, whole / halves / best slices: B1 H16 Nq512 Nk8192 d128 136.7 / 92.1 /
// 43.5 (4 slices); B1 H16 N1111 d128 causal 31.0 / 21.2 / 23.5; B2 H8 N2048 d128 44.3 / 36.7 / 53.7; B1 H6 N3000 d128 causal
// 58.5 / 36.9 / 30.0; B2 H32 Nq300 Nk3000 d64 39.7 / 29.4 / 38.0; B1 H16 N512 d128 12.1 / 12.8 / 17.3.  With more Q tiles than
// CUs and no mask the whole launch was always ahead (B2 H12 N1500 d128, 288 Q tiles: 39.4 / 48.8 / 58.9).
//
// d = 256 has no halves: with one slice and no mask the split launch would be the whole one in the partial-tile kernel, and
// is never taken (B2 H6 N2048: 62.0 whole, 71.8; B1 H8 N4096 136 / 150).  On whole tiles the whole launch chains its Q tiles in
// the kernel without partial tiles, 12 % faster per tile than with them (fit.tile_exact).
//
// Under the causal mask the whole launch runs one workgroup per PAIR of Q tiles; single ones in one slice, longest first,
// fill the CUs better up to about 1000 Q tiles: B1 H12 N3088 d128 (300) 63.7 / 44.5, B5 H2 N6401 d64 (510) 103.5 / 70.1, B5 H24
// N620 d256 (600) 78.6 / 61.3; level from there (B3 H12 N3245 d128, 936 Q tiles: 107.8 / 106.8).  With one to two rounds of
// them the last of the short ones decide, each of which starts behind a longer one (`second`): B8 H12 N512 d128 (384)
// 19.3 / 20.9, B7 H16 N384 d64 (336) 12.6 / 13.2 stay whole.  At d = 256 two more things count, one workgroup per CU: the
// rounds fill worse the more there are, and heads that are no multiple of the 8 XCDs share no L2 (B1 H16 N4096 (512)
// 144 / 160, B3 H6 N3328 (468) 120 / 132, B99 H1 N462 (396) 36.1 / 38.4; but B16 H2 N2272 (576) 176 / 123).
inline SplitPlan split_plan(int B, int H, int Nq, int Nk, int d, bool causal, bool may_slice) {
  const long long heads = (long long)B * H;
  const int n_q = (Nq + kPlanRows - 1) / kPlanRows, n_k = 2 * ((Nk + 127) / 128);
  SplitPlan best{n_k, 1, n_q, false};
  const long long q_tiles = heads * n_q;
  if (n_k <= 4 || q_tiles > (causal ? 4 : 1) * kCUs) return best;
  struct Fit {
    float start, pair;                      // whole launch: start, more of it for a pair's second Q tile
    float tile, tile_exact, tile_shared;    // per tile with one workgroup on a CU (partial / whole tiles), with more
    float start_split, own;                 // split launch: start, the part of it that every workgroup pays
    float step, step_crowd;                 // per step (a tile of either half), more of it at 256 CUs
    float merge;                            // second kernel
    float uneven, astray;                   // more time at 768 workgroups, where heads are no multiple of 8
  };
  const Fit fit = d == 64    ? Fit{4.5f, 3.0f, 0.65f, 0.65f, 0.95f, 6.0f, 3.0f, 0.78f, 0.22f, 5.5f, 0.0f, 0.0f}
                  : d == 128 ? Fit{5.5f, 3.0f, 1.0f, 1.0f, 1.45f, 7.2f, 3.7f, 1.3f, 0.5f, 5.5f, 0.0f, 0.0f}
                             : Fit{7.0f, 7.0f, 1.8f, 1.6f, 2.0f, 8.0f, 6.0f, 1.95f, 0.0f, 3.0f, 0.12f, 0.06f};   // a step is one tile
  // causal: pairs of Q tiles, whose tile counts add up to n_k + 2, with an epilogue each
  const bool pairs = causal && n_q > 1;
  const bool exact = Nq % 128 == 0 && Nk % 128 == 0;
  const float busy = (float)(heads * (pairs ? (n_q + 1) / 2 : n_q)) / kCUs;
  const float tile = busy <= 1.0f ? (exact ? fit.tile_exact : fit.tile) * (1.0f + 0.2f * busy * busy) : fit.tile_shared;
  float least = fit.start + tile * (pairs ? n_k + 2 : n_k) + (pairs ? fit.pair : 0.0f);
  if (d == 256 && busy > 1.0f) least *= busy <= 2.0f ? 2.0f : busy;   // one workgroup per CU: whole rounds
  least *= q_tiles > kCUs ? 0.93f : 0.97f;   // in doubt the whole launch
  const float kv_mb = (float)(heads * Nk) * d * 4e-6f;
  const int rows = n_q > 1 ? kPlanRows : (Nq + 31) / 32 * 32;   // of a workgroup that wavefronts work on
  int last = 0;
  for (int s = 1; s <= n_k / 4; ++s) {
    const int chunk = ((n_k + s - 1) / s + 3) / 4 * 4;
    if (chunk == last) continue;
    last = chunk;
    const int slices = (n_k + chunk - 1) / chunk;
    if (d == 256 && !causal && slices == 1) continue;
    const long long items = causal ? (long long)slices * n_q - (long long)(chunk / 2) * slices * (slices - 1) / 2
                                   : (long long)slices * n_q;
    const long long groups = heads * items;
    if (slices > 1 && (!may_slice || groups > 2 * kCUs || Nk < kSplitMinKeys)) break;
    const float fill = groups < kCUs ? (float)groups / kCUs : 1.0f;
    const float step = fit.step + fit.step_crowd * fill * rows / kPlanRows;
    float time;
    if (causal && slices == 1) {
      // steps of Q tile t (halves: an even number of tiles each)
      auto length = [&](int t) { return fit.own + step * (d == 256 ? 2 * (t + 1) : (2 * (t + 1) + 3) / 4 * 2); };
      float span = length(n_q - 1);
      if (groups > kCUs) {
        // Longest first: workgroup 256 + i, counted from 1, runs behind workgroup 257 - i.  The last one of every Q tile
        // that starts in the second round, or the longest Q tile and one that starts later, bound the span; so does the
        // average over the CUs.
        float total = 0.0f;
        for (int c = 0; c < n_q; ++c) {
          const int t = n_q - 1 - c;
          const long long end = heads * (c + 1);
          total += heads * length(t);
          if (end <= kCUs || heads * c >= 2 * kCUs) continue;
          const long long before = end <= 2 * kCUs ? (2 * kCUs - end) / heads : 0;
          const float second = length(t) + length(n_q - 1 - (int)before);
          if (second > span) span = second;
        }
        if (total / kCUs > span) span = total / kCUs;
        const long long beyond = groups - kCUs < 2 * kCUs ? groups - kCUs : 2 * kCUs;
        span *= (1.0f + fit.uneven * beyond / (2 * kCUs)) * (heads % 8 != 0 ? 1.0f + fit.astray : 1.0f);
      }
      time = fit.start_split - fit.own + span;
    } else {
      const int rounds = (int)((groups + kCUs - 1) / kCUs);
      const int steps = d == 256 ? (chunk < n_k ? chunk : n_k) : chunk / 2;
      // causal: workgroups of all lengths, the longest first, so the CUs end together
      const float work = (float)heads * n_q * (n_q + 2) * (d == 256 ? 1.0f : 0.5f) / kCUs;
      const float length = !causal ? (float)steps * rounds : work > steps ? work : (float)steps;
      float loop = step * length;
      const float memory = kv_mb / 4.5f;   // K and V at 4.5 TB/s: MB per us
      if (loop < memory) loop = memory;
      const float turns = !causal ? (float)rounds : groups > kCUs ? 0.3f + 0.7f * groups / kCUs : 1.0f;
      time = fit.start_split * turns + loop +
             (slices > 1 ? fit.merge + (float)groups * rows * d * 8e-6f / 5.0f : 0.0f);
    }
    if (time < least) {
      least = time;
      best = SplitPlan{chunk, slices, (int)items, true};
    }
  }
  return best;
}

}  // namespace fa2
#endif  // FA2_SPLIT_PLAN_H_
