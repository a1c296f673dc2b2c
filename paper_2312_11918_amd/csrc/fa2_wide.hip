// The 256-row shape of the tile kernel on partial tiles, d = 128.
//
// Sizes that are no whole tiles ran in the 128-row shape, which sends twice the bytes per FLOP from the L2 into LDS and pays a
// prologue and an epilogue for every Q tile.  The 256-row kernel has no register left for a second set of source offsets, those
// of the tiles with rows past the last key.  None is needed: the descriptor's range check turns such rows into zeros in LDS (as good
// as copies of the last key: their columns of S are masked; a tile without any key is not asked for, see wide_staged_tile), and what
// the epilogue derives from the lane is not kept through the loop.  256 registers, no scratch.  Without the mask the bits are those
// of the 128-row shape; under it that one takes the row maximum on every one of its last tiles, this one only on those that the
// diagonal crosses, so where a reference point moves there the last bits differ.  4 % at B8 H16 N2047 (271 -> 261 us, 1022 -> 1066
// TFLOP/s: the clock under N(0,1) operands bounds it from there, as on whole tiles), 6 % under the mask, 9 % at N = 511 (see
// fa2_wide_plan.h).
#include "fa2_wide_plan.h"
#include "fa2_tile_kernel.h"

namespace fa2 {
namespace {

template <int DT, bool kCausal> int launch(const Problem& p) {
  const int n_q = (p.Nq + 255) / 256;
  const int groups = p.B * p.H * (kCausal ? n_q / 2 : n_q);   // whole rounds: a workgroup takes one of every round
  return enqueue(fa2_fwd_kernel<DT, 128, 8, 4, kCausal, true>, kCUs, 512, p.stream, static_cast<const uint16_t*>(p.Q),
                 static_cast<const uint16_t*>(p.K), static_cast<const uint16_t*>(p.V), static_cast<uint16_t*>(p.O), p.LSE, p.H, p.Nq,
                 p.Nk, p.scale_log2e, n_q, kCUs, groups / kCUs, SplitArgs{});
}

}  // namespace

bool wide_tiles(const Problem& p, int* rc) {
  if (!wide_accepts(p.B, p.H, p.Nq, p.Nk, p.d, p.causal)) return false;
  if (p.causal) *rc = p.dtype == FA2_FP16 ? launch<FA2_FP16, true>(p) : launch<FA2_BF16, true>(p);
  else *rc = p.dtype == FA2_FP16 ? launch<FA2_FP16, false>(p) : launch<FA2_BF16, false>(p);
  return true;
}

}  // namespace fa2
