// Which problems on partial tiles run in the 256-row shape (host only, no HIP): see fa2_wide.hip.
#ifndef FA2_WIDE_PLAN_H_
#define FA2_WIDE_PLAN_H_
#include "fa2_split_plan.h"

namespace fa2 {

// d = 128.  The 256-row shape gains where it pads no more than the 128-row one, rows or keys, and where its Q tiles (under the mask
// pairs of them, all complete) fill whole rounds of the CUs, so that one workgroup per CU takes a tile of every round over one
// running K/V stream.  us, 128 rows / 256 rows: B8 H16 N2047 271 / 261, N2000 267 / 257, B4 H16 N4095 516 / 499, B16 H16 N1000 151 / 141,
// B32 H16 N511 96.9 / 88.7, B8 H16 Nq2047 Nk3000 390 / 378, B16 H16 Nq2040 Nk255 112 / 104; causal B8 H16 N2047 166 / 156, B16 H16 N1000
// 107 / 99, B32 H16 N500 77.9 / 75.4, B1 H16 N8100 267 / 258.  More padding: N1900 233 / 235, B16 H24 N640 96 / 130.  Rounds that are not
// whole: B3 H16 N2000 (1.5) 102 / 107, B21 H16 N2040 (10.5) 634 / 647, causal B8 H16 N1500 (1.5) 98.6 / 110.  One tile per head: B64 H16 N250
// 66.5 / 68.8.  A single round of short sequences: B8 H16 Nq500 Nk5000 156 / 157 (of long ones: B2 H16 N2000 69.8 / 68.2).
// Whole rounds are few of all problems, those of powers of two in B H.
inline bool wide_accepts(int B, int H, int Nq, int Nk, int d, bool causal) {
  if (d != 128 || Nq <= 256 || (Nq == Nk && Nq % 256 == 0)) return false;   // (whole square tiles: fa2_fwd.hip)
  const long long n_q = (Nq + 255LL) / 256, heads = (long long)B * H;
  if ((Nq + 127LL) / 128 != 2 * n_q || (Nk + 127LL) / 128 % 2 != 0) return false;
  if (causal && n_q % 2 != 0) return false;
  const long long groups = heads * (causal ? n_q / 2 : n_q);
  return groups <= 0x7fffffffLL && groups % kCUs == 0 && (groups >= 2 * kCUs || Nq >= 1024);
}

// The K/V tile (of 64 keys) that the 256-row shape on partial tiles loads as tile j.  Rows past the last key are left to the descriptor's
// range check, which is specified as lane offset >= range - scalar offset: the scalar offset, that of the tile's first row, has to
// lie within the range itself, past which the difference would wrap.  So a tile without any key, which only rounds the count up
// to four and whose arithmetic is left out, takes the last tile with one.  (Not loading it at all costs a branch per load
// burst: B8 H16 N2047 256.6 -> 258.4 us; this one is within the noise of no check, 256.3.)
constexpr int wide_staged_tile(int j, int Nk) { return j < (Nk - 1) / 64 ? j : (Nk - 1) / 64; }

}  // namespace fa2
#endif  // FA2_WIDE_PLAN_H_
