// Which problems run with the softmax mixed into the MFMAs (host only, no HIP): see fa2_stage.hip.
#ifndef FA2_STAGE_PLAN_H_
#define FA2_STAGE_PLAN_H_
#include "fa2_split_plan.h"

namespace fa2 {

// For a problem that no launch with its keys cut has taken (those are ahead where Q tiles are few: B1 H8 N3000 29 / 55 us).
//
// d = 64.  Without a mask both kernels' times go with the workgroups of the busiest CU: measured over 120 problems, us per K/V
// tile, 1.08, 1.92, 3.0, 3.9 for one to four workgroups of 256 rows, which run two at a time, and 0.565 each for those of 128
// rows in the tile kernel, which run three at a time.  So what decides is how the rows fill rounds of either size; 5 % are
// left to the tile kernel, for starts and ends.  Tile kernel / this one: B2 H6 N9984 (468 workgroups of 256 rows) 350 / 305,
// B4 H16 N2816 (704) 148 / 134, B46 H8 N1024 (1472) 120 / 115, B64 H24 N130 (1536) 34.3 / 31.3; but B6 H2 N6247 (300) 159 / 177,
// B4 H6 N6016 (576) 259 / 282, B13 H32 N384 (832, a quarter of the rows empty) 23.4 / 29.6.
//
// Under the causal mask the diagonal's 256 x 256 block, of which a workgroup runs all four tiles, weighs the more the shorter
// the sequence, and short tiles have to fill the end: 1...20 % ahead from 32 K/V tiles and 512 workgroups on in 30 of 33 problems (B5
// H8 N6656 286 / 237, B2 H12 N5555 143 / 123; three of partial rounds 2...5 % behind), mixed below (B14 H12 N1072 47.0 / 45.1,
// B12 H32 N476 28.1 / 31.5), behind with fewer workgroups (B1 H8 N13184 212 / 242).
//
// d = 256, the same 128 rows per workgroup as in the tile kernel.  Where that one chains its Q tiles over one K/V stream (whole
// tiles, two whole rounds of the CUs or more) they are level at N = 4096 (564 / 567) and this one 1...6 % behind from N = 1024 down
// (B32 H16 N512 202 / 213).  Otherwise, without a mask, 4...16 % ahead in 38 of 38 problems of Q tiles for 200 CUs and more and more than
// 128 keys, level to 1.5 % behind below (B17 H24 N74 23.3 / 23.6).  Under the mask it runs single Q tiles, longest first, against pairs;
// those of up to four rounds are fa2_split.hip's.  With more: 5...27 % ahead from 1536 keys on in 21 of 22 problems (B27 H2 N3524 423 /
// 435), mixed below (B30 H16 N286 116 / 100, B7 H32 N768 126 / 135).
inline bool stage_accepts(int B, int H, int Nq, int Nk, int d, bool causal) {
  if (d != 64 && d != 256) return false;
  const long long heads = (long long)B * H;
  if (d == 256) {
    const long long q_tiles = heads * ((Nq + 127LL) / 128);
    if (q_tiles > 0x7fffffffLL) return false;
    const bool exact = Nq % 128 == 0 && Nk % 128 == 0;
    if (causal) return q_tiles > 4 * kCUs && Nk >= 1536 && !(exact && Nq % 256 == 0 && q_tiles % (2 * kCUs) == 0);
    return Nk > 128 && !(exact && q_tiles > kCUs && q_tiles % kCUs == 0);
  }
  const long long wide = heads * ((Nq + 255LL) / 256), narrow = heads * ((Nq + 127LL) / 128);
  if (wide > 0x7fffffffLL) return false;
  if (causal) return (Nq + 63LL) / 64 >= 32 && wide >= 2 * kCUs;
  const long long mine = (wide + kCUs - 1) / kCUs, other = (narrow + kCUs - 1) / kCUs;
  return 1.05 * (0.96 * mine + (mine % 2 != 0 ? 0.12 : 0.0)) < 0.565 * other;
}

}  // namespace fa2
#endif  // FA2_STAGE_PLAN_H_
