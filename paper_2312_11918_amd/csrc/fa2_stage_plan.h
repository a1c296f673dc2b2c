// Which problems run with the softmax mixed into the MFMAs (host only, no HIP): see fa2_stage.hip.
#ifndef FA2_STAGE_PLAN_H_
#define FA2_STAGE_PLAN_H_
#include "fa2_split_plan.h"

namespace fa2 {

// For a problem that no launch with its keys cut has taken (those are ahead where Q tiles are few: B1 H8 N3000 29 / 55 us).
// Below: tile kernel / this one, us, medians of seven times in turn.
//
// d = 64.  Without a mask both kernels' times go with the workgroups of the busiest CU: measured over 120 problems, us per
// K/V tile, 1.08, 1.92, 3.0, 3.9 for one to four workgroups of 256 rows, which run two at a time, and 0.565 each for those
// of 128 rows in the tile kernel, which run three at a time.  So what decides is how the rows fill rounds of either size;
// 5 % are left to the tile kernel, for starts and ends.  B2 H6 N9984 (468 workgroups of 256 rows) 350 / 305, B4 H16 N2816
// (704) 148 / 134, B46 H8 N1024 (1472) 120 / 115, B64 H24 N130 (1536) 34.3 / 31.3; but B6 H2 N6247 (300) 159 / 177, B4 H6
// N6016 (576) 259 / 282, B13 H32 N384 (832, a quarter of the rows empty) 23.4 / 29.6.
//
// That holds from 20 K/V tiles on (59 of 66 problems that the fit takes are 1...14 % ahead, one 1.7 % behind), for shorter
// ones of one round (71 of 73 are 1...20 % ahead), and where a quarter of every workgroup's rows is empty, which its fourth
// wavefront leaves out (129...192 queries: 31, none behind).  Else a workgroup's start and end count, three of which overlap
// in the tile kernel and two here: with 6 % more left to it, 162 problems run from 11 % ahead to 5 % behind, 112 more than
// 1 % ahead and eight more than 3 % behind.  And an even count of up to six tiles is the tile kernel's, which runs pairs of
// them.  Of 113 problems left to it by these two, 45 are more than 3 % behind here, twelve ahead: B21 H32 Nq256 Nk71
// 15.6 / 17.7, B64 H16 N256 28.8 / 31.1, B78 H12 N512 78.7 / 84.9, B56 H8 N896 108 / 115.
//
// Under the causal mask the diagonal's 256 x 256 block, of which a workgroup runs all four tiles, weighs the more the
// shorter the sequence, and short tiles have to fill the end: from 32 K/V tiles and two workgroups per CU on 1...20 % ahead
// in 173 of 192 problems (B5 H8 N6656 286 / 237, B2 H12 N5555 143 / 123), eight of the others 1...11 % behind (B13 H16 N2688
// 233 / 245, B7 H12 N2176 67 / 75); mixed below (B14 H12 N1072 47.0 / 45.1, B12 H32 N476 28.1 / 31.5), behind with fewer
// workgroups (B1 H8 N13184 212 / 242).  The tile kernel has as many pairs of Q tiles as there are workgroups here, all of
// one length, three at a time: where they are exactly two or three per CU it ends everywhere at once (two: B1 H16 N8036
// 149 / 163, B2 H16 N4096 83.6 / 86.3, 1...10 % behind in 8 of 8; three: B3 H16 N3968 116 / 122, B2 H32 N2944 89 / 93, B8 H2
// N12288 334 / 324, behind in 6 of 9).
//
// d = 256, the same 128 rows per workgroup as in the tile kernel.  Where that one chains its Q tiles over one K/V stream
// (whole tiles, two whole rounds of the CUs or more) they are level at N = 4096 (564 / 567) and this one 1...6 % behind from
// N = 1024 down (B32 H16 N512 202 / 213).  Otherwise, without a mask, 3...18 % ahead with more than 128 keys in 108 of 108
// problems, 85 of them with 1...200 Q tiles (B1 H3 Nq5 Nk206 13.2 / 12.0, B4 H8 Nq377 Nk238 15.7 / 14.6), level to 1.5 %
// behind below (B17 H24 N74 23.3 / 23.6).  Under the mask it runs single Q tiles, longest first, against pairs; those of up
// to four rounds are fa2_split.hip's.  With more: 9...34 % ahead from 1536 keys on in 62 of 62 problems (B27 H2 N3524
// 463 / 423), mixed below (B30 H16 N286 116 / 100, B7 H32 N768 126 / 135).
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
  if (causal) return (Nq + 63LL) / 64 >= 32 && wide > 2 * kCUs && wide != 3 * kCUs;
  const long long mine = (wide + kCUs - 1) / kCUs, other = (narrow + kCUs - 1) / kCUs, tiles = (Nk + 63LL) / 64;
  const bool ends_count = tiles < 20 && mine > 2 && Nq > 192;
  if (ends_count && tiles <= 6 && tiles % 2 == 0) return false;
  return 1.05 * (0.96 * mine + (mine % 2 != 0 ? 0.12 : 0.0)) < (ends_count ? 0.94 : 1.0) * 0.565 * other;
}

}  // namespace fa2
#endif  // FA2_STAGE_PLAN_H_
