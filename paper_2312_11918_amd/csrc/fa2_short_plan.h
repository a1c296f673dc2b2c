// Which problems run with 32 query rows per workgroup and their keys dealt to its wavefronts (host only, no HIP): fa2_short.hip.
#ifndef FA2_SHORT_PLAN_H_
#define FA2_SHORT_PLAN_H_

namespace fa2 {

// How a problem runs there.
struct ShortPlan {
  int waves;    // wavefronts per workgroup; 0: another launch is the better one
  int slices;   // slices of the keys of the longest tile, over workgroups; more than 1 takes a workspace
  int chunk;    // blocks of 32 keys per slice
  int items;    // workgroups per head
};

// The plan for a problem, with or without a workspace for slices.
//
// The lines are drawn from about 900 problems of 2 to 1800 Q tiles of 32 rows and 33 to 8000 keys, N(0,1), timed against what
// ran them before, and leave out what is less than 2 % ahead.  What decides:
//  * Q tiles against CUs.  Up to one tile per CU, this kernel is ahead at every number of keys that the whole or the halved
//    launch of 128 rows would take: us before / now (4 wavefronts) at d = 64, 128, 256: B1 H16 N96 5.0 / 3.8, 6.3 / 4.9, 10.4 / 8.2;
//    B1 H16 N384 7.1 / 5.3, 10.4 / 7.8, 16.4 / 13.7; B1 H4 N1000 12.4 / 7.5, 17.2 / 11.5, 26.9 / 23.4.  With more it reads K and V
//    from the L2 four times as often as tiles of 128 rows and falls behind: B1 H16 N384 (192 tiles) 10.4 / 7.8 at d = 128, H32 (384)
//    10.7 / 10.5, H64 (768) 11.6 / 15.9; a little later where the others' tiles are long (H16 N768 (384) 14.8 / 14.0) and at
//    d = 64, which reads half as much (H32 N512 (512) 9.3 / 7.9, H32 N768 (768) 11.8 / 12.7).
//  * The causal mask: half of the reads, and the 128-row launches take pairs of Q tiles up to 256 keys, two passes one after
//    the other on an idle chip: H24 N205 10.4 / 4.6, 14.4 / 6.3, 24.0 / 10.9; H128 N256 (1024) 11.1 / 8.1 at d = 64, H96 N256 (768)
//    14.9 / 13.5 at d = 128; H16 N1111 (560) 19.7 / 15.3 at d = 128, 14.8 / 10.2 at d = 64; H4 N2688 (336) 30.4 / 20.2 and 20.3 / 13.9.
//  * Blocks in all, each read from the L2 by itself, where the other launch cuts long keys into slices: H2 N2158 d128 (136 tiles
//    of 68 blocks) 20.9 / 16.9, H48 Nq100 Nk2000 (192 of 63) 26.7 / 26.9, H40 Nq248 Nk1728 (320 of 54) 29.6 / 38.6, causal H2 N5000
//    27.8 / 31.1; d = 64: H48 Nq100 Nk4000 24.7 / 33.7.
// Four wavefronts, of which two workgroups share a CU at d = 128 and four at d = 64, are ahead of eight but where few workgroups
// have many keys each: 12.3 / 12.5 us for eight / four at B1 H1 N1300 d128 causal, 7.5 / 8.3 at B1 H4 N1000 d64, 6.7 / 6.9 at N768,
// 5.7 / 5.6 at N512.  At d = 256 square problems of up to 64 tiles without the mask stay with the staged kernel, 13...22 % behind (H4
// N384 16.0 / 13.0): no measurement draws that line.  It keeps small problems of this kind on the bits of an explicit tile shape
// (fa2_fwd_variant), with which they are compared; a sum in parts has others, as problems of more tiles do here.  d = 256:
// four, with two its workgroups fit twice on a CU (H96 N160 causal 18.1 / 14.2, 23.8 before).
inline int short_waves(long long tiles, int Nq, int Nk, int d, bool causal) {
  const bool one_pair = Nk > 128 && Nk <= 256;   // causal: a pair of Q tiles of 128 rows
  const long long blocks = tiles * ((Nk + 31LL) / 32) / (causal ? 2 : 1);
  if (d == 256) {
    if (!causal && Nq == Nk && tiles <= 64) return 0;
    if (causal && Nk <= 256 && tiles > 256) return tiles <= (one_pair ? 1024 : 512) ? 2 : 0;
    if (Nk > 768 && (tiles < 96 || Nk > (causal ? 1600 : 1300) || blocks > 6600)) return 0;
    return tiles <= (!causal ? 256 : Nk >= 384 ? 400 : 300) ? 4 : 0;
  }
  if (Nk > (causal ? 3600 : 2300)) return 0;
  if (blocks > (d == 64 ? (causal ? 30000 : 20000) : (causal ? 20000 : 10500))) return 0;
  long long most;
  if (d == 64) most = causal ? (one_pair ? 1100 : Nk > 256 ? 840 : 512) : Nk > 256 ? 512 : 288;
  else most = causal ? (one_pair ? 900 : Nk > 256 ? 580 : 384) : Nk >= 700 ? 400 : 256;
  if (tiles > most || (d == 64 && !causal && Nk > 1600 && tiles > 256)) return 0;
  return Nk > 768 && tiles <= (!causal ? 256 : Nk > 2300 ? 400 : 288) ? 8 : 4;
}

// Slices: as many as there are CUs for, of eight blocks (two per wavefront) at least; a second kernel (2.5 us) merges them.  us
// before (slices of 128-row tiles) / now: d = 64 H6 Nq300 Nk3000 13.6 / 10.5, H2 Nq32 Nk8000 12.4 / 9.9, H16 Nq64 Nk8000 17.1 / 14.4;
// d = 128 H2 Nq128 Nk1024 12.1 / 8.8, H16 Nq32 Nk3000 15.8 / 12.1, H48 Nq32 Nk4000 37.5 / 26.9, H4 Nq1024 Nk4096 23.6 / 22.1; d = 256 H6
// Nq26 Nk1334 25.1 / 14.5, H2 N1100 28.9 / 19.3, H16 Nq64 Nk8000 47.3 / 37.8; causal H2 N1409 d256 24.3 / 18.8, H2 N2688 d128
// 20.1 / 16.7.  The more blocks in all, the more the reads of 32-row tiles count against the 128 rows of the others, unless those
// are mostly empty: H16 Nq512 Nk8192 (256 tiles of 256 blocks) 45 / 71 at d = 128, 34 / 41 at d = 64, H8 Nq512 Nk2048 d256 32.5 / 30.9.
inline ShortPlan short_plan(int B, int H, int Nq, int Nk, int d, bool causal, bool may_slice) {
  const long long heads = (long long)B * H, n_q = (Nq + 31LL) / 32, n_b = (Nk + 31LL) / 32, tiles = heads * n_q;
  const long long rows128 = (Nq + 127LL) / 128 * 4;   // tiles of 32 rows that those of 128 rows would take
  ShortPlan p{0, 1, (int)n_b, (int)n_q};
  // blocks in all (up to 3 / 2 of them where the rows of the others' tiles are partly empty: B3 H16 Nq40 Nk8040 d64 34.3 / 37.3)
  const long long most = (d == 64 ? 16000 : d == 128 ? 16500 : 8200) * (2 * rows128 >= 3 * n_q ? 3 : 2) / 2;
  if (may_slice && n_b > (d == 64 ? 40 : d == 128 ? 28 : 20) && tiles <= (causal ? 200 : 128) &&
      tiles * n_b / (causal ? 2 : 1) <= most) {
    for (long long s = 2; s <= n_b / 8; ++s) {
      const long long chunk = (n_b + s - 1) / s, slices = (n_b + chunk - 1) / chunk;
      const long long items = causal ? slices * n_q - chunk * (slices * (slices - 1) / 2) : slices * n_q;
      if (heads * items > 256) break;
      p = ShortPlan{0, (int)slices, (int)chunk, (int)items};
    }
    if (p.slices > 1) {
      p.waves = d < 256 && p.chunk > 24 ? 8 : 4;
      return p;
    }
  }
  p.waves = short_waves(tiles, Nq, Nk, d, causal);
  return p;
}

}  // namespace fa2
#endif  // FA2_SHORT_PLAN_H_
