// Which problems run with 32 query rows per workgroup and their keys dealt to its wavefronts (host only, no HIP): fa2_short.hip.
#ifndef FA2_SHORT_PLAN_H_
#define FA2_SHORT_PLAN_H_

namespace fa2 {

// Wavefronts per workgroup of fa2_short_kernel, or 0 where another launch is the better one.  `sliced`: the other launch is the
// one that cuts the keys into slices over workgroups, which a workspace is there for.
//
// The lines are drawn from about 800 problems of 2 to 1800 Q tiles of 32 rows and 33 to 4000 keys, N(0,1), timed against what
// ran them before, and leave out what is less than 2 % ahead.  What decides:
//  * Q tiles against CUs.  Up to one tile per CU, this kernel is ahead at every number of keys that the whole or the halved
//    launch of 128 rows would take: us before / now (4 wavefronts) at d = 64, 128, 256: B1 H16 N96 5.0 / 3.8, 6.3 / 4.9, 10.4 / 8.2;
//    B1 H16 N384 7.1 / 5.3, 10.4 / 7.8, 16.4 / 13.7; B1 H4 N1000 12.4 / 7.5, 17.2 / 11.5, 26.9 / 23.4.  With more it reads K and V
//    from the L2 four times as often as tiles of 128 rows and falls behind: B1 H16 N384 (192 tiles) 10.4 / 7.8 at d = 128, H32 (384)
//    10.7 / 10.5, H64 (768) 11.6 / 15.9; a little later where the others' tiles are long (H16 N768 (384) 14.8 / 14.0) and at
//    d = 64, which reads half as much (H32 N512 (512) 9.3 / 7.9, H32 N768 (768) 11.8 / 12.7).
//  * The causal mask: half of the reads, and the 128-row launches take pairs of Q tiles up to 256 keys, two passes one after
//    the other on an idle chip: H24 N205 10.4 / 4.6, 14.4 / 6.3, 24.0 / 10.9; H128 N256 (1024) 11.1 / 8.1 at d = 64, H96 N256 (768)
//    14.9 / 13.5 at d = 128; H16 N1111 (560) 19.7 / 15.3 at d = 128, 14.8 / 10.2 at d = 64.
//  * Slices cut long keys further than the wavefronts of one workgroup do: B1 H2 Nk4000 d128 Nq64 14.5 / 27 (8 wavefronts).
// Four wavefronts, of which two workgroups share a CU at d = 128 and four at d = 64, are ahead of eight but where few workgroups
// have many keys each: 12.3 / 12.5 us for eight / four at B1 H1 N1300 d128 causal, 7.5 / 8.3 at B1 H4 N1000 d64, 6.7 / 6.9 at N768,
// 5.7 / 5.6 at N512.  At d = 256 square problems of few tiles without the mask stay with the staged kernel, 13...22 % behind (H4 N384
// 16.0 / 13.0), because it gives the bits of an explicit tile shape (fa2_fwd_variant), which a sum in parts cannot.  d = 256: four, with two its workgroups fit twice on a CU (H96 N160 causal 18.1 / 14.2, 23.8 before).
inline int short_waves(int B, int H, int Nq, int Nk, int d, bool causal, bool sliced) {
  const long long tiles = (long long)B * H * ((Nq + 31LL) / 32);
  const bool one_pair = Nk > 128 && Nk <= 256;   // causal: a pair of Q tiles of 128 rows
  if (sliced && Nk >= (d == 64 ? 1400 : causal && d == 128 ? 2300 : 1024)) return 0;
  if (d == 256) {
    if (causal && Nk <= 256 && tiles > 256) return tiles <= (one_pair ? 1024 : 512) ? 2 : 0;
    if (!causal && Nq == Nk && tiles <= 64) return 0;
    if (Nk > 768 && (tiles < 96 || Nk > (causal ? 1600 : 1100))) return 0;
    return tiles <= (!causal ? 256 : Nk >= 384 ? 400 : 300) ? 4 : 0;
  }
  if (Nk > 2300) return 0;
  long long most;
  if (d == 64) most = causal ? (one_pair ? 1100 : Nk > 256 ? 840 : 512) : Nk > 256 ? 512 : 288;
  else most = causal ? (one_pair ? 900 : Nk > 256 ? 580 : 384) : Nk >= 700 ? 400 : 256;
  if (tiles > most || (d == 64 && !causal && Nk > 1600 && tiles > 256)) return 0;
  return Nk > 768 && tiles <= 288 ? 8 : 4;
}

}  // namespace fa2
#endif  // FA2_SHORT_PLAN_H_
