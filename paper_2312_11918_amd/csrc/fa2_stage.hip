// Attention with the softmax mixed into the MFMAs: d = 64 with 64 query rows per wavefront, and d = 256.
//
// At d = 64 the softmax costs a SIMD more issue cycles than the matrix products: per 64 x 64 tile of S and wavefront 224
// vector instructions (1152 cycles, 64 of them exponentials at half rate) beside 32 MFMAs (1024 cycles of the matrix core, 128
// of issue).  Two things kept the tile kernel of fa2_tile_kernel.h from either bound.  Its two or three wavefronts per SIMD run
// whole phases, softmax or MFMAs, which overlap only as it happens; and it reads one 1 KiB fragment from LDS per MFMA.  Here
//  * a wavefront owns two groups of 32 query rows, so that a K or V fragment read from LDS feeds two MFMAs, and a K/V tile
//    staged by a workgroup of four wavefronts serves 256 rows;
//  * the work is a pipeline of stages of 32 keys: stage s runs the softmax of S(s), GEMM-I of S(s+1) and GEMM-II with
//    P~(s-1), and one MFMA alternates with the vector instructions of two elements per lane.
// 212...221 registers, two wavefronts per SIMD, two workgroups per CU.  Bound by vector issue where the loop is long: counted at
// B1 H32 N16384, a tile takes its SIMD 1963 cycles, 1448 of them vector issue (261 instructions and the MFMAs): 74 % of all, 82 %
// of those with both wavefronts there, at 1.74 GHz on N(0,1) inputs.  At B32 H16 N512 it is 45 % and 68 %: starts and ends around
// 16 stages, 1.34 wavefronts per SIMD on average.  The bits are those of the tile kernel (but where the reference point of a
// row moves, which both find out at different keys).  us before and after, in turn in one process: B1 H32 N16384
// 2234 / 2055, B8 H32 N2048 304 / 278, B16 H32 N1024 166 / 156, B32 H16 N512 50.1 / 48.6, B8 H16 N2047 154 / 148, causal B1 H32
// N16384 1160 / 1054, B8 H32 N2048 182 / 175.
//
// At d = 256 O^T alone takes half of the 512 registers that the only wavefront of a SIMD has, so a wavefront owns one group of
// 32 rows, and a stage is GEMM-I of S(s+1), then GEMM-II with P~(s-1), one element of the softmax of S(s) after every second
// MFMA.  The tile kernel's wavefront has nobody to overlap its softmax with.  An MFMA, 32 cycles, takes 71 of its SIMD (34 ns
// settled, at 2.0 GHz); the wavefront issues in 51 % of its cycles, waits for its turn in 24 % and for a counter or
// a barrier in 26 % (counted at B4 H8 N4095).  us before and after: B4 H8 N4095 603 / 561, B6 H12 N1000 122 / 111, B11 H8 N777
// 104 / 92, B2 H16 N1024 41.0 / 39.2, B9 H24 Nq3 Nk355 20.6 / 18.8; causal B4 H32 N1116 157 / 134, B9 H8 N2709 420 / 344.  It
// makes no difference there: 6, 12 or 16 fragments in flight instead of 8 (0...-2 %), the two products mixed (0...-1 %), the
// refills spread over a stage (-1...+1 %).  d = 128 in this form (two groups, one wavefront per SIMD): 6...16 % slower than the
// tile kernel, which has two.
//
// Tried and not kept at d = 64: eight wavefronts (512 rows) per workgroup, level at N = 16384, 4...8 % slower below; two
// wavefronts (128 rows), 6...11 % slower (the K/V refill doubles); one group of rows and three wavefronts per SIMD, 4...9 %
// slower; four K/V buffers instead of two, 0...-4 %; alternating priorities of the two workgroups of a CU, 0...-1 %.
#include "fa2_stage_plan.h"
#include "fa2_tile_kernel.h"

namespace fa2 {
namespace {

constexpr int kStageKeys = 32;                        // keys per stage, half a K/V tile
constexpr int groups_of(int d) { return d == 64 ? 2 : 1; }   // groups of 32 query rows per wavefront
constexpr float kSumLimit = 256.0f;                   // a partial row sum beyond 2^kLazyLog2 moves the reference point

template <int N> using Int = std::integral_constant<int, N>;

// Workgroup -> (head, Q tile); see fa2_fwd_kernel for the operands' layouts, the swizzles, the reference point of the
// exponentials and the epilogue, which are the same.
//
// kCausal: one Q tile per workgroup, the longest first.  kRagged: any Nq and Nk, as in fa2_fwd_kernel, but the count of K/V
// tiles is not padded: a wavefront runs the tiles that its own rows see and only keeps the boundaries of the others.
template <int DT, int kD, bool kCausal, bool kRagged>
__global__ __launch_bounds__(kWaves * 64, kD == 64 ? 2 : 1) void fa2_stage_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V, uint16_t* __restrict__ O,
    float* __restrict__ LSE, int H, int Nq, int Nk, float scale_log2e, int n_qtiles, int total) {
  using E = Elem<DT>;
  using T = Tile<kD>;
  constexpr int kGroups = groups_of(kD);
  constexpr int kWaveRows = 32 * kGroups;
  constexpr int kStageRows = kWaveRows * kWaves;        // query rows per workgroup
  constexpr int kKSteps = kD / 16;                      // MFMA steps along d of GEMM-I: fragments of K per stage
  constexpr int kDBlocks = kD / 32;                     // 32-row blocks of O^T
  constexpr int kVFrags = kStageKeys / 16 * kDBlocks;   // fragments of V per stage
  constexpr int kLoads = T::kLoadsPerWave;              // 1 KiB wavefront loads per tile and wavefront
  using std::false_type;
  using std::true_type;

  // separate objects, so that the compiler can tell a load in flight into one from reads of another
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds0[T::kElems];
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds1[T::kElems];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds0[T::kElems];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds1[T::kElems];
  __shared__ __attribute__((aligned(16))) uint16_t o_slab[kWaves * 1024];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, hh = lane >> 5;   // query within the group, half of the wavefront

  int bh, qt;
  {
    const int xcd = blockIdx.x % kXcds, idx = blockIdx.x / kXcds;
    const int heads = total / n_qtiles;
    if constexpr (!kCausal) {
      // a contiguous range of Q tiles per XCD: those of one head share an L2
      const int per = total / kXcds, rem = total % kXcds;
      const int tile = xcd * per + min(xcd, rem) + idx;
      bh = tile / n_qtiles;
      qt = tile - bh * n_qtiles;
    } else if (heads % kXcds == 0) {
      // Heads stay on one XCD, in groups of 128 workgroups, two rounds of its CUs at d = 64 and four at d = 256 (at least four
      // heads): within a group the longest Q tiles of all heads start first, so that the short ones fill the end, and a group's K and V stay in the L2
      // (all heads as one group: 1...5 % slower at N = 1024...4096).
      const int mine = heads / kXcds;
      const int groups = max(1, mine / max(4, (128 + n_qtiles - 1) / n_qtiles));
      const int size = mine / groups, longer = mine - size * groups;   // the first `longer` groups hold one head more
      int first, n = size;
      if (idx < longer * (size + 1) * n_qtiles) {
        n = size + 1;
        first = idx / (n * n_qtiles) * n;
      } else {
        first = longer + (idx - longer * n_qtiles) / (size * n_qtiles) * size;
      }
      const int at = idx - first * n_qtiles, c = at / n;
      bh = (first + at - c * n) * kXcds + xcd;
      qt = n_qtiles - 1 - c;
    } else {
      const int c = blockIdx.x / heads;
      bh = blockIdx.x - c * heads;
      qt = n_qtiles - 1 - c;
    }
  }

  const size_t row_stride = (size_t)H * kD;
  const size_t q_base = ((size_t)(bh / H) * Nq * H + (size_t)(bh % H)) * kD;
  const size_t kv_base = ((size_t)(bh / H) * Nk * H + (size_t)(bh % H)) * kD;
  const uint32_t head_bytes = (uint32_t)(((size_t)(Nk - 1) * row_stride + kD) * 2);
  const __amdgpu_buffer_rsrc_t k_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(K + kv_base), 0, (int)head_bytes, kBufferFlags);
  const __amdgpu_buffer_rsrc_t v_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(V + kv_base), 0, (int)head_bytes, kBufferFlags);
  const uint32_t row_bytes = (uint32_t)(row_stride * 2), tile_bytes = kBc * row_bytes;

  // Tile j of K or V into LDS, straight from memory; rows past the last key are filled with copies of it.
  auto stage_in = [&](auto is_k, int j, uint16_t* lds_tile) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc = decltype(is_k)::value ? k_rsrc : v_rsrc;
    const bool partial = kRagged && (j + 1) * kBc > Nk;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int chunk = 64 * (wave * kLoads + i) + lane;
      const int row = chunk / T::kChunksPerRow, pos = chunk % T::kChunksPerRow;
      const int swz = decltype(is_k)::value ? T::swz_k(row) : T::swz_v(row);
      uint32_t src = (uint32_t)row * row_bytes + 16u * (uint32_t)(pos ^ swz), at = (uint32_t)j * tile_bytes;
      if (partial) {
        src = (uint32_t)min(j * kBc + row, Nk - 1) * row_bytes + 16u * (uint32_t)(pos ^ swz);
        at = 0;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(lds_tile + 512 * (wave * kLoads + i)), 16, (int)src,
                                               (int)at, 0, 0);
    }
  };

  // Operand fragments from LDS, of the half tile that the pointer names.
  int k_addr[kKSteps], v_addr[kDBlocks];
#pragma unroll
  for (int ks = 0; ks < kKSteps; ++ks) k_addr[ks] = r * kD + 8 * ((2 * ks + hh) ^ T::swz_k(r));
  {
    const int l16 = lane & 15, row0 = 4 * hh + (l16 >> 2);
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db) {
      const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
      v_addr[db] = row0 * kD + 8 * (chunk ^ T::swz_v(row0)) + 4 * (l16 & 1);
    }
  }
  auto k_frag = [&](const uint16_t* kt, int ks) __attribute__((always_inline)) -> u32x4 {
    return *reinterpret_cast<const u32x4*>(kt + k_addr[ks]);
  };
  auto v_frag = [&](const uint16_t* vt, int f) __attribute__((always_inline)) -> u32x4 {
    const uint16_t* p = vt + v_addr[f % kDBlocks] + f / kDBlocks * 16 * kD;
    const u32x2 lo = lds_read_tr16(p), hi = lds_read_tr16(p + 8 * kD);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };

  u32x4 qf[kGroups][kKSteps];
  f32x16 ot[kGroups][kDBlocks];
  f32x16 st[2][kGroups];      // S^T of stage s in st[s % 2]
  u32x4 pf[2][kGroups][2];    // P~ of stage s in pf[s % 2]
  float mc_ref[kGroups], l_run[kGroups];   // reference point of the exponentials (scaled, log2), row sum
  float part[kGroups][2];                  // row sums of the current K/V tile's first half: even and odd elements of a lane

  auto zeros = []() __attribute__((always_inline)) {
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
  };
  // S = -inf where the key comes after `visible` (the key's position in the stage minus 4 hh)
  auto apply_mask = [&](f32x16 (&s)[kGroups], int visible) __attribute__((always_inline)) {
    asm volatile("" : "+v"(visible));   // compared here, not hoisted: 32 comparison results would fill the scalar registers
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v / 4) + (v % 4) > visible + (kCausal ? 32 * g : 0)) s[g][v] = -INFINITY;
  };
  // Element v of S for the softmax.  At d = 256 S is in accumulation registers and is read where it is needed (the compiler
  // reads all of it at the start of a stage).  It does not see that this reads what MFMAs wrote: 16 others stand between.
  auto logit = [&](const f32x16& s, int v) __attribute__((always_inline)) {
    if constexpr (kD == 64) {
      return s[v];
    } else {
      float x;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(s[v]));
      return x;
    }
  };
  // Row maximum of the logits of one group that a lane holds in `s` (without its partner in the other half of the wavefront).
  auto lane_max = [&](f32x16& s) __attribute__((always_inline)) {
    // The wait states that the inline maxima need after an MFMA that wrote S; S goes through the asm, or the maxima could be
    // scheduled before it (a maximum of unfinished sums is still a valid reference, but not the same one in every run).
    if constexpr (kD == 64) asm volatile("s_nop 15\n\ts_nop 3" : "+v"(s));
    else asm volatile("s_nop 15\n\ts_nop 3" : "+a"(s));
    float mx = max2_raw(s[0], s[1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) mx = max3_raw(mx, s[v], s[v + 1]);
    return mx;
  };
  // The reference point for a row maximum.  It stops at the lowest finite number, for logits that overflow once scaled (keys
  // that a caller masks with the type's lowest value).
  auto reference = [&](float mx) __attribute__((always_inline)) {
    return fmaxf(max_with_partner_half_raw(mx) * scale_log2e, kLowest);
  };

  // One stage (parity x), two groups: GEMM-II with pf[1 - x] and the V half tile `vt`, mixed with the softmax of st[x][0] ->
  // pf[x][0], then GEMM-I of the K half tile `kt` -> st[1 - x], mixed with the softmax of st[x][1].  In this order S of group 0 is dead
  // when GEMM-I writes its successor (all at once would take 40 registers too many), and that successor, which the next
  // stage needs first, is done four MFMAs before this stage ends.  The first stage has neither product, the last no GEMM-I.
  auto stage = [&](auto x_tag, auto gemm1_tag, auto gemm2_tag, const uint16_t* kt, const uint16_t* vt)
      __attribute__((always_inline)) {
    constexpr int x = decltype(x_tag)::value;
    constexpr bool kGemm1 = decltype(gemm1_tag)::value, kGemm2 = decltype(gemm2_tag)::value;
    constexpr int kN1 = kGemm1 ? kKSteps : 0, kN2 = kGemm2 ? kVFrags : 0, kFrags = kN1 + kN2;
    constexpr int kRing = kGroups == 2 ? 4 : 8;   // fragments in flight
    static_assert(kGroups == 1 || kKSteps == kRing, "the K fragments are all held, for the second group");
    // two groups: those of V first; one group: those of K
    auto frag = [&](int f) __attribute__((always_inline)) -> u32x4 {
      if constexpr (kGroups == 2) return f < kN2 ? v_frag(vt, f) : k_frag(kt, f - kN2);
      else return f < kN1 ? k_frag(kt, f) : v_frag(vt, f - kN1);
    };
    u32x4 ring[kRing];
#pragma unroll
    for (int f = 0; f < (kFrags < kRing ? kFrags : kRing); ++f) ring[f] = frag(f);

    // The softmax of one group, a pair of elements after each of the 8 MFMAs that `mfma` issues (one group: over four): the
    // exponents of the next pair, the exponentials of this one, sum and P~ of the last one.  Each part is pinned where it stands; left free, the
    // compiler moves all of it behind the MFMAs, to the first use of P~.
    auto softmax = [&](auto g_tag, auto mfma) __attribute__((always_inline)) {
      constexpr int g = decltype(g_tag)::value;
      float e[2][2], p[2][2], sum[2];
      auto exponents = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) e[n & 1][i] = __builtin_fmaf(logit(st[x][g], 2 * n + i), scale_log2e, -mc_ref[g]);
        asm volatile("" : "+v"(e[n & 1][0]), "+v"(e[n & 1][1]));
      };
      auto add_and_pack = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = n > 0 ? sum[i] + p[n & 1][i] : x == 0 ? p[0][i] : part[g][i] + p[0][i];
        uint32_t packed = E::pack2(p[n & 1][0], p[n & 1][1]);
        asm volatile("" : "+v"(packed), "+v"(sum[0]), "+v"(sum[1]));
        pf[x][g][n / 4][n % 4] = packed;
      };
      exponents(0);
      __builtin_amdgcn_sched_barrier(0);
      static_for<8>([&](auto n_tag) __attribute__((always_inline)) {
        constexpr int n = decltype(n_tag)::value;
        auto exponential = [&](int i) __attribute__((always_inline)) {
          p[n & 1][i] = __builtin_amdgcn_exp2f(e[n & 1][i]);
          asm volatile("" : "+v"(p[n & 1][i]));
        };
        if constexpr (kGroups == 2) {
          mfma(n_tag);
          if constexpr (n + 1 < 8) exponents(n + 1);
          exponential(0);
          exponential(1);
          if constexpr (n > 0) add_and_pack(n - 1);
        } else {
          static_assert(kKSteps + kVFrags == 4 * 8);
          mfma(Int<4 * n>{});
          if constexpr (n + 1 < 8) exponents(n + 1);
          __builtin_amdgcn_sched_barrier(0);
          mfma(Int<4 * n + 1>{});
          exponential(0);
          __builtin_amdgcn_sched_barrier(0);
          mfma(Int<4 * n + 2>{});
          exponential(1);
          __builtin_amdgcn_sched_barrier(0);
          mfma(Int<4 * n + 3>{});
          if constexpr (n > 0) add_and_pack(n - 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      add_and_pack(7);
      // A P~ beyond the limit shows in the row's partial sums (of either half of the wavefront).  Then the reference of that
      // row moves, O and its sums are rescaled, and the stage's exponentials are taken again; S is still there, and so far
      // no product has used P~.  The reference only rises: the sums may hold the first half's, and the limit be passed by
      // keys far below it (falling with them, by up to 2^15 a tile, O and l would leave fp32; a row whose keys here are all at
      // or below its reference has P~ <= 1 and stays).
      if (__builtin_amdgcn_ballot_w64(sum[0] + sum[1] > kSumLimit) != 0) {
        const uint32_t u = __builtin_bit_cast(uint32_t, sum[0] + sum[1]);
        const auto both = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        const bool move = __builtin_bit_cast(float, (uint32_t)both[0]) > kSumLimit ||
                          __builtin_bit_cast(float, (uint32_t)both[1]) > kSumLimit;
        const float to = fmaxf(mc_ref[g], reference(lane_max(st[x][g])));
        // a row that stays gets exactly 1: its bits must not depend on the other rows of the wavefront
        const float alpha = move ? __builtin_amdgcn_exp2f(mc_ref[g] - to) : 1.0f;
        if (move) mc_ref[g] = to;
        l_run[g] *= alpha;
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) ot[g][db][v] *= alpha;
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = x == 0 ? 0.f : part[g][i] * alpha;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(st[x][g][2 * n], scale_log2e, -mc_ref[g]));
          const float b = __builtin_amdgcn_exp2f(__builtin_fmaf(st[x][g][2 * n + 1], scale_log2e, -mc_ref[g]));
          sum[0] += a;
          sum[1] += b;
          pf[x][g][n / 4][n % 4] = E::pack2(a, b);
        }
      }
      // (summed tile by tile, in the tile kernel's order: both give the same bits)
      if constexpr (x == 0) {
        part[g][0] = sum[0];
        part[g][1] = sum[1];
      } else {
        l_run[g] += sum[0] + sum[1];
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (kGroups == 2) {
      // fragment f for both groups, then the one kRing ahead into its place
      softmax(Int<0>{}, [&](auto m) __attribute__((always_inline)) {
        constexpr int f = decltype(m)::value / kGroups, g = decltype(m)::value % kGroups;
        if constexpr (kGemm2) {
          ot[g][f % kDBlocks] = E::mfma(ring[f], pf[1 - x][g][f / kDBlocks], ot[g][f % kDBlocks]);
          if constexpr (g == kGroups - 1 && f + kRing < kFrags) ring[f] = frag(f + kRing);
        }
      });
      softmax(Int<1>{}, [&](auto m) __attribute__((always_inline)) {
        constexpr int ks = decltype(m)::value % kKSteps, g = decltype(m)::value / kKSteps;
        if constexpr (kGemm1) st[1 - x][g] = E::mfma(ring[ks], qf[g][ks], ks == 0 ? zeros() : st[1 - x][g]);
      });
    } else {
      softmax(Int<0>{}, [&](auto m) __attribute__((always_inline)) {
        constexpr int i = decltype(m)::value;
        constexpr bool kFirst = i < kKSteps;
        constexpr int n = i - kKSteps;   // of GEMM-II
        if constexpr (kFirst ? kGemm1 : kGemm2) {
          constexpr int f = kGemm1 ? i : n;
          if constexpr (kFirst) st[1 - x][0] = E::mfma(ring[f % kRing], qf[0][i], i == 0 ? zeros() : st[1 - x][0]);
          else ot[0][n % kDBlocks] = E::mfma(ring[f % kRing], pf[1 - x][0][n / kDBlocks], ot[0][n % kDBlocks]);
          if constexpr (f + kRing < kFrags) ring[f % kRing] = frag(f + kRing);
        }
      });
    }
  };

  constexpr int kWaitLoads = 0x0F70;         // s_waitcnt vmcnt(0)
  constexpr int kHalf = kStageKeys * kD;     // elements of half a K/V tile
  const int row_first = qt * kStageRows + wave * kWaveRows;
  const int k_tiles = (Nk + kBc - 1) / kBc;
  const int n_tiles = kCausal ? min((qt + 1) * (kStageRows / kBc), k_tiles) : k_tiles;   // of the workgroup
  // of this wavefront's rows (none if they all lie past the last query)
  const int n_my = kRagged && row_first >= Nq ? 0 : kCausal ? min((row_first + kWaveRows - 1) / kBc + 1, n_tiles) : n_tiles;

  stage_in(true_type{}, 0, k_lds0);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int row = row_first + 32 * g + r;
    const uint16_t* qp = Q + q_base + (size_t)(kRagged ? min(row, Nq - 1) : row) * row_stride + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) qf[g][ks] = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
  }
  stage_in(false_type{}, 0, v_lds0);
  if (n_tiles > 1) {
    stage_in(true_type{}, 1, k_lds1);
    stage_in(false_type{}, 1, v_lds1);
  }
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db) ot[g][db] = zeros();
    l_run[g] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) asm volatile("" : "+v"(qf[g][ks]));   // landed before the loop
  }
  __builtin_amdgcn_s_waitcnt(kWaitLoads);
  __syncthreads();

  // the last key that a lane's row sees, or the last key, minus 4 hh; whether stage s crosses it for some row of the wavefront
  const int last_key = (kCausal ? row_first + r : Nk - 1) - 4 * hh;
  auto mask = [&](auto x_tag, int s) __attribute__((always_inline)) {
    const int end = kStageKeys * (s + 1);
    if (kCausal ? end - 1 > row_first : kRagged && end > Nk) apply_mask(st[decltype(x_tag)::value], last_key - kStageKeys * s);
  };
  int j = 0;   // K/V tile
  if (n_my > 0) {
    // S of K tile 0, both halves, and its row maxima; then stage 0
    static_for<2>([&](auto half) __attribute__((always_inline)) {
      constexpr int x = decltype(half)::value;
#pragma unroll
      for (int ks = 0; ks < kKSteps; ++ks) {
        const u32x4 f = k_frag(k_lds0 + x * kHalf, ks);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) st[x][g] = E::mfma(f, qf[g][ks], ks == 0 ? zeros() : st[x][g]);
      }
    });
    mask(Int<0>{}, 0);
    mask(Int<1>{}, 1);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) mc_ref[g] = reference(max2_raw(lane_max(st[0][g]), lane_max(st[1][g])));
    stage(Int<0>{}, false_type{}, false_type{}, k_lds0, v_lds0);
  }
  __syncthreads();   // K tile 0 is dead
  if (n_tiles > 2) stage_in(true_type{}, 2, k_lds0);

  // Stages 2j + 1 and 2j + 2, which read K tile j + 1 and V tile j.
  auto body = [&](const uint16_t* kt, const uint16_t* vt) __attribute__((always_inline)) {
    mask(Int<1>{}, 2 * j + 1);
    stage(Int<1>{}, true_type{}, true_type{}, kt, vt);
    mask(Int<0>{}, 2 * j + 2);
    stage(Int<0>{}, true_type{}, true_type{}, kt + kHalf, vt + kHalf);
  };
  // After it the tiles of the next body have landed, and those of this one are dead and replaced.
  auto boundary = [&](uint16_t* k_fill, uint16_t* v_fill) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kWaitLoads);
    __syncthreads();
    if (j + 3 < n_tiles) stage_in(true_type{}, j + 3, k_fill);
    if (j + 2 < n_tiles) stage_in(false_type{}, j + 2, v_fill);
    ++j;
  };
  while (j + 1 < n_my) {
    body(k_lds1, v_lds0);
    boundary(k_lds1, v_lds0);
    if (j + 1 >= n_my) break;
    body(k_lds0, v_lds1);
    boundary(k_lds0, v_lds1);
  }
  if (n_my > 0) {
    // the last stage, and GEMM-II of its P~
    const uint16_t* vt = j & 1 ? v_lds1 : v_lds0;
    mask(Int<1>{}, 2 * j + 1);
    stage(Int<1>{}, false_type{}, true_type{}, k_lds0, vt);
#pragma unroll
    for (int f = 0; f < kVFrags; ++f) {
      const u32x4 x = v_frag(vt + kHalf, f);
#pragma unroll
      for (int g = 0; g < kGroups; ++g) ot[g][f % kDBlocks] = E::mfma(x, pf[1][g][f / kDBlocks], ot[g][f % kDBlocks]);
    }
  }
  if constexpr (kCausal || kRagged) {   // the other wavefronts' tiles
    while (j + 1 < n_tiles) boundary(j & 1 ? k_lds0 : k_lds1, j & 1 ? v_lds1 : v_lds0);
  }

  // O / l as 64-byte pieces of rows through the wavefront's LDS slab, and LSE
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int row0 = row_first + 32 * g;
    const float l_tot = sum_with_partner_half(l_run[g]), inv_l = 1.0f / l_tot;
    uint16_t* slab = o_slab + wave * 1024;
    const int rrow = lane >> 2, rchunk = lane & 3;
    uint16_t* orow = O + q_base + (size_t)(row0 + rrow) * row_stride + 8 * rchunk;
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const u32x2 w = {E::pack2(ot[g][db][4 * c + 0] * inv_l, ot[g][db][4 * c + 1] * inv_l),
                         E::pack2(ot[g][db][4 * c + 2] * inv_l, ot[g][db][4 * c + 3] * inv_l)};
        *reinterpret_cast<u32x2*>(slab + r * 32 + 8 * (c ^ ((r >> 2) & 3)) + 4 * hh) = w;
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int row = rrow + 16 * half;
        const u32x4 piece = *reinterpret_cast<const u32x4*>(slab + row * 32 + 8 * (rchunk ^ ((row >> 2) & 3)));
        if (!kRagged || row0 + row < Nq)
          *reinterpret_cast<u32x4*>(orow + (size_t)(16 * half) * row_stride + 32 * db) = piece;
      }
    }
    if (LSE != nullptr && hh == 0 && (!kRagged || row0 + r < Nq))
      LSE[(size_t)bh * Nq + row0 + r] = mc_ref[g] * 0.69314718055994530942f + __builtin_logf(l_tot);
  }
}

template <int DT, int kD, bool kCausal, bool kRagged> int launch(const Problem& p) {
  constexpr int kStageRows = 32 * groups_of(kD) * kWaves;
  const int n_q = (p.Nq + kStageRows - 1) / kStageRows, total = p.B * p.H * n_q;
  return enqueue(fa2_stage_kernel<DT, kD, kCausal, kRagged>, total, kWaves * 64, p.stream, static_cast<const uint16_t*>(p.Q),
                 static_cast<const uint16_t*>(p.K), static_cast<const uint16_t*>(p.V), static_cast<uint16_t*>(p.O), p.LSE, p.H,
                 p.Nq, p.Nk, p.scale_log2e, n_q, total);
}

template <int DT, int kD> int launch(const Problem& p) {
  const bool ragged = p.Nq % (32 * groups_of(kD) * kWaves) != 0 || p.Nk % kBc != 0;
  return p.causal ? (ragged ? launch<DT, kD, true, true>(p) : launch<DT, kD, true, false>(p))
                  : (ragged ? launch<DT, kD, false, true>(p) : launch<DT, kD, false, false>(p));
}

}  // namespace

bool stage_tiles(const Problem& p, int* rc) {
  if (!stage_accepts(p.B, p.H, p.Nq, p.Nk, p.d, p.causal)) return false;
  if (p.d == 64) *rc = p.dtype == FA2_FP16 ? launch<FA2_FP16, 64>(p) : launch<FA2_BF16, 64>(p);
  else *rc = p.dtype == FA2_FP16 ? launch<FA2_FP16, 256>(p) : launch<FA2_BF16, 256>(p);
  return true;
}

}  // namespace fa2
