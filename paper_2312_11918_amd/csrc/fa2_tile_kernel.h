// FlashAttention-2 forward pass for gfx950 (MI355X, CDNA4): the tile kernel of libfa2 (whole launches: fa2_fwd.hip,
// launches with the keys split: fa2_split.hip).
//
// Follows Algorithm 2 of arXiv 2312.11918 (tile of query rows per workgroup, loop over K/V tiles,
// GEMM-I, online softmax, GEMM-II, final division by the row sum) with a data flow designed for
// 64-lane wavefronts and MFMA instead of the paper's Hopper TMA/WGMMA pipeline:
//
//  * Both products are computed TRANSPOSED, S^T = K Q^T and O^T = V^T P^T, with
//    v_mfma_f32_32x32x16.  In the 32x32 accumulator layout a lane owns one column, so with the
//    transposed products every lane owns ONE QUERY: the row maximum and row sum of Algorithm 2 are
//    in-lane reductions plus a single exchange between lane l and lane l+32, the rescale factor
//    exp(m_old - m_new) is a per-lane scalar, and the S^T accumulator registers, rounded to 16 bit,
//    already have the register layout of the B operand of the second product (Section 4.2 of the
//    paper solves the same accumulator-to-operand problem for WGMMA by re-indexing the fragment).
//    The only price is that the key index inside a 16-key MFMA step is permuted; a contraction
//    does not care about the order of its terms, and V is read from LDS with the same permutation.
//  * V is the operand whose contraction index (the key) is not contiguous in memory (Section 4.1
//    of the paper takes a transposed shared-memory view).  Here V stays row-major in LDS and is
//    read with ds_read_b64_tr_b16, the LDS transpose load of gfx950.
//  * K/V tiles are double-buffered (or held in a ring of four) in LDS and the next tiles' global loads are
//    issued before the current tile's MFMAs (the copy/GEMM overlap of Section 6, without TMA or mbarriers;
//    the producer/consumer hand-over is a barrier per tile in one tile shape and counters in LDS in the other).
#ifndef FA2_TILE_KERNEL_H_
#define FA2_TILE_KERNEL_H_
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "fa2_internal.h"
#include "fa2_wide_plan.h"

using fa2::enqueue;
using fa2::kCUs;
using fa2::wide_staged_tile;

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;            // wavefronts per workgroup of the 128-row shape
constexpr int kBr = 32 * kWaves;     // query rows per workgroup (32 per wavefront)
constexpr int kBc = 64;              // keys per K/V tile
constexpr int kSpinLimit = 1 << 18;  // polls of the arrival count before a wavefront gives up (tens of milliseconds)
constexpr int kXcds = 8;             // accelerator complex dies; workgroup i is dispatched to XCD i % 8
constexpr float kLowest = -3.402823466e38f;   // the lowest finite number
constexpr float kLazyLog2 = 8.0f;    // the rowmax reference moves only when exceeded by 2^8

// Element-type specifics: the MFMA flavour and the fp32 -> 16-bit pack (round to nearest even).
// Compile-time loop: calls f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N-1>{}).
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F&&>(f));
}

template <int DT> struct Elem;
template <> struct Elem<FA2_FP16> {
  static __device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    f16x2 r = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, r);
  }
};
template <> struct Elem<FA2_BF16> {
  static __device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    bf16x2 r = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, r);
  }
};

// Value held by the partner lane (l ^ 32): v_permlane32_swap exchanges the upper half of one
// register with the lower half of another, which leaves each half's value broadcast in one result.
__device__ __forceinline__ float sum_with_partner_half(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Maximum of two / three values as single instructions.  fmaxf() makes the compiler quiet possible
// signalling NaNs of every input first (one extra instruction each); inputs here are finite by contract.
__device__ __forceinline__ float max2_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float max3_raw(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float max_with_partner_half_raw(float x) {
  uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return max2_raw(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// LDS transpose load: within each group of 16 lanes the 16 x 4 block of 16-bit elements addressed
// by the lanes (lane p supplies 4 consecutive elements) is transposed, so that lane i receives
// element (i % 4) of lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4.
__device__ __forceinline__ u32x2 lds_read_tr16(const uint16_t* p) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
  return __builtin_bit_cast(u32x2, v);
}

// LDS tile geometry.  A K or V tile is kBc rows of D 16-bit elements, stored row-major WITHOUT
// padding (the direct global->LDS loads write 1 KiB of consecutive LDS per wavefront instruction),
// with the 16-byte chunks of every row permuted by an XOR so that the operand reads are free of
// bank conflicts (the role of the paper's 128-byte shared-memory swizzle, Section 3.2):
//   K is read with 16-byte loads, lane = key row: 16 consecutive rows must land in 16 different
//     16-byte slots of the 256-byte bank period            -> chunk ^= f(row) over the whole period;
//   V is read with the transpose load, 4 key rows x 32 bytes per group of 16 lanes: the 4 rows must
//     land in different 64-byte quarters of the bank period -> chunk ^= g(row) << 2.
template <int D> struct Tile {
  static constexpr int kChunksPerRow = D / 8;                      // 16-byte chunks per row
  static constexpr int kElems = kBc * D;                           // elements per tile
  static constexpr int kLoadsPerWave = kElems * 2 / 1024 / kWaves; // 1 KiB wavefront loads per tile and wave
  static __device__ __forceinline__ int swz_k(int row) { return D >= 128 ? (row & 15) : ((row >> 1) & 7); }
  static __device__ __forceinline__ int swz_v(int row) { return (D >= 128 ? (row & 3) : ((row >> 1) & 1)) << 2; }
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;
constexpr int kBufferFlags = 0x00020000;  // raw buffer descriptor word 3 for gfx9-family: 32-bit data format, no swizzle

// -------------------------------------------------------------------------------------------------
// Kernel with 32 query rows per wavefront.  kWv wavefronts form a workgroup (32*kWv rows); K and V tiles
// cycle through kNBuf LDS buffers each.  Two shapes are instantiated:
//   4 wavefronts, 2 buffers: 128 rows per workgroup, 2 workgroups per CU;
//   8 wavefronts, 4 buffers: 256 rows per workgroup, 1 workgroup per CU, global loads issued three
//                            tiles ahead and half the L2->LDS traffic per FLOP.  This shape has no barrier in
//                            its loop (arrival counters in LDS, see kFlagSync), takes `chain` Q tiles per
//                            workgroup over one running K/V stream (see kChain) and stores O as pieces of rows.
// Either way a SIMD runs two wavefronts, so one wavefront's softmax arithmetic overlaps the other's MFMAs.
// The second has a form for partial tiles (kRagged) at d = 128 (fa2_wide.hip), the first a form with the keys cut (kSplit).
// `total_tiles` is the number of workgroups; `chain` is more than 1 where whole rounds of the CUs are chained: in the 8-wavefront
// shape, and at d = 256 on whole tiles.
//
// kCausal applies the optional mask of S (Section 2 of the paper: entries of S may be set to -inf before the
// softmax; here those with key index > query index).  A Q tile then stops at its diagonal: it visits
// (qt+1)*kNBuf K/V tiles instead of N/kBc, only the last kNBuf of them straddle the diagonal and need the
// element-wise mask, and a workgroup takes two Q tiles of one head, the p-th from the end and the p-th from the
// start, whose tile counts add up to the same number for every p.
//
// kRagged lifts the restriction to whole tiles: Nq query rows and Nk keys of any size >= 1.  Query rows past
// Nq-1 are computed from a copy of the last row and not stored; K/V rows past Nk-1 are staged as copies of
// the last row (finite data; as zeros in the 256-row shape) and their columns of S are set to -inf in the last kNBuf tiles, the only ones
// that can hold them; the tile count is rounded up to a multiple of kNBuf (a padding tile's arithmetic is left out).
//
// kSplit (with kRagged) is for problems whose Q tiles are too few to fill the chip.  Two cuts of the keys:
//  * d <= 128: a workgroup of eight wavefronts for 128 rows.  Wavefronts 0-3 (half 0) take the even K/V tiles, 4-7
//    (half 1) the odd ones, each half with its own LDS buffers, and the two are merged through LDS at the end.  A CU
//    that would hold one workgroup of four wavefronts, one per SIMD, thus has two per SIMD at work;
//  * a workgroup takes a slice of split.chunk K/V tiles only, and leaves O and l unnormalised, with their reference
//    point, in a workspace for fa2_split_merge_kernel.  Tile indices and Nk are then relative to the slice.  A Q tile
//    whose keys all lie in one slice (causal: the first ones) is stored as usual.
// One pass per workgroup; under the causal mask Q tiles are not paired.
//
struct SplitArgs {
  float* part_o = nullptr;   // [Q tile over all heads][slice][wavefront][register quad][lane] of 4: O^T as it is held
  float* part_ml = nullptr;  // [Q tile over all heads][slice][row][2]: reference point (scaled, log2), row sum
  int chunk = 0;             // K/V tiles per slice, a multiple of 4
  int slices = 1;            // slices of the longest Q tile
  int items = 0;             // workgroups per head
};

// Wavefronts per SIMD: at d = 64 the 4-wavefront kernels are held to 168 registers, three workgroups per CU.  With the
// causal mask and partial tiles they took 195 before, two workgroups per CU: B50 H16 N330 fp16 54.7 -> 46.8 us, B60 H24 N140
// fp16 36.2 -> 31.5, B30 H8 N700 bf16 34.7 -> 30.2; level where two workgroups per CU hold the whole grid (see kOneOffset).
template <int DT, int D, int kWv, int kNBuf, bool kCausal, bool kRagged, bool kSplit = false>
__global__ __launch_bounds__(kWv * 64, kWv == 4 && D == 64 ? 3 : kWv == 4 && D <= 128 ? 2 : 1) void fa2_fwd_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ LSE, int H, int Nq, int Nk, float scale_log2e, int n_qtiles,
    int total_tiles, int chain, SplitArgs split) {
  using E = Elem<DT>;
  using T = Tile<D>;
  using std::false_type;
  using std::true_type;
  static_assert(kNBuf == 2 || kNBuf == 4, "two or four LDS buffers per operand");
  constexpr bool kHalves = kSplit && kWv == 8;
  constexpr int kRowWaves = kHalves ? 4 : kWv;   // wavefronts with rows of their own
  constexpr int kRows = 32 * kRowWaves;          // query rows per workgroup
  static_assert(!kSplit || (kRagged && kNBuf == 2), "slices of keys: the 128-row shape with partial tiles");
  static_assert(kRows == kNBuf * kBc, "a Q tile spans exactly kNBuf K/V tiles (the causal tile count relies on it)");
  constexpr int kKSteps = D / 16;   // MFMA steps along d for S^T = K Q^T
  constexpr int kDBlocks = D / 32;  // 32-row blocks of O^T
  constexpr int kKBlocks = kBc / 32;  // 32-key blocks of S^T
  constexpr int kTSteps = kBc / 16;   // MFMA steps along the keys for O^T = V^T P^T
  constexpr int kSteps1 = kKBlocks * kKSteps;  // MFMAs of GEMM-I per tile
  constexpr int kSteps2 = kTSteps * kDBlocks;  // MFMAs of GEMM-II per tile
  constexpr int kRing = 4;                     // operand fragments in flight between LDS and the MFMAs
  constexpr int kLoadsPerWave = T::kElems * 2 / 1024 / kRowWaves;  // 1 KiB wavefront loads per tile and wavefront
  constexpr bool kSplitRefill = kNBuf == 2 && D == 256;    // K and V refills issued as two separate bursts
  // The 8-wavefront shape has no barrier in its loop: its wavefronts count their arrivals at the end of every
  // iteration in LDS and go on as soon as all have finished the iteration BEFORE.  One barrier per tile would
  // start the two wavefronts of every SIMD in the same phase tile after tile, softmax against softmax and MFMAs
  // against MFMAs; with a tile of slack they drift apart and fill each other's gaps.
  constexpr bool kFlagSync = kWv == 8 && !kHalves;
  // A workgroup of that shape takes `chain` Q tiles (under the causal mask: pairs of Q tiles, and the two of a
  // pair as well) one after the other, and the K/V stream runs on
  // from one to the next (after the last K/V tile of one comes the first of the next): only the first Q tile pays
  // for filling the ring, and with one workgroup per CU nothing else would cover that time.  The Q tiles of a
  // workgroup are spaced by the number of workgroups of its XCD, so that at any time the workgroups of an XCD
  // work on neighbouring Q tiles, a few heads whose K and V fit its L2, as they do without chaining.
  // The d = 256 kernel, also one workgroup per CU, chains in the same way when it runs on whole tiles.
  constexpr bool kChain = kFlagSync || (kWv == 4 && D == 256 && !kRagged);

  // The buffers are separate objects on purpose: the compiler then knows that a load in flight into one
  // buffer cannot alias the operand reads from another.  (With kNBuf == 2 the last two pairs are unused.)
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds0[T::kElems * (kHalves ? 2 : 1)];
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds1[T::kElems * (kHalves ? 2 : 1)];
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds2[kNBuf == 4 ? T::kElems : 8];
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds3[kNBuf == 4 ? T::kElems : 8];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds0[T::kElems * (kHalves ? 2 : 1)];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds1[T::kElems * (kHalves ? 2 : 1)];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds2[kNBuf == 4 ? T::kElems : 8];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds3[kNBuf == 4 ? T::kElems : 8];
  __shared__ f32x2 ml_lds[kHalves ? 2 * kRows : 1];  // reference point and row sum of either half, for the other
  // kFlagSync: wavefronts that finished iteration j, counted in entry j % 4.  kHalves: arrivals of either half at its barrier
  // (entries 0 and 1), and whether a wavefront has given up waiting (entry 2)
  __shared__ uint32_t arrivals[4];
  // kRowStores: 32 rows x 32 columns of O per wavefront, through which the result is turned from one query per
  // lane into whole 64-byte pieces of rows before it is stored: a lane-per-query store touches 64 rows per
  // instruction, and the epilogue of a Q tile then costs thousands of cycles that only partly hide behind the other
  // workgroups of the CU (measured: +2 % at N = 2048, +5...10 % at N <= 1024, more with one workgroup per CU)
  // (every kernel but one: the 128-row shape at d = 128 with both the causal mask and partial tiles has no
  // registers left for it)
  constexpr bool kRowStores = kSplit || !(kWv == 4 && D == 128 && kCausal && kRagged);
  __shared__ __attribute__((aligned(16))) uint16_t o_slab[kRowStores ? kWv * 1024 : 8];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform, kept in a scalar register
  const int wave = kHalves ? wave_all % kRowWaves : wave_all;
  const int half = kHalves ? wave_all / kRowWaves : 0;
  const int half_lds = half * T::kElems;  // this half's part of a buffer
  // K/V tile (of the slice) behind this half's tile j
  auto tile_at = [&](int j) { return kHalves ? 2 * j + half : j; };
  const int r = lane & 31;   // column of the 32x32 MFMA tile owned by this lane = query within the wave
  const int hh = lane >> 5;  // which half of the wavefront

  // Q-tile scheduling (Algorithm 2's outer loop, parallel over workgroups).  Workgroups are dealt
  // round-robin to the 8 XCDs, each with its own L2: give every XCD a contiguous range of tiles so
  // that the Q tiles of one head, which all stream the same K and V, share one L2.
  int tile, chain_stride = 0;  // kChain: the Q tile (pair) of chain step c is tile + c * chain_stride, over all heads
  {
    const int wg = blockIdx.x;
    const int per = total_tiles / kXcds, rem = total_tiles % kXcds;
    const int xcd = wg % kXcds, idx = wg / kXcds;
    const int first = xcd * per + (xcd < rem ? xcd : rem);  // first workgroup of this XCD's range
    if constexpr (kChain) {
      tile = first * chain + idx;
      chain_stride = per + (xcd < rem ? 1 : 0);
    } else {
      tile = first + idx;
    }
  }
  // Under the causal mask the work of Q tile qt grows like qt + 1, so a workgroup takes a PAIR of Q tiles of
  // one head, n_qtiles-1-p and then p, one after the other: every workgroup then does the same amount of
  // work (but for the unpaired middle tile when n_qtiles is odd).  total_tiles counts pairs in that case.
  const int n_items = kSplit ? split.items : kCausal ? (n_qtiles + 1) / 2 : n_qtiles;
  int bh = tile / n_items;           // batch entry * H + head (kChain: of the current pass)
  int item = tile - bh * n_items;    // Q tile, or pair of Q tiles (kChain: first Q tile)
  if constexpr (kSplit && kCausal) {
    // the items of a head differ in length: the longest of every head start first, so that the short ones fill the end
    // (a number of heads that is a multiple of 8 still keeps each head on one XCD)
    const int heads = total_tiles / n_items;
    item = blockIdx.x / heads;
    bh = blockIdx.x - item * heads;
  }
  // passes of this workgroup: Q tiles it works through.  A chain longer than 1 under the causal mask is only
  // launched when every pair is complete (n_qtiles even).
  const int n_pass = kSplit ? 1 : kCausal ? (chain > 1 ? 2 * chain : item != n_qtiles - 1 - item ? 2 : 1) : kChain ? chain : 1;
  int qt, q_row, n_tiles;  // set per pass
  // kSplit: the items of a head run slice by slice, so that neighbouring workgroups read the same K and V.  Slice s
  // concerns every Q tile, or under the causal mask those from its own first key on, the last Q tile first.
  int slice = 0, slice_qt = 0;
  if constexpr (kSplit) {
    int rest = item;
    for (int n = n_qtiles; rest >= n;) {
      rest -= n;
      ++slice;
      if constexpr (kCausal) n -= split.chunk / 2;   // (a Q tile is two K/V tiles long)
    }
    slice_qt = kCausal ? n_qtiles - 1 - rest : rest;
  }
  const int first_key = kSplit ? slice * split.chunk * kBc : 0;
  const int nk_all = Nk;   // keys of a batch entry in memory
  if constexpr (kSplit) Nk -= first_key;   // keys from the slice's first one on

  const size_t row_stride = (size_t)H * D;                          // elements between consecutive tokens
  const size_t tile_stride = (size_t)kBc * row_stride;              // elements between consecutive K/V tiles
  // element (b, 0, h, 0) of Q and O / of K and V, for head index bh = b * H + h
  auto q_base_of = [&](int bh_) { return ((size_t)(bh_ / H) * Nq * H + (size_t)(bh_ % H)) * D; };
  auto kv_base_of = [&](int bh_) {
    return (((size_t)(bh_ / H) * nk_all + (kSplit ? first_key : 0)) * H + (size_t)(bh_ % H)) * D;
  };
  size_t head_base = q_base_of(bh);

  // Q_i fragment, held in registers for the whole loop: B operand of S^T = K Q^T.
  u32x4 qf[kKSteps];

  // Direct global->LDS staging (buffer_load ... lds).  Wavefront w issues loads number w*kLoadsPerWave + i
  // of a tile; load n fills LDS bytes [1024 n, 1024 n + 1024) of the tile, lane l the 16-byte chunk
  // 64 n + l.  The chunk's row and (swizzled) position decide which global chunk the lane fetches.
  // Buffer descriptors (base, byte range) of this head's K and V rows: a raw buffer load takes a scalar
  // descriptor, a scalar tile offset and the 32-bit per-lane offset, and its range check turns any
  // offset past the last row into zeros instead of a fault.
  const uint32_t head_bytes = (uint32_t)(((size_t)(Nk - 1) * row_stride + D) * 2);
  auto rsrc_of = [&](const uint16_t* tensor, int bh_) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(tensor + kv_base_of(bh_)), 0, (int)head_bytes,
                                             kBufferFlags);
  };
  __amdgpu_buffer_rsrc_t k_rsrc = rsrc_of(K, bh), v_rsrc = rsrc_of(V, bh);
  // kChain: the head and Q tile of the next pass, whose first K/V tiles the last boundaries of this pass load
  // (their descriptors are made where they are used, not kept in scalar registers through the loop)
  int bh_next = 0, qt_next = 0;
  int stream_base = 0;  // kChain: K/V tiles streamed for the Q tiles this workgroup has finished
  bool more = false;    // kChain: another Q tile follows, so the stream goes on past tile n_tiles - 1
  const uint32_t tile_bytes = (uint32_t)(tile_stride * 2);
  const uint32_t row_bytes = (uint32_t)(row_stride * 2);
  // is_k is a compile-time tag: K and V tiles use different chunk swizzles.  The per-lane source offsets are
  // recomputed at every call (a few integer operations per tile) instead of being kept in registers.
  auto stage_in = [&](auto is_k, __amdgpu_buffer_rsrc_t rsrc, int j, uint16_t* lds_tile) __attribute__((always_inline)) {
    int lane = tid & 63;
    if constexpr (kHalves) {
      j = tile_at(j);
      lds_tile += half_lds;
    }
    // d = 256 with partial tiles has no registers to spare for sixteen loop-invariant source offsets: keep them
    // from being hoisted out of the loop (they cost a few integer operations per load to recompute).  (At d = 128 the
    // registers that this frees, 256 -> 230, would do for kRowStores, but the loop lost 6 % at N = 5000.)
    if constexpr (D == 256 && kRagged) asm volatile("" : "+v"(lane));
    // d = 64 with the causal mask and partial tiles has few to spare at three wavefronts per SIMD: here one offset per
    // operand is kept, and nothing for the last tiles (whose offsets the halves, with two per SIMD, may keep: 2 % at N = 638).
    constexpr bool kOneOffset = D == 64 && kCausal && kRagged;
    if constexpr (kRagged && kFlagSync) j = wide_staged_tile(j, Nk);
    // (the 256-row shape has no registers for these: the range check of the descriptor leaves zeros in LDS for such rows)
    if (kRagged && !kFlagSync && (j + 1) * kBc > Nk) {
      if constexpr (kOneOffset && !kSplit) asm volatile("" : "+v"(lane));
      // a tile with rows past the last key: those rows are filled with copies of the last key's row, so LDS
      // holds finite numbers everywhere (their columns of S are masked; 0 * finite = 0 in GEMM-II)
#pragma unroll
      for (int i = 0; i < kLoadsPerWave; ++i) {
        const int chunk = 64 * (wave * kLoadsPerWave + i) + lane;
        const int row = chunk / T::kChunksPerRow, pos = chunk % T::kChunksPerRow;
        const int swz = decltype(is_k)::value ? T::swz_k(row) : T::swz_v(row);
        const int row_g = min(j * kBc + row, Nk - 1);
        const uint32_t src = (uint32_t)row_g * row_bytes + 16u * (uint32_t)(pos ^ swz);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(lds_tile + 512 * (wave * kLoadsPerWave + i)), 16,
                                                 (int)src, 0, 0, 0);
      }
      return;
    }
    if constexpr (kOneOffset) {
      // The second load is eight rows further on, a scalar distance: V's swizzle repeats there, K's differs in bit 2 of the
      // 16-byte chunk (a row of a head is 128 bytes, so that is bit 6 of the offset).  With all four offsets recomputed at
      // every tile instead, calls of up to two workgroups per CU lost 2...6 % (B7 H16 N412 fp16 14.4 -> 15.3 us, now 14.5;
      // B10 H16 N650 22.2 -> 23.2, now 22.1) and long ones as much (B4 H16 N5001 fp16 251 us, now 232).
      static_assert(!kOneOffset || kLoadsPerWave == 2, "two loads per tile and wavefront");
      const int chunk = 64 * wave * kLoadsPerWave + lane;
      const int row = chunk / T::kChunksPerRow, pos = chunk % T::kChunksPerRow;
      const int swz = decltype(is_k)::value ? T::swz_k(row) : T::swz_v(row);
      const uint32_t src = (uint32_t)row * row_bytes + 16u * (uint32_t)(pos ^ swz);
      uint16_t* const dst = lds_tile + 512 * wave * kLoadsPerWave;
      const uint32_t at = (uint32_t)j * tile_bytes;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)dst, 16, (int)src, (int)at, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + 512), 16,
                                               (int)(decltype(is_k)::value ? src ^ 64u : src), (int)(at + 8u * row_bytes), 0, 0);
      return;
    }
#pragma unroll
    for (int i = 0; i < kLoadsPerWave; ++i) {
      const int chunk = 64 * (wave * kLoadsPerWave + i) + lane;
      const int row = chunk / T::kChunksPerRow, pos = chunk % T::kChunksPerRow;
      const int swz = decltype(is_k)::value ? T::swz_k(row) : T::swz_v(row);
      const uint32_t src = (uint32_t)row * row_bytes + 16u * (uint32_t)(pos ^ swz);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(lds_tile + 512 * (wave * kLoadsPerWave + i)), 16,
                                               (int)src, (int)((uint32_t)j * tile_bytes), 0, 0);
    }
  };

  // Per-lane LDS element offsets of the operand reads (row part + swizzled chunk part).
  // K fragment of MFMA step ks: row r (+32 per key block), chunk 2 ks + hh.  The swizzle only touches the low four
  // bits of the chunk index, so steps 8 apart (d = 256) differ by a constant 16 chunks and share one register.
  constexpr int kKAddrs = kKSteps < 8 ? kKSteps : 8;
  int k_addr[kKAddrs];
#pragma unroll
  for (int ks = 0; ks < kKAddrs; ++ks) k_addr[ks] = half_lds + r * D + 8 * ((2 * ks + hh) ^ T::swz_k(r));
  int v_addr[kDBlocks];  // V fragment of d-block db: row 4 hh + (lane%16)/4 (+16 per step, +8 for the upper half)
  {
    const int l16 = lane & 15;
    const int row0 = 4 * hh + (l16 >> 2);
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db) {
      const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
      v_addr[db] = half_lds + row0 * D + 8 * (chunk ^ T::swz_v(row0)) + 4 * (l16 & 1);
    }
  }

  // Accumulators of Algorithm 2: O^T (fp32), the rowmax reference and the running rowsum.  Each half
  // of the wavefront keeps the partial rowsum of its own keys; the two are added in the epilogue.
  f32x16 ot[kDBlocks];
  f32x16 st[kKBlocks];  // S^T of the tile being processed
  float m_ref;          // reference point of the exponentials, in units of the unscaled logits q.k
  float mc_ref;         // m_ref * scale * log2(e)
  float l_run;

  // Operand fragment of MFMA step `step` of GEMM-I (K rows) / GEMM-II (V columns, transposed by the load).
  auto k_frag = [&](const uint16_t* kt, int step) __attribute__((always_inline)) -> u32x4 {
    const int ks = step / kKBlocks, kb = step % kKBlocks;
    return *reinterpret_cast<const u32x4*>(kt + k_addr[ks % kKAddrs] + (ks / kKAddrs) * 128 + kb * 32 * D);
  };
  auto v_frag = [&](const uint16_t* vt, int step) __attribute__((always_inline)) -> u32x4 {
    const int t = step / kDBlocks, db = step % kDBlocks;
    const uint16_t* p = vt + v_addr[db] + t * 16 * D;
    const u32x2 lo = lds_read_tr16(p);
    const u32x2 hi = lds_read_tr16(p + 8 * D);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };

  // GEMM-I (transposed): S^T[key][query] = K_j Q_i^T, fragments prefetched kRing steps ahead.
  auto gemm1 = [&](const uint16_t* kt) __attribute__((always_inline)) {
    u32x4 ring[kRing];
#pragma unroll
    for (int i = 0; i < kRing; ++i) ring[i] = k_frag(kt, i);
#pragma unroll
    for (int kb = 0; kb < kKBlocks; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) st[kb][v] = 0.f;
#pragma unroll
    for (int i = 0; i < kSteps1; ++i) {
      const int ks = i / kKBlocks, kb = i % kKBlocks;
      st[kb] = E::mfma(ring[i % kRing], qf[ks], st[kb]);
      if (i + kRing < kSteps1) ring[i % kRing] = k_frag(kt, i + kRing);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // One iteration of Algorithm 2's inner loop, software-pipelined by one tile on the K side: softmax of
  // S_j, O += P~_j V_j, then S_{j+1} = K_{j+1} Q^T.  Every iteration thus has one block of softmax
  // arithmetic and one block of back-to-back MFMAs, which the two wavefronts sharing a SIMD overlap.
  // kNext: a tile j+1 exists.
  // mask_tag and straddles: the tile crosses the causal diagonal or the last key; `visible` is then the largest value of
  // 32 kb + 8 (v/4) + v%4 (the key's position in the tile minus this half's 4 hh) that register v of key
  // block kb may have for its key to be at or before this lane's query.
  bool hurry = false;  // kFlagSync: this wavefront did not have to wait at its last boundary, so it is among the slowest
  // kSplitRefill: the K half of the refill, issued inside iteration jj (see stage_ahead there): K tile jj + kNBuf,
  // or, past the end of a chained pass that another one follows, that one's tile
  auto split_k_refill = [&](int jj, uint16_t* k_refill) __attribute__((always_inline)) {
    if (jj + kNBuf < n_tiles) stage_in(true_type{}, k_rsrc, jj + kNBuf, k_refill);
    else if (kChain && more) stage_in(true_type{}, rsrc_of(K, bh_next), jj + kNBuf - n_tiles, k_refill);
  };
  auto iteration = [&](auto next_tag, auto mask_tag, bool straddles, int visible, const uint16_t* v_cur, const uint16_t* k_next,
                       int jj, uint16_t* k_refill) __attribute__((always_inline)) {
    const bool masked = decltype(mask_tag)::value && straddles;   // wavefront-uniform
    if (masked) {
      // S_ij = -inf for j > i: the exponential below turns it into an exact 0 in P~ and in the rowsum.  Key 0
      // is visible to every query, so the reference point is finite from the first tile on.
#pragma unroll
      for (int kb = 0; kb < kKBlocks; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (32 * kb + 8 * (v / 4) + (v % 4) > visible) st[kb][v] = -INFINITY;
    }
    // ---- online softmax for this lane's query (Algorithm 2: rowmax, P~, rowsum, rescale) ----
    // The scale is folded into the exponent, exp(scale*(s - m)) = exp2(s*c - m*c) with c = scale*log2(e), and
    // the maximum is taken on the unscaled logits (valid for scale > 0).
    //
    // The reference point m of the exponentials only has to keep them in range, it need not be the running
    // maximum of Algorithm 2: the result is unchanged because the reference cancels in O / l.  It is moved (and
    // O, l rescaled by exp(m_old - m_new)) only when a tile would otherwise produce a P~ above 2^kLazyLog2.
    if (kFlagSync && hurry) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(0);
    constexpr float kLazyLimit = 256.0f;  // 2^kLazyLog2
    static_assert(kLazyLog2 == 8.0f, "kLazyLimit is 2^kLazyLog2");
    u32x4 ring[kRing];   // operand fragments on their way from LDS to the MFMAs
    float rowsum[2];
    u32x4 pf[kTSteps];

    // Row maximum of this tile (both halves of the wavefront), the move of the reference point for the rows that
    // `moves(mx)` selects, and the rescale of l and O.
    auto update_reference = [&](auto moves) __attribute__((always_inline)) {
      // The maxima below are inline assembly, for which the compiler inserts no wait states: S^T may have been
      // written by an MFMA (8 passes) shortly before, so the distance an MFMA result needs before a vector
      // instruction may read it is put here by hand (this path runs on first, masked and rare tiles only).
      asm volatile("s_nop 15\n\ts_nop 3");
      float mx = max2_raw(st[0][0], st[0][1]);
#pragma unroll
      for (int kb = 0; kb < kKBlocks; ++kb)
#pragma unroll
        for (int v = (kb == 0 ? 2 : 0); v < 16; v += 2) mx = max3_raw(mx, st[kb][v], st[kb][v + 1]);
      mx = max_with_partner_half_raw(mx);
      const bool move = moves(mx);
      // d = 256 takes the maximum on every tile, and a masked tile seldom raises it: mostly no row of the wavefront moves
      constexpr bool kSkipIdleRescale = D == 256 || decltype(mask_tag)::value;
      if (!kSkipIdleRescale || __builtin_amdgcn_ballot_w64(move) != 0) {
        const float m_new = move ? mx : m_ref;
        const float mc_new = kSplit ? fmaxf(m_new * scale_log2e, kLowest) : m_new * scale_log2e;
        // exp(m_old - m_new); 0 on the first tile.  A row that stays (the branch is taken when any row of the
        // wavefront moves) gets exactly 1, not exp2 of a contracted m*c - m*c that may differ from 0 in the last
        // bit: a row's result must not depend on what the other rows of the wavefront hold.
        const float alpha = move ? __builtin_amdgcn_exp2f(mc_ref - mc_new) : 1.0f;
        m_ref = m_new;
        mc_ref = mc_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) ot[db][v] *= alpha;
      }
    };
    // Issued once per tile, right before its first round of exponentials:
    //  * the second half of the refill (kSplitRefill): K tile jj + kNBuf into the buffer that held K tile jj, which
    //    every wavefront finished reading before the barrier that precedes this iteration.  The V half was issued
    //    right after that barrier.  At d = 256 a tile pair is 16 loads per wavefront; issued as one burst they
    //    overrun the queue between the wavefronts and the texture unit, which accepts about four loads per
    //    wavefront at once and then only as fast as the path into LDS drains, and every wavefront of the workgroup
    //    stands still meanwhile;
    //  * the first V fragments of GEMM-II: independent of P~, so their LDS latency hides behind the exponentials.
    auto stage_ahead = [&]() __attribute__((always_inline)) {
      if constexpr (kSplitRefill) split_k_refill(jj, k_refill);
#pragma unroll
      for (int i = 0; i < kRing; ++i) ring[i] = v_frag(v_cur, i);
    };
    // P~ = exp2(s*c - m*c): the rowsum is taken in fp32 from the unrounded values (Algorithm 2 keeps it in
    // the accumulator type); rounded to 16 bit, registers 8t..8t+7 of a 32-key block are the 8 B-operand
    // slots of MFMA step t.
    auto exponentials = [&]() __attribute__((always_inline)) {
      rowsum[0] = 0.f;
      rowsum[1] = 0.f;
#pragma unroll
      for (int kb = 0; kb < kKBlocks; ++kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int v = 8 * t + 2 * c;
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[kb][v], scale_log2e, -mc_ref));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[kb][v + 1], scale_log2e, -mc_ref));
            rowsum[0] += p0;
            rowsum[1] += p1;
            pf[kb * 2 + t][c] = E::pack2(p0, p1);
          }
        }
      }
    };
    // A row moves when its tile maximum is more than 2^kLazyLog2 above the reference (the first tile's reference is
    // -inf, so every row moves there).
    auto exceeds = [&](float mx) __attribute__((always_inline)) { return (mx - m_ref) * scale_log2e > kLazyLog2; };

    if constexpr (D == 256) {
      // One wavefront per SIMD and every register in use: S cannot stay live across a first round of
      // exponentials, so the row maximum is taken on every tile.
      update_reference(exceeds);
      stage_ahead();
      exponentials();
    } else {
      // A tile first exponentiates against the reference it inherits and looks at the partial row sums: a P~
      // above the limit makes the partial row sum of its lane exceed the limit.  Only then -- and on the first
      // tile (reference -inf) and on tiles with masked entries (S holds -inf) -- does the wavefront take the row
      // maximum, move the reference of the rows concerned and exponentiate again.  Which rows move is decided
      // from the row's own values, never from another row's: on first and masked tiles by the maximum, otherwise
      // by the row's two partial sums.  (Finite inputs and a finite reference: the sums are in [0, +inf].)
      stage_ahead();
      bool need_max = masked || jj == 0;   // wavefront-uniform
      float sum_seen = 0.f;
      if (!need_max) {
        exponentials();
        sum_seen = rowsum[0] + rowsum[1];
        need_max = __builtin_amdgcn_ballot_w64(sum_seen > kLazyLimit) != 0;
      }
      if (need_max) {
        update_reference([&](float mx) __attribute__((always_inline)) {
          if (masked || jj == 0) return exceeds(mx);
          const uint32_t u = __builtin_bit_cast(uint32_t, sum_seen);
          const auto both = __builtin_amdgcn_permlane32_swap(u, u, false, false);
          return __builtin_bit_cast(float, (uint32_t)both[0]) > kLazyLimit ||
                 __builtin_bit_cast(float, (uint32_t)both[1]) > kLazyLimit;
        });
        exponentials();
      }
    }
    l_run += rowsum[0] + rowsum[1];
    __builtin_amdgcn_sched_barrier(0);

    // ---- GEMM-II (transposed): O^T[d][query] += V_j^T P~^T.  Slot i of lane-half hh in step t is key
    // 16t + 8(i/4) + 4hh + i%4, the key of accumulator register 8t+i of GEMM-I.  GEMM-I of the next tile
    // follows in the same stream of MFMA steps, so its first K fragments are fetched under the last MFMAs of
    // GEMM-II and no LDS latency is exposed between the two products.
    if (kFlagSync && hurry) __builtin_amdgcn_s_setprio(3);
    else __builtin_amdgcn_s_setprio(1);
    constexpr bool kNext = decltype(next_tag)::value;
    constexpr int kStepsAll = kSteps2 + (kNext ? kSteps1 : 0);
    auto any_frag = [&](int step) __attribute__((always_inline)) -> u32x4 {
      return step < kSteps2 ? v_frag(v_cur, step) : k_frag(k_next, step - kSteps2);
    };
#pragma unroll
    for (int i = 0; i < kStepsAll; ++i) {
      if (i < kSteps2) {
        const int t = i / kDBlocks, db = i % kDBlocks;
        ot[db] = E::mfma(ring[i % kRing], pf[t], ot[db]);
      } else {
        const int i1 = i - kSteps2, ks = i1 / kKBlocks, kb = i1 % kKBlocks;
        if (ks == 0) {
          f32x16 zero;
#pragma unroll
          for (int v = 0; v < 16; ++v) zero[v] = 0.f;
          st[kb] = E::mfma(ring[i % kRing], qf[ks], zero);
        } else {
          st[kb] = E::mfma(ring[i % kRing], qf[ks], st[kb]);
        }
      }
      if (i + kRing < kStepsAll) ring[i % kRing] = any_frag(i + kRing);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // LDS schedule.  K tile t lives in k_lds[t % kNBuf], V tile t in v_lds[t % kNBuf].  Iteration j reads
  // V tile j and K tile j+1.  With a barrier per tile (4-wavefront kernels) those two tiles are dead after the
  // barrier that ends the iteration, and their buffers are refilled with K tile j+1+kNBuf and V tile j+kNBuf;
  // the loads needed by iteration j+1 (K tile j+2, V tile j+1) were issued kNBuf-1 barriers earlier; every
  // barrier issues 2*kLoadsPerWave loads per wavefront, so while every barrier issues its full set it is enough
  // to wait until at most (kNBuf-2)*2*kLoadsPerWave loads are outstanding.  Without barriers (kFlagSync) the
  // refill is one tile behind that, see `boundary`.
  constexpr int kRelaxedVmcnt = (kNBuf - 2) * 2 * kLoadsPerWave;
  static_assert(kRelaxedVmcnt < 64, "vmcnt is a 6-bit counter");
  constexpr int kWaitRelaxed = (kRelaxedVmcnt & 15) | ((kRelaxedVmcnt >> 4) << 14) | 0x0F70;
  constexpr int kWaitAll = 0x0F70;  // vmcnt(0), expcnt and lgkmcnt left alone

  uint16_t* const k_buf[4] = {k_lds0, k_lds1, k_lds2, k_lds3};
  uint16_t* const v_buf[4] = {v_lds0, v_lds1, v_lds2, v_lds3};

  // end of iteration j: publish what iteration j+1 reads, then refill the two dead buffers
  auto boundary = [&](auto relaxed_tag, int j, uint16_t* k_fill, uint16_t* v_fill) __attribute__((always_inline)) {
    if constexpr (kFlagSync) {
      // Arrival j of a wavefront says: my reads of V tile j and K tile j+1 are over, and my share of the loads
      // issued at the previous boundary (K tile j+3, V tile j+2) has landed.  A wavefront leaves boundary j when
      // every wavefront has made arrival j-1: then K tile j+2 and V tile j+1, which iteration j+1 reads, are
      // complete, and V tile j-1 and K tile j are dead, so their buffers (k_fill, v_fill) take K tile j+kNBuf and
      // V tile j-1+kNBuf.  A wavefront makes arrival j before it waits for the others' arrival j-1, so it can be two
      // arrivals ahead of the slowest: arrivals are counted per iteration, iteration j in entry j % 4 (entries are
      // reused four iterations later, far beyond that lead), and arrival j-1 is complete when its entry has
      // reached kWv * ((j-1)/4 + 1).  The wait is bounded: a wavefront that gives up poisons its rowsum, so the
      // error shows in O and LSE instead of hanging the GPU.
      // a first look at the others' count, under way while this wavefront waits for its own loads
      // (with chained Q tiles the iterations are counted along the whole stream: n_tiles is a multiple of 4)
      const int g = stream_base + j;
      uint32_t seen = __hip_atomic_load(&arrivals[(j + 3) & 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_s_waitcnt(kWaitAll);
      if (lane == 0) __hip_atomic_fetch_add(&arrivals[j & 3], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      const uint32_t target = g > 0 ? (uint32_t)(kWv * ((g - 1) / 4 + 1)) : 0u;
      int spins = 0;
      while (seen < target) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > kSpinLimit) {
          l_run = __builtin_nanf("");
          break;
        }
        seen = __hip_atomic_load(&arrivals[(j + 3) & 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // the tiles are read only after the count was seen
      hurry = spins == 0;
      const int kt = j + kNBuf, vt = j - 1 + kNBuf;
      if (kt < n_tiles) stage_in(true_type{}, k_rsrc, kt, k_fill);
      else if (more) stage_in(true_type{}, rsrc_of(K, bh_next), kt - n_tiles, k_fill);
      if (vt < n_tiles) stage_in(false_type{}, v_rsrc, vt, v_fill);
      else if (more) stage_in(false_type{}, rsrc_of(V, bh_next), vt - n_tiles, v_fill);
      return;
    }
    if constexpr (decltype(relaxed_tag)::value) __builtin_amdgcn_s_waitcnt(kWaitRelaxed);
    else __builtin_amdgcn_s_waitcnt(kWaitAll);
    if constexpr (kHalves) {
      // A barrier of this half's four wavefronts, counted in LDS: s_barrier would stop all eight at every tile and keep
      // the two wavefronts of a SIMD, one of either half, in the same phase, softmax against softmax and MFMAs against
      // MFMAs.  The wait is bounded like the one above (without a sleep between polls: about ten milliseconds).  A
      // wavefront that gives up refills buffers that slower ones of its half may still read, so it poisons the row sums
      // of the whole workgroup, not only its own.
      if (lane == 0) __hip_atomic_fetch_add(&arrivals[half], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      int spins = 0;
      while (__hip_atomic_load(&arrivals[half], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <
             (uint32_t)(kRowWaves * (j + 1))) {
        if (++spins > kSpinLimit) {
          __hip_atomic_store(&arrivals[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);   // read in the epilogue
          break;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      __syncthreads();
    }
    // (a chained pass that another one follows goes on with that one's first tiles)
    if constexpr (!kSplitRefill) {
      if (j + 1 + kNBuf < n_tiles) stage_in(true_type{}, k_rsrc, j + 1 + kNBuf, k_fill);
      else if (kChain && more) stage_in(true_type{}, rsrc_of(K, bh_next), j + 1 + kNBuf - n_tiles, k_fill);
    }
    if (j + kNBuf < n_tiles) stage_in(false_type{}, v_rsrc, j + kNBuf, v_fill);
    else if (kChain && more) stage_in(false_type{}, rsrc_of(V, bh_next), j + kNBuf - n_tiles, v_fill);
  };
  // buffers refilled at the boundary after iteration j+i of a group of kNBuf iterations (see `boundary`)
  constexpr int kKFillShift = kFlagSync ? 0 : 1, kVFillShift = kFlagSync ? kNBuf - 1 : 0;

  // Q fragment of Q tile `qtile`: B operand of S^T = K Q^T, straight from global memory into registers
  auto load_q = [&](size_t base, int qtile) __attribute__((always_inline)) {
    const int row = qtile * kRows + wave * 32 + r;
    const int row_ld = kRagged ? min(row, Nq - 1) : row;
    const uint16_t* qp = Q + base + (size_t)row_ld * row_stride + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) qf[ks] = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
  };

  // the arrival counters start at zero; the first pass's barrier publishes them
  if ((kFlagSync || kHalves) && tid < 4) arrivals[tid] = 0;
  for (int pass = 0; pass < n_pass; ++pass) {
    // causal pair: the first Q tile's last K/V reads are over before the buffers are refilled
    if (pass > 0 && !kChain) __syncthreads();
    if constexpr (kChain) {
      // head and Q tile of pass p: chain step p (causal: p / 2, the heavy tile of the pair first, then the light one)
      auto locate = [&](int p, int& bh_, int& qt_) {
        const int t = tile + (kCausal ? p >> 1 : p) * chain_stride;
        bh_ = t / n_items;
        const int it = t - bh_ * n_items;
        qt_ = kCausal ? ((p & 1) == 0 ? n_qtiles - 1 - it : it) : it;
      };
      locate(pass, bh, qt);
      head_base = q_base_of(bh);
      k_rsrc = rsrc_of(K, bh);
      v_rsrc = rsrc_of(V, bh);
      more = pass + 1 < n_pass;
      if (more) locate(pass + 1, bh_next, qt_next);
    } else {
      qt = kSplit ? slice_qt : kCausal ? (pass == 0 ? n_qtiles - 1 - item : item) : item;
    }
    q_row = qt * kRows + wave * 32 + r;
    // a multiple of kNBuf in every case; causal: the keys up to the end of this Q tile
    n_tiles = kCausal ? (qt + 1) * kNBuf : kRagged ? (Nk + kNBuf * kBc - 1) / (kNBuf * kBc) * kNBuf : Nk / kBc;
    if constexpr (kSplit) {
      n_tiles = min((kCausal ? (qt + 1) * 2 : (Nk + 2 * kBc - 1) / (2 * kBc) * 2) - (kCausal ? slice * split.chunk : 0),
                    split.chunk);
      if constexpr (kHalves) n_tiles = (n_tiles + 3) / 4 * 2;   // of each half
    }
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) ot[db][v] = 0.f;
    m_ref = -INFINITY;
    // kSplit: a part of the keys may hold only logits so low that they overflow once scaled (keys that a caller masks with
    // the lowest value of the type, past the last tile of the live ones); its reference stops at the lowest finite number,
    // against which their exponentials are 0.  (A whole launch starts on the first keys, which are live in that use.)
    mc_ref = kSplit ? kLowest : -INFINITY;
    l_run = 0.f;

    // A chained Q tile after the first finds its ring filled, its Q fragment loaded and its first S computed by
    // the end of the pass before it.
    if (!kChain || pass == 0) {
      load_q(head_base, qt);
      static_for<kNBuf>([&](auto t) { stage_in(true_type{}, k_rsrc, decltype(t)::value, k_buf[decltype(t)::value]); });
      static_for<kNBuf - 1>([&](auto t) { stage_in(false_type{}, v_rsrc, decltype(t)::value, v_buf[decltype(t)::value]); });
      // The Q fragment must have landed before the loop so that no wait for it is placed inside the loop.
#pragma unroll
      for (int ks = 0; ks < kKSteps; ++ks) asm volatile("" : "+v"(qf[ks]));
      __builtin_amdgcn_s_waitcnt(kWaitAll);
      __syncthreads();
      gemm1(k_lds0);
      __syncthreads();  // every wavefront has finished reading K tile 0 before its buffer is refilled
      if constexpr (!kFlagSync) {   // (with kFlagSync the first boundary issues these two)
        if constexpr (!kSplitRefill) {
          if (kNBuf < n_tiles) stage_in(true_type{}, k_rsrc, kNBuf, k_lds0);
        }
        if (kNBuf - 1 < n_tiles) stage_in(false_type{}, v_rsrc, kNBuf - 1, v_buf[kNBuf - 1]);
      }
    }

    // partial tiles: wavefronts whose rows all lie past the last query keep the boundaries and skip the arithmetic
    // (not in the partial-tile kernels that have no register left for one more condition)
    constexpr bool kSkipDeadRows = kRagged && D <= 128 && !(D == 128 && kCausal) && !kFlagSync;
    const bool rows_live = !kSkipDeadRows || qt * kRows + wave * 32 < Nq;   // wavefront-uniform
    int j = 0;
    for (; j + kNBuf < n_tiles; j += kNBuf) {  // every barrier of these iterations issues its full set of loads
      static_for<kNBuf>([&](auto t) {
        constexpr int i = decltype(t)::value;
        if (rows_live) iteration(true_type{}, false_type{}, false, 0, v_buf[i], k_buf[(i + 1) % kNBuf], j + i, k_buf[i]);
        boundary(true_type{}, j + i, k_buf[(i + kKFillShift) % kNBuf], v_buf[(i + kVFillShift) % kNBuf]);
      });
    }
    // last kNBuf tiles: wait for everything, and the very last tile has no successor.  Under the causal mask
    // these are exactly the tiles of this Q tile's own rows, the ones the diagonal crosses.
    // Without the causal mask the same tiles are the only ones that can hold keys past Nk-1.
    using mask_tail = std::integral_constant<bool, kCausal || kRagged>;
    static_for<kNBuf>([&](auto t) {
      constexpr int i = decltype(t)::value;
      // causal: (q_row - first key of tile j+i) - 4 hh; a stored row (q_row < Nq = Nk) never sees a key past
      // Nk-1 through it.  Otherwise: (last key - first key of tile j+i) - 4 hh.
      // (kSplit, causal: the same distance, from the slice's first key; a slice that ends before the diagonal masks nothing)
      int visible = kCausal ? (kSplit ? q_row - first_key - tile_at(j + i) * kBc : wave * 32 + r - i * kBc) - 4 * hh
                            : Nk - 1 - tile_at(j + i) * kBc - 4 * hh;
      // computed here, not hoisted above the main loop where 32 comparison results per tile would sit in
      // scalar registers for the whole loop
      if constexpr (mask_tail::value) asm volatile("" : "+v"(visible));
      // Under the causal mask a tile of the Q tile's own rows lies wholly above the diagonal for the wavefronts whose
      // 32 rows come before its first key: for them it would contribute exact zeros, so they leave its arithmetic
      // out (and keep every boundary: the others still count on their loads and arrivals).  The same goes, for every
      // wavefront, for a padding tile that only rounds the tile count up and holds no key at all.
      // And a wavefront whose 32 rows all lie past the last query (partial last Q tile) computes nothing at all.
      const bool live = (!kCausal || (kSplit ? tile_at(j + i) * kBc <= qt * kRows + wave * 32 + 31 - first_key
                                             : i * kBc <= wave * 32 + 31)) &&
                        (!kRagged || tile_at(j + i) * kBc < Nk) && rows_live;
      // ... and only the tile that a wavefront's own rows cross, or that holds the last key, needs the mask and the row
      // maximum: the others of these tiles are wholly visible to it and take the unmasked tile's short path (not where
      // kRowStores is off: no register left for the condition; nor at d = 256, which takes the maximum of every tile
      // anyway and lost 3...5 % by it, nor in the whole launches of d = 64 under the causal mask, where the registers it
      // takes cost a workgroup per CU or 2 %).  With the idle rescale left out as well: B8 H16 N2048
      // d128 bf16 causal 151.6 -> 148.5 us, N = 2047 unmasked 269.6 -> 267.7, the same bits.
      const int tile_end = (kCausal && !kSplit ? i : tile_at(j + i)) * kBc + kBc;   // first key past the tile
      const bool straddles = !kRowStores || D == 256 || (D == 64 && kCausal && !kSplit) || (!kCausal ? tile_end > Nk
                                             : kSplit ? tile_end - 1 > qt * kRows + wave * 32 - first_key
                                                      : tile_end - 1 > wave * 32);
      if constexpr (i + 1 < kNBuf) {
        if (live) iteration(true_type{}, mask_tail{}, straddles, visible, v_buf[i], k_buf[(i + 1) % kNBuf], j + i, k_buf[i]);
        else if constexpr (kSplitRefill) split_k_refill(j + i, k_buf[i]);   // its loads are still this wavefront's
        boundary(false_type{}, j + i, k_buf[(i + kKFillShift) % kNBuf], v_buf[(i + kVFillShift) % kNBuf]);
      } else {
        // Q is last used by the GEMM-I of the iteration before this one: the next Q tile's fragment is fetched
        // under this iteration
        if (kChain && more) load_q(q_base_of(bh_next), qt_next);
        if (live) iteration(false_type{}, mask_tail{}, straddles, visible, v_buf[i], k_buf[(i + 1) % kNBuf], j + i, k_buf[i]);
        else if constexpr (kSplitRefill) split_k_refill(j + i, k_buf[i]);
        if (kChain && more) {
          // S of the next Q tile's first K/V tile (stream tile n_tiles, complete since the boundary two iterations
          // ago), then the boundary that every iteration of the stream ends with.  O, l and the reference of this
          // Q tile are untouched by both and are written out below.
#pragma unroll
          for (int ks = 0; ks < kKSteps; ++ks) asm volatile("" : "+v"(qf[ks]));
          gemm1(k_buf[(i + 1) % kNBuf]);
          boundary(false_type{}, j + i, k_buf[(i + kKFillShift) % kNBuf], v_buf[(i + kVFillShift) % kNBuf]);
        }
      }
    });

    // Epilogue: O_i = O_i / rowsum, LSE_i = m_i + ln(rowsum) (natural log, scaled logits).
    float l_tot = sum_with_partner_half(l_run);
    // kHalves: half 0 goes on with the first kMyBlocks blocks of columns of O, half 1 with the others.
    constexpr int kMyBlocks = kHalves ? kDBlocks / 2 : kDBlocks;
    const int my_column = kHalves ? half * kMyBlocks * 32 : 0;
    if constexpr (kHalves) {
      if (half != 0) {
#pragma unroll
        for (int db = 0; db < kMyBlocks; ++db) {
          const f32x16 x = ot[db];
          ot[db] = ot[db + kMyBlocks];
          ot[db + kMyBlocks] = x;
        }
      }
      __syncthreads();   // the K/V buffers are dead
      // what the other half goes on with, in the registers' own order: 16 bytes per lane, no bank conflicts
      f32x4* const mine = reinterpret_cast<f32x4*>(half == 0 ? k_lds0 : v_lds0) + wave * (kMyBlocks * 4 * 64) + lane;
      const f32x4* const other = reinterpret_cast<f32x4*>(half == 0 ? v_lds0 : k_lds0) + wave * (kMyBlocks * 4 * 64) + lane;
#pragma unroll
      for (int db = 0; db < kMyBlocks; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16& x = ot[db + kMyBlocks];
          mine[(db * 4 + g) * 64] = f32x4{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
        }
      if (hh == 0) ml_lds[half * kRows + wave * 32 + r] = f32x2{mc_ref, l_tot};
      __syncthreads();
      // half 0 always holds a visible key of every row; half 1 may hold none (reference kLowest, sums 0, weight 0)
      const f32x2 ml = ml_lds[(1 - half) * kRows + wave * 32 + r];
      const float m = fmaxf(mc_ref, ml[0]);
      const float w_mine = __builtin_amdgcn_exp2f(mc_ref - m), w_other = __builtin_amdgcn_exp2f(ml[0] - m);
      mc_ref = m;
      l_tot = l_tot * w_mine + ml[1] * w_other;
      if (__hip_atomic_load(&arrivals[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) l_tot = __builtin_nanf("");
#pragma unroll
      for (int db = 0; db < kMyBlocks; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 y = other[(db * 4 + g) * 64];
#pragma unroll
          for (int i = 0; i < 4; ++i) ot[db][4 * g + i] = __builtin_fmaf(y[i], w_other, ot[db][4 * g + i] * w_mine);
        }
    }
    if constexpr (kSplit) {
      if (kCausal ? (qt + 1) * 2 > split.chunk : split.slices > 1) {   // another slice holds keys of this Q tile
        if (qt * kRows + wave * 32 < Nq) {
          const size_t slot = ((size_t)bh * n_qtiles + qt) * split.slices + slice;
          float* po = split.part_o + ((slot * kRowWaves + wave) * kRows / 4 * D + my_column * 32 + lane * 4);
#pragma unroll
          for (int db = 0; db < kMyBlocks; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *reinterpret_cast<f32x4*>(po + (db * 4 + g) * 256) =
                  f32x4{ot[db][4 * g], ot[db][4 * g + 1], ot[db][4 * g + 2], ot[db][4 * g + 3]};
          if (half == 0 && hh == 0)
            *reinterpret_cast<f32x2*>(split.part_ml + 2 * (slot * kRows + wave * 32 + r)) = f32x2{mc_ref, l_tot};
        }
        return;
      }
    }
    const float inv_l = 1.0f / l_tot;
    if (kRowStores || !kRagged || q_row < Nq) {   // (row stores: every lane takes part, rows are checked one by one)
      if constexpr (kRowStores) {
        // Each 32-column block goes through the wavefront's own LDS slab (row r at
        // byte 64 r, its four 16-byte chunks XOR-permuted by (r / 4) % 4 against bank conflicts) and leaves as
        // two stores of 16 rows x 64 bytes.  Only this wavefront touches its slab, and LDS executes a wavefront's
        // accesses in order, so no barrier is involved.
        uint16_t* slab = o_slab + wave_all * 1024;
        int lane_out = lane;
        if constexpr (kFlagSync && kRagged) asm volatile("" : "+v"(lane_out));   // not kept through the loop: no registers
        const int rrow = lane_out >> 2, rchunk = lane_out & 3;   // as a reader: row (+16 for the second half), chunk
        uint16_t* orow = O + head_base + (size_t)(qt * kRows + wave * 32 + rrow) * row_stride + 8 * rchunk + my_column;
#pragma unroll
        for (int db = 0; db < kMyBlocks; ++db) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            // accumulator registers 4g..4g+3 hold d = 32 db + 8 g + 4 hh + (0..3) of this lane's query
            u32x2 w = {E::pack2(ot[db][4 * g + 0] * inv_l, ot[db][4 * g + 1] * inv_l),
                       E::pack2(ot[db][4 * g + 2] * inv_l, ot[db][4 * g + 3] * inv_l)};
            *reinterpret_cast<u32x2*>(slab + r * 32 + 8 * (g ^ ((r >> 2) & 3)) + 4 * hh) = w;
          }
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int row = rrow + 16 * half;
            const u32x4 piece = *reinterpret_cast<const u32x4*>(slab + row * 32 + 8 * (rchunk ^ ((row >> 2) & 3)));
            if (!kRagged || qt * kRows + wave * 32 + row < Nq)
              *reinterpret_cast<u32x4*>(orow + (size_t)(16 * half) * row_stride + 32 * db) = piece;
          }
        }
      } else {
      uint16_t* op = O + head_base + (size_t)q_row * row_stride + 4 * hh;
#pragma unroll
      for (int db = 0; db < kDBlocks; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          // accumulator registers 4g..4g+3 hold d = 32 db + 8 g + 4 hh + (0..3) of this lane's query
          u32x2 w = {E::pack2(ot[db][4 * g + 0] * inv_l, ot[db][4 * g + 1] * inv_l),
                     E::pack2(ot[db][4 * g + 2] * inv_l, ot[db][4 * g + 3] * inv_l)};
          *reinterpret_cast<u32x2*>(op + db * 32 + g * 8) = w;
        }
      }
      }
      if (LSE != nullptr && hh == 0 && half == 0 && (!kRagged || q_row < Nq)) {
        LSE[(size_t)bh * Nq + q_row] = mc_ref * 0.69314718055994530942f + __builtin_logf(l_tot);
      }
    }
    if constexpr (kChain) stream_base += n_tiles;  // every pass's tile count is a multiple of kNBuf
  }  // pass
}

}  // namespace
#endif  // FA2_TILE_KERNEL_H_
