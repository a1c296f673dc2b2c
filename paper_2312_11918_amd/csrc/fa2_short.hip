// Attention of few query rows in all: 32 of them per workgroup, the keys dealt to its wavefronts.
//
// What such a problem takes is a chain: launch, first loads, a K/V tile after the other, epilogue.  The 128-row tile kernel makes it
// long (B1 H16 N384 d128 is 48 workgroups on 256 CUs, each with six tiles to go through), and its halved form half as long.  Here
// the chain is as short as the problem allows: a workgroup has 32 rows, a quarter or an eighth of their keys goes to each
// wavefront, and the wavefronts are merged through LDS at the end.  A wavefront stages its own blocks of 32 keys, and nobody
// else reads them, so the loop has no barrier and waits for nothing but the wavefront's own loads.
//
// The bound of the loop is the path into LDS, 81 GB/s and CU, for every 32 rows read all of their keys: a block per wavefront is 64
// KiB at d = 128 and takes 0.81 us with one workgroup on a CU; at d = 64, half as much, 0.61 us with one (a block's own chain) and
// 0.41 each with two.  The matrix cores need 0.22 us of the 0.81.  The rest of a call is launch, first loads and merge: B1 H16 N512
// d128, four blocks per wavefront, is 3.3 us of loop in 7.8, the matrix cores busy in 12 % of the cycles of busy CUs, 15 bytes into
// LDS in each (35 are 81 GB/s at 2.3 GHz); B1 H16 N1111 causal, up to nine blocks, has 19 % and 24 bytes.  No bank conflicts.  So
// the kernel is for problems whose tiles are about one per CU (short_waves() has the lines and both sides); from there on 128 rows
// per tile read less.
// us a call, 128-row launches before / this kernel: B1 H2 N256 d64 5.7 / 4.4; B1 H16 N1111 d128 causal 19.7 / 15.3; B1 H24 N205
// causal d = 64, 128, 256 10.4 / 4.6, 14.4 / 6.3, 24.0 / 10.9; B1 H2 N1111 d64 13.8 / 7.6; B3 H8 N193 d256 14.7 / 11.4; B1 H2 Nq35
// Nk534 d128 11.7 / 8.0.
//
// Few tiles of many keys: the keys are cut into slices over workgroups as well, where the caller gives a workspace, and a second
// kernel merges their partial O (16 KiB per workgroup at d = 128, a quarter of what slices of 128-row tiles write): B1 H16 Nq32
// Nk3000 d128 15.8 / 12.1, B1 H6 Nq26 Nk1334 d256 25.1 / 14.5, B1 H2 Nq128 Nk1024 d128 12.1 / 8.8.
//
// One buffer per wavefront for K and one for V: the next block of K is requested when this one's fragments have been read, under
// both products and the softmax, the next of V when this one's have, under GEMM-II and the next GEMM-I.  110, 191 and 501 registers at
// d = 64, 128, 256: four, two and one wavefront per SIMD, which is what LDS holds as well.
#include "fa2_tile_kernel.h"

namespace fa2 {
namespace {

constexpr int kShortRows = 32;   // query rows per workgroup
constexpr int kShortKeys = 32;   // keys per block: wavefront w takes blocks w, w + kWv, ...

// See fa2_fwd_kernel for the operands' layouts, the swizzles and the transposed products, which are the same, and for partial
// tiles: rows past Nq - 1 are computed from a copy of the last row and not stored, keys past Nk - 1 masked copies of the last key.
// kCausal: blocks past the diagonal are not visited, and only the tile's own block crosses it.
// A workgroup takes a slice of cut.chunk blocks of its tile's keys (all of them where cut.slices is 1).  A tile whose keys lie in
// several leaves its O^T unnormalised in cut.part_o, with the reference points and sums in cut.part_ml, for fa2_short_merge_kernel.
struct ShortCut {
  float* part_o = nullptr;    // [tile over all heads][slice][register quad][lane] of 4
  float* part_ml = nullptr;   // [tile over all heads][slice][row][2]: reference point (scaled, log2), row sum
  int chunk = 0x7fffffff;     // blocks per slice
  int slices = 1;             // of the longest tile
  int items = 0;              // workgroups per head
};

template <int DT, int kD, int kWv, bool kCausal>
__global__ __launch_bounds__(kWv * 64, kD == 64 ? 4 : kD == 128 ? 2 : 1) void fa2_short_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V, uint16_t* __restrict__ O,
    float* __restrict__ LSE, int H, int Nq, int Nk, float scale_log2e, int n_qtiles, int total, ShortCut cut) {
  using E = Elem<DT>;
  using T = Tile<kD>;
  constexpr int kKSteps = kD / 16;                  // MFMA steps along d of GEMM-I: fragments of K per block
  constexpr int kDBlocks = kD / 32;                 // 32-row blocks of O^T
  constexpr int kVFrags = 2 * kDBlocks;             // fragments of V per block
  constexpr int kElems = kShortKeys * kD;           // elements of a block
  constexpr int kLoads = kElems * 2 / 1024;         // 1 KiB wavefront loads per block
  constexpr int kQuads = kD / 8;                    // register quads of O^T per lane
  using std::false_type;
  using std::true_type;

  // every wavefront's own block of K and of V; at the end its O^T, which takes the same room
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds[kWv * kElems];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds[kWv * kElems];
  __shared__ f32x2 ml_lds[kWv * kShortRows];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, hh = lane >> 5;   // query, half of the wavefront

  // The items of a head run slice by slice, so that neighbouring workgroups read the same keys; slice s concerns every tile, or
  // under the mask those from its own first key on, the last tile first.
  int bh, item;
  if constexpr (kCausal) {   // the longest of every head first
    const int heads = total / cut.items;
    item = blockIdx.x / heads;
    bh = blockIdx.x - item * heads;
  } else {   // a contiguous range per XCD: those of one head share an L2
    const int xcd = blockIdx.x % kXcds, idx = blockIdx.x / kXcds;
    const int per = total / kXcds, rem = total % kXcds;
    const int at = xcd * per + min(xcd, rem) + idx;
    bh = at / cut.items;
    item = at - bh * cut.items;
  }
  int slice = 0;
  for (int n = n_qtiles; item >= n;) {
    item -= n;
    ++slice;
    if constexpr (kCausal) n -= cut.chunk;   // (a tile is one block long)
  }
  const int qt = kCausal ? n_qtiles - 1 - item : item;
  const size_t row_stride = (size_t)H * kD;
  const size_t q_base = ((size_t)(bh / H) * Nq * H + (size_t)(bh % H)) * kD;
  const size_t kv_base = ((size_t)(bh / H) * Nk * H + (size_t)(bh % H)) * kD;
  const uint32_t head_bytes = (uint32_t)(((size_t)(Nk - 1) * row_stride + kD) * 2);
  const __amdgpu_buffer_rsrc_t k_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(K + kv_base), 0, (int)head_bytes, kBufferFlags);
  const __amdgpu_buffer_rsrc_t v_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(V + kv_base), 0, (int)head_bytes, kBufferFlags);
  const uint32_t row_bytes = (uint32_t)(row_stride * 2);

  uint16_t* const k_mine = k_lds + wave * kElems;
  uint16_t* const v_mine = v_lds + wave * kElems;
  // Block j of K or V into this wavefront's LDS; rows past the last key are filled with copies of it.
  auto stage_in = [&](auto is_k, int j) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc = decltype(is_k)::value ? k_rsrc : v_rsrc;
    uint16_t* const dst = decltype(is_k)::value ? k_mine : v_mine;
    const bool partial = (j + 1) * kShortKeys > Nk;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int chunk = 64 * i + lane;
      const int row = chunk / T::kChunksPerRow, pos = chunk % T::kChunksPerRow;
      const int swz = decltype(is_k)::value ? T::swz_k(row) : T::swz_v(row);
      uint32_t src = (uint32_t)row * row_bytes + 16u * (uint32_t)(pos ^ swz), at = (uint32_t)(j * kShortKeys) * row_bytes;
      if (partial) {
        src = (uint32_t)min(j * kShortKeys + row, Nk - 1) * row_bytes + 16u * (uint32_t)(pos ^ swz);
        at = 0;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + 512 * i), 16, (int)src, (int)at, 0, 0);
    }
  };

  int k_addr[kKSteps < 8 ? kKSteps : 8], v_addr[kDBlocks];
#pragma unroll
  for (int ks = 0; ks < (kKSteps < 8 ? kKSteps : 8); ++ks) k_addr[ks] = r * kD + 8 * ((2 * ks + hh) ^ T::swz_k(r));
  {
    const int l16 = lane & 15, row0 = 4 * hh + (l16 >> 2);
#pragma unroll
    for (int db = 0; db < kDBlocks; ++db) {
      const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
      v_addr[db] = row0 * kD + 8 * (chunk ^ T::swz_v(row0)) + 4 * (l16 & 1);
    }
  }

  const int all_blocks = kCausal ? min(qt + 1, (Nk + kShortKeys - 1) / kShortKeys) : (Nk + kShortKeys - 1) / kShortKeys;
  const int first = slice * cut.chunk;   // (0 in the only slice)
  const int n_blocks = min(all_blocks - first, cut.chunk);
  const int row = qt * kShortRows + r;
  u32x4 qf[kKSteps];
  {
    const uint16_t* qp = Q + q_base + (size_t)min(row, Nq - 1) * row_stride + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) qf[ks] = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (wave < n_blocks) {
    stage_in(true_type{}, first + wave);
    stage_in(false_type{}, first + wave);
  }
  __builtin_amdgcn_sched_barrier(0);

  f32x16 ot[kDBlocks];
#pragma unroll
  for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) ot[db][v] = 0.f;
  // The reference point, unscaled and scaled (log2), and the row sum.  The scaled one stops at the lowest finite number, as
  // in the launches that cut the keys: a wavefront without a block, or whose keys' logits overflow once scaled, weighs 0.
  float m_ref = -INFINITY, mc_ref = kLowest, l_run = 0.f;

  constexpr int kWaitLast = (kLoads & 15) | ((kLoads >> 4) << 14) | 0x0F70;   // all but the kLoads last loads have landed
  constexpr int kWaitLoads = 0x0F70, kWaitLds = 0xC07F;                       // vmcnt(0), lgkmcnt(0)
  const int end_block = first + n_blocks;
  for (int j = first + wave; j < end_block; j += kWv) {
    const bool more = j + kWv < end_block;
    // K of this block has landed (its V was requested after it)
    __builtin_amdgcn_s_waitcnt(kWaitLast);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 kf[kKSteps];
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) kf[ks] = *reinterpret_cast<const u32x4*>(k_mine + k_addr[ks % 8] + ks / 8 * 128);
    __builtin_amdgcn_s_waitcnt(kWaitLds);   // the fragments are in registers: the block's place is free
    __builtin_amdgcn_sched_barrier(0);
    if (more) stage_in(true_type{}, j + kWv);
    f32x16 st;
#pragma unroll
    for (int v = 0; v < 16; ++v) st[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) st = E::mfma(kf[ks], qf[ks], st);
    __builtin_amdgcn_sched_barrier(0);
    // V of this block has landed (the next block's K was requested after it); its fragments are read under the softmax
    if (more) __builtin_amdgcn_s_waitcnt(kWaitLast);
    else __builtin_amdgcn_s_waitcnt(kWaitLoads);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 vf[kVFrags];
#pragma unroll
    for (int f = 0; f < kVFrags; ++f) {
      const uint16_t* p = v_mine + v_addr[f % kDBlocks] + f / kDBlocks * 16 * kD;
      const u32x2 lo = lds_read_tr16(p), hi = lds_read_tr16(p + 8 * kD);
      vf[f] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
    const int end = (j + 1) * kShortKeys;
    if (kCausal ? end - 1 > qt * kShortRows : end > Nk) {
      int visible = (kCausal ? row : Nk - 1) - j * kShortKeys - 4 * hh;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v / 4) + (v % 4) > visible) st[v] = -INFINITY;
    }
    float mx = fmaxf(st[0], st[1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) mx = fmaxf(fmaxf(mx, st[v]), st[v + 1]);
    mx = max_with_partner_half_raw(mx);
    // the reference point moves when it is exceeded by 2^8, decided row by row (a row that stays gets exactly 1)
    const bool move = (mx - m_ref) * scale_log2e > kLazyLog2;
    if (__builtin_amdgcn_ballot_w64(move) != 0) {
      const float m_new = move ? mx : m_ref;
      const float mc_new = fmaxf(m_new * scale_log2e, kLowest);
      const float alpha = move ? __builtin_amdgcn_exp2f(mc_ref - mc_new) : 1.0f;
      m_ref = m_new;
      mc_ref = mc_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) ot[db][v] *= alpha;
    }
    float rowsum[2] = {0.f, 0.f};
    u32x4 pf[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int v = 8 * t + 2 * c;
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[v], scale_log2e, -mc_ref));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[v + 1], scale_log2e, -mc_ref));
        rowsum[0] += p0;
        rowsum[1] += p1;
        pf[t][c] = E::pack2(p0, p1);
      }
    l_run += rowsum[0] + rowsum[1];
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    __builtin_amdgcn_sched_barrier(0);
    if (more) stage_in(false_type{}, j + kWv);
#pragma unroll
    for (int f = 0; f < kVFrags; ++f) ot[f % kDBlocks] = E::mfma(vf[f], pf[f / kDBlocks], ot[f % kDBlocks]);
    __builtin_amdgcn_sched_barrier(0);
  }

  // Merge: every wavefront leaves O^T in its own blocks' place, in the registers' order (quad n: registers 4 n ... + 3 of all
  // lanes), and goes on with its share of the quads.  Summed in the wavefronts' order.
  const int parts = min(n_blocks, kWv);
  auto quad_at = [&](int part, int n) __attribute__((always_inline)) {
    uint16_t* const base = n < kQuads / 2 ? k_lds : v_lds;
    return reinterpret_cast<f32x4*>(base + part * kElems) + n % (kQuads / 2) * 64 + lane;
  };
  const float l_mine = sum_with_partner_half(l_run);
  if (wave < parts) {
#pragma unroll
    for (int n = 0; n < kQuads; ++n) {
      const f32x16& x = ot[n / 4];
      *quad_at(wave, n) = f32x4{x[4 * (n % 4)], x[4 * (n % 4) + 1], x[4 * (n % 4) + 2], x[4 * (n % 4) + 3]};
    }
    if (hh == 0) ml_lds[wave * kShortRows + r] = f32x2{mc_ref, l_mine};
  }
  __syncthreads();
  float m = kLowest, l = 0.f, w[kWv];
#pragma unroll
  for (int i = 0; i < kWv; ++i) w[i] = i < parts ? ml_lds[i * kShortRows + r][0] : kLowest;
#pragma unroll
  for (int i = 0; i < kWv; ++i) m = fmaxf(m, w[i]);
#pragma unroll
  for (int i = 0; i < kWv; ++i) {
    w[i] = __builtin_amdgcn_exp2f(w[i] - m);
    if (i < parts) l = __builtin_fmaf(w[i], ml_lds[i * kShortRows + r][1], l);
  }
  constexpr int kMyQuads = kQuads / kWv;
  f32x4 sum[kMyQuads];
#pragma unroll
  for (int n = 0; n < kMyQuads; ++n) sum[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < parts; ++i) {
    float wi = w[0];
#pragma unroll
    for (int x = 1; x < kWv; ++x) wi = i == x ? w[x] : wi;
#pragma unroll
    for (int n = 0; n < kMyQuads; ++n) {
      const f32x4 y = *quad_at(i, wave * kMyQuads + n);
#pragma unroll
      for (int c = 0; c < 4; ++c) sum[n][c] = __builtin_fmaf(wi, y[c], sum[n][c]);
    }
  }
  if (all_blocks > cut.chunk) {
    const size_t slot = ((size_t)bh * n_qtiles + qt) * cut.slices + slice;
    f32x4* const po = reinterpret_cast<f32x4*>(cut.part_o) + (slot * kQuads + wave * kMyQuads) * 64 + lane;
#pragma unroll
    for (int n = 0; n < kMyQuads; ++n) po[n * 64] = sum[n];
    if (wave == 0 && hh == 0) reinterpret_cast<f32x2*>(cut.part_ml)[slot * kShortRows + r] = f32x2{m, l};
    return;
  }
  const float inv_l = 1.0f / l;
  uint16_t* out = O + q_base + (size_t)row * row_stride;
  if constexpr (kMyQuads == 1) {
    const u32x2 x = {E::pack2(sum[0][0] * inv_l, sum[0][1] * inv_l), E::pack2(sum[0][2] * inv_l, sum[0][3] * inv_l)};
    if (row < Nq) *reinterpret_cast<u32x2*>(out + 8 * wave + 4 * hh) = x;
  } else {
    // two quads: the halves of a wavefront exchange theirs, so that each lane holds eight columns
#pragma unroll
    for (int n = 0; n < kMyQuads; n += 2) {
      u32x4 x;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t a = E::pack2(sum[n][2 * c] * inv_l, sum[n][2 * c + 1] * inv_l);
        const uint32_t b = E::pack2(sum[n + 1][2 * c] * inv_l, sum[n + 1][2 * c + 1] * inv_l);
        const auto both = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        x[c] = both[0];
        x[2 + c] = both[1];
      }
      if (row < Nq) *reinterpret_cast<u32x4*>(out + 8 * (wave * kMyQuads + n + hh)) = x;
    }
  }
  if (LSE != nullptr && wave == 0 && hh == 0 && row < Nq)
    LSE[(size_t)bh * Nq + row] = m * 0.69314718055994530942f + __builtin_logf(l);
}

// Merge of the slices of one tile: a wavefront holds one quad of columns, as the kernel above left it.
template <int DT, int kD, bool kCausal>
__global__ __launch_bounds__(256) void fa2_short_merge_kernel(ShortCut cut, uint16_t* __restrict__ O, float* __restrict__ LSE, int H,
                                                              int Nq, int n_qtiles) {
  using E = Elem<DT>;
  constexpr int kQuads = kD / 8;
  const int lane = threadIdx.x & 63, r = lane & 31, hh = lane >> 5;
  const int quad = blockIdx.x % (kQuads / 4) * 4 + (threadIdx.x >> 6), tile = blockIdx.x / (kQuads / 4);
  const int bh = tile / n_qtiles, qt = tile - bh * n_qtiles;
  const int n = kCausal ? (qt + cut.chunk) / cut.chunk : cut.slices;   // slices that hold keys of this tile
  const int row = qt * kShortRows + r;
  if (n == 1 || row >= Nq) return;
  const size_t slot = (size_t)tile * cut.slices;
  const f32x4* po = reinterpret_cast<const f32x4*>(cut.part_o) + (slot * kQuads + quad) * 64 + lane;
  const f32x2* ml = reinterpret_cast<const f32x2*>(cut.part_ml) + slot * kShortRows + r;
  float m = kLowest, l = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  constexpr int kAhead = 4;   // slices whose loads are under way at once
  for (int s = 0; s < n; s += kAhead) {
    f32x4 x[kAhead];
    f32x2 y[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int at = min(s + i, n - 1);
      x[i] = po[(size_t)at * kQuads * 64];
      y[i] = ml[(size_t)at * kShortRows];
    }
    float m_new = m;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) m_new = fmaxf(m_new, y[i][0]);
    const float alpha = __builtin_amdgcn_exp2f(m - m_new);   // reference points are finite (kLowest at least)
    m = m_new;
    l *= alpha;
    o *= alpha;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const float w = s + i < n ? __builtin_amdgcn_exp2f(y[i][0] - m) : 0.f;
      l = __builtin_fmaf(w, y[i][1], l);
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(w, x[i][c], o[c]);
    }
  }
  const float inv_l = 1.0f / l;
  const u32x2 out = {E::pack2(o[0] * inv_l, o[1] * inv_l), E::pack2(o[2] * inv_l, o[3] * inv_l)};
  const int b = bh / H, h = bh - b * H;
  *reinterpret_cast<u32x2*>(O + (((size_t)b * Nq + row) * H + h) * kD + 8 * quad + 4 * hh) = out;
  if (LSE != nullptr && quad == 0 && hh == 0) LSE[(size_t)bh * Nq + row] = m * 0.69314718055994530942f + __builtin_logf(l);
}

template <int DT, int kD, int kWv> int launch(const Problem& p, const ShortPlan& plan, void* workspace) {
  const int n_q = (p.Nq + kShortRows - 1) / kShortRows, heads = p.B * p.H, total = heads * plan.items;
  ShortCut cut;
  cut.items = plan.items;
  if (plan.slices > 1) {
    cut.part_o = static_cast<float*>(workspace);
    cut.part_ml = cut.part_o + (size_t)heads * n_q * plan.slices * kShortRows * kD;
    cut.chunk = plan.chunk;
    cut.slices = plan.slices;
  }
  uint16_t* const o = static_cast<uint16_t*>(p.O);
  auto* kernel = fa2_short_kernel<DT, kD, kWv, true>;
  if constexpr (kWv > 2) {   // (two wavefronts: under the mask only)
    if (!p.causal) kernel = fa2_short_kernel<DT, kD, kWv, false>;
  }
  const int rc = enqueue(kernel, total, kWv * 64, p.stream, static_cast<const uint16_t*>(p.Q), static_cast<const uint16_t*>(p.K),
                         static_cast<const uint16_t*>(p.V), o, p.LSE, p.H, p.Nq, p.Nk, p.scale_log2e, n_q, total, cut);
  if (rc != FA2_OK || plan.slices == 1) return rc;
  return enqueue(p.causal ? fa2_short_merge_kernel<DT, kD, true> : fa2_short_merge_kernel<DT, kD, false>, heads * n_q * (kD / 32), 256,
                 p.stream, cut, o, p.LSE, p.H, p.Nq, n_q);
}

}  // namespace

size_t short_workspace(int B, int H, int Nq, int d, const ShortPlan& plan) {
  const size_t tiles = (size_t)B * H * ((Nq + kShortRows - 1) / kShortRows);
  return plan.slices == 1 ? 0 : tiles * plan.slices * kShortRows * (d + 2) * sizeof(float);
}

int short_tiles(const Problem& p, const ShortPlan& plan, void* workspace) {
  auto go = [&](auto dt) {
    constexpr int kDT = decltype(dt)::value;
    if (p.d == 256) return plan.waves == 2 ? launch<kDT, 256, 2>(p, plan, workspace) : launch<kDT, 256, 4>(p, plan, workspace);
    if (p.d == 128) return plan.waves == 4 ? launch<kDT, 128, 4>(p, plan, workspace) : launch<kDT, 128, 8>(p, plan, workspace);
    return plan.waves == 4 ? launch<kDT, 64, 4>(p, plan, workspace) : launch<kDT, 64, 8>(p, plan, workspace);
  };
  return p.dtype == FA2_FP16 ? go(std::integral_constant<int, FA2_FP16>{}) : go(std::integral_constant<int, FA2_BF16>{});
}

}  // namespace fa2
