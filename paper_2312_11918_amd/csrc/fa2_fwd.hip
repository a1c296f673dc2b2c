// FlashAttention-2 forward pass for gfx950: choice of the tile shape, launches and C ABI of libfa2.
#include "fa2_tile_kernel.h"

namespace {

constexpr int kRows256 = 256;  // query rows per workgroup of the 8-wavefront shape

// One instantiation of the 32-row kernel.
template <int DT, int D, int kWv, int kNBuf, bool kCausal, bool kRagged>
int launch_rows32(const void* Q, const void* K, const void* V, void* O, float* LSE, int H, int Nq, int Nk,
                  float scale_log2e, int n_qtiles, int total, hipStream_t stream, int chain = 1) {
  return enqueue(fa2_fwd_kernel<DT, D, kWv, kNBuf, kCausal, kRagged>, total, kWv * 64, stream,
                 static_cast<const uint16_t*>(Q), static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V),
                 static_cast<uint16_t*>(O), LSE, H, Nq, Nk, scale_log2e, n_qtiles, total, chain, SplitArgs{});
}

template <int DT, int D>
int launch(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int Nq, int Nk, float scale,
           int variant, int mask, hipStream_t stream) {
  const float scale_log2e = scale * 1.44269504088896340736f;
  const bool rows256 = variant == FA2_VARIANT_NARROW8;
  const bool causal = mask == FA2_MASK_CAUSAL;
  const bool ragged = Nq % kBr != 0 || Nk % kBr != 0;  // 128-row shape only (checked by the caller)
  const int rows = rows256 ? kRows256 : kBr;
  const int n_qtiles = (Nq + rows - 1) / rows;
  // causal: one workgroup per pair of Q tiles (n_qtiles-1-p, p)
  const long long total_ll = (long long)B * H * (causal ? (n_qtiles + 1) / 2 : n_qtiles);
  if (total_ll > 0x7fffffffLL) return FA2_ERR_UNSUPPORTED;
  const int total = (int)total_ll;
  if (rows256) {  // exact tiles, d <= 128 (checked by the caller)
    if constexpr (D <= 128) {
      // When the Q tiles (causal: the pairs of Q tiles, all complete) fill whole rounds of the CUs, one workgroup
      // per CU takes a Q tile (pair) of every round.
      const int chain = total % kCUs == 0 && !(causal && n_qtiles % 2 != 0) ? total / kCUs : 1;
      if (causal)
        return launch_rows32<DT, D, 8, 4, true, false>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total / chain,
                                                       stream, chain);
      return launch_rows32<DT, D, 8, 4, false, false>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total / chain,
                                                      stream, chain);
    } else {
      return FA2_ERR_UNSUPPORTED;
    }
  } else if (causal) {
    if (ragged) return launch_rows32<DT, D, 4, 2, true, true>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total, stream);
    // d = 256: pairs chained like the Q tiles of the unmasked case (whole rounds of complete pairs)
    const int chain = D == 256 && total % kCUs == 0 && n_qtiles % 2 == 0 ? total / kCUs : 1;
    return launch_rows32<DT, D, 4, 2, true, false>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total / chain, stream,
                                                   chain);
  }
  if (ragged) return launch_rows32<DT, D, 4, 2, false, true>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total, stream);
  // d = 256 (one workgroup per CU): when the Q tiles fill whole rounds of the CUs, one workgroup per CU takes a Q tile
  // of every round, as in the 256-row shape
  const int chain = D == 256 && total % kCUs == 0 ? total / kCUs : 1;
  return launch_rows32<DT, D, 4, 2, false, false>(Q, K, V, O, LSE, H, Nq, Nk, scale_log2e, n_qtiles, total / chain, stream,
                                                  chain);
}

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// The problems (of positive sizes, with a known mask) that the entry points take.
bool sizes_fit(int B, int H, int Nq, int Nk, int d, int mask) {
  if (d != 64 && d != 128 && d != 256) return false;
  if (mask == FA2_MASK_CAUSAL && Nq != Nk) return false;  // the diagonal is defined for a square S only
  // element offsets are computed in 64 bits; the row index b*N+n must still fit the tile arithmetic
  const int n_max = Nq > Nk ? Nq : Nk;
  if ((long long)B * n_max > 0x7fffffffLL) return false;
  // the K/V rows of one batch entry are addressed with 32-bit byte offsets from a buffer descriptor
  return (unsigned long long)n_max * (unsigned long long)H * (unsigned long long)d * 2ull < (1ull << 32);
}

// The tile shape that FA2_VARIANT_AUTO stands for (sizes already validated by the caller).
int choose_variant(int B, int H, int Nq, int Nk, int d, int mask) {
  // Measured on MI355X with N(0,1) inputs: when its Q tiles fill whole rounds of the chip's 256 CUs (one workgroup
  // per CU, which then takes one Q tile of every round), the 8-wavefront, 256-row shape is faster than the
  // 4-wavefront, 128-row shape by 3-6 % at d = 128 at every N, and by 1-2 % at d = 64 from N = 4096 on (at d = 64
  // below N = 2048 its two wavefronts per SIMD against three lose 2-5 %; what stage_accepts() leaves of d = 64 has one
  // round of it, so that it chains there in an explicit choice only).  With many rounds that are not whole it
  // still gains at d = 128 from N = 2048 on; with few, the 128-row shape, two workgroups per CU, spreads the
  // remainder better.  d = 256 exists in the 128-row shape only, partial tiles in the 256-row shape in fa2_wide.hip's
  // launches only, which come before this choice.
  // Under the causal mask (one workgroup per pair of Q tiles, no chaining) it gains 1-3 % at d = 128 from N = 2048 on.
  const bool causal = mask == FA2_MASK_CAUSAL;
  const long long qt256 = Nq / kRows256;
  const long long wg256 = (long long)B * H * (causal ? (qt256 + 1) / 2 : qt256);
  const bool whole_rounds = wg256 % kCUs == 0;   // unmasked: then one workgroup per CU chains a Q tile of every round
  const bool rows256 = d <= 128 && Nq == Nk && Nq % kRows256 == 0 &&
                       (causal ? d == 128 && Nq >= 2048 && (whole_rounds || wg256 >= 16 * kCUs)
                               : (whole_rounds && (d == 128 || Nq >= 2048)) ||
                                     (d == 128 && wg256 >= 16 * kCUs && Nq >= 2048));
  return rows256 ? FA2_VARIANT_NARROW8 : FA2_VARIANT_NARROW;
}

int run(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int Nq, int Nk, int d,
        float scale, int dtype, int variant, int mask, void* stream, void* workspace = nullptr, size_t workspace_bytes = 0) {
  // All validation happens before the first HIP call: an error launches nothing.
  if (Q == nullptr || K == nullptr || V == nullptr || O == nullptr) return FA2_ERR_INVALID_ARG;
  if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || d <= 0) return FA2_ERR_INVALID_ARG;
  if (!(scale > 0.0f) || !(scale <= 3.0e38f)) return FA2_ERR_INVALID_ARG;  // rejects NaN, inf, <= 0
  if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16) || !aligned(LSE, 4))
    return FA2_ERR_INVALID_ARG;
  if (variant != FA2_VARIANT_AUTO && variant != FA2_VARIANT_NARROW && variant != FA2_VARIANT_NARROW8)
    return FA2_ERR_INVALID_ARG;
  if (mask != FA2_MASK_NONE && mask != FA2_MASK_CAUSAL) return FA2_ERR_INVALID_ARG;
  if (dtype != FA2_FP16 && dtype != FA2_BF16) return FA2_ERR_UNSUPPORTED;
  if (!sizes_fit(B, H, Nq, Nk, d, mask)) return FA2_ERR_UNSUPPORTED;
  if (variant == FA2_VARIANT_AUTO) {
    const fa2::Problem p{Q, K, V, O, LSE, B, H, Nq, Nk, d, scale * 1.44269504088896340736f, dtype, mask == FA2_MASK_CAUSAL,
                         static_cast<hipStream_t>(stream)};
    if (fa2::decode_accepts(B, H, Nq)) return fa2::decode(p, workspace, workspace_bytes);
    int rc;
    fa2::ShortPlan plan = fa2::short_plan(B, H, Nq, Nk, d, p.causal, workspace != nullptr);
    if (plan.slices > 1 && workspace_bytes < fa2::short_workspace(B, H, Nq, d, plan)) {
      // too little is as good as none, also for slices of 128 rows, which may take less (B1 H1 Nq128 Nk8000 d64: 540672 bytes
      // of 946176): what a call computes does not depend on how much it was given
      workspace = nullptr;
      workspace_bytes = 0;
      plan = fa2::short_plan(B, H, Nq, Nk, d, p.causal, false);
    }
    if (plan.waves != 0) return fa2::short_tiles(p, plan, workspace);
    if (fa2::split_tiles(p, workspace, workspace_bytes, &rc) || fa2::stage_tiles(p, &rc) || fa2::wide_tiles(p, &rc)) return rc;
    variant = choose_variant(B, H, Nq, Nk, d, mask);
  }
  if (variant != FA2_VARIANT_NARROW) {
    // the 256-row shape: whole tiles, square, d <= 128
    if (Nq != Nk || Nq % kRows256 != 0 || d == 256) return FA2_ERR_UNSUPPORTED;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (dtype == FA2_FP16) {
    return d == 64    ? launch<FA2_FP16, 64>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s)
           : d == 128 ? launch<FA2_FP16, 128>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s)
                      : launch<FA2_FP16, 256>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s);
  }
  return d == 64    ? launch<FA2_BF16, 64>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s)
         : d == 128 ? launch<FA2_BF16, 128>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s)
                    : launch<FA2_BF16, 256>(Q, K, V, O, LSE, B, H, Nq, Nk, scale, variant, mask, s);
}

}  // namespace

extern "C" int fa2_fwd_variant(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int N,
                               int d, float scale, int dtype, int variant, void* stream) {
  return run(Q, K, V, O, LSE, B, H, N, N, d, scale, dtype, variant, FA2_MASK_NONE, stream);
}

extern "C" int fa2_fwd_masked(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int N,
                              int d, float scale, int dtype, int mask, void* stream) {
  return run(Q, K, V, O, LSE, B, H, N, N, d, scale, dtype, FA2_VARIANT_AUTO, mask, stream);
}

extern "C" int fa2_fwd_qk(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int Nq,
                          int Nk, int d, float scale, int dtype, int mask, void* stream) {
  return run(Q, K, V, O, LSE, B, H, Nq, Nk, d, scale, dtype, FA2_VARIANT_AUTO, mask, stream);
}

extern "C" int fa2_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int N, int d,
                       float scale, int dtype, void* stream) {
  return run(Q, K, V, O, LSE, B, H, N, N, d, scale, dtype, FA2_VARIANT_AUTO, FA2_MASK_NONE, stream);
}

extern "C" int fa2_fwd_ws(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H, int Nq, int Nk,
                          int d, float scale, int dtype, int mask, void* workspace, size_t workspace_bytes, void* stream) {
  if (!aligned(workspace, 16)) return FA2_ERR_INVALID_ARG;
  return run(Q, K, V, O, LSE, B, H, Nq, Nk, d, scale, dtype, FA2_VARIANT_AUTO, mask, stream, workspace, workspace_bytes);
}

extern "C" size_t fa2_workspace_bytes(int B, int H, int Nq, int Nk, int d, int mask) {
  if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || (mask != FA2_MASK_NONE && mask != FA2_MASK_CAUSAL)) return 0;
  if (!sizes_fit(B, H, Nq, Nk, d, mask)) return 0;
  if (fa2::decode_accepts(B, H, Nq)) return fa2::decode_workspace(B, H, Nk, d);
  const bool causal = mask == FA2_MASK_CAUSAL;
  const fa2::ShortPlan plan = fa2::short_plan(B, H, Nq, Nk, d, causal, true);
  return plan.waves != 0 ? fa2::short_workspace(B, H, Nq, d, plan) : fa2::split_workspace(B, H, Nq, Nk, d, causal);
}

extern "C" int fa2_tile_shape(int B, int H, int Nq, int Nk, int d, int mask) {
  if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0) return FA2_ERR_INVALID_ARG;
  if (mask != FA2_MASK_NONE && mask != FA2_MASK_CAUSAL) return FA2_ERR_INVALID_ARG;
  if (d != 64 && d != 128 && d != 256) return FA2_ERR_UNSUPPORTED;
  if (mask == FA2_MASK_CAUSAL && Nq != Nk) return FA2_ERR_UNSUPPORTED;
  return choose_variant(B, H, Nq, Nk, d, mask);
}

extern "C" const char* fa2_strerror(int code) {
  switch (code) {
    case FA2_OK: return "success";
    case FA2_ERR_INVALID_ARG: return "invalid argument (NULL or misaligned pointer, non-positive size, scale not finite and > 0, or unknown variant or mask)";
    case FA2_ERR_UNSUPPORTED: return "unsupported problem (d must be 64, 128 or 256; dtype fp16 or bf16; the causal mask needs Nq == Nk; the 256-row tile shape needs d <= 128 and N a multiple of 256; sizes must fit 32-bit offsets)";
    case FA2_ERR_LAUNCH: return "the HIP runtime refused the kernel launch";
    default: return "unknown fa2 error code";
  }
}

extern "C" int fa2_version(void) { return 600; /* 0.6.0 */ }
