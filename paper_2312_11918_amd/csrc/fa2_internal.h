// What the translation units of libfa2 share: the validated problem and the launchers beside the tile kernels.
#ifndef FA2_INTERNAL_H_
#define FA2_INTERNAL_H_
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <tuple>

#include "fa2.h"
#include "fa2_short_plan.h"
#include "fa2_split_plan.h"

namespace fa2 {

// A problem that has passed validation.
struct Problem {
  const void *Q, *K, *V;
  void* O;
  float* LSE;  // may be null
  int B, H, Nq, Nk, d;
  float scale_log2e;  // scale * log2(e)
  int dtype;
  bool causal;
  hipStream_t stream;
};

// Enqueues `kernel` and reports this launch's own status (not whatever error an earlier, unrelated HIP call left).
template <class... Params, class... Args>
int enqueue(void (*kernel)(Params...), int grid, int block, hipStream_t stream, Args... args) {
  std::tuple<Params...> values{static_cast<Params>(args)...};
  void* ptrs[sizeof...(Params)];
  std::apply([&](auto&... v) { int i = 0; ((ptrs[i++] = &v), ...); }, values);
  const hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)grid), dim3((unsigned)block),
                                         ptrs, 0, stream);
  return err == hipSuccess ? FA2_OK : FA2_ERR_LAUNCH;
}

// fa2_decode.hip: one query per sequence (Nq == 1).  The workspace is used only if it holds decode_workspace bytes.
__attribute__((visibility("hidden"))) bool decode_accepts(int B, int H, int Nq);
__attribute__((visibility("hidden"))) size_t decode_workspace(int B, int H, int Nk, int d);
__attribute__((visibility("hidden"))) int decode(const Problem& p, void* workspace, size_t workspace_bytes);

// fa2_split.hip: several queries, but too few Q tiles to fill the chip.  split_workspace() is 0 when the keys are not cut
// into slices; with fewer bytes than it says they are not either, only into halves.  split_tiles() launches nothing and is
// false where the whole launch is the better one; otherwise *rc is the launch's return code.
__attribute__((visibility("hidden"))) size_t split_workspace(int B, int H, int Nq, int Nk, int d, bool causal);
__attribute__((visibility("hidden"))) bool split_tiles(const Problem& p, void* workspace, size_t workspace_bytes, int* rc);

// fa2_short.hip: few query rows in all, as short_plan() says; returns the launch's return code.  short_workspace(): the bytes that
// the slices of a plan take.
__attribute__((visibility("hidden"))) size_t short_workspace(int B, int H, int Nq, int d, const ShortPlan& plan);
__attribute__((visibility("hidden"))) int short_tiles(const Problem& p, const ShortPlan& plan, void* workspace);

// fa2_wide.hip: d = 128 on partial tiles in the 256-row shape.  Launches nothing and is false where another launch is the better
// one; otherwise *rc is the launch's return code.
__attribute__((visibility("hidden"))) bool wide_tiles(const Problem& p, int* rc);

// fa2_stage.hip: d = 64 with 64 query rows per wavefront, and d = 256.  Launches nothing and is false where the tile kernel's
// whole launch is the better one; otherwise *rc is the launch's return code.
__attribute__((visibility("hidden"))) bool stage_tiles(const Problem& p, int* rc);

}  // namespace fa2
#endif  // FA2_INTERNAL_H_
