// The evaluation kernel of one layout variant and its launch by a run-time
// variant number (the eval_*.hip sources compile disjoint variants).
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "stages.h"

namespace rsl {

// Waves per SIMD a layout's register budget must allow.  The streamed forms up
// to lower degree 32 take at most 168 registers (three waves; a few spilled
// words in the two-slice ones): degree bound 32 went from two waves and 299 us
// to 264 us on 256 pairs of the batch workload, the two-slice ones gained 3-7%.
// Four waves (128 registers) spill the register polynomial: 332 us; at lower
// degrees 40 and 48 already three waves do (394 -> 448 us, 163 -> 434 us on 64
// requests of degrees 8..48).
constexpr int ev_min_waves(int v) { return v >= kEvQ && (v - kEvQ) / 2 < 4 ? 3 : 1; }

template <int V>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ev_min_waves(V)))) void k_eval_ures(const DevProblem* probs, const WorkItem* items, DevTables T) {
  extern __shared__ uint4 lds4[];  // 16-byte aligned: the Horner loop reads uint4 rows
  uint32_t* lds = reinterpret_cast<uint32_t*>(lds4);
  const WorkItem w = items[blockIdx.x];
  stage_eval_variant<V>(probs[w.prob], T, w, lds);
}

// Launch variant V, V + STEP, ... < END that equals `variant`.
template <int V, int END, int STEP = 1>
static void launch_eval_variant(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                                const DevTables& T, hipStream_t st) {
  if (variant == V)
    hipLaunchKernelGGL(k_eval_ures<V>, dim3(nitems), dim3(64), lds, st, probs, items, T);
  else if constexpr (V + STEP < END)
    launch_eval_variant<V + STEP, END, STEP>(variant, probs, items, nitems, lds, T, st);
}

using EvalLaunch = hipError_t(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                              const DevTables& T, hipStream_t st);
EvalLaunch launch_eval_columns, launch_eval_lanes, launch_eval_stream1, launch_eval_stream2;

}  // namespace rsl
