// Evaluation kernels: the lane-pair register forms and the Schur form.
#include "eval_launch.h"

namespace rsl {

hipError_t launch_eval_lanes(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                             const DevTables& T, hipStream_t st) {
  launch_eval_variant<kEvP8, kEvQ>(variant, probs, items, nitems, lds, T, st);
  return hipGetLastError();
}

}  // namespace rsl
