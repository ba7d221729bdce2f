// Evaluation kernels: the LDS-column layouts and the one-lane register form on Horner's rule.
#include "eval_launch.h"

namespace rsl {

hipError_t launch_eval_columns(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                               const DevTables& T, hipStream_t st) {
  launch_eval_variant<kEvBase, kEvP8>(variant, probs, items, nitems, lds, T, st);
  return hipGetLastError();
}

}  // namespace rsl
