// Streamed evaluation kernels with one K slice (x-powers 0..31) per digit product.
#include "eval_launch.h"

namespace rsl {

hipError_t launch_eval_stream1(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                               const DevTables& T, hipStream_t st) {
  launch_eval_variant<kEvQ, kEvNum, 2>(variant, probs, items, nitems, lds, T, st);
  return hipGetLastError();
}

}  // namespace rsl
