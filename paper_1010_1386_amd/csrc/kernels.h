// Host-callable launchers of the device kernels (kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include "device.h"
#include "zgcd.h"

namespace rsl {

// One launch of stage `stage` (see stages.h) over `nitems` work items, one
// block per item.  lds: dynamic LDS bytes; crt_ns: prime slots per lane of the
// CRT kernel (ceil(max primes / 64)); crt_per_block: CRT items per block
// (consecutive items of one problem share the staged constants).  whole: the
// interpolation left each coefficient as one word (staged and plain schedules).
hipError_t launch_stage(int stage, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                        int crt_ns, const DevTables& T, hipStream_t st, int crt_per_block, bool whole);

// The CRT of up to kSlotCrtPrimes primes on the matrix cores, kCrtMmRows
// coefficients per item; max_np: the most primes of any item's problem.
hipError_t launch_crt_mm(const DevProblem* probs, const WorkItem* items, int nitems, int max_np, const DevTables& T,
                         hipStream_t st, bool whole);

// The reduction of problems with digit tiles: items whose sub is spw
// (kReduceSlotsShort for inputs of at most two limbs, kReduceSlotsLong beyond).
hipError_t launch_reduce_tiles(int spw, const DevProblem* probs, const WorkItem* items, int nitems, const DevTables& T,
                               hipStream_t st);

// Evaluation + univariate resultants of items that all have layout `variant`.
hipError_t launch_eval(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                       const DevTables& T, hipStream_t st);

// Pass 0, 1 or 2 of the wide CRT (t values and quotients, column sums, carries
// and output) over `nitems` items; pass 3 is pass 1 on the matrix cores.
hipError_t launch_crt_wide(int pass, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                           const DevTables& T, hipStream_t st, bool whole);

// The wide CRT's digit planes of the M_i limbs, from M (items: problem, 64 primes,
// 64 limbs; lds: the most wide_digits_lds_words of its problems, in bytes).
hipError_t launch_wide_digits(const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                              const DevTables& T, hipStream_t st);

// Pass 0 (reduce u, v over `nitems` items), 1 (Euclid per prime slot), 2 (pack
// the kept scaled gcds) or 3 (G and the cofactors per kept slot) of the modular gcd.
hipError_t launch_zgcd_pass(int pass, const ZgcdDesc& Z, const WorkItem* items, int nitems, const DevTables& T,
                            hipStream_t st);

// Interpolation on the matrix cores, items (problem, slot, tile of 256): which =
// 0, Newton coefficients and segment polynomials; 1, the basis change.  maxD:
// the largest degree bound of the items.
hipError_t launch_interp(int which, const DevProblem* probs, const WorkItem* items, int nitems, int maxD,
                         const DevTables& T, hipStream_t st);

// Stirling numbers of the first kind mod p_g for g in [g0, g0+count), rows 0..scap.
hipError_t launch_stirling_build(uint32_t* stir, int64_t sstride, const PrimeConst* pcs, int g0,
                                 int count, int scap, hipStream_t st);

// dst[t] = src[t] (or 0 when src is null) for t < n words.
hipError_t launch_copy_words(uint32_t* dst, const uint32_t* src, size_t n, hipStream_t st);

}  // namespace rsl
