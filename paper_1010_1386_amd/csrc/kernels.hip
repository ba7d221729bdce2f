// HIP kernels of the modular resultant pipeline for gfx950 (wave64).
//
// Every stage kernel walks a host-built list of work items, one item per
// block, so that one launch per stage serves any number of problems of
// different shapes (a single problem is a batch of one).
//
//   reduce      coefficients (multi-limb) -> residues c R^2 mod p, transposed tiles
//                                                         (paper Sec. 4.1, step 1)
//   eval_ures   one lane per (prime, point): Horner evaluation at x_i and the
//               univariate resultant over Z_p             (Sec. 4.1, steps 1-2)
//   interp      Newton forward differences on consecutive points and segment
//               polynomials; falling-factorial -> monomial basis
//   interp_newton divided differences on a gapped point set (bad points replaced)
//                                                         (Sec. 4.1, step 3)
//   crt_mm      direct form, limb sums on the matrix cores, an undecided quotient settled by
//               the sign of Y - M                        (Sec. 4.1, step 3)
//   crt         direct form by column sums with Garner fallback (gcds and jobs without room for
//               the digits, the Garner hook); crt_wide_* beyond 512 primes
//   crt_wide_*  the direct form in three passes for problems with many primes
//   stirling_build  per-prime table of Stirling numbers of the first kind
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "eval_launch.h"
#include "kernels.h"
#include "stages.h"
#include "zgcd.h"

namespace rsl {

static_assert(kCrtWaves == kCrtBlockCoeffs, "one coefficient per wave of a CRT block");

__global__ __launch_bounds__(256) void k_reduce(const DevProblem* probs, const WorkItem* items, DevTables T) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  if (w.sub)
    stage_reduce_ml(probs[w.prob], T, w, lds);
  else
    stage_reduce(probs[w.prob], T, w, true);
}

// Digit tiles (items ordered by their sub, the prime slots per wave)
template <int SPW>
__global__ __launch_bounds__(256) void k_reduce_tiles(const DevProblem* probs, const WorkItem* items, DevTables T) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  stage_reduce_tiles<SPW>(probs[w.prob], T, w, lds);
}

hipError_t launch_reduce_tiles(int spw, const DevProblem* probs, const WorkItem* items, int nitems, const DevTables& T,
                               hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  const dim3 g(nitems), b(256);
  if (spw == kReduceSlotsShort) hipLaunchKernelGGL(k_reduce_tiles<kReduceSlotsShort>, g, b, 0, st, probs, items, T);
  else if (spw == kReduceSlotsLong)
    hipLaunchKernelGGL(k_reduce_tiles<kReduceSlotsLong>, g, b, reduce_tiles_lds_words() * 4, st, probs, items, T);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_eval(int variant, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                       const DevTables& T, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  if (variant < 0 || variant >= kEvNum) return hipErrorInvalidValue;
  const auto launch = variant < kEvP8 ? launch_eval_columns
                      : variant < kEvQ ? launch_eval_lanes
                      : (variant - kEvQ) % 2 ? launch_eval_stream2 : launch_eval_stream1;
  return launch(variant, probs, items, nitems, lds, T, st);
}

template <int WHICH, int KS>
__global__ __launch_bounds__(64 * KS) void k_interp(const DevProblem* probs, const WorkItem* items, DevTables T) {
  extern __shared__ uint4 lds4[];
  uint32_t* lds = reinterpret_cast<uint32_t*>(lds4);
  const WorkItem w = items[blockIdx.x];
  if constexpr (WHICH == 0) stage_interp_coeffs<KS>(probs[w.prob], T, w, lds);
  else stage_interp_basis<KS>(probs[w.prob], T, w, lds);
}

hipError_t launch_interp(int which, const DevProblem* probs, const WorkItem* items, int nitems, int maxD,
                         const DevTables& T, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  const int ks = nitems < kInterpSplitItems ? 4 : 1;
  const size_t lds = static_cast<size_t>(which == 0 ? interp_coeffs_lds_words(maxD, ks) : interp_basis_lds_words(ks)) * 4;
  const dim3 g(nitems), b(64 * ks);
  if (which == 0 && ks == 4) hipLaunchKernelGGL((k_interp<0, 4>), g, b, lds, st, probs, items, T);
  else if (which == 0) hipLaunchKernelGGL((k_interp<0, 1>), g, b, lds, st, probs, items, T);
  else if (ks == 4) hipLaunchKernelGGL((k_interp<1, 4>), g, b, lds, st, probs, items, T);
  else hipLaunchKernelGGL((k_interp<1, 1>), g, b, lds, st, probs, items, T);
  return hipGetLastError();
}

__global__ __launch_bounds__(1024) void k_interp_newton(const DevProblem* probs, const WorkItem* items, DevTables T,
                                                        bool whole) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  stage_interp_newton(probs[w.prob], T, w, lds, whole);
}

template <int NS>
__global__ __launch_bounds__(512) void k_crt(const DevProblem* probs, const WorkItem* items, int nitems, int per,
                                             DevTables T, bool whole) {
  extern __shared__ uint32_t lds[];
  // items blockIdx.x * per .. + per - 1 (one problem's items are consecutive:
  // the constants and limb table are staged again only when the problem changes)
  for (int b = 0; b < per; ++b) {
    const int idx = blockIdx.x * per + b;
    if (idx >= nitems) break;  // block-uniform
    const WorkItem w = items[idx];
    const bool fresh = b == 0 || items[idx - 1].prob != w.prob;
    if (b > 0) __syncthreads();  // the previous item's waves are done with the LDS
    stage_crt<NS>(probs[w.prob], T, w, lds, kCrtBlockCoeffs / static_cast<int>(blockDim.x >> 6), fresh, whole);
  }
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void k_crt_mm(const DevProblem* probs, const WorkItem* items, DevTables T,
                                                    bool whole) {
  extern __shared__ uint4 lds4[];
  const WorkItem w = items[blockIdx.x];
  stage_crt_mm<NW>(probs[w.prob], T, w, reinterpret_cast<uint32_t*>(lds4), whole);
}

hipError_t launch_crt_mm(const DevProblem* probs, const WorkItem* items, int nitems, int max_np, const DevTables& T,
                         hipStream_t st, bool whole) {
  if (nitems <= 0) return hipSuccess;
  const int nw = nitems < kCrtMmSplitItems ? 4 : 1;
  const size_t lds = static_cast<size_t>(crt_mm_lds_words(max_np, nw)) * 4;
  const dim3 g(nitems), b(64 * nw);
  if (nw == 4) hipLaunchKernelGGL(k_crt_mm<4>, g, b, lds, st, probs, items, T, whole);
  else hipLaunchKernelGGL(k_crt_mm<1>, g, b, lds, st, probs, items, T, whole);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_crt_wide_t(const DevProblem* probs, const WorkItem* items, DevTables T,
                                                     bool whole) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  stage_crt_wide_t(probs[w.prob], T, w, lds, whole);
}

__global__ __launch_bounds__(kWideHT) void k_crt_wide_sum(const DevProblem* probs, const WorkItem* items) {
  extern __shared__ uint4 lds4[];  // 16-byte aligned: rows of t values are read as uint4
  const WorkItem w = items[blockIdx.x];
  stage_crt_wide_sum(probs[w.prob], w, reinterpret_cast<uint32_t*>(lds4));
}

__global__ __launch_bounds__(64) void k_crt_wide_fin(const DevProblem* probs, const WorkItem* items) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  stage_crt_wide_fin(probs[w.prob], w, lds);
}

__global__ __launch_bounds__(256) void k_crt_wide_sum_mfma(const DevProblem* probs, const WorkItem* items) {
  extern __shared__ uint4 lds4[];
  const WorkItem w = items[blockIdx.x];
  stage_crt_wide_sum_mfma(probs[w.prob], w, reinterpret_cast<uint32_t*>(lds4));
}

__global__ __launch_bounds__(256) void k_wide_digits(const DevProblem* probs, const WorkItem* items, DevTables T) {
  extern __shared__ uint32_t lds[];
  const WorkItem w = items[blockIdx.x];
  stage_wide_digits(probs[w.prob], T, w, lds);
}

hipError_t launch_wide_digits(const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                              const DevTables& T, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_wide_digits, dim3(nitems), dim3(256), lds, st, probs, items, T);
  return hipGetLastError();
}

hipError_t launch_crt_wide(int pass, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                           const DevTables& T, hipStream_t st, bool whole) {
  if (nitems <= 0) return hipSuccess;
  const dim3 g(nitems);
  switch (pass) {
    case 0: hipLaunchKernelGGL(k_crt_wide_t, g, dim3(256), lds, st, probs, items, T, whole); break;
    case 1: hipLaunchKernelGGL(k_crt_wide_sum, g, dim3(kWideHT), lds, st, probs, items); break;
    case 2: hipLaunchKernelGGL(k_crt_wide_fin, g, dim3(64), lds, st, probs, items); break;
    case 3: hipLaunchKernelGGL(k_crt_wide_sum_mfma, g, dim3(256), lds, st, probs, items); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(kZThreads) void k_zreduce(ZgcdDesc Z, const WorkItem* items, DevTables T) {
  stage_zreduce(Z, T, items[blockIdx.x]);
}
__global__ __launch_bounds__(kZThreads) void k_zgcd(ZgcdDesc Z, DevTables T) {
  extern __shared__ uint32_t lds[];
  stage_zgcd(Z, T, blockIdx.x, lds);
}
__global__ __launch_bounds__(kZThreads) void k_zpack(ZgcdDesc Z, DevTables T) { stage_zpack(Z, T, blockIdx.x); }
__global__ __launch_bounds__(kZThreads) void k_zcof(ZgcdDesc Z, DevTables T) {
  extern __shared__ uint32_t lds[];
  stage_zcof(Z, T, blockIdx.x >> 1, blockIdx.x & 1, lds);
}

hipError_t launch_zgcd_pass(int pass, const ZgcdDesc& Z, const WorkItem* items, int nitems, const DevTables& T,
                            hipStream_t st) {
  const dim3 b(kZThreads);
  switch (pass) {
    case 0:
      if (nitems <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_zreduce, dim3(nitems), b, 0, st, Z, items, T);
      break;
    case 1:
      if (Z.np <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_zgcd, dim3(Z.np), b, static_cast<size_t>(zgcd_lds_words(Z)) * 4, st, Z, T);
      break;
    case 2:
      if (Z.nk <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_zpack, dim3(Z.nk), b, 0, st, Z, T);
      break;
    case 3:
      if (Z.nk <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_zcof, dim3(2 * Z.nk), b, static_cast<size_t>(zcof_lds_words(Z)) * 4, st, Z, T);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// s(k+1, j) = s(k, j-1) - k s(k, j); one block per prime, rows in LDS.
__global__ __launch_bounds__(1024) void k_stirling_build(uint32_t* stir, int64_t sstride,
                                                         const PrimeConst* pcs, int g0, int scap) {
  extern __shared__ uint32_t sm[];
  const int g = g0 + blockIdx.x;
  const PrimeConst pc = pcs[g];
  uint32_t* cur = sm;
  uint32_t* nxt = sm + (scap + 2);
  uint32_t* S = stir + static_cast<int64_t>(g) * sstride;
  if (threadIdx.x == 0) { cur[0] = pc.r1; S[0] = pc.r1; }
  __syncthreads();
  for (int k = 0; k < scap; ++k) {
    const uint32_t kt = mmul(static_cast<uint32_t>(k), pc.r2, pc.p, pc.pinv);
    const bool keep = ((k + 1) % kCkpt) == 0;  // a checkpoint row
    uint32_t* row = S + ckpt_rowoff((k + 1) / kCkpt);
    for (int j = threadIdx.x; j <= k + 1; j += 1024) {
      const uint32_t left = (j > 0) ? cur[j - 1] : 0u;
      const uint32_t mid = (j <= k) ? cur[j] : 0u;
      const uint32_t v = msubm(left, mmul(mid, kt, pc.p, pc.pinv), pc.p);
      nxt[j] = v;
      if (keep) row[j] = v;
    }
    __syncthreads();
    uint32_t* t = cur; cur = nxt; nxt = t;
  }
}

// ------------------------------------------------------------ launchers

hipError_t launch_stage(int stage, const DevProblem* probs, const WorkItem* items, int nitems, size_t lds,
                        int crt_ns, const DevTables& T, hipStream_t st, int crt_per_block, bool whole) {
  if (nitems <= 0) return hipSuccess;
  const dim3 g(nitems);
  const int per = crt_per_block > 1 ? crt_per_block : 1;
  const dim3 gc((nitems + per - 1) / per);
  switch (stage) {
    case kStageReduce: hipLaunchKernelGGL(k_reduce, g, dim3(256), lds, st, probs, items, T); break;
    case kStageEval: return hipErrorInvalidValue;  // launch_eval: one kernel per layout
    case kStageConv: return hipErrorInvalidValue;  // launch_interp
    case kStageStir: return hipErrorInvalidValue;
    case kStageNewton: hipLaunchKernelGGL(k_interp_newton, g, dim3(1024), lds, st, probs, items, T, whole); break;
    case kStageCrt:
      switch (crt_ns) {
        case 1: hipLaunchKernelGGL(k_crt<1>, gc, dim3(kCrtWaves * 64), lds, st, probs, items, nitems, per, T, whole); break;
        case 2: hipLaunchKernelGGL(k_crt<2>, gc, dim3(kCrtWaves * 64), lds, st, probs, items, nitems, per, T, whole); break;
        case 3: hipLaunchKernelGGL(k_crt<3>, gc, dim3(kCrtWaves * 64), lds, st, probs, items, nitems, per, T, whole); break;
        case 4: hipLaunchKernelGGL(k_crt<4>, gc, dim3(kCrtWaves * 64), lds, st, probs, items, nitems, per, T, whole); break;
        case 6:
          hipLaunchKernelGGL(k_crt<6>, gc, dim3(crt_block_waves(6) * 64), lds, st, probs, items, nitems, per, T, whole);
          break;
        case 8:
          hipLaunchKernelGGL(k_crt<8>, gc, dim3(crt_block_waves(8) * 64), lds, st, probs, items, nitems, per, T, whole);
          break;
        default: return hipErrorInvalidValue;
      }
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Device-to-device word copy / fill, launched as kernels so that a resident
// job's per-run resets are plain kernel nodes when the run is captured in a graph.
__global__ __launch_bounds__(256) void k_copy_words(uint32_t* dst, const uint32_t* src, size_t n) {
  for (size_t t = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; t < n;
       t += static_cast<size_t>(gridDim.x) * blockDim.x)
    dst[t] = src ? src[t] : 0u;
}

hipError_t launch_copy_words(uint32_t* dst, const uint32_t* src, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(k_copy_words, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, dst, src, n);
  return hipGetLastError();
}

hipError_t launch_stirling_build(uint32_t* stir, int64_t sstride, const PrimeConst* pcs, int g0,
                                 int count, int scap, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_stirling_build, dim3(count), dim3(1024),
                     static_cast<size_t>(2) * (scap + 2) * sizeof(uint32_t), st, stir, sstride, pcs, g0, scap);
  return hipGetLastError();
}

}  // namespace rsl
