// Modular gcd over Z[x] for the square-free step after the resultant (the
// Project step of the paper's Sec. 3.2 takes a square-free factorisation of
// R by Yun's algorithm, i.e. gcds of R and its derivatives; the outlook of
// Sec. 6 proposes the modular route for it).  Device stages, per prime slot:
//   zreduce  u, v mod p (two's complement limbs, division-free)
//   zgcd     Euclid's algorithm over Z_p in LDS, one block per prime,
//            division-free steps; the gcd made monic and scaled by
//            ell = gcd(lc u, lc v) mod p
//   zpack    the kept slots' scaled gcds in the CRT input layout
//   zcof     G mod p = scaled gcd / (signed content), then the exact quotients
//            u / G and v / G by long division over Z_p (a nonzero remainder
//            flags a certificate failure)
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "modarith.h"
#include "stages.h"

namespace rsl {

struct ZgcdDesc {
  int nu, nv;           // degrees of u and v (nv = -1: v is zero)
  int Lu, Lv;           // limbs per coefficient
  int np;               // prime slots of the first pass
  int gs;               // row stride of the scaled gcds
  const uint32_t* u;    // (nu + 1) * Lu
  const uint32_t* v;    // (nv + 1) * Lv
  const int* pidx;      // np global prime indices
  const uint32_t* ell;  // np: ell mod p (normal form)
  uint32_t* up;         // np * (nu + 1) residues, normal form
  uint32_t* vp;         // np * (nv + 1)
  uint32_t* gt;         // np * gs: ell * (monic gcd mod p), normal form
  int* gdeg;            // np: degree of the gcd mod p
  // kept slots (least gcd degree)
  int nk, dg;           // kept slots, degree of G
  const int* kept;      // nk slot indices
  const uint32_t* smod; // nk: signed content of the scaled gcd mod p, normal form
  uint64_t* c0;         // nk * (dg + 1): scaled gcd, CRT input layout (Montgomery form)
  uint64_t* cg;         // nk * (dg + 1): G mod p
  uint64_t* ca;         // nk * (nu - dg + 1): u / G mod p
  uint64_t* cb;         // nk * (nv - dg + 1): v / G mod p (nv >= dg)
  int* rem;             // [0] set when a division leaves a remainder
};

constexpr int kZThreads = 256;  // threads of a block of every pass

// residues of u (sub 0) or v (sub 1): item slot, block of 256 coefficients
__device__ inline void stage_zreduce(const ZgcdDesc& Z, const DevTables& T, const WorkItem& w) {
  const int n = w.sub ? Z.nv : Z.nu, L = w.sub ? Z.Lv : Z.Lu;
  const int t = w.blk * kZThreads + static_cast<int>(threadIdx.x);
  if (t > n) return;
  const PrimeConst pc = T.pc[Z.pidx[w.slot]];
  const uint32_t* src = (w.sub ? Z.v : Z.u) + static_cast<size_t>(t) * L;
  uint32_t* dst = w.sub ? Z.vp : Z.up;
  dst[static_cast<size_t>(w.slot) * (n + 1) + t] = limbs_mod_p(src, L, pc);
}

__host__ __device__ inline int zgcd_lds_words(const ZgcdDesc& Z) { return (Z.nu + 1) + (Z.nv + 2); }

// Degree of a[0..d-1] (its entries below d): the highest nonzero, found 64
// entries at a time by a wave ballot (-1 when all are zero).  Wave-uniform.
__device__ inline int zdeg_below(const uint32_t* a, int d) {
  const int lane = threadIdx.x & 63;
  for (int top = d; top > 0; top -= 64) {
    const int j = top - 64 + lane;
    const uint64_t nz = __ballot(j >= 0 && a[j] != 0u);
    if (nz) return top - 64 + (63 - __clzll(static_cast<long long>(nz)));
  }
  return -1;
}

// One block per prime slot.  Pseudo-remainder steps without divisions keep A a
// nonzero multiple of the remainder sequence's members, so the last nonzero one
// is a multiple of the gcd; one inversion at the end makes it monic.  In the
// generic pattern (deg A = deg B + 1) one pass takes the two eliminations at
// once, as in the evaluation,
//   A[j] <- L^2 A[j] - L lc(A) B[j-1] - (L A[b] - lc(A) B[b-1]) B[j],  L = lc(B),
// with one barrier: a step's scalars and every B[j] come from entries it does
// not write.  Bound by the latency of a step, so a step is one LDS round trip
// (a thread's first kZHold entries are read together with the scalars' operands)
// and one product for all three scalars, a lane each.  A polynomial of degree 360
// and its derivative: 92 us, 0.25 us a step (115 us with the scalars as three
// products and the entries read after them; 326 us with one wave per prime and
// one elimination per pass, six coefficients a lane going through every step).
constexpr int kZHold = 2;
__device__ inline void stage_zgcd(const ZgcdDesc& Z, const DevTables& T, int slot, uint32_t* lds) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const PrimeConst pc = T.pc[Z.pidx[slot]];
  const uint32_t p = pc.p, pinv = pc.pinv, one = pc.r1;
  uint32_t* X = lds;                 // nu + 1 words
  uint32_t* Y = lds + (Z.nu + 1);    // nv + 1 words
  for (int k = tid; k <= Z.nu; k += nt) X[k] = mmul(Z.up[static_cast<size_t>(slot) * (Z.nu + 1) + k], pc.r2, p, pinv);
  for (int k = tid; k <= Z.nv; k += nt) Y[k] = mmul(Z.vp[static_cast<size_t>(slot) * (Z.nv + 1) + k], pc.r2, p, pinv);
  __syncthreads();
  uint32_t* A = X;
  uint32_t* B = Y;
  // degrees, the same in every wave: read from LDS between barriers
  int da = zdeg_below(X, Z.nu + 1), db = (Z.nv >= 0) ? zdeg_below(Y, Z.nv + 1) : -1;
  if (da < db) {
    uint32_t* t = A; A = B; B = t;
    const int d = da; da = db; db = d;
  }
  while (db > 0) {
    if (da == db + 1) {
      uint32_t av[kZHold], bv[kZHold], bl[kZHold];
#pragma unroll
      for (int r = 0; r < kZHold; ++r) {
        const int j = tid + r * nt, jj = j < db ? j : 0;
        av[r] = A[jj];
        bv[r] = B[jj];
        bl[r] = B[jj > 0 ? jj - 1 : 0];
      }
      const uint32_t L = B[db], lcA = A[da], Ab = A[db], Bb = B[db - 1];
      if (L == 0u) {  // the last remainder dropped by more than one degree
        db = zdeg_below(B, db);
        continue;
      }
      // lane 0: L L, lane 1: -L lc(A), lane 2: lc(A) B[b-1] - L A[b], as x y - u w
      const int ln = tid & 3;
      const uint32_t v = mmulsub(ln == 0 ? L : ln == 1 ? 0u : lcA, ln == 0 ? L : Bb, ln == 0 ? 0u : L, ln == 1 ? lcA : Ab,
                                 p, pinv);
      const uint32_t al = __builtin_amdgcn_readlane(v, 0), be = __builtin_amdgcn_readlane(v, 1),
                     ga = __builtin_amdgcn_readlane(v, 2);
#pragma unroll
      for (int r = 0; r < kZHold; ++r) {
        const int j = tid + r * nt;
        if (j < db) A[j] = mmad3(al, av[r], be, j > 0 ? bl[r] : 0u, ga, bv[r], p, pinv);
      }
      for (int j = tid + kZHold * nt; j < db; j += nt) A[j] = mmad3(al, A[j], be, B[j - 1], ga, B[j], p, pinv);
      __syncthreads();
      da = db;
      db -= 1;  // at most: the next step sees a zero leading coefficient
    } else {
      const uint32_t L = B[db];
      for (int d = da; d >= db; --d) {
        const uint32_t la = A[d];
        const int s = d - db;
        for (int j = tid; j < d; j += nt)
          A[j] = (j >= s) ? mmulsub(L, A[j], la, B[j - s], p, pinv) : mmul(L, A[j], p, pinv);
        __syncthreads();
      }
      da = db;
      db = zdeg_below(A, db);
    }
    uint32_t* t = A; A = B; B = t;
  }
  if (db == 0 && B[0] != 0u) {  // a nonzero constant: the gcd
    A = B;
    da = 0;
  }
  const uint32_t inv = (da >= 0) ? minv(A[da], one, p, pinv) : 0u;
  for (int k = tid; k <= da; k += nt)
    Z.gt[static_cast<size_t>(slot) * Z.gs + k] = mmul(mmul(A[k], inv, p, pinv), Z.ell[slot], p, pinv);
  if (tid == 0) Z.gdeg[slot] = da;
}

// kept slot i: the scaled gcd in the CRT input layout (Montgomery form: the
// CRT reduces each entry once)
__device__ inline void stage_zpack(const ZgcdDesc& Z, const DevTables& T, int i) {
  const int slot = Z.kept[i];
  const PrimeConst pc = T.pc[Z.pidx[slot]];
  for (int k = threadIdx.x; k <= Z.dg; k += blockDim.x)
    Z.c0[static_cast<size_t>(i) * (Z.dg + 1) + k] =
        mmul(Z.gt[static_cast<size_t>(slot) * Z.gs + k], pc.r2, pc.p, pc.pinv);
}

__host__ __device__ inline int zcof_lds_words(const ZgcdDesc& Z) {
  const int n = Z.nu > Z.nv ? Z.nu : Z.nv;
  return (n + 1) + (Z.dg + 1);
}

// Long division of W (degree n, Montgomery) by G (degree dg, Montgomery,
// inverse leading coefficient ginv): quotient coefficients to q[0..n-dg]
// (Montgomery form, the CRT input layout), remainder check.  One barrier per
// quotient coefficient; the row taken off is W[k+dg] (G / lc G), one product
// behind the barrier, and a thread's first kZHold entries of G / lc G stay in
// registers.
__device__ inline void zdivide(uint32_t* W, int n, uint32_t* G, int dg, uint32_t ginv, uint64_t* q,
                               int* rem, const PrimeConst& pc) {
  const uint32_t p = pc.p, pinv = pc.pinv;
  const int tid = threadIdx.x, nt = blockDim.x;
  __syncthreads();  // every thread has read lc G
  for (int j = tid; j < dg; j += nt) G[j] = mmul(G[j], ginv, p, pinv);
  uint32_t gv[kZHold];
#pragma unroll
  for (int r = 0; r < kZHold; ++r) gv[r] = tid + r * nt < dg ? G[tid + r * nt] : 0u;
  for (int k = n - dg; k >= 0; --k) {
    uint32_t wv[kZHold];
#pragma unroll
    for (int r = 0; r < kZHold; ++r) wv[r] = tid + r * nt < dg ? W[k + tid + r * nt] : 0u;
    const uint32_t top = W[k + dg];
#pragma unroll
    for (int r = 0; r < kZHold; ++r)
      if (tid + r * nt < dg) W[k + tid + r * nt] = msubm(wv[r], mmul(top, gv[r], p, pinv), p);
    for (int j = tid + kZHold * nt; j < dg; j += nt) W[k + j] = msubm(W[k + j], mmul(top, G[j], p, pinv), p);
    __syncthreads();
  }
  // the tops stayed where they were; stores inside the loop would each be waited
  // for at its barrier
  for (int k = tid; k <= n - dg; k += nt) q[k] = mmul(W[k + dg], ginv, p, pinv);
  if (zdeg_below(W, dg) >= 0 && tid == 0) rem[0] = 1;
}

// Kept slot i: G mod p, then u / G (part 0) or v / G (part 1), a block each:
// bound by the latency of a quotient coefficient like the steps above.  Degree
// 360: 43 us (53 us with two products behind each barrier and the quotient stored
// as it came; 114 us with one wave per prime and the divisions in turn).
__device__ inline void stage_zcof(const ZgcdDesc& Z, const DevTables& T, int i, int part, uint32_t* lds) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int slot = Z.kept[i];
  const PrimeConst pc = T.pc[Z.pidx[slot]];
  const uint32_t p = pc.p, pinv = pc.pinv, one = pc.r1;
  const int n = part ? Z.nv : Z.nu;
  if (n < Z.dg) return;  // v = 0 (no cofactor)
  uint32_t* W = lds;              // n + 1 words
  uint32_t* G = lds + (n + 1);    // dg + 1 words
  const uint32_t sM = minv(mmul(Z.smod[i], pc.r2, p, pinv), one, p, pinv);
  for (int k = tid; k <= Z.dg; k += nt) {
    const uint32_t g = mmul(mmul(Z.gt[static_cast<size_t>(slot) * Z.gs + k], pc.r2, p, pinv), sM, p, pinv);
    G[k] = g;
    if (part == 0) Z.cg[static_cast<size_t>(i) * (Z.dg + 1) + k] = g;
  }
  const uint32_t* src = (part ? Z.vp : Z.up) + static_cast<size_t>(slot) * (n + 1);
  for (int k = tid; k <= n; k += nt) W[k] = mmul(src[k], pc.r2, p, pinv);
  __syncthreads();
  const uint32_t ginv = minv(G[Z.dg], one, p, pinv);
  uint64_t* q = (part ? Z.cb : Z.ca) + static_cast<size_t>(i) * (n - Z.dg + 1);
  zdivide(W, n, G, Z.dg, ginv, q, Z.rem, pc);
}

}  // namespace rsl
