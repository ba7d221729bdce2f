// Device code of the pipeline stages.  Each stage_* function processes one
// work item with one thread block; the stage kernels (kernels.hip) and the
// persistent batched kernel call the same functions.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "device.h"
#include "ures.h"
#include "ures_regs.h"

namespace rsl {

enum : int {
  kStageReduce = 0,
  kStageEval = 1,
  kStageConv = 2,
  kStageStir = 3,
  kStageNewton = 4,
  kStageCrt = 5,
  kNumStages = 6,
};

constexpr int kCrtWaves = 8;          // waves of a CRT block (one coefficient each)
// waves of a CRT block with ns prime slots per lane (more slots: fewer waves,
// two coefficients each, to stay within the LDS of a block)
__host__ __device__ inline int crt_block_waves(int ns) { return ns > 4 ? 4 : kCrtWaves; }
constexpr int kLdsWords = 16384;      // 64 KB of dynamic LDS per block at most

// ------------------------------------------------------------------ helpers

// acc + x y with acc kept below p 2^32 (one conditional subtraction on the high word)
__device__ __forceinline__ uint64_t mac_fold(uint64_t acc, uint32_t x, uint32_t y, uint32_t p) {
  acc += static_cast<uint64_t>(x) * y;
  uint32_t hi = static_cast<uint32_t>(acc >> 32);
  hi = umin32(hi, hi - p);
  return (static_cast<uint64_t>(hi) << 32) | static_cast<uint32_t>(acc);
}

// a + b for a, b < p 2^32, result < p 2^32
__device__ __forceinline__ uint64_t add_fold(uint64_t a, uint64_t b, uint32_t p) {
  const uint64_t s = a + b;
  uint32_t hi = static_cast<uint32_t>(s >> 32);
  hi = umin32(hi, hi - p);
  return (static_cast<uint64_t>(hi) << 32) | static_cast<uint32_t>(s);
}

// Lazy Horner steps acc <- REDC(acc x~ + c) with acc kept in [0, 2p): the
// input stays below 2p^2 + p < p 2^32, so REDC's bound holds without the final
// conditional subtraction.  The phases of the independent chains are written
// interleaved so that each dependent instruction has others to hide behind.
__device__ __forceinline__ void horner_step4(uint32_t* a, const uint4 c, uint32_t xt, uint32_t p, uint32_t pinv) {
  const uint64_t t0 = static_cast<uint64_t>(a[0]) * xt + c.x;
  const uint64_t t1 = static_cast<uint64_t>(a[1]) * xt + c.y;
  const uint64_t t2 = static_cast<uint64_t>(a[2]) * xt + c.z;
  const uint64_t t3 = static_cast<uint64_t>(a[3]) * xt + c.w;
  const uint32_t m0 = static_cast<uint32_t>(t0) * pinv, m1 = static_cast<uint32_t>(t1) * pinv;
  const uint32_t m2 = static_cast<uint32_t>(t2) * pinv, m3 = static_cast<uint32_t>(t3) * pinv;
  a[0] = static_cast<uint32_t>((t0 + static_cast<uint64_t>(m0) * p) >> 32);
  a[1] = static_cast<uint32_t>((t1 + static_cast<uint64_t>(m1) * p) >> 32);
  a[2] = static_cast<uint32_t>((t2 + static_cast<uint64_t>(m2) * p) >> 32);
  a[3] = static_cast<uint32_t>((t3 + static_cast<uint64_t>(m3) * p) >> 32);
}

__device__ __forceinline__ void horner_step8(uint32_t* a, uint32_t* b, const uint4 c, const uint4 d, uint32_t xt,
                                             uint32_t p, uint32_t pinv) {
  const uint64_t t0 = static_cast<uint64_t>(a[0]) * xt + c.x;
  const uint64_t t1 = static_cast<uint64_t>(a[1]) * xt + c.y;
  const uint64_t t2 = static_cast<uint64_t>(a[2]) * xt + c.z;
  const uint64_t t3 = static_cast<uint64_t>(a[3]) * xt + c.w;
  const uint64_t t4 = static_cast<uint64_t>(b[0]) * xt + d.x;
  const uint64_t t5 = static_cast<uint64_t>(b[1]) * xt + d.y;
  const uint64_t t6 = static_cast<uint64_t>(b[2]) * xt + d.z;
  const uint64_t t7 = static_cast<uint64_t>(b[3]) * xt + d.w;
  const uint32_t m0 = static_cast<uint32_t>(t0) * pinv, m1 = static_cast<uint32_t>(t1) * pinv;
  const uint32_t m2 = static_cast<uint32_t>(t2) * pinv, m3 = static_cast<uint32_t>(t3) * pinv;
  const uint32_t m4 = static_cast<uint32_t>(t4) * pinv, m5 = static_cast<uint32_t>(t5) * pinv;
  const uint32_t m6 = static_cast<uint32_t>(t6) * pinv, m7 = static_cast<uint32_t>(t7) * pinv;
  a[0] = static_cast<uint32_t>((t0 + static_cast<uint64_t>(m0) * p) >> 32);
  a[1] = static_cast<uint32_t>((t1 + static_cast<uint64_t>(m1) * p) >> 32);
  a[2] = static_cast<uint32_t>((t2 + static_cast<uint64_t>(m2) * p) >> 32);
  a[3] = static_cast<uint32_t>((t3 + static_cast<uint64_t>(m3) * p) >> 32);
  b[0] = static_cast<uint32_t>((t4 + static_cast<uint64_t>(m4) * p) >> 32);
  b[1] = static_cast<uint32_t>((t5 + static_cast<uint64_t>(m5) * p) >> 32);
  b[2] = static_cast<uint32_t>((t6 + static_cast<uint64_t>(m6) * p) >> 32);
  b[3] = static_cast<uint32_t>((t7 + static_cast<uint64_t>(m7) * p) >> 32);
}

// Two and four chains of the same lazy Horner step (lane-pair layout).
__device__ __forceinline__ void horner_step2(uint32_t* a, uint32_t c0, uint32_t c1, uint32_t xt, uint32_t p,
                                             uint32_t pinv) {
  const uint64_t t0 = static_cast<uint64_t>(a[0]) * xt + c0;
  const uint64_t t1 = static_cast<uint64_t>(a[1]) * xt + c1;
  const uint32_t m0 = static_cast<uint32_t>(t0) * pinv, m1 = static_cast<uint32_t>(t1) * pinv;
  a[0] = static_cast<uint32_t>((t0 + static_cast<uint64_t>(m0) * p) >> 32);
  a[1] = static_cast<uint32_t>((t1 + static_cast<uint64_t>(m1) * p) >> 32);
}
__device__ __forceinline__ void horner_step2x2(uint32_t* a, uint32_t* b, uint32_t c0, uint32_t c1, uint32_t d0,
                                               uint32_t d1, uint32_t xt, uint32_t p, uint32_t pinv) {
  const uint64_t t0 = static_cast<uint64_t>(a[0]) * xt + c0;
  const uint64_t t1 = static_cast<uint64_t>(a[1]) * xt + c1;
  const uint64_t t2 = static_cast<uint64_t>(b[0]) * xt + d0;
  const uint64_t t3 = static_cast<uint64_t>(b[1]) * xt + d1;
  const uint32_t m0 = static_cast<uint32_t>(t0) * pinv, m1 = static_cast<uint32_t>(t1) * pinv;
  const uint32_t m2 = static_cast<uint32_t>(t2) * pinv, m3 = static_cast<uint32_t>(t3) * pinv;
  a[0] = static_cast<uint32_t>((t0 + static_cast<uint64_t>(m0) * p) >> 32);
  a[1] = static_cast<uint32_t>((t1 + static_cast<uint64_t>(m1) * p) >> 32);
  b[0] = static_cast<uint32_t>((t2 + static_cast<uint64_t>(m2) * p) >> 32);
  b[1] = static_cast<uint32_t>((t3 + static_cast<uint64_t>(m3) * p) >> 32);
}

// ------------------------------------------------------------------ reduce

// Coefficient t of the prime's transposed tile: f part [i][j] (j padded to
// myp), then g part [i][j] (j padded to nyp).  Stores c R^2 mod p (0 for padding).
// With zero_status, the block of (slot 0, block 0) also clears the problem's
// status words (a launch that runs before every other stage of the problem).
// A two's complement value of L limbs mod p, without divisions: the signed top
// limb plus 2p lies in (0, 4p) since p > 2^30; each lower limb w (< 2^32 < 4p)
// enters as r <- r 2^32 + w, with r 2^32 mod p = mmul(r, R^2).
__device__ inline uint32_t limbs_mod_p(const uint32_t* wd, int L, const PrimeConst& pc) {
  const uint32_t p = pc.p;
  const int32_t top = static_cast<int32_t>(wd[L - 1]);
  uint64_t x = static_cast<uint64_t>(static_cast<int64_t>(top) + 2 * static_cast<int64_t>(p));  // < 4p
  x = (x >= 2ull * p) ? x - 2ull * p : x;
  x = (x >= p) ? x - p : x;
  uint32_t r = static_cast<uint32_t>(x);
  for (int l = L - 2; l >= 0; --l) {
    uint32_t wl = wd[l];
    wl = umin32(wl, wl - p);
    wl = umin32(wl, wl - p);
    wl = umin32(wl, wl - p);
    r = maddm(mmul(r, pc.r2, p, pc.pinv), wl, p);
  }
  return r;
}

// Position in the partner's tiles (the system eliminated in x) of the
// coefficient at tile position t (inside the f or g rectangle): x^i y^j there
// is y'^i x'^j, so [x-power i][row j] becomes [x'-power j][row i].
__device__ inline int partner_pos(const DevProblem& P, int t) {
  if (t < P.goff) {
    const int i = t / P.myp, j = t - i * P.myp;
    return j * P.pmyp + i;
  }
  const int u = t - P.goff;
  const int i = u / P.nyp, j = u - i * P.nyp;
  return P.pgoff + j * P.pnyp + i;
}

// Tile position t -> the input coefficient's index, -1 for a padding position.
__device__ inline int tile_input(const DevProblem& P, int t) {
  if (t >= P.CS) return -1;
  if (t < P.goff) {
    const int i = t / P.myp, j = t - i * P.myp;
    return (j <= P.my) ? j * P.rowf + i : -1;
  }
  const int u = t - P.goff;
  const int i = u / P.nyp, j = u - i * P.nyp;
  return (i < P.rowg && j <= P.ny) ? (P.my + 1) * P.rowf + j * P.rowg + i : -1;
}

// Digit tiles (evaluation on the matrix cores).  The residue c mod p of the
// coefficient at x-power i < 32 KH (KH = 1 or 2 K slices of 32) and row j is
// kept as four balanced base-256 digits, c = sum_b c_b 256^b, -128 <= c_b <= 127
// (a residue below p is within their range 127 (1 + 256 + 256^2 + 256^3); the
// earlier five 7-bit digits took 25 digit products instead of 16).  The tile of
// rows 16 t .. 16 t + 15 (g's tiles follow f's) holds the B operands of
// v_mfma_i32_16x16x64_i8, lane l = (j mod 16) + 16 ((i mod 32) / 8) reading its
// bytes as 16-byte loads:
//   KH = 1: digits 3, 2, 1, 0 of x-powers 8 (l / 16) .. + 7, eight bytes each
//   KH = 2: digits 0, 1, 2, 3, sixteen bytes each: x-powers 8 (l / 16) .. + 7,
//           then 32 + 8 (l / 16) .. + 7
__host__ __device__ inline int dig_rt(int rows) { return (rows + 15) / 16; }
constexpr int kEvDigits = 4;
// balanced base-256 digits of v (|v| <= 0x7F7F7F7F) as the bytes of a word
__host__ __device__ __forceinline__ uint32_t balanced_digits(uint32_t v) { return (v + 0x80808080u) ^ 0x80808080u; }
// out[a] = byte a of w0, w1, w2, w3 (lowest first)
__device__ __forceinline__ void byte_transpose4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t* out) {
  const uint32_t t0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), t1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
  const uint32_t t2 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), t3 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}
__device__ inline void stage_reduce(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                    bool zero_status = false) {
  if (zero_status && w.slot == 0 && w.blk == 0)
    for (int i = threadIdx.x; i < 2 * P.np + 2; i += blockDim.x) P.status[i] = 0;
  const int t = w.blk * blockDim.x + threadIdx.x;
  if (t >= P.CS) return;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const int in = tile_input(P, t);
  uint32_t v = 0;
  if (in >= 0) {
    const uint32_t r = limbs_mod_p(P.coeff + static_cast<size_t>(in) * P.L_in, P.L_in, pc);
    v = mmul(r, pc.r3, pc.p, pc.pinv);
    if (w.slot < P.pshared) P.presid[static_cast<size_t>(w.slot) * P.pCS + partner_pos(P, t)] = v;
  }
  P.resid[static_cast<size_t>(w.slot) * P.CS + t] = v;
}

// Problems whose evaluation takes its sums from the matrix cores: whole digit
// tiles, written every run (padding included, so nothing is cleared before).  A
// lane owns one K run of 8 x-powers of one row -- 8 coefficients, their four
// digits 32 bytes of the tile -- and each of the block's four waves SPW prime
// slots.  In signed residues a limb w = w_s + 2^32 b (w_s its signed value) takes
//   r <- sredc((r + b) R^2 + w_s R) = r 2^32 + w mod p,
// five instructions per limb, coefficient and prime (|r| <= 0.9 p with the two
// constants centred).  Inputs of more than two limbs pass through LDS 16 limbs
// at a time, read once per block for its 4 SPW primes, each limb below the top
// less 2^31 (its top bit flipped: a signed word without a carry), two limbs a
// step,
//   r <- sredc(r R^3 + w_1 R^2 + w_0 R) = r 2^64 + w_1 2^32 + w_0 mod p,
// five instructions per two limbs (|r| <= 1.2 p); the same steps on zero
// coefficients (off) give what the offsets add, taken off at the end: 10 pairs of
// degree 15 with 2^2048 coefficients 190 -> 151 us.  Item (first slot, block of
// 64 lanes, sub = SPW).
//
// Short inputs: the lanes walk the tiles in order, padding runs as zeros (a
// separate pass over the padding cost more than the idle lanes: 41 -> 48 us on 256
// pairs of the batch workload).  Long ones: the runs with coefficients first, the
// padding in blocks of its own, which skip the limb loop (258 -> 193 us on 10
// pairs of degree 15 with 2^2048 coefficients, of whose tile runs a quarter hold
// coefficients).  Against byte or 8-byte stores of canonical residues with 14
// instructions per limb, and a clearing launch per upload: 256 pairs 80 -> 41 us,
// 64 requests of degrees 8..48 75 -> 38, the 2^2048 set 368 -> 193 (one limb a
// step); the launch saved 3-9 us per call.
constexpr int kReduceChunk = 16;  // limbs per LDS chunk
// Prime slots per wave for inputs of up to two limbs (2, 3, 4: 7.4, 8.1, 8.5 us on
// the degree-24 pair, 41, 37, 38 us on 256 pairs) and of more (3, 4: 162, 151 us
// on the 2^2048 set, 23, 24.5 us on 10 pairs of degree 9 with 2^512; 5, 6 and 8
// were no better than 4 with one limb a step).
constexpr int kReduceSlotsShort = 2, kReduceSlotsLong = 4;
// runs with coefficients, and all runs of a slot's tiles
__host__ __device__ inline int reduce_runs(const DevProblem& P) {
  return (P.my + 1) * ((P.rowf + 7) / 8) + (P.ny + 1) * ((P.rowg + 7) / 8);
}
__host__ __device__ inline int reduce_tile_runs(const DevProblem& P) { return (P.dRTf + P.dRTg) * 64 * P.dkh; }
__host__ __device__ inline int reduce_tile_blocks(const DevProblem& P) {
  return (P.L_in > 2 ? (reduce_runs(P) + 63) / 64 : 0) + reduce_tile_runs(P) / 64;
}
__host__ __device__ inline int reduce_tiles_lds_words() { return kReduceChunk * 8 * 64; }
template <int SPW>
__device__ inline void stage_reduce_tiles(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (w.slot == 0 && w.blk == 0)
    for (int i = threadIdx.x; i < 2 * P.np + 2; i += blockDim.x) P.status[i] = 0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kh = P.dkh, s0 = w.slot + wave * SPW;
  // run of 8 x-powers k8 of row j of polynomial gp -> its place in the slot's tiles
  auto place = [&](int gp, int j, int k8) {
    return reinterpret_cast<uint8_t*>(P.dig + static_cast<size_t>(s0) * P.dfr * 64) +
           (static_cast<size_t>((gp ? P.dRTf : 0) + (j >> 4)) * 64 + (j & 15) + 16 * (k8 & 3)) * (32 * kh) +
           8 * (k8 >> 2);
  };
  auto store = [&](uint8_t* at, const uint32_t (&lo)[kEvDigits], const uint32_t (&hi)[kEvDigits]) {
    if (kh == 1) {
      reinterpret_cast<uint4*>(at)[0] = make_uint4(lo[3], hi[3], lo[2], hi[2]);
      reinterpret_cast<uint4*>(at)[1] = make_uint4(lo[1], hi[1], lo[0], hi[0]);
    } else {
#pragma unroll
      for (int b = 0; b < kEvDigits; ++b)
        *reinterpret_cast<uint64_t*>(at + 16 * b) = (static_cast<uint64_t>(hi[b]) << 32) | lo[b];
    }
  };
  const size_t slot_bytes = static_cast<size_t>(P.dfr) * 512;
  int gp, j, k8, nv;
  auto tile_run = [&](int t) {  // run t of the tiles in order
    const int unit = t >> (kh - 1), tile = unit >> 6, ln = unit & 63;
    gp = tile >= P.dRTf ? 1 : 0;
    j = 16 * (tile - (gp ? P.dRTf : 0)) + (ln & 15);
    k8 = (ln >> 4) + 4 * (t & (kh - 1));
    nv = j <= (gp ? P.ny : P.my) ? (gp ? P.rowg : P.rowf) - 8 * k8 : 0;
  };
  bool mine = true;
  if constexpr (SPW == kReduceSlotsLong) {
    const int nruns = reduce_runs(P), nb = (nruns + 63) / 64;
    if (w.blk >= nb) {  // runs without coefficients: zero
      tile_run((w.blk - nb) * 64 + lane);
      if (nv > 0) return;
      const uint32_t zero[kEvDigits] = {0u, 0u, 0u, 0u};
      uint8_t* at = place(gp, j, k8);
      for (int s = 0; s < SPW && s0 + s < P.np; ++s) store(at + s * slot_bytes, zero, zero);
      return;
    }
    // runs with coefficients, consecutive lanes taking consecutive rows
    const int t = w.blk * 64 + lane, nf = (P.my + 1) * ((P.rowf + 7) / 8);
    gp = t >= nf ? 1 : 0;
    const int u = gp ? t - nf : t, rows = gp ? P.ny + 1 : P.my + 1;
    k8 = u / rows;
    j = u - k8 * rows;
    mine = t < nruns;
    nv = mine ? (gp ? P.rowg : P.rowf) - 8 * k8 : 0;
  } else {
    tile_run(w.blk * 64 + lane);
  }
  nv = nv < 0 ? 0 : nv > 8 ? 8 : nv;  // coefficients of the run
  const int i0 = 8 * k8, len = gp ? P.rowg : P.rowf;
  const int L = P.L_in;
  const uint32_t* src =
      P.coeff + (static_cast<size_t>(gp ? (P.my + 1) * P.rowf : 0) + static_cast<size_t>(j) * len + i0) * L;
  SignedMod M[SPW];
  int32_t r1[SPW], r2[SPW], r3[SPW], off[SPW], acc[SPW][8];
  constexpr int32_t kMin = INT32_MIN;
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    const PrimeConst pc = T.pc[P.pidx[s0 + s < P.np ? s0 + s : P.np - 1]];
    M[s] = signed_mod(pc);
    r1[s] = scenter(static_cast<int32_t>(pc.r1), M[s]);
    r2[s] = scenter(static_cast<int32_t>(pc.r2), M[s]);
    r3[s] = scenter(static_cast<int32_t>(pc.r3), M[s]);
    off[s] = 0;
  }
  auto top = [&](const uint32_t (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int s = 0; s < SPW; ++s) acc[s][e] = smul(static_cast<int32_t>(v[e]), r1[s], M[s]);
  };
  auto next = [&](const uint32_t (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int32_t b = static_cast<int32_t>(v[e] >> 31);
#pragma unroll
      for (int s = 0; s < SPW; ++s)
        acc[s][e] = sredc(smad(acc[s][e] + b, r2[s], smad(static_cast<int32_t>(v[e]), r1[s], 0)), M[s]);
    }
  };
  uint32_t v[8];
  if (L <= 2) {
    uint32_t lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = e < nv ? src[e * L + L - 1] : 0u;
      lo[e] = (L == 2 && e < nv) ? src[2 * e] : 0u;
    }
    top(v);
    if (L == 2) next(lo);
  } else {
    for (int l1 = L; l1 > 0; l1 -= kReduceChunk) {  // limbs [l0, l1), top chunk first
      const int l0 = l1 > kReduceChunk ? l1 - kReduceChunk : 0;
      __syncthreads();
      // wave q brings limbs l0 + 4 q .. + 3 of every lane's coefficients
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int u = 0; u < kReduceChunk / 4; ++u) {
          const int l = 4 * wave + u;
          const uint32_t x = (e < nv && l0 + l < l1) ? src[static_cast<size_t>(e) * L + l0 + l] : 0u;
          lds[(l * 8 + e) * 64 + lane] = l0 + l < L - 1 ? x ^ 0x80000000u : x;
        }
      __syncthreads();
      int l = l1 - l0 - 1;
      if (l1 == L) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = lds[(l * 8 + e) * 64 + lane];
        top(v);
        --l;
      }
      if (l >= 0 && (l & 1) == 0) {  // an odd number of limbs: one by itself
#pragma unroll
        for (int s = 0; s < SPW; ++s) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            acc[s][e] = sredc(smad(acc[s][e], r2[s], smad(static_cast<int32_t>(lds[(l * 8 + e) * 64 + lane]), r1[s], 0)), M[s]);
          off[s] = sredc(smad(off[s], r2[s], smad(kMin, r1[s], 0)), M[s]);
        }
        --l;
      }
      for (; l > 0; l -= 2) {
        uint32_t lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = lds[(l * 8 + e) * 64 + lane];
          lo[e] = lds[(l * 8 - 8 + e) * 64 + lane];
        }
#pragma unroll
        for (int s = 0; s < SPW; ++s) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            acc[s][e] = sredc(smad(acc[s][e], r3[s], smad(static_cast<int32_t>(v[e]), r2[s],
                                                          smad(static_cast<int32_t>(lo[e]), r1[s], 0))), M[s]);
          off[s] = sredc(smad(off[s], r3[s], smad(kMin, r2[s], smad(kMin, r1[s], 0))), M[s]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < SPW; ++s) {
      const int32_t o = scenter(off[s], M[s]);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[s][e] = scenter(scenter(acc[s][e], M[s]) - o, M[s]);
    }
  }
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    if (s0 + s >= P.np || !mine) break;
    uint32_t lo[kEvDigits], hi[kEvDigits], d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = balanced_digits(static_cast<uint32_t>(acc[s][e]));
    byte_transpose4(d[0], d[1], d[2], d[3], lo);
    byte_transpose4(d[4], d[5], d[6], d[7], hi);
    store(place(gp, j, k8) + s * slot_bytes, lo, hi);
  }
}

// Multi-limb inputs: a block takes 64 transposed positions and 32 prime slots
// (item: slot = first slot, blk = position block, sub = 1).  The 64
// coefficients' limbs are staged in LDS 64 limbs at a time (coalesced reads of
// each coefficient's limb run, stored [limb][coefficient] with a padded row);
// thread (c, q) runs the Horner steps of the limbs, top limb first, for slots
// slot + q + 4 r, r < 8: eight independent chains.
constexpr int kReduceMlCoeffs = 64;
constexpr int kReduceMlSlots = 32;
constexpr int kReduceMlLimbs = 64;
__host__ __device__ inline int reduce_ml_lds_words() { return kReduceMlLimbs * (kReduceMlCoeffs + 1); }

__device__ inline void stage_reduce_ml(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (w.slot == 0 && w.blk == 0)
    for (int i = threadIdx.x; i < 2 * P.np + 2; i += blockDim.x) P.status[i] = 0;
  constexpr int kPer = kReduceMlSlots / 4;
  const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int t = w.blk * kReduceMlCoeffs + c;
  const int in = tile_input(P, t);
  uint32_t p[kPer], pinv[kPer], r2[kPer], r3[kPer], acc[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const int sl = w.slot + q + 4 * r;
    const PrimeConst pc = T.pc[P.pidx[sl < P.np ? sl : 0]];
    p[r] = pc.p;
    pinv[r] = pc.pinv;
    r2[r] = pc.r2;
    r3[r] = pc.r3;
    acc[r] = 0u;
  }
  const int L = P.L_in;
  for (int l1 = L; l1 > 0; l1 -= kReduceMlLimbs) {  // limbs [l0, l1), top chunk first
    const int l0 = l1 > kReduceMlLimbs ? l1 - kReduceMlLimbs : 0, nl = l1 - l0;
    __syncthreads();
    for (int e = threadIdx.x; e < kReduceMlCoeffs * nl; e += blockDim.x) {
      const int cc = e / nl, l = e - cc * nl;
      const int ci = tile_input(P, w.blk * kReduceMlCoeffs + cc);
      lds[l * (kReduceMlCoeffs + 1) + cc] = (ci >= 0) ? P.coeff[static_cast<size_t>(ci) * L + l0 + l] : 0u;
    }
    __syncthreads();
    for (int l = nl - 1; l >= 0; --l) {
      const uint32_t wd = lds[l * (kReduceMlCoeffs + 1) + c];
      if (l0 + l == L - 1) {
        // the signed top limb plus 2p lies in (0, 4p) since p > 2^30
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
          uint64_t x = static_cast<uint64_t>(static_cast<int64_t>(static_cast<int32_t>(wd)) + 2 * static_cast<int64_t>(p[r]));
          x = (x >= 2ull * p[r]) ? x - 2ull * p[r] : x;
          x = (x >= p[r]) ? x - p[r] : x;
          acc[r] = static_cast<uint32_t>(x);
        }
      } else {
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
          uint32_t wl = umin32(wd, wd - p[r]);
          wl = umin32(wl, wl - p[r]);
          wl = umin32(wl, wl - p[r]);
          acc[r] = maddm(mmul(acc[r], r2[r], p[r], pinv[r]), wl, p[r]);
        }
      }
    }
  }
  if (t >= P.CS) return;
  const int tp = (in >= 0 && w.slot < P.pshared) ? partner_pos(P, t) : 0;
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const int sl = w.slot + q + 4 * r;
    if (sl < P.np) {
      const uint32_t v = (in >= 0) ? mmul(acc[r], r3[r], p[r], pinv[r]) : 0u;
      P.resid[static_cast<size_t>(sl) * P.CS + t] = v;
      if (in >= 0 && sl < P.pshared) P.presid[static_cast<size_t>(sl) * P.pCS + tp] = v;
    }
  }
}

// -------------------------------------------------------------- eval + ures

// Bad-pair bookkeeping of one eval wave: the count, and a per-prime flag set
// when a bad point lies among 0..D (the interpolation then needs the gapped
// point set).
__device__ inline void eval_report_bad(const DevProblem& P, int slot, int pt, bool live, bool bad) {
  const uint64_t nbad = __ballot(live && bad);
  const uint64_t early = __ballot(live && bad && pt <= P.D);
  if ((threadIdx.x & 63) == 0) {
    if (nbad) atomicAdd(P.status + 1 + P.np, static_cast<int>(__popcll(nbad)));
    if (early) atomicOr(P.status + 2 + P.np + slot, 1);
  }
}

// LDS words needed by one eval block (one wave).
__host__ __device__ inline int eval_lds_words(const DevProblem& P) {
  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  return P.CS + 2 * nm1 * 64;
}

// One wave: 64 consecutive points of one prime.  The prime's coefficient tile
// is copied to LDS once; Horner then runs on kRowGroup rows of f and of g at a
// time (eight independent chains per lane), each step reading kRowGroup
// coefficients with one broadcast LDS load.  The values f_j(x_i), g_j(x_i) go
// to two LDS columns per lane and the univariate resultant runs there.
__device__ inline void stage_eval_ures(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  const int lane = threadIdx.x;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const uint32_t p = pc.p, pinv = pc.pinv;
  uint32_t* tile = lds;
  const uint32_t* src = P.resid + static_cast<size_t>(w.slot) * P.CS;
  for (int t = lane; t < P.CS; t += 64) tile[t] = src[t];
  __syncthreads();

  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  uint32_t* cols = lds + P.CS;
  Column<64> A{cols + lane};
  Column<64> B{cols + nm1 * 64 + lane};
  const int pt = w.blk * 64 + lane;
  const uint32_t x = static_cast<uint32_t>(P.origin + (pt < P.E ? pt : P.E));
  const uint32_t xt = mmul(x, pc.r2, p, pinv);

  const int gf = P.myp / kRowGroup, gg = P.nyp / kRowGroup;
  const int ng = gf > gg ? gf : gg;
  const uint32_t* ftile = tile;
  const uint32_t* gtile = tile + P.goff;
  for (int q = 0; q < ng; ++q) {
    // group degrees are uniform: keep them (and the loop bounds) in SGPRs
    const int df = __builtin_amdgcn_readfirstlane((q < gf) ? P.gdeg[q] : -1);
    const int dg = __builtin_amdgcn_readfirstlane((q < gg) ? P.gdeg[gf + q] : -1);
    const int dboth = df < dg ? df : dg;
    uint32_t a[4] = {0, 0, 0, 0}, b[4] = {0, 0, 0, 0};
    const uint32_t* fq = ftile + kRowGroup * q;
    const uint32_t* gq = gtile + kRowGroup * q;
    int i = df > dg ? df : dg;
    for (; i > dboth; --i) {  // only the higher-degree tile is active
      if (i <= df) horner_step4(a, *reinterpret_cast<const uint4*>(fq + i * P.myp), xt, p, pinv);
      else horner_step4(b, *reinterpret_cast<const uint4*>(gq + i * P.nyp), xt, p, pinv);
    }
    if (i >= 0) {  // both tiles: eight independent chains, next rows prefetched
      uint4 cf = *reinterpret_cast<const uint4*>(fq + i * P.myp);
      uint4 cg = *reinterpret_cast<const uint4*>(gq + i * P.nyp);
      for (; i > 0; --i) {
        const uint4 nf = *reinterpret_cast<const uint4*>(fq + (i - 1) * P.myp);
        const uint4 ng = *reinterpret_cast<const uint4*>(gq + (i - 1) * P.nyp);
        horner_step8(a, b, cf, cg, xt, p, pinv);
        cf = nf;
        cg = ng;
      }
      horner_step8(a, b, cf, cg, xt, p, pinv);
    }
    const int j = kRowGroup * q;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (j + r <= P.my) A[j + r] = umin32(a[r], a[r] - p);  // Horner keeps values below 2p
      if (j + r <= P.ny) B[j + r] = umin32(b[r], b[r] - p);
    }
  }
  bool bad = false;
  const uint32_t r = ures_formal(A, B, P.my, P.ny, pc, &bad);
  const bool live = pt <= P.E;
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, p, pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// LDS words of a grouped eval block (K lanes per pair, 64/K pairs).
__host__ __device__ inline int eval_group_lds_words(const DevProblem& P, int K) {
  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  return P.CS + 2 * nm1 * (64 / K);
}

// Lanes of one wave meet here: LDS operations of a wave execute in program
// order, so the fences only keep the compiler from moving memory operations
// across this point.
struct WaveSync {
  __device__ void operator()() const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

// One wave, K lanes per (prime, point) pair: 64/K consecutive points of one
// prime.  Lane l of a pair evaluates rows j = 4q + l + K r (r < 4/K) of every
// row group q, so all lanes walk the same group degrees; the columns hold pair
// q at LDS word q + j (64/K), which makes the K lanes' accesses to one j-slice
// conflict-free.  The K lanes then run ures_group on the shared columns.
template <int K>
__device__ inline void stage_eval_ures_group(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                             uint32_t* lds) {
  constexpr int PB = 64 / K;            // pairs per block
  constexpr int R = kRowGroup / K;      // rows of a group per lane
  constexpr int NG = (R == 1) ? 2 : 1;  // groups per Horner pass (four chains per lane)
  const int lane = threadIdx.x;
  const int l = lane / PB, q = lane % PB;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const uint32_t p = pc.p, pinv = pc.pinv;
  uint32_t* tile = lds;
  {
    const uint4* src = reinterpret_cast<const uint4*>(P.resid + static_cast<size_t>(w.slot) * P.CS);
    uint4* dst = reinterpret_cast<uint4*>(tile);
    for (int t = lane; t < P.CS / 4; t += 64) dst[t] = src[t];
  }
  __syncthreads();

  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  uint32_t* cols = lds + P.CS;
  Column<PB> A{cols + q};
  Column<PB> B{cols + nm1 * PB + q};
  const int pt = w.blk * PB + q;
  const uint32_t x = static_cast<uint32_t>(P.origin + (pt < P.E ? pt : P.E));
  const uint32_t xt = mmul(x, pc.r2, p, pinv);

  const int gf = P.myp / kRowGroup, gg = P.nyp / kRowGroup;
  const int ng = gf > gg ? gf : gg;
  for (int q0 = 0; q0 < ng; q0 += NG) {
    // chains: [group][f or g][row]; a missing group reads column l of row 0
    // (in the tile) and is never stored
    int deg[NG][2];
    const uint32_t* base[NG][2];
    int stride[2] = {P.myp, P.nyp};
    int top = -1;
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const int qq = q0 + gi;
      deg[gi][0] = __builtin_amdgcn_readfirstlane((qq < gf) ? P.gdeg[qq] : -1);
      deg[gi][1] = __builtin_amdgcn_readfirstlane((qq < gg) ? P.gdeg[gf + qq] : -1);
      base[gi][0] = tile + ((qq < gf) ? kRowGroup * qq : 0) + l;
      base[gi][1] = tile + P.goff + ((qq < gg) ? kRowGroup * qq : 0) + l;
      top = deg[gi][0] > top ? deg[gi][0] : top;
      top = deg[gi][1] > top ? deg[gi][1] : top;
    }
    uint32_t acc[NG][2][R];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[gi][s][r] = 0u;
    for (int i = top; i >= 0; --i) {
      uint32_t c[NG][2][R];
#pragma unroll
      for (int gi = 0; gi < NG; ++gi)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const bool on = i <= deg[gi][s];  // uniform; rows above a chain's degree add zeros
          const uint32_t* rowp = base[gi][s] + (on ? i : 0) * stride[s];
#pragma unroll
          for (int r = 0; r < R; ++r) c[gi][s][r] = on ? rowp[K * r] : 0u;
        }
      uint64_t t[NG][2][R];
#pragma unroll
      for (int gi = 0; gi < NG; ++gi)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int r = 0; r < R; ++r) t[gi][s][r] = static_cast<uint64_t>(acc[gi][s][r]) * xt + c[gi][s][r];
      uint32_t mm[NG][2][R];
#pragma unroll
      for (int gi = 0; gi < NG; ++gi)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int r = 0; r < R; ++r) mm[gi][s][r] = static_cast<uint32_t>(t[gi][s][r]) * pinv;
#pragma unroll
      for (int gi = 0; gi < NG; ++gi)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc[gi][s][r] = static_cast<uint32_t>((t[gi][s][r] + static_cast<uint64_t>(mm[gi][s][r]) * p) >> 32);
    }
#pragma unroll
    for (int gi = 0; gi < NG; ++gi)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int j = kRowGroup * (q0 + gi) + l + K * r;
        const uint32_t va = acc[gi][0][r], vb = acc[gi][1][r];
        if (q0 + gi < gf && j <= P.my) A[j] = umin32(va, va - p);  // Horner keeps values below 2p
        if (q0 + gi < gg && j <= P.ny) B[j] = umin32(vb, vb - p);
      }
  }
  WaveSync sync;
  sync();
  bool bad = false;
  const uint32_t r = ures_group<K>(A, B, P.my, P.ny, pc, l, &bad, sync);
  const bool live = pt <= P.E && l == 0;
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, p, pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// LDS words of a register-form eval block: the tile plus two scratch columns
// of NMAX + 1 entries per lane for lanes that leave the register path.
__host__ __device__ inline int eval_regs_lds_words(const DevProblem& P, int nmax) {
  return P.CS + 2 * (nmax + 1) * 64;
}

// One wave, one lane per (prime, point) pair, the two polynomials in registers
// (ures_regs): Horner as in stage_eval_ures, then the unrolled remainder
// sequence; no LDS traffic after the tile except for lanes that fall back.
template <int NMAX>
__device__ inline void stage_eval_ures_regs(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                            uint32_t* lds) {
  constexpr int N = RegPoly<NMAX>::kN;
  const int lane = threadIdx.x;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const uint32_t p = pc.p, pinv = pc.pinv;
  uint32_t* tile = lds;
  {
    const uint4* src = reinterpret_cast<const uint4*>(P.resid + static_cast<size_t>(w.slot) * P.CS);
    uint4* dst = reinterpret_cast<uint4*>(tile);
    for (int t = lane; t < P.CS / 4; t += 64) dst[t] = src[t];
  }
  __syncthreads();
  uint32_t* cols = lds + P.CS;
  const int pt = w.blk * 64 + lane;
  const uint32_t x = static_cast<uint32_t>(P.origin + (pt < P.E ? pt : P.E));
  const uint32_t xt = mmul(x, pc.r2, p, pinv);

  uint32_t X[N], Y[N];
  const int gf = P.myp / kRowGroup, gg = P.nyp / kRowGroup;
  const int ng = gf > gg ? gf : gg;
  const uint32_t* ftile = tile;
  const uint32_t* gtile = tile + P.goff;
#pragma unroll
  for (int q = 0; q < N / kRowGroup; ++q) {
    uint32_t a[4] = {0, 0, 0, 0}, b[4] = {0, 0, 0, 0};
    if (q < ng) {
      const int df = __builtin_amdgcn_readfirstlane((q < gf) ? P.gdeg[q] : -1);
      const int dg = __builtin_amdgcn_readfirstlane((q < gg) ? P.gdeg[gf + q] : -1);
      const int dboth = df < dg ? df : dg;
      const uint32_t* fq = ftile + kRowGroup * q;
      const uint32_t* gq = gtile + kRowGroup * q;
      int i = df > dg ? df : dg;
      for (; i > dboth; --i) {
        if (i <= df) horner_step4(a, *reinterpret_cast<const uint4*>(fq + i * P.myp), xt, p, pinv);
        else horner_step4(b, *reinterpret_cast<const uint4*>(gq + i * P.nyp), xt, p, pinv);
      }
      if (i >= 0) {
        uint4 cf = *reinterpret_cast<const uint4*>(fq + i * P.myp);
        uint4 cg = *reinterpret_cast<const uint4*>(gq + i * P.nyp);
        for (; i > 0; --i) {
          const uint4 nf = *reinterpret_cast<const uint4*>(fq + (i - 1) * P.myp);
          const uint4 ngv = *reinterpret_cast<const uint4*>(gq + (i - 1) * P.nyp);
          horner_step8(a, b, cf, cg, xt, p, pinv);
          cf = nf;
          cg = ngv;
        }
        horner_step8(a, b, cf, cg, xt, p, pinv);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = kRowGroup * q + r;
      X[j] = (j <= P.my) ? umin32(a[r], a[r] - p) : 0u;  // Horner keeps values below 2p
      Y[j] = (j <= P.ny) ? umin32(b[r], b[r] - p) : 0u;
    }
  }
  bool bad = false;
  uint32_t r;
  if (P.my - P.ny > 1 || P.ny - P.my > 1) {
    // the long shapes: the values go to the lane's own two columns for the
    // first division (ures_regs_long), the chain then runs in registers
    Column<64> CA{cols + lane}, CB{cols + (NMAX + 1) * 64 + lane};
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (j <= NMAX) {
        if (j <= P.my) CA[j] = X[j];
        if (j <= P.ny) CB[j] = Y[j];
      }
    r = ures_regs_long<NMAX>(CA, CB, P.my, P.ny, pc, &bad);
  } else {
    r = ures_regs<NMAX>(X, Y, P.my, P.ny, pc, &bad, Column<64>{cols + lane},
                        Column<64>{cols + (NMAX + 1) * 64 + lane});
  }
  const bool live = pt <= P.E;
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, p, pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// LDS words of a two-lanes-per-pair register-form block (32 pairs).
__host__ __device__ inline int eval_regs2_lds_words(const DevProblem& P, int nmax) {
  return P.CS + 2 * (nmax + 1) * 32;
}

// Exchange with the partner lane of a lane pair (lanes 2q and 2q + 1).
struct PairSwap {
  __device__ uint32_t operator()(uint32_t v) const {
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0xB1 /* quad_perm 1,0,3,2 */, 0xF,
                                                          0xF, false));
  }
};

// One wave, two lanes per (prime, point) pair (32 pairs): lane l of pair q
// evaluates rows j = 4 g + 2 r + l of every row group g and keeps row j in
// element j / 2, then the pair runs ures_regs2.
template <int NMAX>
__device__ inline void stage_eval_ures_regs2(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                             uint32_t* lds) {
  constexpr int N2 = RegPoly2<NMAX>::kN;
  const int lane = threadIdx.x;
  const int l = lane & 1, q = lane >> 1;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const uint32_t p = pc.p, pinv = pc.pinv;
  uint32_t* tile = lds;
  {
    const uint4* src = reinterpret_cast<const uint4*>(P.resid + static_cast<size_t>(w.slot) * P.CS);
    uint4* dst = reinterpret_cast<uint4*>(tile);
    for (int t = lane; t < P.CS / 4; t += 64) dst[t] = src[t];
  }
  __syncthreads();
  uint32_t* cols = lds + P.CS;
  const int pt = w.blk * 32 + q;
  const uint32_t x = static_cast<uint32_t>(P.origin + (pt < P.E ? pt : P.E));
  const uint32_t xt = mmul(x, pc.r2, p, pinv);

  uint32_t X[N2], Y[N2];
  const int gf = P.myp / kRowGroup, gg = P.nyp / kRowGroup;
  const int ng = gf > gg ? gf : gg;
  const uint32_t* ftile = tile;
  const uint32_t* gtile = tile + P.goff;
  // one row group per pass (rows 4 g + l and 4 g + 2 + l of f and of g: four
  // chains): first the steps where only the higher-degree polynomial's rows
  // are nonzero, then all four chains with the next row's values prefetched
#pragma unroll
  for (int gq = 0; gq < N2 / 2; ++gq) {
    uint32_t a[2] = {0u, 0u}, b[2] = {0u, 0u};
    if (gq < ng) {
      const int df = __builtin_amdgcn_readfirstlane((gq < gf) ? P.gdeg[gq] : -1);
      const int dg = __builtin_amdgcn_readfirstlane((gq < gg) ? P.gdeg[gf + gq] : -1);
      const uint32_t* fq = ftile + kRowGroup * (gq < gf ? gq : 0) + l;
      const uint32_t* gqp = gtile + kRowGroup * (gq < gg ? gq : 0) + l;
      const int dboth = df < dg ? df : dg;
      int i = df > dg ? df : dg;
      for (; i > dboth; --i) {
        if (i <= df) {
          const uint32_t* fr = fq + i * P.myp;
          horner_step2(a, fr[0], fr[2], xt, p, pinv);
        } else {
          const uint32_t* gr = gqp + i * P.nyp;
          horner_step2(b, gr[0], gr[2], xt, p, pinv);
        }
      }
      if (i >= 0) {
        const uint32_t* fr = fq + i * P.myp;
        const uint32_t* gr = gqp + i * P.nyp;
        uint32_t f0 = fr[0], f1 = fr[2], g0 = gr[0], g1 = gr[2];
        for (; i > 0; --i) {
          const uint32_t* fn = fq + (i - 1) * P.myp;
          const uint32_t* gn = gqp + (i - 1) * P.nyp;
          const uint32_t nf0 = fn[0], nf1 = fn[2], ng0 = gn[0], ng1 = gn[2];
          horner_step2x2(a, b, f0, f1, g0, g1, xt, p, pinv);
          f0 = nf0;
          f1 = nf1;
          g0 = ng0;
          g1 = ng1;
        }
        horner_step2x2(a, b, f0, f1, g0, g1, xt, p, pinv);
      }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = 2 * gq + r;  // element: row 4 gq + 2 r + l
      const int j = 2 * k + l;
      X[k] = (gq < gf && j <= P.my) ? umin32(a[r], a[r] - p) : 0u;
      Y[k] = (gq < gg && j <= P.ny) ? umin32(b[r], b[r] - p) : 0u;
    }
  }
  bool bad = false;
  const uint32_t r = ures_regs2<NMAX>(X, Y, P.my, P.ny, l, pc, &bad, Column<32>{cols + q},
                                      Column<32>{cols + (NMAX + 1) * 32 + q}, PairSwap(), WaveSync());
  const bool live = pt <= P.E && l == 0;
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, p, pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// ------------------------------------------------ eval on the matrix cores
// The values f_j(x_k) = sum_i c_ij x_k^i mod p of 16 points and 16 rows j are
// the product of the power matrix V[k][i] = x_k^i mod p with the residue
// matrix C[i][j] (i < 32 KH: the K dimension).  Both split into four balanced
// base-256 digits (int8 operands); the digit products V_a C_b accumulate on
// the matrix cores into the seven anti-diagonal sums S_s = sum_{a+b=s} V_a C_b,
// |S_s| <= 4 * 64 * 128^2 = 2^22, and
//   f_j(x_k) R mod p = sredc(sum_s S_s w_s),  w_s = 2^{8s} R^2 mod p, centred
// (at most 0.51 p).  Lane l of a 16x16x64 product holds A row l mod 16 (a
// point) and B column l mod 16 (a row) for one quarter of K, and gets the
// outputs [4 (l / 16) + r][l mod 16], r < 4.  With one K slice of 32 two digit
// products of one anti-diagonal share an instruction (their K ranges side by
// side): 10 products per tile; with two slices 16.  The 16x16x64 form issues at
// the rate of 16x16x32, so both take twice the work per instruction.
typedef int ev_v4i __attribute__((ext_vector_type(4)));
typedef uint32_t ev_v4u __attribute__((ext_vector_type(4)));
__host__ __device__ inline int ev_tile_products(int kh) { return kh == 1 ? 10 : 16; }
__host__ __device__ inline int eval_mfma_row_stride(const DevProblem& P) {
  return ((P.my > P.ny ? P.my : P.ny) + 1) | 1;
}

// A operands of one 16-point tile: the digits of x^(8 g + e) (and x^(32 + 8 g + e)),
// e < 8, of the lane's point and K quarter g = lane / 16.  KH = 1: digits
// (0, 1), (2, 3); KH = 2: one operand per digit.
template <int KH>
__device__ __forceinline__ void ev_powers(const DevProblem& P, int pt, const PrimeConst& pc, const SignedMod& M,
                                          ev_v4i (&A)[2 * KH]) {
  const int g = (threadIdx.x & 63) >> 4;
  const int32_t x = P.origin + (pt < P.E ? pt : P.E);
  const int32_t xt = smul(x, static_cast<int32_t>(pc.r2), M);
  const int32_t x2 = smul(xt, xt, M), x4 = smul(x2, x2, M), x8 = smul(x4, x4, M), x16 = smul(x8, x8, M);
  // normal form x^(8 g): a product with the Montgomery form x R stays in normal form
  const int32_t x24 = smul(x16, x8, M);
  int32_t first = smul(g == 1 ? x8 : g == 2 ? x16 : x24, 1, M);
  if (g == 0) first = 1;
#pragma unroll
  for (int half = 0; half < KH; ++half) {
    uint32_t w[8], lo[kEvDigits], hi[kEvDigits];
    int32_t v = first;
    if (half == 1) v = smul(first, smul(x16, x16, M), M);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      w[e] = balanced_digits(static_cast<uint32_t>(v));
      if (e < 7) v = smul(v, xt, M);
    }
    byte_transpose4(w[0], w[1], w[2], w[3], lo);
    byte_transpose4(w[4], w[5], w[6], w[7], hi);
#pragma unroll
    for (int a = 0; a < kEvDigits; ++a) {
      const int q = KH == 1 ? a >> 1 : a, o = KH == 1 ? 2 * (a & 1) : 2 * half;
      A[q][o] = static_cast<int>(lo[a]);
      A[q][o + 1] = static_cast<int>(hi[a]);
    }
  }
}

// Recombination weights (block-uniform).
struct EvWeights {
  int32_t w[2 * kEvDigits - 1];
};
__device__ __forceinline__ EvWeights ev_weights(const PrimeConst& pc, const SignedMod& M) {
  EvWeights W;
  int32_t v = scenter(static_cast<int32_t>(pc.r2), M);
  const int32_t t256 = smul(256, static_cast<int32_t>(pc.r2), M);
#pragma unroll
  for (int s = 0; s < 2 * kEvDigits - 1; ++s) {
    W.w[s] = __builtin_amdgcn_readfirstlane(v);
    v = scenter(smul(v, t256, M), M);
  }
  return W;
}

// Values of rows 0 .. deg of one polynomial (its digit tiles at `tile`, nrt of
// them) at the 16 H points of A, to F[point][row] (row stride SR): signed, or
// canonical residues.
template <int KH, int H, bool CANON>
__device__ __forceinline__ void ev_sums(const uint4* tile, int nrt, int deg, const ev_v4i (&A)[H][2 * KH],
                                        const EvWeights& W, const SignedMod& M, uint32_t* F, int SR) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  typedef const __attribute__((address_space(1))) ev_v4u* gptr;  // global loads (not flat)
  const gptr src = (gptr)(tile) + lane * (2 * KH);
  ev_v4u nx[2 * KH];
#pragma unroll
  for (int q = 0; q < 2 * KH; ++q) nx[q] = src[q];
  for (int rt = 0; rt < nrt; ++rt) {
    ev_v4u b[2 * KH];
#pragma unroll
    for (int q = 0; q < 2 * KH; ++q) b[q] = nx[q];
    if (rt + 1 < nrt) {  // the next tile's loads go out ahead of this tile's products
#pragma unroll
      for (int q = 0; q < 2 * KH; ++q) nx[q] = src[(rt + 1) * 64 * 2 * KH + q];
    }
    const int row = 16 * rt + (lane & 15);
    const bool keep = row <= deg;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      ev_v4i S[2 * kEvDigits - 1];
#pragma unroll
      for (int s = 0; s < 2 * kEvDigits - 1; ++s) S[s] = ev_v4i{0, 0, 0, 0};
      auto mm = [](ev_v4i a, ev_v4i bb, ev_v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bb, c, 0, 0, 0); };
      if constexpr (KH == 1) {
        // operand pairs [B_hi | B_lo] against [A_0 | A_1] and [A_2 | A_3]
        const int z = 0;
        const ev_v4i b03{z, z, (int)b[0].x, (int)b[0].y};                                  // 0, 3
        const ev_v4i b32{(int)b[0].x, (int)b[0].y, (int)b[0].z, (int)b[0].w};              // 3, 2
        const ev_v4i b21{(int)b[0].z, (int)b[0].w, (int)b[1].x, (int)b[1].y};              // 2, 1
        const ev_v4i b10{(int)b[1].x, (int)b[1].y, (int)b[1].z, (int)b[1].w};              // 1, 0
        const ev_v4i b0z{(int)b[1].z, (int)b[1].w, z, z};                                  // 0, -
        S[0] = mm(A[h][0], b0z, S[0]);
        S[1] = mm(A[h][0], b10, S[1]);
        S[2] = mm(A[h][0], b21, S[2]);
        S[3] = mm(A[h][0], b32, S[3]);
        S[4] = mm(A[h][0], b03, S[4]);
        S[2] = mm(A[h][1], b0z, S[2]);
        S[3] = mm(A[h][1], b10, S[3]);
        S[4] = mm(A[h][1], b21, S[4]);
        S[5] = mm(A[h][1], b32, S[5]);
        S[6] = mm(A[h][1], b03, S[6]);
      } else {
#pragma unroll
        for (int a = 0; a < kEvDigits; ++a)
#pragma unroll
          for (int d = 0; d < kEvDigits; ++d)
            S[a + d] = mm(A[h][a], ev_v4i{(int)b[d].x, (int)b[d].y, (int)b[d].z, (int)b[d].w}, S[a + d]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int64_t t = 0;
#pragma unroll
        for (int s = 0; s < 2 * kEvDigits - 1; ++s) t = smad(S[s][r], W.w[s], t);
        const int32_t v = sredc(t, M);
        if (keep) F[(16 * h + 4 * g + r) * SR + row] = CANON ? scanon(v, M) : static_cast<uint32_t>(v);
      }
    }
  }
}

__device__ __forceinline__ const uint4* ev_tiles(const DevProblem& P, int slot, int gp) {
  return reinterpret_cast<const uint4*>(P.dig + static_cast<size_t>(slot) * P.dfr * 64) +
         (gp ? static_cast<size_t>(P.dRTf) * 128 * P.dkh : 0);
}

// One lane per (prime, point) pair, 64 points per wave: the streamed form
// (ures_stream).  The lower-degree polynomial's values pass through LDS into
// the lane's registers, then the higher one's values take the same LDS, one row
// per lane, from where the division reads them once.  So a wave holds one
// polynomial's values only -- the LDS per wave is half that of keeping both --
// and any higher degree up to kStreamLongMax fits.  A lane that leaves the
// generic pattern (or whose leading coefficient vanishes) starts over: the
// values of both polynomials are formed again, 32 points at a time, in the
// same LDS, and the general column code runs on them in place.
// Bound by VALU issue: 0.86 of the 4-cycle rate at lower degrees up to 24 and 32 on the
// 512 pairs of the batch workload (4.2 K and 5.1 K instructions per 64 pairs, 469 and
// 366 us), 0.64-0.71 with two K slices where the launch fills the chip (64 requests of
// degrees 8..48, lower degrees up to 32, 40 and 48: 180, 387 and 161 us); the matrix
// cores are busy for an eighth to a sixth of it.  256 pairs went from 1394 us (both
// values in LDS, five 7-bit digits, canonical residues, long divisions from LDS) to
// 0.9 ms.
// LDS: 64 rows of kStreamFront zeros and the values, at an odd stride.
__host__ __device__ inline int eval_stream_row_stride(const DevProblem& P) {
  return ((P.my > P.ny ? P.my : P.ny) + 1 + kStreamFront) | 1;
}
__host__ __device__ inline int eval_stream_lds_words(const DevProblem& P) { return 64 * eval_stream_row_stride(P); }

template <int NMAX, int KH>
__device__ inline void stage_eval_ures_stream(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                              uint32_t* lds) {
  const int lane = threadIdx.x;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const SignedMod M = signed_mod(pc);
  const EvWeights W = ev_weights(pc, M);
  const int SR = eval_stream_row_stride(P);
  const bool swap = P.my < P.ny;  // A: the higher degree m, B: the lower degree n
  const int m = swap ? P.ny : P.my, n = swap ? P.my : P.ny;
  const int rtA = swap ? P.dRTg : P.dRTf, rtB = swap ? P.dRTf : P.dRTg;
  const int pt0 = w.blk * 64, pt = pt0 + lane;
  uint32_t* vals = lds + kStreamFront;
  uint32_t* row = vals + lane * SR;
#pragma unroll
  for (int j = 1; j <= kStreamFront; ++j) row[-j] = 0u;

  int32_t X[NMAX];
  int32_t L;
  {
    ev_v4i A[4][2 * KH];
#pragma unroll
    for (int h = 0; h < 4; ++h) ev_powers<KH>(P, pt0 + 16 * h + (lane & 15), pc, M, A[h]);
    ev_sums<KH, 4, false>(ev_tiles(P, w.slot, swap ? 0 : 1), rtB, n, A, W, M, vals, SR);
    WaveSync()();
    const int pad = stream_pad(n);
    const uint32_t* src = row - pad;
#pragma unroll
    for (int q = 0; q < NMAX / 4; ++q)
      if (4 * q < n + pad) {
#pragma unroll
        for (int j = 4 * q; j < 4 * q + 4; ++j) X[j] = static_cast<int32_t>(src[j]);
      }
    L = static_cast<int32_t>(row[n]);
    WaveSync()();
    ev_sums<KH, 4, false>(ev_tiles(P, w.slot, swap ? 1 : 0), rtA, m, A, W, M, vals, SR);
    WaveSync()();
  }
  const bool bad = L == 0 || row[m] == 0u;
  bool ok;
  uint32_t r = ures_stream<NMAX>(X, L, Column<1>{row}, m, n, pc, &ok);
  if (swap && ((m * n) & 1)) r = mneg(r, pc.p);  // Res(f, g) = (-1)^{mn} Res(g, f)
  ok = ok && !bad;
  const uint64_t redo = __ballot(!ok);
  if (redo) {
    for (int half = 0; half < 2; ++half) {
      if (((redo >> (32 * half)) & 0xFFFFFFFFu) == 0u) continue;  // wave-uniform
      WaveSync()();
      ev_v4i A[2][2 * KH];
#pragma unroll
      for (int h = 0; h < 2; ++h) ev_powers<KH>(P, pt0 + 32 * half + 16 * h + (lane & 15), pc, M, A[h]);
      ev_sums<KH, 2, true>(ev_tiles(P, w.slot, 0), P.dRTf, P.my, A, W, M, vals, SR);
      ev_sums<KH, 2, true>(ev_tiles(P, w.slot, 1), P.dRTg, P.ny, A, W, M, vals + 32 * SR, SR);
      WaveSync()();
      if (!ok && (lane >> 5) == half) {
        bool b2 = false;
        r = ures_formal(Column<1>{vals + (lane & 31) * SR}, Column<1>{vals + (32 + (lane & 31)) * SR}, P.my, P.ny, pc,
                        &b2);
      }
    }
  }
  const bool live = pt <= P.E;
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, pc.p, pc.pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// A lane pair per (prime, point), 32 points per wave, both polynomials' values
// [poly][point][row] in LDS, then the branch-free pair chain
// (ures_regs2_generic); in the same LDS words the two scratch columns per pair
// of the restart path (written only after the restarting pairs have their
// values back in registers).  Taken when two lanes per pair are asked for.
__host__ __device__ inline int eval_mfma2_lds_words(const DevProblem& P, int nmax) {
  const int vals = 2 * 32 * eval_mfma_row_stride(P), cols = 2 * (nmax + 1) * 32;
  return vals > cols ? vals : cols;
}

template <int NMAX, int KH>
__device__ inline void stage_eval_ures_mfma2(const DevProblem& P, const DevTables& T, const WorkItem& w,
                                             uint32_t* lds) {
  constexpr int PTS = 32;
  const int lane = threadIdx.x;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const SignedMod M = signed_mod(pc);
  const int SR = eval_mfma_row_stride(P);
  uint32_t* Fv[2] = {lds, lds + PTS * SR};
  uint32_t* cols = lds;  // restart path only
  {
    const EvWeights W = ev_weights(pc, M);
    ev_v4i A[2][2 * KH];
#pragma unroll
    for (int h = 0; h < 2; ++h) ev_powers<KH>(P, w.blk * PTS + 16 * h + (lane & 15), pc, M, A[h]);
    ev_sums<KH, 2, true>(ev_tiles(P, w.slot, 0), P.dRTf, P.my, A, W, M, Fv[0], SR);
    ev_sums<KH, 2, true>(ev_tiles(P, w.slot, 1), P.dRTg, P.ny, A, W, M, Fv[1], SR);
  }
  WaveSync()();
  constexpr int N2 = RegPoly2<NMAX>::kN;
  const int l = lane & 1, q = lane >> 1;
  const int pt = w.blk * PTS + q;
  const bool live = pt <= P.E && l == 0;
  bool ok, bad;
  uint32_t X[N2], Y[N2];
  auto load = [&] {
#pragma unroll
    for (int k = 0; k < N2; ++k) {
      const int j = 2 * k + l;
      X[k] = (j <= P.my) ? Fv[0][q * SR + j] : 0u;
      Y[k] = (j <= P.ny) ? Fv[1][q * SR + j] : 0u;
    }
  };
  load();
  uint32_t r = ures_regs2_generic<NMAX>(X, Y, P.my, P.ny, l, pc, &ok, &bad, PairSwap());
  if (!ok) {
    load();
    WaveSync()();  // every restarting pair has its values before the columns overwrite them
    r = ures2_columns<NMAX>(X, Y, P.my, P.ny, l, pc, Column<32>{cols + q}, Column<32>{cols + (NMAX + 1) * 32 + q},
                            PairSwap(), WaveSync());
  }
  if (live) {
    const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
    P.zval[o] = redc(r, pc.p, pc.pinv);
    P.zbad[o] = bad ? 1 : 0;
  }
  eval_report_bad(P, w.slot, pt, live, bad);
}

// ------------------------------------------------ eval + Schur (Sec. 4.1)
// The univariate resultant as the determinant of the Sylvester matrix S
// (n_y rows of f's coefficients, then m_y rows of g's), triangularised by the
// generalised Schur algorithm on its displacement generators.  With K the
// down-shift inside each of the two row blocks and Z the column shift,
//   S - K S Z^T = G B^T,  G = [e_0, e_n],  B = [row 0 of S, row n of S],
// a rank-2 displacement (a single generator when one block is empty).  Step
// k reads the pivot row (g0, b0) of the current generators, d = g0 . b0, and
// forms the generators of the Schur complement without divisions:
//   G' = [ g0_1 G_0 - g0_0 G_1 ,  (f d e_0 + K' G b0) ],
//   B' = [ b0_1 B_0 - b0_0 B_1 ,  d e_0 + Z' (B g0) ],
// which represent d times the complement of the represented matrix; so the
// pivots of S are d_k / sigma_k with sigma_{k+1} = d_k sigma_k, and
// det S = prod d_k / prod sigma_k (one inversion at the end).  (f = 1 when
// rows k and k+1 lie in the same block; K' shifts inside blocks.)  A zero
// pivot before the last step (a vanishing leading minor) ends the recursion:
// the point then goes through the remainder sequence, as do bad points and
// problems with an empty block.
//
// One wave per (prime, point); lane l holds row l of both generators (degree
// sum m_y + n_y <= 64); the points of a block (kSchurPts) run one after the
// other over the prime's tile, staged once.  Lane j evaluates the
// coefficients a_{m-j} = f_{m-j}(x_i) and b_{n-j} = g_{n-j}(x_i).
constexpr int kSchurPts = 16;
constexpr int kSchurMaxR = 64;
__host__ __device__ inline int eval_schur_lds_words(const DevProblem& P) {
  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  return P.CS + 2 * nm1;
}

__device__ inline void stage_eval_schur(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  const int lane = threadIdx.x;
  const PrimeConst pc = T.pc[P.pidx[w.slot]];
  const uint32_t p = pc.p, pinv = pc.pinv, one = pc.r1;
  uint32_t* tile = lds;
  const uint32_t* src = P.resid + static_cast<size_t>(w.slot) * P.CS;
  for (int t = lane; t < P.CS; t += 64) tile[t] = src[t];
  const int nm1 = (P.my > P.ny ? P.my : P.ny) + 1;
  uint32_t* colA = lds + P.CS;  // columns of the one-lane fallback
  uint32_t* colB = colA + nm1;
  __syncthreads();
  const int m = P.my, n = P.ny, r = m + n;
  const bool two = n > 0 && m > 0;
  const int nxa = P.rowf, nxb = P.rowg;
  const int nx = nxa > nxb ? nxa : nxb;
  const int ra = m - lane, rb = n - lane;  // this lane's rows of f and g
  for (int s = 0; s < kSchurPts; ++s) {
    const int pt = w.blk * kSchurPts + s;
    if (pt > P.E) break;
    const uint32_t x = static_cast<uint32_t>(P.origin + pt);
    const uint32_t xt = mmul(x, pc.r2, p, pinv);
    // Horner in x over every power (zero coefficients beyond a row's degree);
    // values stay below 2p as in horner_step4
    auto hstep = [&](uint32_t acc, uint32_t c) {
      const uint64_t t = static_cast<uint64_t>(acc) * xt + c;
      const uint32_t mq = static_cast<uint32_t>(t) * pinv;
      return static_cast<uint32_t>((t + static_cast<uint64_t>(mq) * p) >> 32);
    };
    uint32_t av = 0u, bv = 0u;
    for (int i = nx - 1; i >= 0; --i) {
      av = hstep(av, (ra >= 0 && i < nxa) ? tile[i * P.myp + ra] : 0u);
      bv = hstep(bv, (rb >= 0 && i < nxb) ? tile[P.goff + i * P.nyp + rb] : 0u);
    }
    av = umin32(av, av - p);
    bv = umin32(bv, bv - p);
    const uint32_t lcf = __builtin_amdgcn_readlane(av, 0), lcg = __builtin_amdgcn_readlane(bv, 0);
    bool bad = (lcf == 0u) || (lcg == 0u);
    uint32_t res = 0u;
    bool done = false;
    if (!bad && two && r <= kSchurMaxR) {
      uint32_t G0 = (lane == 0) ? one : 0u, G1 = (lane == n) ? one : 0u;
      uint32_t B0 = av, B1 = bv;  // S[0][l] = a_{m-l}, S[n][l] = b_{n-l}
      uint32_t num = one, den = one, sigma = one;
      done = true;
      for (int k = 0; k < r; ++k) {
        const uint32_t ga = __builtin_amdgcn_readlane(G0, k), gb = __builtin_amdgcn_readlane(G1, k);
        const uint32_t ba = __builtin_amdgcn_readlane(B0, k), bb = __builtin_amdgcn_readlane(B1, k);
        const uint32_t d = mmulsub(ga, ba, mneg(gb, p), bb, p, pinv);  // ga ba + gb bb
        num = mmul(num, d, p, pinv);
        den = mmul(den, sigma, p, pinv);
        if (k == r - 1) break;
        if (d == 0u) {  // a vanishing leading minor
          done = false;
          break;
        }
        const uint32_t xg = mmulsub(gb, G0, ga, G1, p, pinv);
        const uint32_t yb = mmulsub(bb, B0, ba, B1, p, pinv);
        const uint32_t c = mmulsub(G0, ba, mneg(G1, p), bb, p, pinv);  // G b0
        const uint32_t u = mmulsub(ga, B0, mneg(gb, p), B1, p, pinv);  // B g0
        const uint32_t cprev = static_cast<uint32_t>(__shfl_up(static_cast<int>(c), 1, 64));
        const uint32_t uprev = static_cast<uint32_t>(__shfl_up(static_cast<int>(u), 1, 64));
        if (lane > k) {
          G0 = xg;
          G1 = (lane == n) ? 0u : ((lane == k + 1) ? d : cprev);
          B0 = yb;
          B1 = (lane == k + 1) ? d : uprev;
        }
        sigma = mmul(sigma, d, p, pinv);
      }
      if (done) res = (num == 0u) ? 0u : mmul(num, minv(den, one, p, pinv), p, pinv);
    }
    if (!done) {
      // remainder sequence in lane 0 on the evaluated coefficients
      if (ra >= 0) colA[ra] = av;
      if (rb >= 0) colB[rb] = bv;
      WaveSync()();
      if (lane == 0) res = ures_formal(Column<1>{colA}, Column<1>{colB}, m, n, pc, &bad);
      WaveSync()();
    }
    if (lane == 0) {
      const size_t o = static_cast<size_t>(w.slot) * (P.E + 1) + pt;
      P.zval[o] = redc(res, p, pinv);
      P.zbad[o] = bad ? 1 : 0;
    }
    eval_report_bad(P, w.slot, pt, lane == 0, bad);
  }
}

// LDS words of the evaluation launch for the problem's layout.
__host__ __device__ inline int eval_stage_lds_words(const DevProblem& P) {
  if (P.schur) return eval_schur_lds_words(P);
  if (P.evmf) return P.evk == 2 ? eval_mfma2_lds_words(P, P.regn) : eval_stream_lds_words(P);
  if (P.evk == 2 && P.regn) return eval_regs2_lds_words(P, P.regn);
  if (P.evk > 1) return eval_group_lds_words(P, P.evk);
  return P.regn ? eval_regs_lds_words(P, P.regn) : eval_lds_words(P);
}

// Evaluation layouts; each has a kernel of its own (own register budget).
enum : int {
  kEvBase = 0,  // one lane per pair, LDS columns
  kEvG2,        // two lanes per pair, LDS columns
  kEvG4,        // four lanes per pair, LDS columns
  kEvR8, kEvR16, kEvR24, kEvR32,  // one lane per pair, registers (degree bound)
  kEvP8, kEvP16, kEvP24, kEvP32,  // two lanes per pair, registers
  kEvSchur,     // one wave per pair, Schur algorithm on the Sylvester generators
  kEvM,         // two lanes per pair, registers, sums on the matrix cores: + 2 (regn / 8 - 1) + dkh - 1
  kEvQ = kEvM + 8,   // one lane per pair, streamed, sums on the matrix cores: + 2 (regn / 8 - 1) + dkh - 1
  kEvNum = kEvQ + 12
};
constexpr int kStreamDegMax = 48;   // lower degree of the streamed form (registers)
constexpr int kStreamLongMax = 63;  // higher degree (its values stay in LDS: 17 KB per wave)
constexpr int kMfmaXPowers = 64;    // x-powers of the matrix-core sums (two K slices of 32)
__host__ __device__ inline int eval_variant(const DevProblem& P) {
  if (P.schur) return kEvSchur;
  if (P.evmf) return (P.evk == 2 ? kEvM : kEvQ) + 2 * (P.regn / 8 - 1) + P.dkh - 1;
  const int r = P.regn == 8 ? 0 : P.regn == 16 ? 1 : P.regn == 24 ? 2 : 3;
  if (P.evk == 2 && P.regn) return kEvP8 + r;
  if (P.evk == 2) return kEvG2;
  if (P.evk == 4) return kEvG4;
  if (P.regn) return kEvR8 + r;
  return kEvBase;
}
template <int V>
__device__ inline void stage_eval_variant(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if constexpr (V == kEvBase) stage_eval_ures(P, T, w, lds);
  else if constexpr (V == kEvG2) stage_eval_ures_group<2>(P, T, w, lds);
  else if constexpr (V == kEvG4) stage_eval_ures_group<4>(P, T, w, lds);
  else if constexpr (V >= kEvR8 && V <= kEvR32) stage_eval_ures_regs<8 * (V - kEvR8 + 1)>(P, T, w, lds);
  else if constexpr (V == kEvSchur) stage_eval_schur(P, T, w, lds);
  else if constexpr (V >= kEvQ) stage_eval_ures_stream<8 * ((V - kEvQ) / 2 + 1), (V - kEvQ) % 2 + 1>(P, T, w, lds);
  else if constexpr (V >= kEvM) stage_eval_ures_mfma2<8 * ((V - kEvM) / 2 + 1), (V - kEvM) % 2 + 1>(P, T, w, lds);
  else stage_eval_ures_regs2<8 * (V - kEvP8 + 1)>(P, T, w, lds);
}

// The persistent schedule's dispatch (block-uniform): the LDS-column code,
// which keeps the register budget of a kernel that also runs the other stages
// small.
__device__ inline void stage_eval_columns(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  switch (P.evk) {
    case 2: stage_eval_ures_group<2>(P, T, w, lds); return;
    case 4: stage_eval_ures_group<4>(P, T, w, lds); return;
    default: stage_eval_ures(P, T, w, lds); return;
  }
}

// ------------------------------------------------------------ interpolation

// The consecutive fast path applies when the D+1 points used are origin ..
// origin + D: always with formal-degree values, otherwise when none of them
// was flagged bad (the evaluation stage sets a per-prime flag).  It
// interpolates in t = x - origin; for a shifted origin the Newton stage takes
// the result back to x.
__device__ inline bool fast_prime(const DevProblem& P, int slot) {
  if (P.newton_all) return false;
  if (P.formal) return true;
  return __builtin_amdgcn_readfirstlane(P.status[2 + P.np + slot]) == 0;
}

// Newton forward differences at 0..D as a convolution, one i-chunk of it:
//   a_k = Delta^k z_0 / k! = sum_{i<=k} (z_i / i!) ((-1)^(k-i) / (k-i)!)
// Each thread owns one k; the chunk's partial sum is stored unreduced
// (below p 2^32; REDC of the sum over chunks is a_k).
__device__ inline void stage_interp_conv(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (!fast_prime(P, w.slot)) return;
  const int g = P.pidx[w.slot];
  const PrimeConst pc = T.pc[g];
  const uint32_t p = pc.p, pinv = pc.pinv;
  const uint32_t* ifact = T.ifact + static_cast<size_t>(g) * T.kstride;
  const int nt = blockDim.x;
  const int k0 = w.blk * nt;
  const int kmax = (k0 + nt - 1 < P.D) ? k0 + nt - 1 : P.D;
  const int ib = w.sub * P.cchunk;
  const int ie = (ib + P.cchunk - 1 < kmax) ? ib + P.cchunk - 1 : kmax;  // last i used by this block
  // alpha_i = z_i / i! for i in [ib, ie]; beta_t = (-1)^t / t! R for t in [k0 - ie, kmax - ib]
  const int tb = (k0 - ie > 0) ? k0 - ie : 0;
  const int te = kmax - ib;
  const int na = ie - ib + 1 > 0 ? ie - ib + 1 : 0;
  const int nb = te - tb + 1 > 0 ? te - tb + 1 : 0;
  uint32_t* alpha = lds;
  uint32_t* beta = lds + na;
  const uint32_t* z = P.zval + static_cast<size_t>(w.slot) * (P.E + 1);
  // alpha then beta as one index range, two entries per thread per pass so
  // that their loads are in flight together
  for (int base = threadIdx.x; base < na + nb; base += 2 * nt) {
    uint32_t zv[2], fv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = base + u * nt;
      const int ec = e < na + nb ? e : na + nb - 1;
      const int idx = ec < na ? ib + ec : tb + (ec - na);
      fv[u] = ifact[idx];
      zv[u] = ec < na ? z[idx] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = base + u * nt;
      if (e < na) {
        alpha[e] = mmul(zv[u], fv[u], p, pinv);
      } else if (e < na + nb) {
        const int t = tb + (e - na);
        beta[e - na] = (t & 1) ? mneg(fv[u], p) : fv[u];
      }
    }
  }
  __syncthreads();
  const int k = k0 + threadIdx.x;
  if (k > P.D) return;
  const int iend = (ie < k) ? ie : k;
  uint64_t c0 = 0, c1 = 0, c2 = 0, c3 = 0;
  int i = ib;
  for (; i + 3 <= iend; i += 4) {
    c0 = mac_fold(c0, alpha[i - ib], beta[k - i - tb], p);
    c1 = mac_fold(c1, alpha[i + 1 - ib], beta[k - i - 1 - tb], p);
    c2 = mac_fold(c2, alpha[i + 2 - ib], beta[k - i - 2 - tb], p);
    c3 = mac_fold(c3, alpha[i + 3 - ib], beta[k - i - 3 - tb], p);
  }
  for (; i <= iend; ++i) c0 = mac_fold(c0, alpha[i - ib], beta[k - i - tb], p);
  const uint64_t acc = add_fold(add_fold(c0, c1, p), add_fold(c2, c3, p), p);
  P.aconv[(static_cast<size_t>(w.sub) * P.np + w.slot) * (P.D + 1) + k] = acc;
}

// Falling-factorial basis -> monomials, one k-chunk of the sum
//   c_j = sum_{k >= j} a_k s(k, j)
// written as partial sums per chunk (REDC of the sum over the chunks that
// reach j is c_j).  The context keeps only every kCkpt-th row of the Stirling
// triangle.  The rows k0 .. k0 + kCkpt - 1 after a checkpoint row k0 follow
// from it by x^(k0 + t) = x^(k0) (x - k0)^(t) (falling factorials), so their
// contribution to c_j is a short convolution with that row:
//   sum_t a_{k0+t} s(k0 + t, j) = sum_{i < kCkpt} h_i s(k0, j - i),
// h = the monomial coefficients of sum_t a_{k0+t} (x - k0)^(t).  A segment's h
// is expanded once by Horner's rule (h <- h (x - k0 - t) + a_{k0+t}, one
// coefficient per lane of a half wave) into `hseg`; the basis change then
// streams only checkpoint rows: one column per thread, the row's window and
// the members' h in LDS.

// a_k = REDC(sum of the convolution chunks that reach k) for k in [kb, ke]
// (0 beyond the problem's degree bound), into dst[k - kb].
__device__ inline void load_newton_coeffs(const DevProblem& P, int slot, const PrimeConst& pc, int kb, int ke,
                                          uint32_t* dst) {
  const uint32_t p = pc.p;
  const uint64_t* ap = P.aconv + static_cast<size_t>(slot) * (P.D + 1);
  const size_t astride = static_cast<size_t>(P.np) * (P.D + 1);
  for (int k = kb + static_cast<int>(threadIdx.x); k <= ke; k += blockDim.x) {
    uint32_t v = 0u;
    if (k <= P.D) {
      const int nch = k / P.cchunk + 1;
      uint64_t q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = ap[(u < nch ? u : nch - 1) * astride + k];
      uint64_t sacc = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u < nch) sacc = add_fold(sacc, q[u], p);
      for (int ch = 8; ch < nch; ++ch) sacc = add_fold(sacc, ap[ch * astride + k], p);
      v = redc(sacc, p, pc.pinv);
    }
    dst[k - kb] = v;
  }
}

// h of the segment starting at k0 (rows k0 .. min(k0 + kCkpt - 1, ke), a_k at
// a[k - kb]) by one half wave: lane i of the half gets h_i.
__device__ inline uint32_t segment_h(const uint32_t* a, int kb, int k0, int ke, const PrimeConst& pc) {
  const uint32_t p = pc.p, pinv = pc.pinv;
  const int i = threadIdx.x & (kCkpt - 1);
  uint32_t h = 0u;
  uint32_t ct = mmul(static_cast<uint32_t>(k0 + kCkpt - 1), pc.r2, p, pinv);  // (k0 + t) R mod p
  for (int t = kCkpt - 1; t >= 0; --t) {
    const int k = k0 + t;
    const uint32_t av = (k <= ke) ? a[k - kb] : 0u;
    const uint32_t prev = static_cast<uint32_t>(__shfl_up(static_cast<int>(h), 1, kCkpt));
    h = msubm(i > 0 ? prev : 0u, mmul(h, ct, p, pinv), p);
    if (i == 0) h = maddm(h, av, p);
    ct = msubm(ct, pc.r1, p);
  }
  return h;
}

// Rows [k1, ke] (k1 a multiple of kCkpt) into the partial sum acc of column
// j0 + threadIdx.x; the block's threads are its columns.  The segments' h are
// expanded here from a_k at lds_a[k - kb].  LDS: lh (kCkpt words), lw
// (blockDim + kCkpt - 1).
__device__ inline uint64_t basis_block(const uint32_t* S, int j0, int k1, int ke, int kb, const uint32_t* lds_a,
                                       const PrimeConst& pc, uint32_t* lh, uint32_t* lw) {
  const int nt = blockDim.x, tid = threadIdx.x;
  uint64_t acc = 0u;
  // the next segment's row window (two values per thread, nt >= kCkpt - 1) is
  // loaded into registers while the current segment is convolved
  uint32_t nw0 = 0u, nw1 = 0u;
  auto fetch = [&](int k0) {
    const uint32_t* row = S + ckpt_rowoff(k0 / kCkpt);
    const int ja = j0 - (kCkpt - 1) + tid, jb = ja + nt;
    nw0 = (ja >= 0 && ja <= k0) ? row[ja] : 0u;
    nw1 = (tid < kCkpt - 1 && jb >= 0 && jb <= k0) ? row[jb] : 0u;
  };
  if (k1 <= ke) fetch(k1);
  for (int k0 = k1; k0 <= ke; k0 += kCkpt) {
    if (tid < kCkpt) lh[tid] = segment_h(lds_a, kb, k0, ke, pc);
    lw[tid] = nw0;
    if (tid < kCkpt - 1) lw[nt + tid] = nw1;
    __syncthreads();
    if (k0 + kCkpt <= ke) fetch(k0 + kCkpt);
#pragma unroll 8
    for (int i = 0; i < kCkpt; ++i) acc = mac_fold(acc, lh[i], lw[tid + kCkpt - 1 - i], pc.p);  // s(k0, j - i)
    __syncthreads();  // the next segment overwrites lh and lw
  }
  return acc;
}

// ------------------------------------- interpolation on the matrix cores
// The staged and plain schedules.  Both triangular factors of the consecutive
// points' interpolation act on one (problem, prime) column by sums of the form
//   out_k = sum_i A(k - i) d_i,
// A Toeplitz: the forward differences (A(x) = (-1)^x / x!, d = z_i / i!) and, per
// checkpoint row k0 of the Stirling triangle, the segment's polynomial
// (A = h_{k0}, d = s(k0, .)).  Written over blocks of 16, k = 16 a + b and
// i = 16 u + v, with D = a - u,
//   out[b][a] = sum_{D, v} A(16 D + b - v) d[16 (a - D) + v]:
// a matrix product with 16 rows b, 16 block columns a and K = (D, v), whose left
// operand does not depend on a.  So one column fills the 16 x 16 output tile of
// the matrix cores by itself (the earlier form put the columns of 16 problems
// side by side, and left 14 of 16 idle on a single system), the operand tiles
// are built once per wave, and nothing has to be grouped by primes.  Both sides
// split into four balanced base-256 digits (16 int8 16x16x64 products per K
// slice of 64); the seven anti-diagonal sums stay below 4 * 3840 * 2^14 < 2^28
// for the differences and 4 * 48 * 120 * 2^14 < 2^29 for the basis change.
//
// Each takes a tile of 256 outputs per item (problem, slot, tile), KS waves
// splitting the K range (KS = 4 for jobs with few tiles).  Measured, both
// products and the segment polynomials between them: 256 pairs of the batch
// workload 497 -> 220 us (against 16-column tiles with five 7-bit digits), 64
// requests of degrees 8..48 1170 -> 253, curve analysis 130 -> 35, the degree-24
// pair 35 -> 17 us (against the vector-ALU sums).
constexpr int kTile = 256;
// Fewer tiles than one per SIMD: four waves share a tile's K range (curve
// analysis, 756 tiles: 14.9 + 20.2 us against 25.3 + 38.3 with one wave each);
// from there on one wave per tile, which forms the sums once (24 pairs of the
// batch workload, about 1900 tiles: 28.0 + 36.2 us against 30.3 + 38.6; 256
// pairs: 104.7 + 115.6 against 153.6 + 195.3).
constexpr int kInterpSplitItems = 1024;
constexpr int kConvFront = 18;  // zero blocks of 16 below index 0 of d (the tile's columns reach -288)
constexpr int kSegWords = 21;   // 16-byte groups of one segment's reversed digits with their padding
__host__ __device__ inline int interp_coeffs_lds_words(int D, int ks) {
  const int kt = D / kTile * kTile;
  const int w = 16 * (kt / 16 + 16 + kConvFront) + 16 * (4 * (D / 64 + 1) + 1);
  const int red = ks > 1 ? 512 * ks : 768;  // the partial sums, then the segments' scratch
  return w > red ? w : red;
}
__host__ __device__ inline int interp_basis_lds_words(int ks) { return 8 * kSegWords * 4 * ks; }

// digits of four consecutive values: out[d] = digit d of v0, v1, v2, v3
__device__ __forceinline__ void digits4(int32_t v0, int32_t v1, int32_t v2, int32_t v3, uint32_t* out) {
  byte_transpose4(balanced_digits(static_cast<uint32_t>(v0)), balanced_digits(static_cast<uint32_t>(v1)),
                  balanced_digits(static_cast<uint32_t>(v2)), balanced_digits(static_cast<uint32_t>(v3)), out);
}

// Toeplitz operand of a K slice: bytes start .. start + 15 of each digit's
// reversed run, stored as groups of 4 bytes of each digit (16 bytes per group).
__device__ __forceinline__ void toeplitz_operand(const uint4* groups, int start, ev_v4i (&A)[kEvDigits]) {
  const uint4* g = groups + (start >> 2);
  const uint32_t sh = static_cast<uint32_t>(start) & 3u;
  uint4 r[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) r[j] = g[j];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    A[0][j] = static_cast<int>(__builtin_amdgcn_alignbyte(r[j + 1].x, r[j].x, sh));
    A[1][j] = static_cast<int>(__builtin_amdgcn_alignbyte(r[j + 1].y, r[j].y, sh));
    A[2][j] = static_cast<int>(__builtin_amdgcn_alignbyte(r[j + 1].z, r[j].z, sh));
    A[3][j] = static_cast<int>(__builtin_amdgcn_alignbyte(r[j + 1].w, r[j].w, sh));
  }
}

__device__ __forceinline__ void digit_products(const ev_v4i (&A)[kEvDigits], const ev_v4i (&B)[kEvDigits],
                                               ev_v4i (&S)[2 * kEvDigits - 1]) {
#pragma unroll
  for (int a = 0; a < kEvDigits; ++a)
#pragma unroll
    for (int b = 0; b < kEvDigits; ++b)
      S[a + b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[a], B[b], S[a + b], 0, 0, 0);
}

// sum_s S_s 2^(8 s) of the lane's four outputs (rows 4 (l / 16) + r of column l
// mod 16), with weights 2^(8 s) mod p, summed over the KS waves: wave 0 returns
// true and the sums.
template <int KS>
__device__ __forceinline__ bool interp_sums(const ev_v4i (&S)[2 * kEvDigits - 1], const PrimeConst& pc,
                                            const SignedMod& M, uint32_t* lds, int64_t (&t)[4]) {
  int32_t w = 1;
  const int32_t t256 = smul(256, static_cast<int32_t>(pc.r2), M);
#pragma unroll
  for (int r = 0; r < 4; ++r) t[r] = 0;
#pragma unroll
  for (int s = 0; s < 2 * kEvDigits - 1; ++s) {
    const int32_t wu = __builtin_amdgcn_readfirstlane(w);
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = smad(S[s][r], wu, t[r]);
    w = scenter(smul(w, t256, M), M);
  }
  if constexpr (KS > 1) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t* red = reinterpret_cast<int64_t*>(lds) + lane * 4;
    __syncthreads();  // the operands in LDS are consumed
    if (wave > 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave * 256 + r] = t[r];
    }
    __syncthreads();
    if (wave > 0) return false;
#pragma unroll
    for (int v = 1; v < KS; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) t[r] += red[v * 256 + r];
  }
  WaveSync()();
  return true;
}

// Newton coefficients a_k = Delta^k z_0 / k! of a tile of 256 k's, and from them
// the segments' polynomials of the basis change: rows k0 .. k0 + 31 after a
// checkpoint row k0 contribute sum_t a_{k0+t} x^(k0+t) = x^(k0) H(x),
//   H(x) = sum_t a_{k0+t} (x - k0)(x - k0 - 1) .. (x - k0 - t + 1),
// and H's monomial coefficients h_0..h_31 go to hseg (signed, |h| <= p / 2).
// Horner's rule in x over quads of factors: with the quartic of four factors,
// h_i <- h_{i-4} + e1 h_{i-3} + e2 h_{i-2} + e3 h_{i-1} + e4 h_i + l_i, a lane
// keeping four entries of one of the tile's eight segments; the quartics and
// the low parts l are formed by one lane each beforehand.  Against one factor
// per step with one entry per lane (32 shuffled steps, 629 instructions per 64
// coefficients): about 600 per 256.
template <int KS>
__device__ inline void stage_interp_coeffs(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (!fast_prime(P, w.slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NT = 64 * KS;
  const int g = P.pidx[w.slot];
  const PrimeConst pc = T.pc[g];
  const SignedMod M = signed_mod(pc);
  const uint32_t* ifact = T.ifact + static_cast<size_t>(g) * T.kstride;
  const uint32_t* z = P.zval + static_cast<size_t>(w.slot) * (P.E + 1);
  const int k0t = kTile * w.blk;
  const int kend = (k0t + kTile - 1 < P.D) ? k0t + kTile - 1 : P.D;
  const int nsl = kend / 64 + 1;         // K slices: D = 0 .. 4 nsl - 1
  const int nu = k0t / 16 + 16 + kConvFront;
  uint32_t* yw = lds;                    // [block of 16][digit][4 words]
  uint4* tw = reinterpret_cast<uint4*>(lds + 16 * nu);  // [group of 4][digit]
  for (int q = tid; q < 4 * nu; q += NT) {
    const int i0 = 4 * q - 16 * kConvFront;
    int32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = (i0 >= 0 && i0 + e <= kend)
                 ? smul(static_cast<int32_t>(z[i0 + e]), static_cast<int32_t>(ifact[i0 + e]), M) : 0;
    uint32_t o[kEvDigits];
    digits4(v[0], v[1], v[2], v[3], o);
#pragma unroll
    for (int d = 0; d < kEvDigits; ++d) yw[(q >> 2) * 16 + 4 * d + (q & 3)] = o[d];
  }
  const int C = 16 * (4 * nsl - 1) + 15;
  for (int q = tid; q < 4 * (4 * nsl + 1); q += NT) {
    int32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int x = C - (4 * q + e);
      const int32_t f = (x >= 0 && x <= kend) ? static_cast<int32_t>(ifact[x]) : 0;
      v[e] = (x & 1) ? -f : f;
    }
    uint32_t o[kEvDigits];
    digits4(v[0], v[1], v[2], v[3], o);
    tw[q] = make_uint4(o[0], o[1], o[2], o[3]);
  }
  if constexpr (KS > 1) __syncthreads();
  else WaveSync()();

  ev_v4i S[2 * kEvDigits - 1];
#pragma unroll
  for (int s = 0; s < 2 * kEvDigits - 1; ++s) S[s] = ev_v4i{0, 0, 0, 0};
  const int b = lane & 15, q4 = lane >> 4;  // row b (left operand), block column b (right operand), K quarter
  for (int s = wave; s < nsl; s += KS) {
    const int d = 4 * s + q4;
    ev_v4i A[kEvDigits], B[kEvDigits];
    const ev_v4i* src = reinterpret_cast<const ev_v4i*>(yw) + 4 * (k0t / 16 + b - d + kConvFront);
#pragma unroll
    for (int e = 0; e < kEvDigits; ++e) B[e] = src[e];
    toeplitz_operand(tw, C - 16 * d - b, A);
    digit_products(A, B, S);
  }
  int64_t t[4];
  if (!interp_sums<KS>(S, pc, M, lds, t)) return;

  int4* av = reinterpret_cast<int4*>(lds);        // the tile's a_k
  int4* lowp = reinterpret_cast<int4*>(lds) + 64; // [segment][quad] low parts
  int4* quart = lowp + 64;                        // [segment][quad] quartics
  {
    int32_t a[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = (k0t + 16 * b + 4 * q4 + r <= P.D) ? sredc(t[r], M) : 0;
    WaveSync()();
    av[4 * b + q4] = make_int4(a[0], a[1], a[2], a[3]);
  }
  WaveSync()();
  const int e = lane & 7;  // segment lane / 8; quad (rows k0 + 4 e ..) and entries 4 e .. 4 e + 3
  {
    const int64_t c0 = k0t + 4 * lane, c1 = c0 + 1, c2 = c0 + 2, c3 = c0 + 3;
    // x R mod p, centred, for |x| < 2^50
    auto mont = [&](int64_t x) { return scenter(smul(sredc(x, M), static_cast<int32_t>(pc.r3), M), M); };
    const int64_t s2 = c0 + c1, p2 = c0 * c1, s3 = s2 + c2, q3 = p2 + s2 * c2, p3 = p2 * c2;
    const int4 a = av[lane];
    const int32_t p3m = mont(p3), q3m = mont(q3), s3m = mont(s3);
    int4 l;
    l.x = scenter(a.x + sredc(smad(-mont(c0), a.y, smad(mont(p2), a.z, smad(-p3m, a.w, 0))), M), M);
    l.y = scenter(a.y + sredc(smad(-mont(s2), a.z, smad(q3m, a.w, 0)), M), M);
    l.z = scenter(a.z + sredc(smad(-s3m, a.w, 0), M), M);
    l.w = scenter(a.w, M);
    lowp[lane] = l;
    quart[lane] = make_int4(mont(-(s3 + c3)), mont(q3 + s3 * c3), mont(-(p3 + q3 * c3)), mont(p3 * c3));
  }
  WaveSync()();
  int32_t h0 = 0, h1 = 0, h2 = 0, h3 = 0;
  auto from_left = [](int32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x111 /* row_shr:1 */, 0xF, 0xF, true); };
#pragma unroll
  for (int Q = 7; Q >= 0; --Q) {
    const int4 l = lowp[(lane & 56) + Q], c = quart[(lane & 56) + Q];
    const int32_t q0 = from_left(h0), q1 = from_left(h1), q2 = from_left(h2), q3 = from_left(h3);
    const bool first = e == 0;
    const int32_t z1 = first ? 0 : q1, z2 = first ? 0 : q2, z3 = first ? 0 : q3;
    const int32_t n0 = sredc(smad(c.x, z1, smad(c.y, z2, smad(c.z, z3, smad(c.w, h0, 0)))), M) + (first ? l.x : q0);
    const int32_t n1 = sredc(smad(c.x, z2, smad(c.y, z3, smad(c.z, h0, smad(c.w, h1, 0)))), M) + (first ? l.y : q1);
    const int32_t n2 = sredc(smad(c.x, z3, smad(c.y, h0, smad(c.z, h1, smad(c.w, h2, 0)))), M) + (first ? l.z : q2);
    const int32_t n3 = sredc(smad(c.x, h0, smad(c.y, h1, smad(c.z, h2, smad(c.w, h3, 0)))), M) + (first ? l.w : q3);
    h0 = scenter(n0, M);  // |n| <= (4 / 4 / 3 + 1 / 2 + 1 / 2) p < 1.5 p
    h1 = scenter(n1, M);
    h2 = scenter(n2, M);
    h3 = scenter(n3, M);
  }
  const int at = k0t + 4 * lane;
  if (at < P.hstride)
    *reinterpret_cast<int4*>(P.hseg + static_cast<size_t>(w.slot) * P.hstride + at) = make_int4(h0, h1, h2, h3);
}

// Falling factorials -> monomials, a tile of 256 coefficients:
//   c_j = sum_{k0} sum_{i < 32} h_{k0,i} s(k0, j - i)
// over the checkpoint rows k0 >= the tile's first j.  The segments' operands are
// built in LDS eight at a time; the row's digits are split in registers from
// the 16 words a lane loads one segment ahead.  Written as c_j 2^32, the only
// word the CRT reads for j.  Bound by the digit splitting of the rows (about 90
// VALU instructions against 16 products per segment).
alignas(16) __device__ const uint32_t kZeroRow[16] = {};
template <int KS>
__device__ inline void stage_interp_basis(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (!fast_prime(P, w.slot)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = P.pidx[w.slot];
  const PrimeConst pc = T.pc[g];
  const SignedMod M = signed_mod(pc);
  const uint32_t* stir = T.stir + static_cast<size_t>(g) * T.sstride;
  const uint32_t* hrow = P.hseg + static_cast<size_t>(w.slot) * P.hstride;
  const int j0 = kTile * w.blk, D = P.D;
  uint4* seg = reinterpret_cast<uint4*>(lds) + wave * 8 * kSegWords;  // this wave's eight segments
  for (int t = lane; t < 8 * kSegWords; t += 64) seg[t] = make_uint4(0u, 0u, 0u, 0u);
  ev_v4i S[2 * kEvDigits - 1];
#pragma unroll
  for (int s = 0; s < 2 * kEvDigits - 1; ++s) S[s] = ev_v4i{0, 0, 0, 0};
  const int b = lane & 15, q4 = lane >> 4;
  const int J = j0 + 16 * (b - q4);  // first index of the lane's 16 row entries
  typedef const __attribute__((address_space(1))) ev_v4u* gptr;
  // the 16 row entries of segment s (k0 = 32 s): zero outside 0 .. k0
  auto load_row = [&](int s, ev_v4u (&r)[4]) {
    const uint32_t* src = (J >= 0 && J <= 32 * s) ? stir + ckpt_rowoff(s) + J : kZeroRow;
    const gptr p4 = (gptr)(src);
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = p4[u];
  };
  const int sfirst = j0 / 32, slast = D / 32;
  for (int s0 = sfirst + 8 * wave; s0 <= slast; s0 += 8 * KS) {
    WaveSync()();  // the previous segments' operands are consumed
    const int x = 32 * s0 + 4 * lane;  // entries 4 (lane mod 8) .. + 3 of segment s0 + lane / 8
    int4 h = make_int4(0, 0, 0, 0);
    if (x < P.hstride) h = *reinterpret_cast<const int4*>(hrow + x);
    ev_v4u nx[4];
    load_row(s0, nx);
    uint32_t o[kEvDigits];
    digits4(h.w, h.z, h.y, h.x, o);
    seg[(lane >> 3) * kSegWords + 15 - (lane & 7)] = make_uint4(o[0], o[1], o[2], o[3]);
    WaveSync()();
    const int ns = slast - s0 + 1 < 8 ? slast - s0 + 1 : 8;
    for (int u = 0; u < ns; ++u) {
      ev_v4u r[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) r[v] = nx[v];
      if (u + 1 < ns) load_row(s0 + u + 1, nx);
      const int k0 = 32 * (s0 + u);
      if (k0 < j0 + kTile && J == k0) {  // the row ends at its entry k0: words beyond it are not part of the table
        r[0].y = r[0].z = r[0].w = 0u;
#pragma unroll
        for (int v = 1; v < 4; ++v) r[v].x = r[v].y = r[v].z = r[v].w = 0u;
      }
      ev_v4i A[kEvDigits], B[kEvDigits];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        uint32_t dg[kEvDigits];
        digits4(static_cast<int32_t>(r[v].x), static_cast<int32_t>(r[v].y), static_cast<int32_t>(r[v].z),
                static_cast<int32_t>(r[v].w), dg);
#pragma unroll
        for (int d = 0; d < kEvDigits; ++d) B[d][v] = static_cast<int>(dg[d]);
      }
      toeplitz_operand(seg + u * kSegWords, 63 - 16 * q4 - b, A);
      digit_products(A, B, S);
    }
  }
  int64_t t[4];
  if (!interp_sums<KS>(S, pc, M, lds, t)) return;
  uint64_t* cp = P.cpart + static_cast<size_t>(w.slot) * (D + 1);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int j = j0 + 16 * b + 4 * q4 + r;
    if (j <= D) cp[j] = static_cast<uint64_t>(scanon(sredc(t[r], M), M)) << 32;
  }
}

// LDS words of a basis-change block of the persistent schedule: a segment's h,
// the row window and the chunk's a_k.
__host__ __device__ inline int basis_lds_words(int nthreads, int K) { return kCkpt + nthreads + kCkpt - 1 + K; }

// The persistent schedule's basis change: (problem, slot, block of blockDim
// columns, chunk).
__device__ inline void stage_interp_stir(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds) {
  if (!fast_prime(P, w.slot)) return;
  const int g = P.pidx[w.slot];
  const PrimeConst pc = T.pc[g];
  const int nt = blockDim.x;
  const int kb = w.sub * P.kchunk;
  const int ke = (kb + P.kchunk - 1 < P.D) ? kb + P.kchunk - 1 : P.D;
  const int j0 = w.blk * nt;
  uint32_t* lh = lds;
  uint32_t* lw = lds + kCkpt;
  uint32_t* la = lw + nt + kCkpt - 1;
  load_newton_coeffs(P, w.slot, pc, kb, ke, la);
  __syncthreads();
  if (j0 > ke || j0 > P.D) return;  // block-uniform: no row of the chunk reaches these columns
  // rows below j0 contribute nothing to them: start at j0's checkpoint
  const int jc = (j0 / kCkpt) * kCkpt;
  const int k1 = kb > jc ? kb : jc;
  const uint64_t acc = basis_block(T.stir + static_cast<int64_t>(g) * T.sstride, j0, k1, ke, kb, la, pc, lh, lw);
  const int j = j0 + static_cast<int>(threadIdx.x);
  if (j <= P.D) P.cpart[(static_cast<size_t>(w.sub) * P.np + w.slot) * (P.D + 1) + j] = acc;
}

// LDS words of the gapped-interpolation block.
__host__ __device__ inline int newton_lds_words(const DevProblem& P, int nthreads) {
  const int e1 = P.E + 1;
  return 3 * e1 + (e1 > nthreads ? e1 : nthreads);
}

// The partial-sum chunks of a run: the problem's layout in the persistent
// schedule, one whole chunk in the staged and plain ones.
struct Chunks {
  int n, len;
};
__device__ inline Chunks chunks_of(const DevProblem& P, bool whole) {
  return whole ? Chunks{1, P.D + 1} : Chunks{P.nchunk, P.kchunk};
}

// Consecutive points from a shifted origin o: the fast path left the
// coefficients ct_k of R(t + o) in the slot's partial sums; R(x) has
//   c_j = sum_{k >= j} C(k, j) (-o)^(k-j) ct_k,
// a correlation j! c_j = sum_d u_{j+d} v_d with u_k = k! ct_k and
// v_d = (-o)^d / d! (a Taylor shift), one thread per j.  Written as the
// Newton stage writes its result: c_j 2^32 in the first chunk the CRT reads
// for j, zero in the later ones.  LDS: 2 (D+1) words.
__device__ inline void shift_origin(const DevProblem& P, const DevTables& T, int slot, uint32_t* lds, Chunks ck) {
  const int tid = threadIdx.x, nt = blockDim.x, D = P.D;
  const int g = P.pidx[slot];
  const PrimeConst pc = T.pc[g];
  const uint32_t p = pc.p, pinv = pc.pinv;
  const uint32_t* fact = T.fact + static_cast<size_t>(g) * T.kstride;
  const uint32_t* ifact = T.ifact + static_cast<size_t>(g) * T.kstride;
  const size_t cstride = static_cast<size_t>(P.np) * (D + 1);
  uint64_t* cp = P.cpart + static_cast<size_t>(slot) * (D + 1);
  uint32_t* u = lds;
  uint32_t* v = lds + (D + 1);
  const uint32_t mo = mmul(p - static_cast<uint32_t>(P.origin), pc.r2, p, pinv);  // -o R (o < 2^24 < p)
  for (int k = tid; k <= D; k += nt) {
    uint64_t cs = 0;
    for (int ch = k / ck.len; ch < ck.n; ++ch) cs = add_fold(cs, cp[ch * cstride + k], p);
    u[k] = mmul(redc(cs, p, pinv), fact[k], p, pinv);  // k! ct_k
    uint32_t pw = pc.r1, base = mo;                     // (-o)^k R by squaring
    for (int e = k; e; e >>= 1) {
      if (e & 1) pw = mmul(pw, base, p, pinv);
      base = mmul(base, base, p, pinv);
    }
    v[k] = mmul(pw, ifact[k], p, pinv);  // (-o)^k / k! R
  }
  __syncthreads();  // every partial sum is read before any is overwritten
  for (int j = tid; j <= D; j += nt) {
    uint64_t acc = 0;
    for (int d = 0; d <= D - j; ++d) acc = mac_fold(acc, u[j + d], v[d], p);
    const uint32_t c = mmul(redc(acc, p, pinv), ifact[j], p, pinv);
    const int ch0 = j / ck.len;
    cp[ch0 * cstride + j] = static_cast<uint64_t>(c) << 32;
    for (int ch = ch0 + 1; ch < ck.n; ++ch) cp[ch * cstride + j] = 0;
  }
}

// Gapped point sets (bad points replaced): one block per prime; select the
// first D+1 usable points, Newton divided differences, then the Newton form
// expanded in the monomial basis by Horner.  Slots that took the consecutive
// path need only the shift back from a nonzero origin.
__device__ inline void stage_interp_newton(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds,
                                           bool whole) {
  const Chunks ck = chunks_of(P, whole);
  const int tid = threadIdx.x, nt = blockDim.x;
  const int slot = w.slot;
  const bool fast = fast_prime(P, slot);
  if (tid == 0) P.status[1 + slot] = fast ? 0 : 1;
  if (fast) {
    if (P.origin != 0) shift_origin(P, T, slot, lds, ck);
    return;
  }
  const int g = P.pidx[slot];
  const PrimeConst pc = T.pc[g];
  const uint32_t p = pc.p, pinv = pc.pinv;
  const int E = P.E, D = P.D;
  const uint32_t* fact = T.fact + static_cast<size_t>(g) * T.kstride;
  const uint32_t* ifact = T.ifact + static_cast<size_t>(g) * T.kstride;
  const uint32_t* z = P.zval + static_cast<size_t>(slot) * (E + 1);
  const uint8_t* zb = P.zbad + static_cast<size_t>(slot) * (E + 1);

  uint32_t* xs = lds;                 // E+1: selected point indices
  uint32_t* d0 = xs + (E + 1);        // E+1
  uint32_t* invt = d0 + (E + 1);      // E+1: 1/t R mod p
  uint32_t* d1 = invt + (E + 1);      // max(E+1, nt); also the scan buffer
  int* cnt = reinterpret_cast<int*>(d1);

  for (int t = tid + 1; t <= E; t += nt) invt[t] = mmul(ifact[t], fact[t - 1], p, pinv);

  // selection: first D+1 usable points (all points in formal mode)
  const int chunk = (E + 1 + nt - 1) / nt;
  const int lo = tid * chunk;
  const int hi = (lo + chunk < E + 1) ? lo + chunk : E + 1;
  int c = 0;
  for (int i = lo; i < hi; ++i) c += (P.formal || !zb[i]) ? 1 : 0;
  cnt[tid] = c;
  __syncthreads();
  for (int off = 1; off < nt; off <<= 1) {  // inclusive Hillis-Steele scan
    const int v = (tid >= off) ? cnt[tid - off] : 0;
    __syncthreads();
    cnt[tid] += v;
    __syncthreads();
  }
  const int total = cnt[nt - 1];
  int q = cnt[tid] - c;
  __syncthreads();
  if (total < D + 1) {
    if (tid == 0) atomicOr(P.status, kErrTooFewGoodPoints);
    return;  // block-uniform
  }
  for (int i = lo; i < hi && q <= D; ++i)
    if (P.formal || !zb[i]) {
      xs[q] = static_cast<uint32_t>(i);
      d0[q] = z[i];
      ++q;
    }
  __syncthreads();

  // divided differences, level by level (ping-pong buffers)
  uint32_t* cur = d0;
  uint32_t* nxt = d1;
  for (int k = 1; k <= D; ++k) {
    for (int i = tid; i <= D; i += nt) {
      if (i >= k) {
        const uint32_t diff = msubm(cur[i], cur[i - 1], p);
        nxt[i] = mmul(diff, invt[xs[i] - xs[i - k]], p, pinv);
      } else {
        nxt[i] = cur[i];
      }
    }
    __syncthreads();
    uint32_t* t = cur; cur = nxt; nxt = t;
  }
  // Newton form -> monomials: P <- P (x - x_k) + a_k, k = D-1 .. 0
  uint32_t* coef = invt;  // the inverse table is no longer needed
  for (int i = tid; i <= D; i += nt) coef[i] = cur[i];
  __syncthreads();
  uint32_t* pa = nxt;
  uint32_t* pb = cur;
  if (tid == 0) pa[0] = coef[D];
  __syncthreads();
  for (int k = D - 1; k >= 0; --k) {
    const uint32_t xk = static_cast<uint32_t>(P.origin) + xs[k];
    const uint32_t xkt = mmul(xk, pc.r2, p, pinv);
    const int deg = D - k;  // degree after this step
    for (int j = tid; j <= deg; j += nt) {
      const uint32_t left = (j > 0) ? pa[j - 1] : 0u;
      const uint32_t mid = (j < deg) ? pa[j] : 0u;
      uint32_t v = msubm(left, mmul(mid, xkt, p, pinv), p);
      if (j == 0) v = maddm(v, coef[k], p);
      pb[j] = v;
    }
    __syncthreads();
    uint32_t* t = pa; pa = pb; pb = t;
  }
  // the first chunk the CRT reads for coefficient j carries c_j 2^32 (REDC gives
  // c_j); the later chunks are zero
  for (int j = tid; j <= D; j += nt) {
    const int ch0 = j / ck.len;
    P.cpart[(static_cast<size_t>(ch0) * P.np + slot) * (D + 1) + j] = static_cast<uint64_t>(pa[j]) << 32;
    for (int ch = ch0 + 1; ch < ck.n; ++ch)
      P.cpart[(static_cast<size_t>(ch) * P.np + slot) * (D + 1) + j] = 0;
  }
}

// ----------------------------------------------------------------------- CRT

// dst[t] = src(t) for t < n with the block's threads; every thread issues up
// to eight loads (clamped to valid indices) before storing any, so a small
// table costs about one memory latency.
template <class F>
__device__ inline void block_stage(uint32_t* dst, int n, F src) {
  const int nt = blockDim.x;
  for (int base = threadIdx.x; base < n; base += 8 * nt) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = base + u * nt;
      v[u] = src(t < n ? t : n - 1);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = base + u * nt;
      if (t < n) dst[t] = v[u];
    }
  }
}

// Residues of the block's coefficients (kCrtBlockCoeffs per block) are
// staged in LDS first: [coefficient][prime].
constexpr int kCrtBlockCoeffs = 8;
constexpr int kCrtConsts = 6;  // per prime: p, -p^{-1}, Garner inverse, w, r_lo, r_hi
__host__ __device__ inline int crt_wave_words(int ns) { return 3 * 64 * ns + 4; }
__host__ __device__ inline int crt_base_words(const DevProblem& P, int ns, int nwaves) {
  return nwaves * crt_wave_words(ns) + kCrtBlockCoeffs * P.np + kCrtConsts * P.np;
}
// The table of the M / p_j limbs is staged in LDS when it fits.
__host__ __device__ inline bool crt_stage_mi(const DevProblem& P, int ns, int nwaves) {
  return P.np * P.L_out + crt_base_words(P, ns, nwaves) <= kLdsWords;
}
__host__ __device__ inline int crt_lds_words(const DevProblem& P, int ns, int nwaves) {
  return (crt_stage_mi(P, ns, nwaves) ? P.np * P.L_out : 0) + crt_base_words(P, ns, nwaves);
}

// Sum of a 32-bit value over the 64 lanes of a wave (every lane gets it).
__device__ inline uint32_t wave_sum32(uint32_t v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), m, 64));
  return v;
}

// Radix conversion of one coefficient (lanes own output limbs t = lane + 64 r):
//   Z_t = init_t + sum_j v_j tab[j][t]   (96-bit column sums),
// carries resolved with wave ballots; writes Z mod 2^(32 L_out).
// Each v_j < 2^32 comes in 16-bit halves -- the caller leaves lo16(v_j) in
// vbuf[j] and hi16(v_j) in sb[j] (sb is free until the carry phase) -- so that
// the column sums
//   A_t = sum_j lo16(v_j) tab[j][t],  B_t = sum_j hi16(v_j) tab[j][t]
// take one 64-bit multiply-add per term with no carry handling: every term is
// below 2^48 and at most 512 primes come here, so both sums stay below 2^57.
// Then Z_t = init_t + A_t + 2^16 B_t, formed once per limb in 96 bits.
template <int NS>
__device__ inline void crt_radix(const DevProblem& P, int k, bool valid, const uint32_t* vbuf, const uint32_t* tab,
                                 int tstride, const uint64_t* init, uint32_t* sb, uint32_t* sc) {
  const int lane = threadIdx.x & 63;
  const int np = P.np, L = P.L_out;
  // two independent accumulator pairs per limb (short dependency chains)
  uint64_t A0[NS], B0[NS], A1[NS], B1[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) A0[r] = B0[r] = A1[r] = B1[r] = 0u;
  int j = 0;
  for (; j + 4 <= np; j += 4) {
    const uint64_t l0 = vbuf[j], l1 = vbuf[j + 1], l2 = vbuf[j + 2], l3 = vbuf[j + 3];
    const uint64_t h0 = sb[j], h1 = sb[j + 1], h2 = sb[j + 2], h3 = sb[j + 3];
    const uint32_t* p0 = tab + static_cast<size_t>(j) * tstride;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int t = lane + 64 * r;
      if (t < L) {
        const uint64_t w0 = p0[t], w1 = p0[tstride + t], w2 = p0[2 * tstride + t], w3 = p0[3 * tstride + t];
        A0[r] += l0 * w0;
        B0[r] += h0 * w0;
        A1[r] += l1 * w1;
        B1[r] += h1 * w1;
        A0[r] += l2 * w2;
        B0[r] += h2 * w2;
        A1[r] += l3 * w3;
        B1[r] += h3 * w3;
      }
    }
  }
  for (; j < np; ++j) {
    const uint64_t l0 = vbuf[j], h0 = sb[j];
    const uint32_t* p0 = tab + static_cast<size_t>(j) * tstride;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int t = lane + 64 * r;
      if (t < L) {
        const uint64_t w0 = p0[t];
        A0[r] += l0 * w0;
        B0[r] += h0 * w0;
      }
    }
  }
  uint64_t lo[NS];
  uint32_t hc[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const uint64_t A = A0[r] + A1[r], B = B0[r] + B1[r];  // each < 2^58
    uint64_t z = init[r] + A;
    uint32_t h = z < A ? 1u : 0u;
    const uint64_t Bs = B << 16;
    z += Bs;
    h += (z < Bs ? 1u : 0u) + static_cast<uint32_t>(B >> 48);
    lo[r] = z;
    hc[r] = h;
  }
  // limb t receives lo32(S_t) + hi32(S_{t-1}) + top32(S_{t-2})
  WaveSync sync;
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int t = lane + 64 * r;
    sb[t + 1] = static_cast<uint32_t>(lo[r] >> 32);
    sc[t + 2] = hc[r];
  }
  if (lane == 0) {
    sb[0] = 0;
    sc[0] = 0;
    sc[1] = 0;
  }
  sync();
  uint32_t l1[NS], h1[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int t = lane + 64 * r;
    const uint64_t wv = static_cast<uint64_t>(static_cast<uint32_t>(lo[r])) + sb[t] + sc[t];
    l1[r] = static_cast<uint32_t>(wv);
    h1[r] = static_cast<uint32_t>(wv >> 32);  // <= 2
  }
  sync();
#pragma unroll
  for (int r = 0; r < NS; ++r) sb[lane + 64 * r + 1] = h1[r];
  sync();
  uint64_t cin = 0;
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int t = lane + 64 * r;
    const uint64_t x2 = static_cast<uint64_t>(l1[r]) + sb[t];
    const uint32_t l2 = static_cast<uint32_t>(x2);
    const bool gen = (x2 >> 32) != 0 && t < L;
    const bool prop = (l2 == 0xFFFFFFFFu) && t < L;
    const uint64_t G = __ballot(gen);
    const uint64_t Pm = __ballot(prop);
    const uint64_t X = G | Pm;
    const unsigned __int128 tot = static_cast<unsigned __int128>(X) + G + cin;
    const uint64_t S = static_cast<uint64_t>(tot);
    const uint64_t C = S ^ X ^ G;  // carry into each limb of this group
    cin = static_cast<uint64_t>(tot >> 64);
    const uint32_t limb = l2 + static_cast<uint32_t>((C >> lane) & 1u);
    if (valid && t < L) P.out[static_cast<size_t>(k) * L + t] = limb;
  }
}

// One wave per coefficient k; lanes own primes (slot i = lane + 64 r) with the
// shifted residues u_i = c_k + H mod p_i, H = (M-1)/2, so that Y = c_k + H lies
// in [0, M) and c_k = Y - H is the symmetric residue.
//
// Direct form: with M_i = M / p_i and t_i = u_i (M_i^{-1} mod p_i),
//   Y = sum_i t_i M_i - q M,  q = floor(sum_i t_i / p_i).
// q is found from 32-bit fixed-point parts f_i = floor(t_i floor(2^64/p_i) / 2^32),
// which undershoot t_i 2^32 / p_i by less than 2 each: q = floor(sum f_i / 2^32)
// whenever the fraction of that sum is below 2^32 - 2 np.  Otherwise (rare)
// the wave computes Y by Garner's mixed-radix digits instead: digit v_j is
// formed in lane j and broadcast, every lane i > j adds v_j (prod_{l<j} p_l
// mod p_i), and Y = sum_j v_j prod_{l<j} p_l.
// The output Z = Y - H mod 2^(32 L_out) is formed by crt_radix with
// init = 2^(32 L_out) - H (+ q (2^(32 L_out) - M) in the direct form).
template <int NS>
__device__ inline void crt_one(const DevProblem& P, int k_raw, const uint32_t* mi, int mstride, uint32_t* wb,
                               const uint32_t* ures, const uint32_t* pconst) {
  const int lane = threadIdx.x & 63;
  const bool valid = k_raw <= P.D;
  const int k = valid ? k_raw : P.D;
  const int np = P.np;
  const int L = P.L_out;
  uint32_t* vbuf = wb;
  uint32_t* sb = wb + 64 * NS;
  uint32_t* sc = sb + 64 * NS + 2;
  const uint32_t* cp = pconst;               // p
  const uint32_t* cpinv = pconst + np;       // -p^{-1} mod 2^32
  const uint32_t* cinvm = pconst + 2 * np;   // Garner inverse (Montgomery)
  const uint32_t* cw = pconst + 3 * np;      // (M / p_i)^{-1} mod p_i (Montgomery)
  const uint32_t* crlo = pconst + 4 * np;    // floor(2^64 / p_i), low word
  const uint32_t* crhi = pconst + 5 * np;    //                    high word

  uint32_t u[NS];
  // f_i < 2^32 split as fa + fb 2^16: both halves summed over up to 512 primes
  // stay below 2^25, so the 32-bit wave sums cannot wrap
  uint32_t fa = 0u, fb = 0u;
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int i = lane + 64 * r;
    u[r] = 0u;
    if (i < np) {
      u[r] = ures[i];
      const uint32_t p = cp[i];
      const uint32_t t = mmul(u[r], cw[i], p, cpinv[i]);
      vbuf[i] = t & 0xFFFFu;  // the halves crt_radix multiplies with
      sb[i] = t >> 16;
      const uint64_t f = static_cast<uint64_t>(t) * crhi[i] + __umulhi(t, crlo[i]);
      fa += static_cast<uint32_t>(f) & 0xFFFFu;
      fb += static_cast<uint32_t>(f >> 16);
    }
  }
  const uint64_t Sf = static_cast<uint64_t>(wave_sum32(fa)) + (static_cast<uint64_t>(wave_sum32(fb)) << 16);
  const uint32_t q = static_cast<uint32_t>(Sf >> 32);
  const bool direct = static_cast<uint32_t>(Sf) < 0xFFFFFFFFu - 2u * static_cast<uint32_t>(np) && !P.crt_garner;
  uint64_t init[NS];
  if (__builtin_amdgcn_readfirstlane(direct ? 1 : 0)) {
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int t = lane + 64 * r;
      init[r] = (t < L) ? static_cast<uint64_t>(P.NH[t]) + static_cast<uint64_t>(q) * P.negM[t] : 0u;
    }
    WaveSync()();
    crt_radix<NS>(P, k, valid, vbuf, mi, mstride, init, sb, sc);
    return;
  }
  // Garner fallback (tables read from global memory)
  uint32_t acc[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) acc[r] = 0u;
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    for (int jj = 0; jj < 64; ++jj) {
      const int j = r * 64 + jj;
      if (j >= np) break;
      const int i0 = lane + 64 * r;
      const uint32_t pr = i0 < np ? cp[i0] : 3u, pir = i0 < np ? cpinv[i0] : 0u;
      const uint32_t im = i0 < np ? cinvm[i0] : 0u;
      const uint32_t vloc = mmul(msubm(u[r], acc[r], pr), im, pr, pir);
      const uint32_t vj = __builtin_amdgcn_readlane(vloc, jj);
      if (lane == 0) {
        vbuf[j] = vj & 0xFFFFu;
        sb[j] = vj >> 16;
      }
#pragma unroll
      for (int rr = r; rr < NS; ++rr) {
        const int i = lane + 64 * rr;
        if (i > j && i < np) {
          const uint32_t tji = P.Tg[static_cast<size_t>(j) * P.tgs + i];
          acc[rr] = maddm(acc[rr], mmul(vj, tji, cp[i], cpinv[i]), cp[i]);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NS; ++r) {
    const int t = lane + 64 * r;
    init[r] = (t < L) ? P.NH[t] : 0u;
  }
  WaveSync()();
  crt_radix<NS>(P, k, valid, vbuf, P.Plimb, P.LP, init, sb, sc);
}

// Coefficient k modulo a prime (cpp: its first chunk's entry).  Whole runs hold
// c_k 2^32, read as its high word.
__device__ __forceinline__ uint32_t coeff_of(const DevProblem& P, const uint64_t* cpp, size_t cstride, int k,
                                             uint32_t p, uint32_t pinv, bool whole) {
  if (whole) return reinterpret_cast<const uint32_t*>(cpp)[1];
  if (P.nchunk == 1) return redc(*cpp, p, pinv);
  const int ch0 = k / P.kchunk;
  uint64_t q[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int ch = ch0 + u < P.nchunk ? ch0 + u : P.nchunk - 1;
    q[u] = cpp[ch * cstride];
  }
  uint64_t cs = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (ch0 + u < P.nchunk) cs = add_fold(cs, q[u], p);
  for (int ch = ch0 + 8; ch < P.nchunk; ++ch) cs = add_fold(cs, cpp[ch * cstride], p);
  return redc(cs, p, pinv);
}

// One item: kCrtBlockCoeffs coefficients, `cpw` per wave,
// k = (blk * waves + wave) * cpw + c (waves * cpw = kCrtBlockCoeffs).  With
// `fresh` the per-prime constants and (when it fits) the M / p_j limb table
// are staged in LDS first; a block that takes several items of one problem
// in a row (the staged launch) stages them once.  The residues u_i of the
// item's coefficients are summed from the basis-change partial sums, with the
// block's threads reading kCrtBlockCoeffs consecutive coefficients of one
// prime together.
constexpr int kCrtItemsPerBlock = 4;  // items per block of the staged launch, from 1024 items on
template <int NS>
__device__ inline void stage_crt(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds,
                                 int cpw, bool fresh, bool whole) {
  const int nw = blockDim.x >> 6;
  const int wave = threadIdx.x >> 6;
  const int np = P.np;
  const bool staged_mi = crt_stage_mi(P, NS, nw);
  const int L = P.L_out;
  uint32_t* mis = lds;
  uint32_t* wbase = lds + (staged_mi ? np * L : 0);
  uint32_t* wb = wbase + wave * crt_wave_words(NS);
  uint32_t* ures = wbase + nw * crt_wave_words(NS);  // [kCrtBlockCoeffs][np]
  uint32_t* pconst = ures + kCrtBlockCoeffs * np;     // [kCrtConsts][np]
  const size_t cstride = static_cast<size_t>(np) * (P.D + 1);
  const int kbase = w.blk * kCrtBlockCoeffs;
  if (fresh && staged_mi)
    block_stage(mis, np * L, [&](int t) {
      const int j = t / L, l = t - j * L;
      return P.Mi[static_cast<size_t>(j) * L + l];
    });
  {
    for (int t = threadIdx.x; t < np * kCrtBlockCoeffs; t += blockDim.x) {
      const int i = t / kCrtBlockCoeffs, c = t - i * kCrtBlockCoeffs;
      const int k = (kbase + c <= P.D) ? kbase + c : P.D;
      const uint64_t* cpp = P.cpart + static_cast<size_t>(i) * (P.D + 1) + k;
      const PrimeConst pc = T.pc[P.pidx[i]];
      ures[c * np + i] = maddm(coeff_of(P, cpp, cstride, k, pc.p, pc.pinv, whole), P.Hm[i], pc.p);
      if (c == 0 && fresh) {
        pconst[i] = pc.p;
        pconst[np + i] = pc.pinv;
        pconst[2 * np + i] = P.invM[i];
        pconst[3 * np + i] = P.wdir[i];
        pconst[4 * np + i] = P.rinv[2 * i];
        pconst[5 * np + i] = P.rinv[2 * i + 1];
      }
    }
    __syncthreads();
    // two calls rather than one with a selected pointer: with the table in
    // LDS the compiler then reads it with LDS instructions, not flat loads
    for (int c = 0; c < cpw; ++c) {
      const int local = wave * cpw + c;
      if (staged_mi)
        crt_one<NS>(P, kbase + local, mis, L, wb, ures + local * np, pconst);
      else
        crt_one<NS>(P, kbase + local, P.Mi, L, wb, ures + local * np, pconst);
    }
  }
}

// ---------------------------------------------------- CRT on the matrix cores
// The direct form Y = sum_i t_i M_i - q M of the per-lane-slot path (up to
// kSlotCrtPrimes primes), with the limb sums as matrix products: coefficients x
// primes times primes x limbs.  t_i < p_i splits into four balanced base-256
// digits, and so does each 32-bit limb of M_i once the number is written with
// signed limbs: adding 0x80808080 to every limb (with carries) and flipping the
// top bit of each byte gives digits in -128..127 whose value is M_i exactly
// (CrtConst::dig, in operand order).  The seven anti-diagonal sums stay below
// 4 * 512 * 2^14 = 2^25, so
//   V_l = A_l + 2^32 B_l,  A_l = D_0 + .. + 2^24 D_3,  B_l = D_4 + .. + 2^16 D_6
// are 64-bit signed numbers, and one lane per coefficient walks the limbs with
// a signed carry: limb l is the low word of A_l + B_{l-1} + NH_l + q negM_l +
// carry.  Against one wave per coefficient with two multiply-adds per (prime,
// limb) and ballots for the carries (725 instructions per coefficient on the
// batch workload): 191 -> 63 us on 256 pairs, 137 -> 48 on 64 requests of
// degrees 8..48, 259 -> 44 on 10 pairs of degree 9 with 2^512 coefficients.
//
// An item is 16 coefficients of a problem.  One wave takes it whole, 16 limbs per
// step; with NW = 4 (few items) four waves share the primes of the t digits and
// take 64 limbs per step, and the first walks their carries.
//
// Quotient: q is floor(sum f / 2^32) or one more (the f_i undershoot); a wave
// with an undecided coefficient first walks the limbs of Y0 - M with no output,
// whose final carry is its sign.
constexpr int kCrtMmRows = 16;
// Fewer items than four per SIMD: four waves each (10 pairs of degree 9 with
// 2^512 coefficients, 60 items of 310 primes: 43.5 against 112 us; the
// degree-24 pair 8.9 against 16.2; 60 pairs of the batch workload, about 1300
// items: 25.9 against 38).  At 2900 items they tie (47.5, 49.4); from 5600 on
// one wave each is faster (62.8 against 68.0 on 256 pairs).
constexpr int kCrtMmSplitItems = 4096;
constexpr int kCrtMmSums = 16 * 17;  // [limb][row], odd row count of 8-byte words
__host__ __device__ inline int crt_mm_lds_words(int np, int nw) {
  return (np + 63) / 64 * 64 * kCrtMmRows + 4 * kCrtMmSums * nw;
}

// Word of digit d, row r and the 4 primes 4 w .. 4 w + 3 of a 64-prime chunk:
// 64-byte rows of four 16-byte units, the units of a row permuted so that
// neither the word stores down the rows nor the 16-byte operand reads collide
// in a bank.
__device__ __forceinline__ int crt_mm_word(int d, int r, int w) {
  return (d * kCrtMmRows + r) * 16 + (((w >> 2) ^ ((r >> 2) & 3)) << 2) + (w & 3);
}

template <int NW>
__device__ inline void stage_crt_mm(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds,
                                    bool whole) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15, q4 = lane >> 4;
  const int np = P.np, L = P.L_out, nkc = (np + 63) / 64;
  auto sync = [] {
    if constexpr (NW > 1) __syncthreads();
    else WaveSync()();
  };
  uint32_t* tdig = lds;
  int64_t* sumA = reinterpret_cast<int64_t*>(tdig + nkc * 64 * kCrtMmRows);  // [limb of the step][row]
  int64_t* sumB = sumA + kCrtMmSums * NW;
  const int kbase = w.blk * kCrtMmRows;
  const size_t cstride = static_cast<size_t>(np) * (P.D + 1);

  // t_i and the fixed-point parts: lane = (coefficient row, every fourth quad of primes)
  const int k = (kbase + row <= P.D) ? kbase + row : P.D;
  uint64_t f = 0;
  for (int quad = q4 + 4 * wave; quad < nkc * 16; quad += 4 * NW) {
    int32_t t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * quad + e;
      t[e] = 0;
      if (i < np) {
        const PrimeConst pc = T.pc[P.pidx[i]];
        const uint64_t* cpp = P.cpart + static_cast<size_t>(i) * (P.D + 1) + k;
        const uint32_t u = maddm(coeff_of(P, cpp, cstride, k, pc.p, pc.pinv, whole), P.Hm[i], pc.p);
        const uint32_t tv = mmul(u, P.wdir[i], pc.p, pc.pinv);
        f += static_cast<uint64_t>(tv) * P.rinv[2 * i + 1] + __umulhi(tv, P.rinv[2 * i]);
        t[e] = static_cast<int32_t>(tv);
      }
    }
    uint32_t o[kEvDigits];
    digits4(t[0], t[1], t[2], t[3], o);
#pragma unroll
    for (int d = 0; d < kEvDigits; ++d) tdig[(quad >> 4) * 64 * kCrtMmRows + crt_mm_word(d, row, quad & 15)] = o[d];
  }
  f += static_cast<uint64_t>(__shfl_xor(static_cast<long long>(f), 16, 64));
  f += static_cast<uint64_t>(__shfl_xor(static_cast<long long>(f), 32, 64));
  if constexpr (NW > 1) {  // the waves' parts
    uint64_t* fp = reinterpret_cast<uint64_t*>(sumA);
    if (lane < kCrtMmRows) fp[16 * wave + lane] = f;
    __syncthreads();
    f = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) f += fp[16 * v + row];
  }
  uint32_t q = static_cast<uint32_t>(f >> 32);  // of coefficient row `row`, in its four lanes of every wave
  const bool undecided = static_cast<uint32_t>(f) >= 0xFFFFFFFFu - 2u * static_cast<uint32_t>(np);
  sync();

  const ev_v4i* md = reinterpret_cast<const ev_v4i*>(P.Mdig) + row;
  const int nq = (np + 15) / 16;  // groups of 16 primes
  auto load_b = [&](int u, ev_v4i (&B)[kEvDigits]) {  // u = limb tile * nkc + chunk
    const int lt = u / nkc, qu = 4 * (u - lt * nkc) + q4;
    const int at = lt * nq + (qu < nq ? qu : nq - 1);  // beyond the last prime: any digits, the t digits are zero
#pragma unroll
    for (int d = 0; d < kEvDigits; ++d) B[d] = md[(at * kEvDigits + d) * 16];
  };
  const int ntile = (L + 15) / 16;
  for (int pass = __ballot(undecided) ? 0 : 1; pass < 2; ++pass) {  // block-uniform
    int64_t carry = 0, lastB = 0;
    int32_t qr[4];  // multiplier of M for the lane's four output rows
#pragma unroll
    for (int r = 0; r < 4; ++r) qr[r] = __shfl(static_cast<int>(q), 4 * q4 + r, 64) + (pass == 0 ? 1 : 0);
    ev_v4i nx[kEvDigits];
    if (wave < ntile) load_b(wave * nkc, nx);
    for (int t0 = 0; t0 < ntile; t0 += NW) {
      const int tile = t0 + wave;
      const int l = 16 * tile + row;  // the lane's limb (output column)
      const int64_t nm = l < L ? static_cast<int64_t>(P.negM[l]) : 0;
      const int64_t nh = l < L && pass ? static_cast<int64_t>(P.NH[l]) : 0;
      ev_v4i S[2 * kEvDigits - 1];
#pragma unroll
      for (int s = 0; s < 2 * kEvDigits - 1; ++s) S[s] = ev_v4i{0, 0, 0, 0};
      if (tile < ntile)
        for (int kc = 0; kc < nkc; ++kc) {
          ev_v4i A[kEvDigits], B[kEvDigits];
#pragma unroll
          for (int d = 0; d < kEvDigits; ++d) B[d] = nx[d];
          const int u = kc + 1 < nkc ? tile * nkc + kc + 1 : (tile + NW) * nkc;
          if (u < ntile * nkc) load_b(u, nx);
#pragma unroll
          for (int d = 0; d < kEvDigits; ++d)
            A[d] = *reinterpret_cast<const ev_v4i*>(tdig + kc * 64 * kCrtMmRows + crt_mm_word(d, row, 4 * q4));
          digit_products(A, B, S);
        }
      sync();  // the previous step's sums are consumed
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = (16 * wave + row) * 17 + 4 * q4 + r;
        sumA[at] = smad(S[3][r], 1 << 24, smad(S[2][r], 1 << 16, smad(S[1][r], 1 << 8, S[0][r]))) + nh + qr[r] * nm;
        sumB[at] = smad(S[6][r], 1 << 16, smad(S[5][r], 1 << 8, S[4][r]));
      }
      sync();
      if (threadIdx.x < kCrtMmRows) {
        uint32_t* dst = P.out + static_cast<size_t>(kbase + lane) * L + 16 * t0;
        const bool put = pass == 1 && kbase + lane <= P.D;
        for (int v = 0; v < NW && t0 + v < ntile; ++v) {
          const int n = L - 16 * (t0 + v) < 16 ? L - 16 * (t0 + v) : 16;
          int64_t a[16], b[16];
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            a[j] = sumA[(16 * v + j) * 17 + lane];
            b[j] = sumB[(16 * v + j) * 17 + lane];
          }
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            if (j < n) {
              const int64_t s = a[j] + lastB + carry;
              lastB = b[j];
              carry = s >> 32;
              if (put) dst[16 * v + j] = static_cast<uint32_t>(s);
            }
          }
        }
      }
    }
    // Y0 - M = sum_l (..) 2^(32 l) - (q + 1) 2^(32 L): its sign is that of the carry out less q + 1
    if (pass == 0) {
      if (carry + lastB >= static_cast<int64_t>(q) + 1) q += 1u;  // lanes 0..15 of the first wave
      if constexpr (NW > 1) {
        __syncthreads();
        if (threadIdx.x < kCrtMmRows) sumA[lane] = q;
        __syncthreads();
        q = static_cast<uint32_t>(sumA[row]);
      } else {
        q = static_cast<uint32_t>(__shfl(static_cast<int>(q), row, 64));
      }
    }
  }
}

// ------------------------------------------------------------------ wide CRT
// Problems with more primes than the per-lane slots cover.  The same direct
// form Y = sum_i t_i M_i - q M (M_i = M / p_i, t_i = u_i M_i^{-1} mod p_i) in
// three passes over device memory:
//   1. per coefficient k: t_{k,i} for every prime, and the quotient estimate
//      q_k = floor(sum_i f_{k,i} / 2^32) from the fixed-point parts, which is
//      the true quotient or one short of it (each f undershoots by < 2);
//   2. the integer contraction S[k][h] = sum_i t_{k,i} m_{i,h} over 16-bit
//      halves m_{i,h} of the M_i limbs (each term < 2^47, so 4096 primes sum
//      below 2^59 without carries), tiled 16 coefficients x 256 limbs;
//   3. one wave per coefficient: Y0 = sum_h S[k][h] 2^(16 h) + q_k (2^(32 Lw) - M)
//      mod 2^(32 Lw), which lies in [0, 2M) (Lw = L_out + 1 limbs hold it),
//      compared with M; the output is Y0 - H (- M when Y0 >= M) mod 2^(32 L_out).
constexpr int kWideTCoeffs = 8;    // coefficients per block of pass 1 (256 threads)
constexpr int kWideKT = 16;        // coefficients per block of pass 2
constexpr int kWideHT = 256;       // limbs per block of pass 2 (one per thread)
constexpr int kWideChunk = 64;     // primes per LDS chunk of pass 2
constexpr int kWideDigits = 4;     // base-256 digits of t and of the M_i limbs (matrix-core pass 2)
constexpr uint32_t kWideOffset = 0x80808080u;  // a limb's digits in -128..127 are those of the limb less this

__host__ __device__ inline int wide_t_lds_words() { return 4 * 4 * kWideTCoeffs; }
__host__ __device__ inline int wide_sum_lds_words() { return kWideChunk * kWideKT; }
__host__ __device__ inline int wide_fin_lds_words(const DevProblem& P) { return P.Lw; }

// Carry into this lane when every lane adds its `gen` (carry out of its own
// limb) and passes an incoming carry on when `prop` (limb all ones); `cin` is
// the carry into lane 0 and becomes the carry out of lane 63.
__device__ inline uint32_t wave_carry_in(bool gen, bool prop, uint64_t* cin) {
  const int lane = threadIdx.x & 63;
  const uint64_t G = __ballot(gen);
  const uint64_t X = G | __ballot(prop);
  const unsigned __int128 tot = static_cast<unsigned __int128>(X) + G + *cin;
  const uint64_t C = static_cast<uint64_t>(tot) ^ X ^ G;
  *cin = static_cast<uint64_t>(tot >> 64);
  return static_cast<uint32_t>((C >> lane) & 1u);
}

// Pass 1: block item blk covers coefficients blk*8 .. blk*8+7; thread owns
// coefficient c = tid mod 8 and primes tid/8 + 32 r, kWideTPrimes of them at a
// time: a prime's constants are three dependent loads, which bound the pass (ten
// resultants of degree 225 over 2025 primes: one prime at a time 99 us, four 59, eight 55).
constexpr int kWideTPrimes = 8;
__device__ inline void stage_crt_wide_t(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* lds,
                                        bool whole) {
  const int c = threadIdx.x & (kWideTCoeffs - 1);
  const int k_raw = w.blk * kWideTCoeffs + c;
  const bool valid = k_raw <= P.D;
  const int k = valid ? k_raw : P.D;
  const int np = P.np;
  const size_t cstride = static_cast<size_t>(np) * (P.D + 1);
  uint32_t fa = 0u, fb = 0u;  // 16-bit halves of the f parts, summed
  uint32_t ta = 0u, tb = 0u;  // and of the t
  const int step = blockDim.x / kWideTCoeffs;
  for (int i0 = threadIdx.x / kWideTCoeffs; i0 < np; i0 += kWideTPrimes * step) {
    uint32_t t[kWideTPrimes];
    uint64_t f[kWideTPrimes];
#pragma unroll
    for (int v = 0; v < kWideTPrimes; ++v) {
      const int i = min(i0 + v * step, np - 1);
      const uint64_t* cpp = P.cpart + static_cast<size_t>(i) * (P.D + 1) + k;
      const PrimeConst pc = T.pc[P.pidx[i]];
      const uint32_t u = maddm(coeff_of(P, cpp, cstride, k, pc.p, pc.pinv, whole), P.Hm[i], pc.p);  // c_k + H mod p
      t[v] = mmul(u, P.wdir[i], pc.p, pc.pinv);
      f[v] = static_cast<uint64_t>(t[v]) * P.rinv[2 * i + 1] + __umulhi(t[v], P.rinv[2 * i]);
    }
#pragma unroll
    for (int v = 0; v < kWideTPrimes; ++v) {
      const int i = i0 + v * step;
      if (i >= np) break;
      if (valid) P.wT[static_cast<size_t>(k) * P.wnpad + i] = t[v];
      fa += static_cast<uint32_t>(f[v]) & 0xFFFFu;
      fb += static_cast<uint32_t>(f[v] >> 16);
      ta += t[v] & 0xFFFFu;
      tb += t[v] >> 16;
    }
  }
  // lanes of one coefficient differ in lane bits 3..5
#pragma unroll
  for (int m = kWideTCoeffs; m < 64; m <<= 1) {
    fa += static_cast<uint32_t>(__shfl_xor(static_cast<int>(fa), m, 64));
    fb += static_cast<uint32_t>(__shfl_xor(static_cast<int>(fb), m, 64));
    ta += static_cast<uint32_t>(__shfl_xor(static_cast<int>(ta), m, 64));
    tb += static_cast<uint32_t>(__shfl_xor(static_cast<int>(tb), m, 64));
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  if (lane < kWideTCoeffs) {
    uint32_t* at = lds + wave * 4 * kWideTCoeffs + lane;
    at[0] = fa;
    at[kWideTCoeffs] = fb;
    at[2 * kWideTCoeffs] = ta;
    at[3 * kWideTCoeffs] = tb;
  }
  __syncthreads();
  if (threadIdx.x < kWideTCoeffs && valid) {
    uint64_t sa = 0, sb = 0, ua = 0, ub = 0;
    for (int v = 0; v < nw; ++v) {
      const uint32_t* at = lds + v * 4 * kWideTCoeffs + c;
      sa += at[0];
      sb += at[kWideTCoeffs];
      ua += at[2 * kWideTCoeffs];
      ub += at[3 * kWideTCoeffs];
    }
    P.wq[k] = static_cast<uint32_t>((sa + (sb << 16)) >> 32);
    if (P.wide_mfma) P.wsum[k] = ua + (ub << 16);
  }
}

// Pass 2: item (blk = coefficient tile, sub = limb tile); the block's t values
// for 64 primes at a time are staged in LDS as [prime][coefficient] (read
// back as broadcasts); each thread streams one limb column of the M_i table
// and splits it into its two 16-bit halves, so every t value feeds two
// multiply-adds.  Loads go out a group of 8 primes ahead of their use, from
// clamped (always valid) addresses.
__device__ inline void stage_crt_wide_sum(const DevProblem& P, const WorkItem& w, uint32_t* lds) {
  constexpr int G = 8;
  const int np = P.np, Lw = P.Lw, nh = 2 * Lw;
  const int k0 = w.blk * kWideKT;
  const int t = w.sub * kWideHT + static_cast<int>(threadIdx.x);
  const bool tv_ok = t < Lw;
  const uint32_t* Mcol = P.Mi + (tv_ok ? t : Lw - 1);
  uint64_t alo[kWideKT], ahi[kWideKT];
#pragma unroll
  for (int c = 0; c < kWideKT; ++c) alo[c] = ahi[c] = 0u;
  // no masks needed: the staged t values are zero beyond the last prime, and
  // lanes beyond the last limb store nothing
  auto load_group = [&](int ibase, uint32_t* m) {
#pragma unroll
    for (int u = 0; u < G; ++u) m[u] = Mcol[static_cast<size_t>(min(ibase + u, np - 1)) * Lw];
  };
  uint32_t mcur[G], mnext[G];
  load_group(0, mcur);
  for (int i0 = 0; i0 < np; i0 += kWideChunk) {
    __syncthreads();  // the previous chunk is consumed
    for (int e = threadIdx.x; e < kWideChunk * kWideKT; e += blockDim.x) {
      const int c = e / kWideChunk, ii = e - c * kWideChunk;  // coalesced along the primes of one row
      const int i = i0 + ii, k = k0 + c;
      lds[ii * kWideKT + c] = (i < np && k <= P.D) ? P.wT[static_cast<size_t>(k) * P.wnpad + i] : 0u;
    }
    __syncthreads();
    const int n = min(kWideChunk, np - i0);
    for (int ii = 0; ii < n; ii += G) {
      load_group(i0 + ii + G, mnext);  // beyond np: clamped (their t values are zero)
      __builtin_amdgcn_sched_barrier(0);  // issue them before this group's arithmetic
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const uint32_t lo = mcur[u] & 0xFFFFu, hi = mcur[u] >> 16;
        const uint4* tv = reinterpret_cast<const uint4*>(lds + (ii + u) * kWideKT);
#pragma unroll
        for (int q4 = 0; q4 < kWideKT / 4; ++q4) {
          const uint4 t4 = tv[q4];
          alo[4 * q4 + 0] += static_cast<uint64_t>(t4.x) * lo;
          ahi[4 * q4 + 0] += static_cast<uint64_t>(t4.x) * hi;
          alo[4 * q4 + 1] += static_cast<uint64_t>(t4.y) * lo;
          ahi[4 * q4 + 1] += static_cast<uint64_t>(t4.y) * hi;
          alo[4 * q4 + 2] += static_cast<uint64_t>(t4.z) * lo;
          ahi[4 * q4 + 2] += static_cast<uint64_t>(t4.z) * hi;
          alo[4 * q4 + 3] += static_cast<uint64_t>(t4.w) * lo;
          ahi[4 * q4 + 3] += static_cast<uint64_t>(t4.w) * hi;
        }
      }
#pragma unroll
      for (int u = 0; u < G; ++u) mcur[u] = mnext[u];
    }
  }
  if (tv_ok)
#pragma unroll
    for (int c = 0; c < kWideKT; ++c)
      if (k0 + c <= P.D) {  // column sum of limb t: alo + ahi 2^16 (< 2^76) as (low, high) words
        const unsigned __int128 v = static_cast<unsigned __int128>(alo[c]) + (static_cast<unsigned __int128>(ahi[c]) << 16);
        uint64_t* dst = P.wS + static_cast<size_t>(k0 + c) * nh + 2 * t;
        dst[0] = static_cast<uint64_t>(v);
        dst[1] = static_cast<uint64_t>(v >> 64);
      }
}

// Pass 2 on the matrix cores, in base-256 digits of -128..127: t < 2^31 has four
// (t = sum_a t_a 2^(8a)), and so has a limb less kWideOffset (its bytes with the
// top bit flipped, no carry to the next limb), whose products fall short of the
// column sum by kWideOffset sum_i t_i, added at the end from pass 1's sum of the
// t.  The int8 MFMA (16 x 16 outputs, 64 primes per step) accumulates
// sum_i t_a m_b in int32 per anti-diagonal s = a + b: at most 4 * 2^14 * 4096 =
// 2^28 for 4096 primes, exact.  Sixteen products a step; five 7-bit digits,
// which need no offset, take 25 (ten
// resultants of degree 225 over 2025 primes: 289 -> 215 us).  The column sum is
// below 2^85.  The limb digits are planes Md[b][t][i] (a limb's primes
// contiguous); the block stages its 32 limbs x 64 primes x 4 digits in LDS once
// per step for its four waves.  The t values come from wT (beyond the last prime it
// holds anything, which meets the zero digits that stage_wide_digits writes there)
// and are split into digits in registers.  Wave w takes coefficients
// k0 + 16 w ... (one 16-row tile) and the block's 32 limbs (two 16-column
// tiles); a lane holds row r of A and column r of B for the 16 primes of its
// quarter kg (any fixed assignment of primes to the K slots serves, as long
// as A and B use the same one).
constexpr int kWideMfmaK = 64;   // primes per MFMA step (planes padded to a multiple)
constexpr int kWideMfmaKT = 64;  // coefficients per block (four waves)
constexpr int kWideMfmaTT = 32;  // limbs per block
__host__ __device__ inline int wide_mfma_lds_words() { return kWideDigits * kWideMfmaTT * kWideMfmaK / 4; }
typedef int wide_v4i __attribute__((ext_vector_type(4)));

// The digit planes Md[b][t][i] of M_i = M / p_i, from the limbs of M alone: item
// (problem, blk = 64 primes, sub = 64 limbs).  Limb t of an exact quotient comes
// from limb t of M and the borrow into it,
//   q = (m_t - b) / p mod 2^32,  b' = (q p - (m_t - b)) / 2^32,
// and the borrow into the block's first limb t0 is -(M mod 2^(32 t0)) 2^(-32 t0)
// mod p: a reduction chain over the limbs below, a quarter of them per wave (a
// lane per prime), joined by the power 2^(-8 t0).  So every block starts by
// itself, and the M_i, np times as long as M, are neither uploaded nor stored.
// Wave 0 then walks the block's 64 limbs, and the digits go out as 16-byte
// words of 16 primes: zero beyond the last prime, which the contraction relies on (it
// reads t values there that nothing writes); those beyond the last limb are not used.
// Bound by the chains'
// latency, 27 us for 2025 primes and 1925 limbs; as a transposition of uploaded
// M_i it took 19 us, behind 0.55 ms for their 15.6 MB (image and transfer).
constexpr int kWideDigitLimbs = 64;
__host__ __device__ inline int wide_digits_lds_words(const DevProblem& P) {
  return P.wlpad + kWideDigitLimbs + kWideMfmaK * (kWideDigitLimbs + 1) + 4 * kWideMfmaK;
}
__device__ inline void stage_wide_digits(const DevProblem& P, const DevTables& T, const WorkItem& w, uint32_t* smem) {
  const int i0 = w.blk * kWideMfmaK, t0 = w.sub * kWideDigitLimbs;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* lds = smem;                                             // [prime][limb]
  uint32_t* part = lds + kWideMfmaK * (kWideDigitLimbs + 1);        // [quarter][prime]
  uint32_t* m32 = part + 4 * kWideMfmaK;                            // limbs of M, zero above
  for (int t = threadIdx.x; t < t0 + kWideDigitLimbs; t += blockDim.x) m32[t] = t < P.Lw ? P.Mw[t] : 0u;
  __syncthreads();
  const bool on = i0 + lane < P.np;
  const PrimeConst pc = T.pc[P.pidx[on ? i0 + lane : 0]];
  const uint32_t p = pc.p, pinv = pc.pinv;
  const int len = t0 / 4;
  {
    uint32_t r = 0;  // at most p + 1 between limbs
    const uint32_t* seg = m32 + wave * len;
#pragma unroll 4
    for (int t = 0; t < len; ++t) {
      const uint64_t x = static_cast<uint64_t>(r) + seg[t];
      r = static_cast<uint32_t>((x + static_cast<uint64_t>(static_cast<uint32_t>(x) * pinv) * p) >> 32);
    }
    part[wave * kWideMfmaK + lane] = r >= p ? r - p : r;
  }
  __syncthreads();
  if (wave == 0) {
    const uint32_t f = mpow(1u, static_cast<uint32_t>(len), pc.r1, p, pinv);  // 2^(-32 len), Montgomery form
    uint32_t r = part[lane];
#pragma unroll
    for (int j = 1; j < 4; ++j) {
      r = mmul(r, f, p, pinv) + part[j * kWideMfmaK + lane];
      r = r >= p ? r - p : r;
    }
    uint32_t b = r ? p - r : 0u;
    const uint32_t pi = 0u - pinv;  // 1 / p mod 2^32
#pragma unroll 4
    for (int t = 0; t < kWideDigitLimbs; ++t) {
      const uint32_t m = m32[t0 + t], q = (m - b) * pi;
      b = static_cast<uint32_t>((static_cast<uint64_t>(q) * p) >> 32) + (m < b ? 1u : 0u);
      lds[lane * (kWideDigitLimbs + 1) + t] = on ? q ^ kWideOffset : 0u;
    }
  }
  __syncthreads();
  const size_t plane = static_cast<size_t>(P.wlpad) * P.wnpad;
  const int q = threadIdx.x & 3, tt = threadIdx.x >> 2;  // 16 primes of one limb, every digit
  if (t0 + tt >= P.wlpad) return;
  uint32_t dg[4][kWideDigits];  // [4 primes][digit]
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t* m = lds + (16 * q + 4 * v) * (kWideDigitLimbs + 1) + tt;
    byte_transpose4(m[0], m[kWideDigitLimbs + 1], m[2 * (kWideDigitLimbs + 1)], m[3 * (kWideDigitLimbs + 1)], dg[v]);
  }
  int8_t* dst = P.wMd + static_cast<size_t>(t0 + tt) * P.wnpad + i0 + 16 * q;
#pragma unroll
  for (int d = 0; d < kWideDigits; ++d)
    *reinterpret_cast<uint4*>(dst + d * plane) = make_uint4(dg[0][d], dg[1][d], dg[2][d], dg[3][d]);
}

__device__ inline void stage_crt_wide_sum_mfma(const DevProblem& P, const WorkItem& w, uint32_t* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int Lw = P.Lw, nh = 2 * Lw;
  const int k0 = w.blk * kWideMfmaKT + 16 * wave;  // this wave's coefficient tile
  const int t0 = w.sub * kWideMfmaTT;
  const int r = lane & 15, kg = lane >> 4;
  const size_t mplane = static_cast<size_t>(P.wlpad) * P.wnpad;
  const uint32_t* trow = P.wT + static_cast<size_t>(k0 + r) * P.wnpad + 16 * kg;
  uint4* bl = reinterpret_cast<uint4*>(lds);  // [digit][limb][prime quarter]
  wide_v4i acc[2][2 * kWideDigits - 1];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int d = 0; d < 2 * kWideDigits - 1; ++d) acc[u][d] = wide_v4i{0, 0, 0, 0};
  for (int i0 = 0; i0 < P.wnpad; i0 += kWideMfmaK) {
    __syncthreads();  // the previous step's tile is consumed
    for (int e = threadIdx.x; e < kWideDigits * kWideMfmaTT * 4; e += blockDim.x) {
      const int d = e / (kWideMfmaTT * 4), rem = e - d * (kWideMfmaTT * 4), tl = rem >> 2, q = rem & 3;
      bl[e] = *reinterpret_cast<const uint4*>(P.wMd + d * mplane + static_cast<size_t>(t0 + tl) * P.wnpad + i0 + 16 * q);
    }
    // the wave's A: 16 t values, split into digit bytes
    uint32_t tv[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 v = *reinterpret_cast<const uint4*>(trow + i0 + 4 * q);
      tv[4 * q] = v.x;
      tv[4 * q + 1] = v.y;
      tv[4 * q + 2] = v.z;
      tv[4 * q + 3] = v.w;
    }
    wide_v4i a[kWideDigits];
#pragma unroll
    for (int wd = 0; wd < 4; ++wd) {
      uint32_t o[kWideDigits];
      digits4(static_cast<int32_t>(tv[4 * wd]), static_cast<int32_t>(tv[4 * wd + 1]),
              static_cast<int32_t>(tv[4 * wd + 2]), static_cast<int32_t>(tv[4 * wd + 3]), o);
#pragma unroll
      for (int d = 0; d < kWideDigits; ++d) a[d][wd] = static_cast<int>(o[d]);
    }
    __syncthreads();
#pragma unroll
    for (int db = 0; db < kWideDigits; ++db) {
      const wide_v4i b0 = *reinterpret_cast<const wide_v4i*>(&bl[(db * kWideMfmaTT + r) * 4 + kg]);
      const wide_v4i b1 = *reinterpret_cast<const wide_v4i*>(&bl[(db * kWideMfmaTT + 16 + r) * 4 + kg]);
#pragma unroll
      for (int da = 0; da < kWideDigits; ++da) {
        acc[0][da + db] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[da], b0, acc[0][da + db], 0, 0, 0);
        acc[1][da + db] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[da], b1, acc[1][da + db], 0, 0, 0);
      }
    }
  }
  // lane holds rows 4 kg + e (coefficients) of column r (limb) of each tile
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int t = t0 + 16 * u + r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + 4 * kg + e;
      if (k <= P.D && t < Lw) {
        __int128 v = static_cast<__int128>(P.wsum[k]) * kWideOffset;
#pragma unroll
        for (int d = 0; d < 2 * kWideDigits - 1; ++d) v += static_cast<__int128>(acc[u][d][e]) * (1ll << (8 * d));
        uint64_t* dst = P.wS + static_cast<size_t>(k) * nh + 2 * t;
        dst[0] = static_cast<uint64_t>(v);
        dst[1] = static_cast<uint64_t>(v >> 64);
      }
    }
  }
}

// Pass 3: one wave (the whole block) per coefficient k = blk.
__device__ inline void stage_crt_wide_fin(const DevProblem& P, const WorkItem& w, uint32_t* lds) {
  const int lane = threadIdx.x & 63;
  const int k = w.blk;
  const int Lw = P.Lw, L = P.L_out;
  const uint64_t* S = P.wS + static_cast<size_t>(k) * 2 * Lw;
  const uint32_t q = P.wq[k];
  uint32_t* y = lds;
  // Y0 limbs, 64 at a time; V_t = (column sum of limb t) + q negM_t < 2^86 is
  // (lo: 64 bits, hi: 32 bits), and limb t is lo32(V_t) + mid32(V_{t-1}) +
  // hi(V_{t-2}) plus carries; the values of lanes 62 and 63 carry over
  uint32_t pm = 0u, ph1 = 0u, ph2 = 0u, pc1 = 0u;
  uint64_t cin = 0u;
  for (int t0 = 0; t0 < Lw; t0 += 64) {
    const int t = t0 + lane;
    uint64_t lo = 0u;
    uint32_t hi = 0u;
    if (t < Lw) {
      lo = S[2 * t];
      hi = static_cast<uint32_t>(S[2 * t + 1]);
      const uint64_t b = static_cast<uint64_t>(q) * P.negM[t];
      lo += b;
      hi += (lo < b) ? 1u : 0u;
    }
    const uint32_t mid = static_cast<uint32_t>(lo >> 32);
    uint32_t mprev = static_cast<uint32_t>(__shfl_up(static_cast<int>(mid), 1, 64));
    uint32_t hprev2 = static_cast<uint32_t>(__shfl_up(static_cast<int>(hi), 2, 64));
    if (lane == 0) {
      mprev = pm;
      hprev2 = ph2;
    }
    if (lane == 1) hprev2 = ph1;
    const uint64_t s = static_cast<uint64_t>(static_cast<uint32_t>(lo)) + mprev + hprev2;
    const uint32_t l1 = static_cast<uint32_t>(s), h1 = static_cast<uint32_t>(s >> 32);  // h1 <= 2
    uint32_t h1prev = static_cast<uint32_t>(__shfl_up(static_cast<int>(h1), 1, 64));
    if (lane == 0) h1prev = pc1;
    const uint64_t x2 = static_cast<uint64_t>(l1) + h1prev;
    const uint32_t l2 = static_cast<uint32_t>(x2);
    const uint32_t cy = wave_carry_in((x2 >> 32) != 0, l2 == 0xFFFFFFFFu, &cin);
    if (t < Lw) y[t] = l2 + cy;
    pm = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mid), 63));
    ph1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(hi), 63));
    ph2 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(hi), 62));
    pc1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(h1), 63));
  }
  WaveSync()();
  // Y0 >= M ?  (top limbs first; equal counts as >=)
  int ge = 1;
  for (int t0 = ((Lw - 1) / 64) * 64; t0 >= 0; t0 -= 64) {
    const int t = t0 + lane;
    const uint32_t yv = (t < Lw) ? y[t] : 0u, mv = (t < Lw) ? P.Mw[t] : 0u;
    const uint64_t gt = __ballot(yv > mv), lt = __ballot(yv < mv);
    const uint64_t d = gt | lt;
    if (d) {
      const int top = 63 - __clzll(static_cast<long long>(d));
      ge = static_cast<int>((gt >> top) & 1u);
      break;
    }
  }
  // output: Y0 - H (- M) mod 2^(32 L_out)
  const uint32_t* A = ge ? P.NHM : P.NH;
  cin = 0u;
  for (int t0 = 0; t0 < L; t0 += 64) {
    const int t = t0 + lane;
    const uint64_t x = (t < L) ? static_cast<uint64_t>(y[t]) + A[t] : 0u;
    const uint32_t l = static_cast<uint32_t>(x);
    const uint32_t cy = wave_carry_in((x >> 32) != 0, l == 0xFFFFFFFFu && t < L, &cin);
    if (t < L) P.out[static_cast<size_t>(k) * L + t] = l + cy;
  }
}

}  // namespace rsl
