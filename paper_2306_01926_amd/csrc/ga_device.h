// Device helpers shared by the gfx950 kernel files: bf16 conversions, the
// canonical |r|^2 split, the MFMA 32x32x16 scoring of 32 keys against blocks of
// 32 groups with the packed top-2 reduction, and the exact fp64 argmin used for
// keys whose MFMA decision is not certified.  Included inside
// namespace ga { namespace { ... } } by each kernel file.
#pragma once

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
// Round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// Storage-dtype traits: load as float, representative rounding, store.
struct F32 {
  using T = float;
  static constexpr int kBits = 32;
  __device__ static float load(const float* p, int64_t i) { return p[i]; }
  __device__ static float rep(float c) { return c; }
  __device__ static void store(float* p, int64_t i, float r) { p[i] = r; }
};
struct BF16 {
  using T = uint16_t;
  static constexpr int kBits = 16;
  __device__ static float load(const uint16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
  __device__ static float rep(float c) { return bf16_to_f32(f32_to_bf16(c)); }
  __device__ static void store(uint16_t* p, int64_t i, float r) { p[i] = (uint16_t)(__float_as_uint(r) >> 16); }
};

// min / max of finite scores as a median of three with -FLT_MAX / FLT_MAX:
// one v_med3_f32 each, without the NaN canonicalisation fminf / fmaxf need.
__device__ __forceinline__ float min2(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, -FLT_MAX); }
__device__ __forceinline__ float max2(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, FLT_MAX); }

// v_min3_f32 without the NaN canonicalisation the compiler adds around
// fminf-based min3 (the operands are finite scores).  Never an MFMA's result
// itself: the wait states between an MFMA and a VALU read of its registers are
// not kept for inline assembly (the packed scores are VALU results); min3m is
// for those.
__device__ __forceinline__ float min3f(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// v_minimum3_f32 (no NaN canonicalisation either).
__device__ __forceinline__ float min3m(float a, float b, float c) {
  return __builtin_elementwise_minimum(__builtin_elementwise_minimum(a, b), c);
}

__device__ __forceinline__ float readlane_f(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// (value of lane q, value of lane q + 32) in every lane l, q = l % 32.
__device__ __forceinline__ u32x2 halves(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return u32x2{r[0], r[1]};
}

// Lane exchanges by DPP (VALU, no LDS round trip): within 8 lanes as the xors
// 1, 2 and (equal to 4 once the quads agree) the half-row mirror.
template <int CTRL>
__device__ __forceinline__ int dpp(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const long long b = __double_as_longlong(x);
  const uint32_t lo = (uint32_t)dpp<CTRL>((int)(uint32_t)b), hi = (uint32_t)dpp<CTRL>((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

// The largest of the 64 lanes' values, in every lane.
__device__ __forceinline__ float wave_max(float x) {
  x = max2(x, __int_as_float(dpp<kXor1>(__float_as_int(x))));
  x = max2(x, __int_as_float(dpp<kXor2>(__float_as_int(x))));
  x = max2(x, __int_as_float(dpp<kHalfMirror>(__float_as_int(x))));
  x = max2(x, __int_as_float(dpp<kMirror>(__float_as_int(x))));
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = max2(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const u32x2 q = halves(__float_as_uint(x));
  return max2(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// The largest of the 64 lanes' words, in every lane.
__device__ __forceinline__ uint32_t wave_max_bits(uint32_t x) {
  x = max(x, (uint32_t)dpp<kXor1>((int)x));
  x = max(x, (uint32_t)dpp<kXor2>((int)x));
  x = max(x, (uint32_t)dpp<kHalfMirror>((int)x));
  x = max(x, (uint32_t)dpp<kMirror>((int)x));
  const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = max(p[0], p[1]);
  const u32x2 q = halves(x);
  return max(q[0], q[1]);
}

// The smallest of the 64 lanes' scores and its index (the lowest among equals),
// in every lane.
__device__ __forceinline__ void wave_argmin(double& best, int& bj) {
  auto take = [&](double ob, int oj) __attribute__((always_inline)) {
    if (ob < best || (ob == best && oj < bj)) {
      best = ob;
      bj = oj;
    }
  };
  take(dpp<kXor1>(best), dpp<kXor1>(bj));
  take(dpp<kXor2>(best), dpp<kXor2>(bj));
  take(dpp<kHalfMirror>(best), dpp<kHalfMirror>(bj));
  take(dpp<kMirror>(best), dpp<kMirror>(bj));
  auto halves2 = [&](uint32_t lo, uint32_t hi) __attribute__((always_inline)) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
  };
  {
    const long long b = __double_as_longlong(best);
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto u = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    const auto j = __builtin_amdgcn_permlane16_swap((uint32_t)bj, (uint32_t)bj, false, false);
    best = halves2(l[0], u[0]);
    bj = (int)j[0];
    take(halves2(l[1], u[1]), (int)j[1]);
  }
  {
    const long long b = __double_as_longlong(best);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto u = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    const auto j = __builtin_amdgcn_permlane32_swap((uint32_t)bj, (uint32_t)bj, false, false);
    best = halves2(l[0], u[0]);
    bj = (int)j[0];
    take(halves2(l[1], u[1]), (int)j[1]);
  }
}

// |r|^2 of a bf16 row split over the eight lanes 8 k .. 8 k + 7 (rc: this lane's
// eight features), in all of them.  The canonical value is the fp64 fma chain
// over c = 0..63.  Each square of a bf16 number is exact in fp64 (16 significant
// bits); if the nonzero squares of a row span at most 31 binades, every partial
// sum in any order is a multiple of the smallest square's last bit and below
// 2^53 of it, so every partial sum is exact and any summation order gives the
// chain's bits.  False: not provably so, the caller runs the chain.
__device__ __forceinline__ int sq_exp(double x) {  // biased exponent of a square (0 for 0)
  return (int)((__double_as_longlong(x) >> 52) & 2047);
}
__device__ __forceinline__ bool norm8(const double (&rc)[8], double& nrm) {
  double acc = 0.0;
  int emax = 0, emin = 4096;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double q = rc[e] * rc[e];  // exact
    acc += q;
    if (q != 0.0) {
      emax = max(emax, sq_exp(q));
      emin = min(emin, sq_exp(q));
    }
  }
  acc += dpp<kXor1>(acc);
  acc += dpp<kXor2>(acc);
  acc += dpp<kHalfMirror>(acc);
  emax = max(emax, dpp<kXor1>(emax));
  emin = min(emin, dpp<kXor1>(emin));
  emax = max(emax, dpp<kXor2>(emax));
  emin = min(emin, dpp<kXor2>(emin));
  emax = max(emax, dpp<kHalfMirror>(emax));
  emin = min(emin, dpp<kHalfMirror>(emin));
  nrm = acc;
  return emin == 4096 || emax - emin <= 31;
}

// |r|^2 as an fp64 fma chain over c = 0..63 (lane c holds r_c); same value in all lanes.
__device__ double canon_nrm_wave(float r) {
  double acc = 0.0;
#pragma unroll 8
  for (int c = 0; c < 64; ++c) {
    const double rc = (double)readlane_f(r, c);
    acc = fma(rc, rc, acc);
  }
  return acc;
}

// |r|^2 as three bf16 terms hi + mid + lo (each the bf16 rounding of the
// remainder; the two subtractions are exact), |sum - nrm| <= ~2^-24 nrm.  The
// assign kernel adds them to the scores through one extra MFMA k-step.
__device__ void write_nsplit(double nrm, uint16_t* dst) {
  const uint32_t hi = f32_to_bf16((float)nrm);
  const double r1 = nrm - (double)bf16_to_f32(hi);
  const uint32_t mid = f32_to_bf16((float)r1);
  const double r2 = r1 - (double)bf16_to_f32(mid);
  const uint32_t lo = f32_to_bf16((float)r2);
  *(u32x4*)dst = u32x4{hi | (mid << 16), lo, 0u, 0u};
}


// The assign kernel's LDS copy of -2R stores 16-byte chunk c of row r at chunk
// c ^ ((r >> 1) & 7) of a 128-byte row: 16 consecutive rows reading the same
// logical chunk then hit 16 distinct groups of 4 banks (no padding needed).
__device__ __forceinline__ int swz(int r, int c) { return r * 64 + 8 * (c ^ ((r >> 1) & 7)); }

// Exact assignment of NK bf16 keys at once by a whole wave, the
// representatives read from the LDS copy of -2R.  The canonical
// definition (score fma(-2, k.r, |r|^2) with k.r an fp64 fma chain over
// c = 0..63, lowest index among minima): x = -2r is exact in bf16 and every
// partial sum of the chain over k_c x_c is exactly -2 times the one over
// k_c r_c (the partial sums stay far from the fp64 subnormal range), so the
// score is |r|^2 + (chain over k_c x_c) with one rounding.  kd: the keys as
// fp64 rows [NK][64] in LDS (the same words in every lane).  Lane l takes
// groups l, l + 64, l + 128, ... in ascending order, two at a time, and each
// converts its representatives' features once for all NK keys.
template <int NK>
__device__ void exact_argmin_keys(const double* kd, const uint16_t* Rs, const double* __restrict__ nrm, int N,
                                  int* jb) {
  const int lane = threadIdx.x & 63;
  double best[NK];
  int bj[NK];
#pragma unroll
  for (int b = 0; b < NK; ++b) {
    best[b] = INFINITY;
    bj[b] = 0x7fffffff;
  }
  for (int j0 = lane; j0 < N; j0 += 128) {
    const int j1 = j0 + 64;
    const bool two = j1 < N;
    const int j1r = two ? j1 : j0;  // a row that exists
    const double n0 = nrm[j0], n1 = nrm[j1r];  // in flight during the dot products
    double d0[NK], d1[NK];
#pragma unroll
    for (int b = 0; b < NK; ++b) d0[b] = d1[b] = 0.0;
#pragma unroll 2
    for (int i = 0; i < 8; ++i) {
      const u32x4 w0 = *(const u32x4*)(Rs + swz(j0, i)), w1 = *(const u32x4*)(Rs + swz(j1r, i));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double x0 = (double)bf16_to_f32(w0[e] & 0xffffu), y0 = (double)bf16_to_f32(w0[e] >> 16);
        const double x1 = (double)bf16_to_f32(w1[e] & 0xffffu), y1 = (double)bf16_to_f32(w1[e] >> 16);
#pragma unroll
        for (int b = 0; b < NK; ++b) {
          const f64x2 kk = *(const f64x2*)(kd + b * 64 + 8 * i + 2 * e);
          d0[b] = fma(kk[0], x0, d0[b]);
          d0[b] = fma(kk[1], y0, d0[b]);
          d1[b] = fma(kk[0], x1, d1[b]);
          d1[b] = fma(kk[1], y1, d1[b]);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NK; ++b) {
      const double s0 = n0 + d0[b];
      if (s0 < best[b]) {
        best[b] = s0;
        bj[b] = j0;
      }
      const double s1 = n1 + d1[b];
      if (two && s1 < best[b]) {
        best[b] = s1;
        bj[b] = j1;
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NK; ++b) {
    wave_argmin(best[b], bj[b]);
    jb[b] = bj[b];
  }
}

// Scores are ranked as packed floats: the low 4 mantissa bits of a score are
// replaced by its accumulator register index v (0..15), so one min/med3 chain
// keeps value and register of the best two.  The block of the best is tracked
// beside it and the lane half is resolved when the halves merge, so the
// group of a packed best (v, block b, half h) is 32 b + 8 (v/4) + 4 h + v%4.
constexpr uint32_t kPackMask = 15u;

// Top-2 of one block's 16 scores folded into the running (M1, M2, B1 = block
// of M1).  Over quads: with m1 <= m2 the two smallest so far and
// a = min3(m1, x0, x1), the two smallest of {m1, m2, x0, x1, x2, x3} are
// min3(a, x2, x3) and min3(m2, med3(m1, x0, x1), med3(a, x2, x3)).  A packed
// value equal to M1 from a later block keeps the earlier block; such a key is
// never certified (its gap is 0), so the choice does not matter.
__device__ __forceinline__ void reduce_block(const f32x16& acc, int blk, float& M1, float& M2, int& B1) {
  const float prev = M1;
#pragma unroll
  for (int v = 0; v < 16; v += 4) {
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x[e] = __uint_as_float((__float_as_uint(acc[v + e]) & ~kPackMask) | (uint32_t)(v + e));
    const float t01 = __builtin_amdgcn_fmed3f(M1, x[0], x[1]);
    const float a = min3f(M1, x[0], x[1]);
    const float t23 = __builtin_amdgcn_fmed3f(a, x[2], x[3]);
    M1 = min3f(a, x[2], x[3]);
    M2 = min3f(M2, t01, t23);
  }
  B1 = M1 < prev ? blk : B1;
}

// The two smallest of K class minima, ranked as packed floats: the low 3
// mantissa bits are replaced by the class (K <= 8), so one min / med3 chain keeps
// the best's value and class and the second best's value.
constexpr uint32_t kClassMask = 7u;
template <int K>
__device__ __forceinline__ void top2_classes(const float (&m)[K], float& M1, float& M2) {
  float x[K];
#pragma unroll
  for (int k = 0; k < K; ++k) x[k] = __uint_as_float((__float_as_uint(m[k]) & ~kClassMask) | (uint32_t)k);
  M1 = min2(x[0], x[1]);
  M2 = max2(x[0], x[1]);
#pragma unroll
  for (int k = 2; k + 1 < K; k += 2) {
    const float t = __builtin_amdgcn_fmed3f(M1, x[k], x[k + 1]);
    M1 = min3m(M1, x[k], x[k + 1]);
    M2 = min2(M2, t);
  }
}

// Two partitions of a lane's scores, one running minimum per class, in place of
// a top-2 chain over all of them: 8 classes by accumulator register % 8 (over
// all blocks) and one class per half block (registers 0-7 and 8-15).  A class of
// the first and a class of the second share exactly one group, so any group but
// the best differs from it in one of the two, and the smaller of the two
// partitions' second best bounds every other group's score.  Certification: the
// packed minima of the 8 classes are off by at most 2^-20 relative, half of the
// bound's cp (the half blocks are not packed); a best group outside the winning
// class of a partition would need that partition's second best within
// 2 (cm M + packing) of its best, which differs from the packed best by at most the
// packing error, so the bound E with cp = 2^-19 covers all of it.  1.4 VALU
// operations per score, 2.4 for the packed chain of reduce_block.
//
// fold_block: one block's 16 scores into the 8 classes, and the minima of its
// two halves.
__device__ __forceinline__ void fold_block(const f32x16& x, float (&mA)[8], float& lo, float& hi) {
#pragma unroll
  for (int k = 0; k < 8; ++k) mA[k] = min3m(mA[k], x[k], x[k + 8]);
  lo = min3m(min3m(min3m(min3m(x[0], x[1], x[2]), x[3], x[4]), x[5], x[6]), x[7], x[7]);
  hi = min3m(min3m(min3m(min3m(x[8], x[9], x[10]), x[11], x[12]), x[13], x[14]), x[15], x[15]);
}

// The lane-local group index (without the lane half's 4 h) of register v of
// block b: 32 b + 8 (v / 4) + v % 4.
__device__ __forceinline__ int local_group(int b, int v) { return 32 * b + v + (v & 12); }

// Bounds shared by every tile of a slice: the largest |r|^2 and |r| (with
// margins for their fp32 evaluation) and the error constants of the launch.
struct Certify {
  float nmaxf, rmaxf, cm, cp;
};

// Upper bound of |k| for the key whose 64 bf16 features are split over lanes
// q and q + 32 (32 each, as MFMA fragments); the same value in both lanes.
__device__ __forceinline__ float key_norm_bound(const u32x4 (&f)[4]) {
  float ss = 0.f;
#pragma unroll
  for (int s2 = 0; s2 < 4; ++s2)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = bf16_to_f32(f[s2][e] & 0xffffu), hi = bf16_to_f32(f[s2][e] >> 16);
      ss = fmaf(lo, lo, ss);
      ss = fmaf(hi, hi, ss);
    }
  const u32x2 p = halves(__float_as_uint(ss));
  return sqrtf(__uint_as_float(p[0]) + __uint_as_float(p[1])) * (1.0f + 0x1p-16f);
}

// Append this lane's entry if `mine`; the region's count `n` is wave-uniform.
__device__ __forceinline__ void wave_append(bool mine, uint32_t rec, uint32_t* region, int& n) {
  const uint64_t mask = __ballot(mine);
  if (mine)
    region[n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] =
        rec;
  n += (int)__popcll(mask);
}

// The |r|^2 part of every score: block b's MFMA of the split row (A) with
// ones in the first three k slots of lanes h = 0 (B), the same for every tile.
template <int NB>
__device__ __forceinline__ void norm_terms(const u32x4 (&an)[NB], const u32x4& ones, f32x16 (&nacc)[NB]) {
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int b = 0; b < NB; ++b)
    nacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, an[b]),
                                                      __builtin_bit_cast(bf16x8, ones), zero, 0, 0, 0);
}

// Scores of one tile against all NB blocks of groups and the lane's top-2.
// HOISTED: the |r|^2 parts (norm_terms) were formed once per workgroup and
// start each block's accumulation (four MFMAs per block); else they are the
// block's fifth MFMA, after the four k-steps (an order the error bound allows:
// it holds for any order of the terms).  Block b + 1's MFMAs are interleaved
// with block b's reduction (all in one straight-line region), so the matrix
// cores and the VALU work together.
template <int NB, bool HOISTED>
__device__ __forceinline__ void score_tile(const u32x4 (&af)[NB][4], const u32x4 (&an)[NB], const u32x4& ones,
                                           const f32x16 (&nacc)[NB], const u32x4 (&kf)[4], float& M1, float& M2,
                                           int& B1) {
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int kM = HOISTED ? 4 : 5;  // MFMAs per block
  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    acc[b] = HOISTED ? nacc[b] : zero;
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2)
      acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[b][s2]),
                                                       __builtin_bit_cast(bf16x8, kf[s2]), acc[b], 0, 0, 0);
    if (!HOISTED)
      acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, an[b]),
                                                       __builtin_bit_cast(bf16x8, ones), acc[b], 0, 0, 0);
  }
  M1 = FLT_MAX;
  M2 = FLT_MAX;
  B1 = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) reduce_block(acc[b], b, M1, M2, B1);
  __builtin_amdgcn_sched_group_barrier(0x008, kM, 0);  // block 0's MFMAs
#pragma unroll
  for (int b = 1; b < NB; ++b)
#pragma unroll
    for (int g = 0; g < kM; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // one MFMA of block b
      __builtin_amdgcn_sched_group_barrier(0x002, HOISTED ? 10 : 8, 0);  // VALU of block b - 1
    }
}
