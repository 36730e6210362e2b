// fp32 path of the grouping and the attention (gfx950): MFMA scores in fp32
// whose argmin is certified against the exact fp64 definition, the ordered
// fp64 member sums, and the fp32 group attention.
#include <hip/hip_runtime.h>

#include <float.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "ga_internal.h"

namespace ga {
namespace {

#include "ga_device.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS row stride (floats) of the MFMA A operand: 16 consecutive rows reading
// one 16-byte chunk then hit all 64 banks once.
constexpr int kRow = 68;
constexpr int kAsgChunk = 128;  // groups staged at a time by k_assign_f32
constexpr int kAttChunk = 64;   // by k_attend_f32
constexpr int kExactK = 4;      // uncertain keys decided together by one wave

// This lane's half row (features 32 h .. 32 h + 31) times `mul`.
__device__ __forceinline__ void load_half(const float* __restrict__ row, int h, float mul, f32x4 (&f)[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = *(const f32x4*)(row + 32 * h + 4 * s) * mul;
}

// acc += A (32 rows of an LDS tile) x B (32 columns held as half rows): 32 MFMA
// 32x32x2 steps; lanes h = 0 and 1 supply features c and 32 + c on both sides.
__device__ __forceinline__ f32x16 mfma_rows(const float* rows, int q, int h, const f32x4 (&b)[8], f32x16 acc) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const f32x4 a = *(const f32x4*)(rows + q * kRow + 32 * h + 4 * s);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[s][e], acc, 0, 0, 0);
  }
  return acc;
}

// ------------------------------------------------------------------ assign
// The canonical decision of NK keys (rows k[b], wave-uniform) by one wave:
// lanes take groups lane, lane + 64, ...; the dot product an fp64 fma chain
// over c = 0..63, the score fma(-2, dot, |r|^2), lowest index among minima.
template <int NK>
__device__ __forceinline__ void exact_keys(const float* const (&k)[kExactK], const float* __restrict__ Rbh,
                                           const double* __restrict__ nrm, int N, int (&jb)[kExactK]) {
  const int lane = threadIdx.x & 63;
  double best[NK];
#pragma unroll
  for (int b = 0; b < NK; ++b) {
    best[b] = INFINITY;
    jb[b] = 0x7fffffff;
  }
  for (int j = lane; j < N; j += 64) {
    const float* r = Rbh + (int64_t)j * 64;
    const double nj = nrm[j];
    double dot[NK];
#pragma unroll
    for (int b = 0; b < NK; ++b) dot[b] = 0.0;
#pragma unroll 2
    for (int c = 0; c < 64; c += 8) {
      const f32x4 r0 = *(const f32x4*)(r + c), r1 = *(const f32x4*)(r + c + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double x = (double)(e < 4 ? r0[e & 3] : r1[e & 3]);
#pragma unroll
        for (int b = 0; b < NK; ++b) dot[b] = fma((double)k[b][c + e], x, dot[b]);
      }
    }
#pragma unroll
    for (int b = 0; b < NK; ++b) {
      const double s = fma(-2.0, dot[b], nj);
      if (s < best[b]) {
        best[b] = s;
        jb[b] = j;
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NK; ++b) wave_argmin(best[b], jb[b]);
}

// k_assign_f32: grid (ceil(tiles / (4 tpw)), BH), 256 threads; each wave
// scores tpw tiles of 32 keys against all groups (staged kAsgChunk at a time)
// with MFMA 32x32x2 fp32: s^ = |r|^2 + sum r_c (-2 k_c), |r|^2 (rounded to
// fp32) as the accumulator's start, then the packed top-2 of reduce_block.
// The bound E of certified decisions is the bf16 path's: each of the 64
// products and the start added with at most one rounding (truncation
// included) is within cm M, cm = (d + 4) 2^-23, M = max |r|^2 + 2 |k| max |r|.
// Keys that it does not certify (0.07% on mixtures of 64 groups), among them
// every key that a NaN, an infinity or an overflow touches (E is then no
// finite number) or whose scores underflow (E >= 1e-30), are queued and decided by
// exact_keys, so the groups are those of the fp64 definition.  Bound by the
// MFMA rate (157 TFLOP/s in fp32) at full grids: 32 slices of 2000 keys against
// 64 groups 148 -> 17 us (event times, with about 5 us of event overhead), 128
// slices of 8000 against 128 groups 163 us (103 TFLOP/s), where an fp64 fma
// chain for every (key, group) took 148 us and several milliseconds.
__global__ __launch_bounds__(256) void k_assign_f32(const float* __restrict__ K, const float* __restrict__ R,
                                                    const double* __restrict__ nrm64, int32_t* __restrict__ belong,
                                                    int n, int N, int tpw, float cm, float cp) {
  __shared__ __align__(16) float Rl[kAsgChunk * kRow];
  __shared__ __align__(16) float Nl[kAsgChunk];
  __shared__ uint32_t nbits;  // largest |r|^2 as bits (a NaN's are larger than any number's)
  __shared__ int nq;
  extern __shared__ int32_t queue[];  // [4 tpw 32] local indices of uncertain keys
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, q = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t bh = blockIdx.y;
  const int64_t key0 = (int64_t)blockIdx.x * 4 * tpw * 32;
  const float* Kbh = K + bh * (int64_t)n * 64;
  const float* Rbh = R + bh * (int64_t)N * 64;
  const double* nrm_bh = nrm64 + bh * N;
  if (tid == 0) {
    nbits = 0;
    nq = 0;
  }
  for (int t = 0; t < tpw; ++t) {
    // the waves' tiles of one pass are neighbours; every wave runs every pass (barriers below)
    const int lk = (t * 4 + wave) * 32 + q;
    const int64_t key = key0 + lk;
    if (key0 + (int64_t)t * 128 >= n) break;  // uniform
    f32x4 kf[8];
    load_half(Kbh + min(key, (int64_t)n - 1) * 64, h, -2.0f, kf);
    float M1 = FLT_MAX, M2 = FLT_MAX;
    int B1 = 0;
    for (int g0 = 0; g0 < N; g0 += kAsgChunk) {
      const int ng = min(kAsgChunk, N - g0), nblk = (ng + 31) >> 5;
      if (t == 0 || N > kAsgChunk) {
        __syncthreads();
        for (int x = tid; x < nblk * 32 * 16; x += 256) {
          const int r = x >> 4, ch = x & 15;
          *(f32x4*)(Rl + r * kRow + 4 * ch) = *(const f32x4*)(Rbh + (int64_t)(g0 + min(r, ng - 1)) * 64 + 4 * ch);
        }
        if (tid < nblk * 32) {
          const float v = tid < ng ? (float)nrm_bh[g0 + tid] : 3.0e38f;  // a padded group never wins
          Nl[tid] = v;
          if (tid < ng) atomicMax(&nbits, __float_as_uint(v));
        }
        __syncthreads();
      }
      for (int b = 0; b < nblk; ++b) {
        f32x16 acc;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const f32x4 nv = *(const f32x4*)(Nl + b * 32 + 8 * w + 4 * h);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[4 * w + e] = nv[e];
        }
        acc = mfma_rows(Rl + b * 32 * kRow, q, h, kf, acc);
        reduce_block(acc, (g0 >> 5) + b, M1, M2, B1);
      }
    }
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) ss = fmaf(kf[s][e], kf[s][e], ss);
    const u32x2 ps = halves(__float_as_uint(ss)), p1 = halves(__float_as_uint(M1)), p2 = halves(__float_as_uint(M2)),
                pb = halves((uint32_t)B1);
    const float k2 = sqrtf(__uint_as_float(ps[0]) + __uint_as_float(ps[1])) * (1.0f + 0x1p-16f);  // 2 |k|
    const float a1 = __uint_as_float(p1[0]), b1 = __uint_as_float(p1[1]);
    const bool hi_wins = b1 < a1;
    const uint32_t vw = __float_as_uint(hi_wins ? b1 : a1) & kPackMask;
    const int jstar = 32 * (int)(hi_wins ? pb[1] : pb[0]) + 8 * (int)(vw >> 2) + (hi_wins ? 4 : 0) + (int)(vw & 3);
    const float best = min2(a1, b1);
    const float second = min2(max2(a1, b1), min2(__uint_as_float(p2[0]), __uint_as_float(p2[1])));
    const float nmaxf = __uint_as_float(nbits) * (1.0f + 0x1p-20f);
    const float Mk = nmaxf + k2 * (sqrtf(nmaxf) * (1.0f + 0x1p-20f));
    const float aM1 = fabsf(best);
    const float E = (cm * Mk + cp * (aM1 + 3.0f * cm * Mk)) * (1.0f + 0x1p-20f) + 0x1p-22f * aM1 + 1e-30f;
    const bool certain = (second > best + 2.0f * E) && (E < FLT_MAX) && (jstar < N);
    if (h == 0 && key < n) {
      if (certain)
        belong[bh * n + key] = jstar;
      else
        queue[atomicAdd(&nq, 1)] = lk;
    }
  }
  __syncthreads();
  const int nu = nq;
  for (int u0 = wave * kExactK; u0 < nu; u0 += 4 * kExactK) {
    const int nb = min(kExactK, nu - u0);
    int64_t kk[kExactK];
    const float* rows[kExactK];
    int jb[kExactK];
#pragma unroll
    for (int b = 0; b < kExactK; ++b) {
      kk[b] = key0 + __builtin_amdgcn_readfirstlane(queue[u0 + min(b, nb - 1)]);
      rows[b] = Kbh + kk[b] * 64;
    }
    if (nb == 1)
      exact_keys<1>(rows, Rbh, nrm_bh, N, jb);
    else
      exact_keys<kExactK>(rows, Rbh, nrm_bh, N, jb);
    if (lane == 0)
#pragma unroll
      for (int b = 0; b < kExactK; ++b)
        if (b < nb) belong[bh * n + kk[b]] = jb[b];
  }
}

// ------------------------------------------------------------------ ordered sums
__device__ __forceinline__ int wave_incl_scan(int x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(x, d);
    if (lane >= d) x += t;
  }
  return x;
}

// Stable counting sort of one slice's keys by group; grid BH, 1024 threads.
// LDS: per-wave 64-bit lane masks [16][N], counts [N], running offsets [N].
// Within a 1024-key chunk, a key's rank among same-group keys is the number
// of lower lanes in its wave with the same group (popcount of the OR-ed lane
// mask) plus the members of that group in the lower waves of the chunk.
// Entries of belong outside [0, N) are left out.
__global__ __launch_bounds__(1024) void k_bucket(const int32_t* __restrict__ belong, int n, int N,
                                                 int32_t* __restrict__ perm, int32_t* __restrict__ goff,
                                                 int32_t* __restrict__ count) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int wsum[16];
  unsigned long long* wmask = (unsigned long long*)smem;
  int32_t* cnt = (int32_t*)(wmask + 16 * N);
  int32_t* run = cnt + N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t bh = blockIdx.x;
  const int32_t* a = belong + bh * n;

  for (int g = tid; g < N; g += 1024) cnt[g] = 0;
  for (int x = tid; x < 16 * N; x += 1024) wmask[x] = 0ull;
  __syncthreads();
  for (int i = tid; i < n; i += 1024) {
    const int g = a[i];
    if ((unsigned)g < (unsigned)N) atomicAdd(&cnt[g], 1);
  }
  __syncthreads();
  const int v = tid < N ? cnt[tid] : 0;
  const int incl = wave_incl_scan(v);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int t = lane < 16 ? wsum[lane] : 0;
    const int ti = wave_incl_scan(t);
    if (lane < 16) wsum[lane] = ti - t;
  }
  __syncthreads();
  if (tid < N) {
    const int ex = incl - v + wsum[wave];
    run[tid] = ex;
    goff[bh * N + tid] = ex;
    count[bh * N + tid] = v;
  }
  __syncthreads();

  const unsigned long long below = (1ull << lane) - 1ull;
  for (int base = 0; base < n; base += 1024) {
    const int i = base + tid;
    const int g = i < n ? a[i] : -1;
    const bool ok = (unsigned)g < (unsigned)N;
    if (ok) atomicOr(&wmask[wave * N + g], 1ull << lane);
    __syncthreads();
    unsigned long long m = 0ull;
    int rank = 0;
    if (ok) {
      m = wmask[wave * N + g];
      rank = __popcll(m & below);
      int pre = 0;
      for (int w2 = 0; w2 < wave; ++w2) pre += __popcll(wmask[w2 * N + g]);
      perm[bh * n + run[g] + pre + rank] = i;
    }
    __syncthreads();
    if (ok && rank == 0) {
      atomicAdd(&run[g], __popcll(m));
      wmask[wave * N + g] = 0ull;
    }
    __syncthreads();
  }
}

// k_segsum: grid (ceil(N/4), BH), 256 threads: one wave per group, lane =
// feature.  The wave adds the rows of its group's members in ascending key order
// in fp64 (fp32 sums need not be exact, so the order is part of the
// definition).  UPDATE: count, centroid = (float)(sum / count) (an empty group
// keeps its centroid), representative and |r|^2; otherwise the fp32 rounding of
// the value sum.  SORTED: the members are perm[goff .. goff + count) (k_bucket);
// otherwise the wave finds them itself: it scans the slice's groups 64 keys at
// a time and appends the keys of its group to a list in LDS (a ballot gives
// their places, so the list ascends), added whenever 64 are there and at the
// end.  Entries of belong outside [0, N) are ignored.
//
// Bound by latency: kScanU loads of 64 groups are in flight in the scan, and a
// batch of kSegU rows while the one before it is added (all 64 rows of a full
// list at once: no faster, and 98 against 78 us at 128 slices of 8000 keys, 128
// groups, where fewer waves are resident).  Groups of up to kSegU members load by
// the quad, not whole batches (scan of 512 slices of 300 keys, 256 groups 43 -> 33
// us; sorted, 512 slices of 1000, 512 groups 82 -> 67).  Which of the two: see
// sums_sorted.
constexpr int kSegU = 16;
constexpr int kSegS = 4;
constexpr int kScanU = 8;
template <bool UPDATE, bool SORTED>
__global__ __launch_bounds__(256) void k_segsum(const float* __restrict__ X, const int32_t* __restrict__ belong,
                                                const int32_t* __restrict__ perm, const int32_t* __restrict__ goff,
                                                int n, int N, int32_t* __restrict__ count, float* __restrict__ out,
                                                float* __restrict__ R, double* __restrict__ nrm64) {
  __shared__ int32_t list[SORTED ? 1 : 4][SORTED ? 1 : 128];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = blockIdx.x * 4 + wave;
  const int64_t bh = blockIdx.y;
  if (g >= N) return;
  const int64_t row = bh * N + g;
  const float* Xb = X + bh * (int64_t)n * 64 + lane;
  double acc = 0.0;
  int cnt = 0;  // members
  // adds the rows idx of the lanes 0 .. m - 1 (1 .. 64) in order
  auto sum = [&](int idx, int m) {
    auto load = [&](int x, auto& v) {  // past the end: the last member again, not added
      constexpr int U = sizeof(v) / sizeof(float);
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = Xb[(int64_t)__builtin_amdgcn_readlane(idx, x + u) * 64];
    };
    auto add = [&](int x, const auto& v) {
      constexpr int U = sizeof(v) / sizeof(float);
      if (x + U <= m) {
#pragma unroll
        for (int u = 0; u < U; ++u) acc += (double)v[u];
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (x + u < m) acc += (double)v[u];
      }
    };
    if (!SORTED && m <= 4 * kSegS) {  // few members: only as many loads as there are quads of them
      float v0[kSegS], v1[kSegS], v2[kSegS], v3[kSegS];
      load(0, v0);
      if (m > kSegS) load(kSegS, v1);
      if (m > 2 * kSegS) load(2 * kSegS, v2);
      if (m > 3 * kSegS) load(3 * kSegS, v3);
      add(0, v0);
      if (m > kSegS) add(kSegS, v1);
      if (m > 2 * kSegS) add(2 * kSegS, v2);
      if (m > 3 * kSegS) add(3 * kSegS, v3);
      return;
    }
    float va[kSegU], vb[kSegU];
    load(0, va);
    if (m > kSegU) load(kSegU, vb);
    add(0, va);
    if (m <= kSegU) return;
    if (m > 2 * kSegU) load(2 * kSegU, va);
    add(kSegU, vb);
    if (m <= 2 * kSegU) return;
    if (m > 3 * kSegU) load(3 * kSegU, vb);
    add(2 * kSegU, va);
    if (m > 3 * kSegU) add(3 * kSegU, vb);
  };
  if constexpr (SORTED) {
    cnt = __builtin_amdgcn_readfirstlane(count[row]);
    const int32_t* P = perm + bh * n + __builtin_amdgcn_readfirstlane(goff[row]);
    if (cnt <= kSegU) {
      int x = 0;
      for (; x + kSegS <= cnt; x += kSegS) {
        float v[kSegS];
#pragma unroll
        for (int u = 0; u < kSegS; ++u) v[u] = Xb[(int64_t)P[x + u] * 64];
#pragma unroll
        for (int u = 0; u < kSegS; ++u) acc += (double)v[u];
      }
      for (; x < cnt; ++x) acc += (double)Xb[(int64_t)P[x] * 64];
    } else {
      int next = P[min(lane, cnt - 1)];
      for (int x = 0; x < cnt; x += 64) {
        const int idx = next;
        next = P[min(x + 64 + lane, cnt - 1)];
        sum(idx, min(64, cnt - x));
      }
    }
  } else {
    const int32_t* bel = belong + bh * n;
    int32_t* L = list[wave];
    int held = 0;  // members in the list
    for (int base = 0; base < n; base += 64 * kScanU) {
      int b[kScanU];
#pragma unroll
      for (int u = 0; u < kScanU; ++u) b[u] = bel[min(base + 64 * u + lane, n - 1)];
#pragma unroll
      for (int u = 0; u < kScanU; ++u) {
        const int key = base + 64 * u + lane;
        const bool mine = key < n && b[u] == g;
        const uint64_t mask = __ballot(mine);
        if (mask == 0) continue;  // uniform
        if (mine)
          L[held + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = key;
        held += (int)__popcll(mask);
        if (held >= 64) {
          cnt += 64;
          held -= 64;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          sum(L[lane], 64);
          const int rest = L[64 + lane];  // at most 63 of these are members
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          L[lane] = rest;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    cnt += held;
    if (held > 0) sum(L[min(lane, held - 1)], held);
  }
  if (!UPDATE) {
    out[row * 64 + lane] = (float)acc;
    return;
  }
  if (!SORTED && lane == 0) count[row] = cnt;
  float c;
  if (cnt > 0) {
    c = (float)(acc / (double)cnt);
    out[row * 64 + lane] = c;
  } else {
    c = out[row * 64 + lane];
  }
  R[row * 64 + lane] = c;
  const double nrm = canon_nrm_wave(c);
  if (lane == 0) nrm64[row] = nrm;
}

// ------------------------------------------------------------------ attention
// k_attend_f32: grid (ceil(tiles / (4 tpw)), BH), 256 threads; each wave takes
// tiles of 32 queries (lane l: query l % 32, h = l / 32).  Per 32-group block:
// scores by MFMA 32x32x2 fp32 (A = centroid rows from LDS, B = the query), the
// running-maximum softmax, and the combine by MFMA again: the exponentials
// leave the first product's registers as the second one's B operand (step v
// contracts groups 8 (v / 4) + v % 4 and + 4, which registers v of lanes h = 0
// and 1 hold), A = the value sums.  Everything is fp32, as is the denominator;
// the count enters only there.
__global__ __launch_bounds__(256) void k_attend_f32(const float* __restrict__ Q, const float* __restrict__ centroid,
                                                    const int32_t* __restrict__ count,
                                                    const float* __restrict__ vsum, int n, int N, float scale,
                                                    int tpw, float* __restrict__ O) {
  __shared__ __align__(16) float Rs[kAttChunk * kRow];
  __shared__ __align__(16) float Vs[kAttChunk * 64];
  __shared__ __align__(16) float Cs[kAttChunk];  // member counts, 0 for an empty or padded group
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, q = lane & 31;
  const int wave = tid >> 6;
  const int64_t bh = blockIdx.y;
  const int64_t q0 = (int64_t)blockIdx.x * 4 * tpw * 32;
  const float* Rbh = centroid + bh * (int64_t)N * 64;
  const float* Vbh = vsum + bh * (int64_t)N * 64;
  for (int t = 0; t < tpw; ++t) {
    if (q0 + (int64_t)t * 128 >= n) break;  // uniform
    const int64_t qi = q0 + (t * 4 + wave) * 32 + q;
    f32x4 qf[8];
    load_half(Q + (bh * n + min(qi, (int64_t)n - 1)) * 64, h, 1.0f, qf);
    f32x16 o0, o1;
#pragma unroll
    for (int v = 0; v < 16; ++v) o0[v] = o1[v] = 0.f;
    float m = -INFINITY, ssum = 0.f;  // ssum: this lane's half of the groups
    for (int g0 = 0; g0 < N; g0 += kAttChunk) {
      const int ng = min(kAttChunk, N - g0), nblk = (ng + 31) >> 5;
      if (t == 0 || N > kAttChunk) {
        __syncthreads();
        for (int x = tid; x < nblk * 32 * 16; x += 256) {
          const int r = x >> 4, ch = x & 15;
          const int64_t src = (int64_t)(g0 + min(r, ng - 1)) * 64 + 4 * ch;
          *(f32x4*)(Rs + r * kRow + 4 * ch) = *(const f32x4*)(Rbh + src);
          const f32x4 vv = *(const f32x4*)(Vbh + src);
          *(f32x4*)(Vs + r * 64 + 4 * ch) = r < ng && count[bh * N + g0 + r] > 0 ? vv : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (tid < nblk * 32) Cs[tid] = tid < ng ? (float)max(count[bh * N + g0 + tid], 0) : 0.f;
        __syncthreads();
      }
      for (int b = 0; b < nblk; ++b) {
        f32x16 p;
        float cj[16];
        bool some = false;  // a non-empty group in the block (the same for both halves, below)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const f32x4 cv = *(const f32x4*)(Cs + b * 32 + 8 * w + 4 * h);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            cj[4 * w + e] = cv[e];
            some |= cv[e] > 0.f;
            p[4 * w + e] = 0.f;
          }
        }
        if (!__any(some)) continue;
        p = mfma_rows(Rs + b * 32 * kRow, q, h, qf, p);
        float bm = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          p[v] = cj[v] > 0.f ? scale * p[v] : -INFINITY;
          bm = fmaxf(bm, p[v]);
        }
        const u32x2 pm = halves(__float_as_uint(bm));
        const float mn = fmaxf(m, fmaxf(__uint_as_float(pm[0]), __uint_as_float(pm[1])));
        if (__any(mn != m)) {
          const float alpha = expf(m - mn);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            o0[v] *= alpha;
            o1[v] *= alpha;
          }
          ssum *= alpha;
          m = mn;
        }
        const float* vr = Vs + (b * 32 + 4 * h) * 64 + q;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float e = cj[v] > 0.f ? expf(p[v] - m) : 0.f;
          ssum = fmaf(cj[v], e, ssum);
          const float* vg = vr + (8 * (v >> 2) + (v & 3)) * 64;
          o0 = __builtin_amdgcn_mfma_f32_32x32x2f32(vg[0], e, o0, 0, 0, 0);
          o1 = __builtin_amdgcn_mfma_f32_32x32x2f32(vg[32], e, o1, 0, 0, 0);
        }
      }
    }
    const u32x2 ps = halves(__float_as_uint(ssum));
    const float stot = __uint_as_float(ps[0]) + __uint_as_float(ps[1]);
    const float inv = stot > 0.f ? 1.0f / stot : 0.f;
    if (qi < n) {
      float* orow = O + (bh * n + qi) * 64 + 4 * h;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        *(f32x4*)(orow + 8 * w) = f32x4{o0[4 * w], o0[4 * w + 1], o0[4 * w + 2], o0[4 * w + 3]} * inv;
        *(f32x4*)(orow + 32 + 8 * w) = f32x4{o1[4 * w], o1[4 * w + 1], o1[4 * w + 2], o1[4 * w + 3]} * inv;
      }
    }
  }
}

// Passes of four 32-row tiles per workgroup: one while the grid has at most
// about three workgroups per compute unit (the staged groups then cost less
// than an idle unit), more beyond that.
int passes(int64_t tiles, int64_t BH, int cap) {
  const int64_t wgs = ((tiles + 3) / 4) * BH;
  const int64_t p = (wgs + 767) / 768;
  return (int)(p < 1 ? 1 : p > cap ? cap : p);
}

}  // namespace

hipError_t launch_assign_f32(const Dims& d, const float* K, const float* R, const double* nrm64, int32_t* belong,
                             bool first, hipStream_t st) {
  TimedLaunch timed(first ? "assign_first" : "assign", st);
  const int64_t tiles = ((int64_t)d.n + 31) / 32;
  const int tpw = passes(tiles, d.BH, 16);
  const float cm = (float)(kD + 4) * 0x1p-23f * (1.0f + 0x1p-10f) * cert_widen();
  const float cp = 0x1p-19f * (1.0f + 0x1p-10f) * cert_widen();
  const dim3 grid((unsigned)((tiles + 4 * tpw - 1) / (4 * tpw)), (unsigned)d.BH);
  hipLaunchKernelGGL(k_assign_f32, grid, dim3(256), (size_t)4 * tpw * 32 * 4, st, K, R, nrm64, belong, d.n, d.N, tpw,
                     cm, cp);
  return hipGetLastError();
}

// Whether the ordered sums sort the keys by group first.  The scan of k_segsum
// reads a slice's groups once for every group: with few (group, key) pairs it is
// hidden behind the rows' latency and saves the sort's launch, with many it is the
// longest part.  Aggregate, us, scan : sort, at the edge and on both sides of it: 32
// slices of 20000 keys, 128 groups 47 : 58, 256 groups 65 : 59, 1024 groups 170 :
// 61; 32 of 2000, 256 groups 10 : 13, 512 groups 12.7 : 13.3, 1024 groups 21 : 15;
// 512 of 300, 128 groups 20 : 22, 256 groups 33 : 33.  Beyond 4000 keys both grow
// alike.
static bool sums_sorted(const Dims& d) {
  return d.BH * d.N * (d.n < 4000 ? d.n : 4000) >= 32000000;
}

static size_t bucket_lds(int N) { return (size_t)16 * N * 8 + (size_t)2 * N * 4; }

// The slices' keys sorted by group into w.mrec's first half (perm; its second half
// takes goff), which only the bf16 path uses otherwise.
static hipError_t launch_sort(const Dims& d, const int32_t* belong, const Workspace& w, int32_t* count,
                              hipStream_t st) {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute((const void*)k_bucket, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)bucket_lds(kMaxGroups));
  });
  TimedLaunch timed("bucket", st);
  hipLaunchKernelGGL(k_bucket, dim3((unsigned)d.BH), dim3(1024), bucket_lds(d.N), st, belong, d.n, d.N,
                     (int32_t*)w.mrec, (int32_t*)w.mrec + d.BH * d.n, count);
  return hipGetLastError();
}

template <bool UPDATE>
static hipError_t launch_segsum(const Dims& d, bool sorted, const float* X, const int32_t* belong, const Workspace& w,
                                int32_t* count, float* out, hipStream_t st) {
  TimedLaunch timed(UPDATE ? "update" : "valuesum", st);
  const auto kern = sorted ? k_segsum<UPDATE, true> : k_segsum<UPDATE, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)((d.N + 3) / 4), (unsigned)d.BH), dim3(256), 0, st, X, belong,
                     (const int32_t*)w.mrec, (const int32_t*)w.mrec + d.BH * d.n, d.n, d.N, count, out, (float*)w.R,
                     w.nrm64);
  return hipGetLastError();
}

hipError_t launch_update_f32(const Dims& d, const float* K, const int32_t* belong, const Workspace& w, int32_t* count,
                             float* C, hipStream_t st) {
  const bool sorted = sums_sorted(d);
  if (sorted) {
    const hipError_t e = launch_sort(d, belong, w, count, st);
    if (e != hipSuccess) return e;
  }
  return launch_segsum<true>(d, sorted, K, belong, w, count, C, st);
}

hipError_t launch_valuesum_f32(const Dims& d, const float* V, const int32_t* belong, bool updated, const Workspace& w,
                               int32_t* count, float* vsum, hipStream_t st) {
  const bool sorted = sums_sorted(d);
  if (sorted && !updated) {
    const hipError_t e = launch_sort(d, belong, w, count, st);
    if (e != hipSuccess) return e;
  }
  return launch_segsum<false>(d, sorted, V, belong, w, count, vsum, st);
}

hipError_t launch_attend_f32(const Dims& d, const float* Q, const float* centroid, const int32_t* count,
                             const float* vsum, float scale, float* O, hipStream_t st) {
  TimedLaunch timed("attend", st);
  const int64_t tiles = ((int64_t)d.n + 31) / 32;
  const int tpw = passes(tiles, d.BH, 16);
  hipLaunchKernelGGL(k_attend_f32, dim3((unsigned)((tiles + 4 * tpw - 1) / (4 * tpw)), (unsigned)d.BH), dim3(256), 0,
                     st, Q, centroid, count, vsum, d.n, d.N, scale, tpw, O);
  return hipGetLastError();
}

}  // namespace ga
