// Query statistics of the calibration block on the device, from the second
// moment M of a head's Queries (Eq. 6): channel sensitivities w (Eq. 8), the
// full metric's matrix, and the principal basis U_r with its eigenvalues
// (Eq. 15), all in fp64. One workgroup per head:
//
//  1. Householder tridiagonalisation T = Q^T M Q. M lives in registers (each
//     thread holds D/8 columns of D/64 rows); a step applies the previous
//     reflection's rank-2 update and multiplies by the new vector in one sweep,
//     and only the vectors go through LDS. Between two barriers one wave turns
//     the product into the next reflection.
//  2. The r largest eigenvalues of T by multisection on Sturm counts: 32 lanes
//     per eigenvalue narrow its interval 33-fold per round.
//  3. Eigenvectors of T by two rounds of inverse iteration (LU with partial
//     pivoting, one lane per eigenvalue) from fixed start vectors, each round
//     followed by modified Gram-Schmidt (twice) in order of the eigenvalues,
//     so close or equal eigenvalues still give an orthonormal set.
//  4. Back-transformation by the stored reflections, 16 lanes per vector.
//
// Latency bounds it (a chain of D reflections, 11 Sturm sweeps and a few solves
// of length D); only the first r of the D eigenpairs are needed, which is why
// neither QL on all vectors nor Jacobi sweeps (about 1,000 dependent rotation
// rounds at D = 128) is used: a host Jacobi took 15 ms per head, all heads of a
// launch together take 0.33 ms here (r = 8; 0.39 ms for r = 16) at D = 128. Every loop has a fixed trip count, so non-finite
// input ends too. All sums have a fixed order: equal M give equal bits.
#include "qwm_common.h"

#include <atomic>

namespace qwm {
namespace {

constexpr int kLanes = 512;   // threads of the workgroup
constexpr int kMaxRank = 32;

template <int CTRL>
__device__ inline double dpp(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(u)), CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, uint64_t(hi) << 32 | lo);
}
// x plus the value of the lane N away inside its group of 2N (every lane of the
// group ends with the same sum, since a + b and b + a round alike)
template <int N>
__device__ inline double add_step(double x) {
  if constexpr (N == 1) return x + dpp<0xB1>(x);        // quad_perm 1,0,3,2
  else if constexpr (N == 2) return x + dpp<0x4E>(x);   // quad_perm 2,3,0,1
  else if constexpr (N == 4) return x + dpp<0x141>(x);  // row_half_mirror
  else if constexpr (N == 8) return x + dpp<0x140>(x);  // row_mirror
  else {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t l = uint32_t(u), h = uint32_t(u >> 32);
    if constexpr (N == 16) {
      const auto a = __builtin_amdgcn_permlane16_swap(l, l, false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(h, h, false, false);
      return __builtin_bit_cast(double, uint64_t(b[0]) << 32 | a[0]) +
             __builtin_bit_cast(double, uint64_t(b[1]) << 32 | a[1]);
    } else {
      const auto a = __builtin_amdgcn_permlane32_swap(l, l, false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(h, h, false, false);
      return __builtin_bit_cast(double, uint64_t(b[0]) << 32 | a[0]) +
             __builtin_bit_cast(double, uint64_t(b[1]) << 32 | a[1]);
    }
  }
}
// sum over groups of N lanes, the same bits on every lane of the group
template <int N>
__device__ inline double group_sum(double x) {
  if constexpr (N >= 2) x = add_step<1>(x);
  if constexpr (N >= 4) x = add_step<2>(x);
  if constexpr (N >= 8) x = add_step<4>(x);
  if constexpr (N >= 16) x = add_step<8>(x);
  if constexpr (N >= 32) x = add_step<16>(x);
  if constexpr (N >= 64) x = add_step<32>(x);
  return x;
}
__device__ inline double lane_value(double x, int lane) {  // lane: wave-uniform
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane(int(uint32_t(u)), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(int(uint32_t(u >> 32)), lane);
  return __builtin_bit_cast(double, uint64_t(hi) << 32 | lo);
}
// 1 / x to about one ulp (v_rcp_f64 holds about 24 bits; two Newton steps)
__device__ inline double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// sqrt(x), x > 0, to about one ulp (v_rsq_f64 and two Newton steps)
__device__ inline double root(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = __builtin_fma(__builtin_fma(-x * y, y, 1.0), 0.5 * y, y);
  const double r = x * y;
  return __builtin_fma(__builtin_fma(-r, r, x), 0.5 * y, r);
}

// double -> bf16 with one rounding (nearest, ties to even), for normal values.
__device__ inline void store_rn(float* p, double x) { *p = (float)x; }
__device__ inline void store_rn(bf16* p, double x) {
  uint64_t u = __builtin_bit_cast(uint64_t, x);
  u += (uint64_t(1) << 44) - 1 + ((u >> 45) & 1);
  u &= ~((uint64_t(1) << 45) - 1);
  *p = bf16((float)__builtin_bit_cast(double, u));  // exact: the value already fits bf16
}

typedef double f64x2 __attribute__((ext_vector_type(2)));

template <int D>
struct BasisLds {
  double row[D], vn[D], v[D], w[D], p[D];  // next row of M, vectors of the reflections, M v
  double al[D], be[D], bt[D];              // T (diagonal, off-diagonal) and 2 / v^T v of each reflection
  double lam[kMaxRank];
  double red[kLanes / 64];
  double fd[D][kMaxRank], fu[D][kMaxRank], fl[D][kMaxRank];  // LU of T - lam: 1 / pivot, first super-diagonal, multipliers
  double z[kMaxRank][D + 2];                                 // vectors, one row per eigenvalue
};

// m_in: [BH][D][D], divided by div unless that is 0 (not read at cold start); scratch:
// [BH][D][D], may be m_in itself (the reflection vectors replace M).
template <typename T, int D>
__global__ __launch_bounds__(kLanes) void basis_kernel(const double* m_in, int64_t div, int cold,
                                                       double* scratch, uint8_t* calib, quantwm_calib_layout C, int r,
                                                       int full) {
  constexpr int R = D / 64, P = D / 16, NE = D / 64;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  BasisLds<D>& S = *reinterpret_cast<BasisLds<D>*>(smem_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = tid >> 3, sub = tid & 7;
  const int64_t bh = blockIdx.x;
  uint8_t* slab = calib + bh * C.slab_bytes;
  float* wo = reinterpret_cast<float*>(slab + C.w);
  float* lo_ = reinterpret_cast<float*>(slab + C.lam);
  T* uo = reinterpret_cast<T*>(slab + C.u_t);
  float* mo = reinterpret_cast<float*>(slab + C.m);
  const double* mi = m_in + bh * D * D;
  double* vecs = scratch + bh * D * D;

  // ---- M: row row0 + 64 j, columns 2 sub + 16 m + {0, 1}
  f64x2 a[R][P];
  double amax = 0.0;
  if (!cold) {
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int m = 0; m < P; ++m) {
        f64x2 x = *reinterpret_cast<const f64x2*>(mi + (row0 + 64 * j) * D + 2 * sub + 16 * m);
        if (div) x = x / (double)div;
        a[j][m] = x;
        amax = fmax(amax, fmax(fabs(x.x), fabs(x.y)));
        const int c = 2 * sub + 16 * m, i = row0 + 64 * j;
        if (i == c) S.row[i] = x.x;
        if (i == c + 1) S.row[i] = x.y;
      }
  } else if (tid < D) {
    S.row[tid] = 0.0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmax(amax, __shfl_xor(amax, o));
  if (lane == 0) S.red[wave] = amax;
  __syncthreads();
  double tr = 0.0;
  for (int k = 0; k < D; ++k) tr += S.row[k];
  if (tr == 0.0) {  // cold start: uniform sensitivity, PSAC inactive
    if (tid < D) wo[tid] = 1.0f;
    if (tid < r) lo_[tid] = 0.0f;
    for (int i = tid; i < r * D; i += kLanes) uo[i] = T(0.0f);
    if (full)
      for (int i = tid; i < D * D; i += kLanes) mo[i] = i / D == i % D ? 1.0f : 0.0f;
    return;
  }
  const double mean = tr / (double)D;
  if (tid < D) wo[tid] = (float)(S.row[tid] / mean);
  if (full) {
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int m = 0; m < P; ++m) {
        float* q = mo + (row0 + 64 * j) * D + 2 * sub + 16 * m;
        q[0] = (float)(a[j][m].x / mean);
        q[1] = (float)(a[j][m].y / mean);
      }
  }
  if (r == 0) return;
  // scaled by a power of two to magnitude 1 (exact), so that no square under- or overflows
  for (int i = 0; i < kLanes / 64; ++i) amax = fmax(amax, S.red[i]);
  int ex = 0;
  if (amax > 0.0 && amax < __builtin_inf()) (void)frexp(amax, &ex);
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int m = 0; m < P; ++m) {
      a[j][m].x = ldexp(a[j][m].x, -ex);
      a[j][m].y = ldexp(a[j][m].y, -ex);
    }
  __syncthreads();  // everyone has read the diagonal
  // row 0 for the first reflection, nothing pending
  if (row0 == 0)
#pragma unroll
    for (int m = 0; m < P; ++m) *reinterpret_cast<f64x2*>(&S.row[2 * sub + 16 * m]) = a[0][m];
  if (tid < D) S.v[tid] = S.w[tid] = S.p[tid] = S.vn[tid] = 0.0;
  __syncthreads();

  // ---- 1. tridiagonalisation
  double beta = 0.0;
  for (int k = 0; k < D; ++k) {
    if (wave == 0) {
      // the previous reflection's rank-2 form: w = p - (beta/2 p^T v) v
      double v[NE], w[NE], x[NE], s = 0.0;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        v[e] = S.vn[lane + 64 * e];
        w[e] = S.p[lane + 64 * e];
        x[e] = S.row[lane + 64 * e];
        s = __builtin_fma(v[e], w[e], s);
      }
      const double K = 0.5 * beta * group_sum<64>(s);
      double vk = 0.0, wk = 0.0, xk = 0.0, x1 = 0.0, q = 0.0;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        w[e] = __builtin_fma(-K, v[e], w[e]);
        S.v[lane + 64 * e] = v[e];
        S.w[lane + 64 * e] = w[e];
        if ((k >> 6) == e) { vk = lane_value(v[e], k & 63); wk = lane_value(w[e], k & 63); }
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int t = lane + 64 * e;
        x[e] = __builtin_fma(-vk, w[e], __builtin_fma(-wk, v[e], x[e]));
        if ((k >> 6) == e) xk = lane_value(x[e], k & 63);
        if (((k + 1) >> 6) == e) x1 = lane_value(x[e], (k + 1) & 63);
        if (t > k + 1) q = __builtin_fma(x[e], x[e], q);
      }
      const double sigma = group_sum<64>(q);
      double off = k + 1 < D ? x1 : 0.0, v1 = 0.0;
      beta = 0.0;
      if (sigma > 0.0) {
        const double nrm = root(__builtin_fma(x1, x1, sigma));
        off = x1 > 0.0 ? -nrm : nrm;
        v1 = x1 - off;
        beta = 2.0 * recip(__builtin_fma(v1, v1, sigma));
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int t = lane + 64 * e;
        const double y = beta == 0.0 || t <= k ? 0.0 : (t == k + 1 ? v1 : x[e]);
        S.vn[t] = y;
        vecs[k * D + t] = y;
      }
      if (lane == 0) {
        S.al[k] = xk;
        S.be[k] = off;
        S.bt[k] = beta;
      }
    }
    __syncthreads();
    // the pending update of the previous reflection, and M v of the new one
    const double bk = S.bt[k];
    double acc[R], vi[R], wi[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      acc[j] = 0.0;
      vi[j] = S.v[row0 + 64 * j];
      wi[j] = S.w[row0 + 64 * j];
    }
#pragma unroll
    for (int m = 0; m < P; ++m) {
      if (16 * m + 15 <= k) continue;  // columns that are done
      const int c = 2 * sub + 16 * m;
      const f64x2 vc = *reinterpret_cast<const f64x2*>(&S.v[c]), wc = *reinterpret_cast<const f64x2*>(&S.w[c]),
                  nc = *reinterpret_cast<const f64x2*>(&S.vn[c]);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        if (64 * j + 63 <= k) continue;
        f64x2 y = a[j][m];
        y.x = __builtin_fma(-vi[j], wc.x, __builtin_fma(-wi[j], vc.x, y.x));
        y.y = __builtin_fma(-vi[j], wc.y, __builtin_fma(-wi[j], vc.y, y.y));
        a[j][m] = y;
        acc[j] = __builtin_fma(y.x, nc.x, __builtin_fma(y.y, nc.y, acc[j]));
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int i = row0 + 64 * j;
      const double s = group_sum<8>(acc[j]);
      if (sub == 0) S.p[i] = i > k ? bk * s : 0.0;
      if (i == k + 1)
#pragma unroll
        for (int m = 0; m < P; ++m) *reinterpret_cast<f64x2*>(&S.row[2 * sub + 16 * m]) = a[j][m];
    }
    __syncthreads();
  }

  // ---- 2. the r largest eigenvalues of T
  double gl = __builtin_inf(), gu = -__builtin_inf();
  for (int i = 0; i < D; ++i) {
    const double rad = (i > 0 ? fabs(S.be[i - 1]) : 0.0) + (i + 1 < D ? fabs(S.be[i]) : 0.0);
    gl = fmin(gl, S.al[i] - rad);
    gu = fmax(gu, S.al[i] + rad);
  }
  const double tnorm = fmax(fabs(gl), fabs(gu));
  const double tiny = fmax(tnorm, 0x1p-900) * 0x1p-104;  // stands in for a zero pivot
  gl -= tnorm * 0x1p-46;
  gu += tnorm * 0x1p-46;
  const int g32 = tid >> 5, l32 = tid & 31;
  for (int e = g32; e < kMaxRank; e += kLanes / 32) {
    if (e - (g32 & 1) >= r) break;  // wave-uniform: both 32-lane groups of the wave are past r
    const int want = D - 1 - e;     // eigenvalue e from the top has `want` below it
    double lo = gl, hi = gu;
    for (int round = 0; round < 11; ++round) {
      const double step = (hi - lo) * (1.0 / 33.0);
      const double x = __builtin_fma(step, (double)(l32 + 1), lo);
      int below = 0;
      double q = 1.0, b2 = 0.0;
      // q <- al - x - b2 / q, with 1 / q = y (1 + e + e^2) from a 24-bit y: the
      // chain is v_rcp_f64 and three fmas
#pragma unroll 16
      for (int i = 0; i < D; ++i) {
        const double y = __builtin_amdgcn_rcp(q), f = S.al[i] - x, t = b2 * y;
        const double e = __builtin_fma(-q, y, 1.0);
        q = __builtin_fma(-t, __builtin_fma(e, e, e), f - t);
        q = fabs(q) < tiny ? -tiny : q;
        below += q < 0.0;
        b2 = S.be[i] * S.be[i];
      }
      const uint64_t bal = __ballot(below > want);
      const uint32_t mine = uint32_t(bal >> (lane & 32));
      const int first = mine ? __ffs(mine) - 1 : 32;  // first point above the eigenvalue
      const double nlo = first > 0 ? __builtin_fma(step, (double)first, lo) : lo;
      hi = first < 32 ? __builtin_fma(step, (double)(first + 1), lo) : hi;
      lo = nlo;
    }
    if (l32 == 0 && e < r) S.lam[e] = 0.5 * (lo + hi);
  }
  __syncthreads();

  // ---- 3. eigenvectors of T. Rows of T - lam eliminated with partial pivoting:
  // row i of U is (1 / fd, fu, and T's next off-diagonal if rows i and i + 1
  // were swapped); bit i of `swaps` says so.
  uint64_t swaps[D / 64];
  const bool solver = wave == 0 && lane < r;
  if (solver) {
    const double lam = S.lam[lane];
    double p = S.al[0] - lam, u = S.be[0];
#pragma unroll
    for (int blk = 0; blk < D / 64; ++blk) {
      uint64_t sw = 0;
      for (int ii = 0; ii < 64; ++ii) {
        const int i = blk * 64 + ii;
        if (i + 1 < D) {
          const double b = S.be[i], an = S.al[i + 1] - lam, un = i + 2 < D ? S.be[i + 1] : 0.0;
          const bool s = fabs(b) > fabs(p);
          if (!s && fabs(p) < tiny) p = tiny;
          const double rp = recip(s ? b : p), l = (s ? p : b) * rp;
          S.fd[i][lane] = rp;
          S.fu[i][lane] = s ? an : u;
          S.fl[i][lane] = l;
          p = s ? __builtin_fma(-l, an, u) : __builtin_fma(-l, u, an);
          u = s ? -l * un : un;
          if (s) sw |= uint64_t(1) << ii;
        } else {
          if (fabs(p) < tiny) p = tiny;
          S.fd[i][lane] = recip(p);
        }
      }
      swaps[blk] = sw;
    }
  }
  for (int round = 0; round < 2; ++round) {
    if (solver) {
      // forward: L y = b. The first round's b is a fixed pseudo-random vector per eigenvalue
      double y = 0.0;
      uint32_t rng = 0x9e3779b9u * (uint32_t(lane) + 1u);
      auto rhs = [&](int i) -> double {
        if (round > 0) return S.z[lane][i];
        rng = rng * 1664525u + 1013904223u;
        return (double)int32_t(rng) * 0x1p-31 + (rng & 1024 ? 0.25 : -0.25);
      };
      y = rhs(0);
#pragma unroll
      for (int blk = 0; blk < D / 64; ++blk)
        for (int ii = 0; ii < 64; ++ii) {
          const int i = blk * 64 + ii;
          if (i + 1 >= D) break;
          const bool s = (swaps[blk] >> ii) & 1;
          const double bn = rhs(i + 1), l = S.fl[i][lane];
          S.z[lane][i] = s ? bn : y;
          y = s ? __builtin_fma(-l, bn, y) : __builtin_fma(-l, y, bn);
        }
      // backward: U x = y; the largest magnitude normalises against overflow
      double x1 = y * S.fd[D - 1][lane], x2 = 0.0, mx = fabs(x1);
      S.z[lane][D - 1] = x1;
#pragma unroll
      for (int blk = D / 64 - 1; blk >= 0; --blk)
        for (int ii = 63; ii >= 0; --ii) {
          const int i = blk * 64 + ii;
          if (i + 1 >= D) continue;
          const bool s = (swaps[blk] >> ii) & 1;
          double t = __builtin_fma(-S.fu[i][lane], x1, S.z[lane][i]);
          if (s && i + 2 < D) t = __builtin_fma(-S.be[i + 1], x2, t);
          x2 = x1;
          x1 = t * S.fd[i][lane];
          S.z[lane][i] = x1;
          mx = fmax(mx, fabs(x1));
        }
      const double sc = mx > 0.0 && mx < __builtin_inf() ? recip(mx) : 1.0;
      for (int i = 0; i < D; ++i) S.z[lane][i] *= sc;
    }
    __syncthreads();
    // modified Gram-Schmidt in order of decreasing eigenvalue, the whole set twice:
    // wave w holds vectors w, w + 8, ... in registers; vector e becomes a unit
    // vector and goes through LDS to the waves, which take its part out of theirs
    constexpr int NW = kLanes / 64, NV = kMaxRank / NW;
    double z[NV][NE];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int q = 0; q < NE; ++q) z[v][q] = v * NW + wave < r ? S.z[v * NW + wave][lane + 64 * q] : 0.0;
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int ev = 0; ev < NV; ++ev)
        for (int ew = 0; ew < NW; ++ew) {
          const int e = ev * NW + ew;
          if (e >= r) break;
          if (wave == ew) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NE; ++q) s = __builtin_fma(z[ev][q], z[ev][q], s);
            s = group_sum<64>(s);
            const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
            for (int q = 0; q < NE; ++q) {
              z[ev][q] *= inv;
              S.z[e][lane + 64 * q] = z[ev][q];
            }
          }
          __syncthreads();
          double u[NE];
#pragma unroll
          for (int q = 0; q < NE; ++q) u[q] = S.z[e][lane + 64 * q];
#pragma unroll
          for (int v = ev; v < NV; ++v) {
            if (v * NW + wave <= e) continue;
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NE; ++q) s = __builtin_fma(u[q], z[v][q], s);
            s = group_sum<64>(s);
#pragma unroll
            for (int q = 0; q < NE; ++q) z[v][q] = __builtin_fma(-s, u[q], z[v][q]);
          }
        }
    }
    __syncthreads();
  }

  // ---- 4. back-transformation z := H_0 ... H_{D-3} z: 16 lanes per vector, lane
  // l of the group holding elements 2 l + 32 m + {0, 1}
  constexpr int B = D / 32;
  const int e = tid >> 4, l16 = tid & 15;
  f64x2 z[B];
#pragma unroll
  for (int m = 0; m < B; ++m) z[m] = *reinterpret_cast<const f64x2*>(&S.z[e][2 * l16 + 32 * m]);
  if (wave * 4 < r) {
    f64x2 v[B];
    auto load = [&](int k) {
#pragma unroll
      for (int m = 0; m < B; ++m) v[m] = *reinterpret_cast<const f64x2*>(vecs + k * D + 2 * l16 + 32 * m);
    };
#pragma unroll 4
    for (int k = D - 3; k >= 0; --k) {
      load(k);
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < B; ++m) s = __builtin_fma(v[m].x, z[m].x, __builtin_fma(v[m].y, z[m].y, s));
      s = group_sum<16>(s) * S.bt[k];
#pragma unroll
      for (int m = 0; m < B; ++m) {
        z[m].x = __builtin_fma(-s, v[m].x, z[m].x);
        z[m].y = __builtin_fma(-s, v[m].y, z[m].y);
      }
    }
    // largest-magnitude entry positive, the lowest index on ties
    double big = -1.0, val = 0.0;
    int at = 0;
#pragma unroll
    for (int m = 0; m < B; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const double x = q ? z[m].y : z[m].x;
        if (fabs(x) > big) { big = fabs(x); val = x; at = 2 * l16 + 32 * m + q; }
      }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      const double ob = __shfl_xor(big, o), ov = __shfl_xor(val, o);
      const int oa = __shfl_xor(at, o);
      if (ob > big || (ob == big && oa < at)) { big = ob; val = ov; at = oa; }
    }
    const double sg = val < 0.0 ? -1.0 : 1.0;
    if (e < r) {
#pragma unroll
      for (int m = 0; m < B; ++m) {
        store_rn(uo + e * D + 2 * l16 + 32 * m, sg * z[m].x);
        store_rn(uo + e * D + 2 * l16 + 32 * m + 1, sg * z[m].y);
      }
      if (l16 == 0) lo_[e] = (float)ldexp(S.lam[e], ex);
    }
  }
}

template <typename T, int D>
hipError_t launch_basis_td(const quantwm_config& c, const double* m, int64_t div, bool cold, double* scratch,
                           uint8_t* calib, hipStream_t s) {
  static_assert(sizeof(BasisLds<D>) <= 160 * 1024, "LDS of one workgroup");
  // the dynamic LDS limit is raised once per device for this instance
  static std::atomic<uint64_t> raised{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
  if (!bit || !(raised.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)basis_kernel<T, D>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            int(sizeof(BasisLds<D>)));
    if (e != hipSuccess) return e;
    raised.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL((basis_kernel<T, D>), dim3((unsigned)(c.batch * c.heads)), dim3(kLanes), sizeof(BasisLds<D>), s,
                     m, div, int(cold), scratch, calib, calib_layout(c), c.rank, int(c.metric == QWM_METRIC_FULL));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_basis(const quantwm_config& c, const double* m, int64_t div, bool cold, double* scratch,
                        uint8_t* calib, hipStream_t s) {
  const bool bf = c.dtype == QWM_BF16;
  if (c.head_dim == 64)
    return bf ? launch_basis_td<bf16, 64>(c, m, div, cold, scratch, calib, s)
              : launch_basis_td<float, 64>(c, m, div, cold, scratch, calib, s);
  return bf ? launch_basis_td<bf16, 128>(c, m, div, cold, scratch, calib, s)
            : launch_basis_td<float, 128>(c, m, div, cold, scratch, calib, s);
}

}  // namespace qwm
