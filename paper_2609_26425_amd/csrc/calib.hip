// Calibration kernels for gfx950: the calibration block (centroids, channel
// sensitivities, principal basis) and the constants the append search derives
// from it; the historical Query second moment (Eq. 6) in fp64; and
// deterministic Lloyd K-means for the centroids (Eq. 3).
#include "qwm_common.h"

namespace qwm {
namespace {

__device__ inline float ldf(const float* p) { return *p; }
__device__ inline float ldf(const bf16* p) { return (float)*p; }

// double -> bf16 with one rounding (nearest, ties to even), for normal values.
__device__ inline bf16 to_bf16_rn(double x) {
  uint64_t u = __double_as_longlong(x);
  const uint64_t lsb = (u >> 45) & 1;
  u += (uint64_t(1) << 44) - 1 + lsb;
  u &= ~((uint64_t(1) << 45) - 1);
  return bf16((float)__longlong_as_double(u));  // exact: the value already fits bf16
}
__device__ inline void store_rn(float* p, double x) { *p = (float)x; }
__device__ inline void store_rn(bf16* p, double x) { *p = to_bf16_rn(x); }

// Eq. 12 group sums W_g, the expanded-distance constants of Eq. 9
// (a_jc = -2 (w_c mu_jc), b_j = sum_c (w_c mu_jc) mu_jc; Values use w = 1) and
// U_r in [d][r] order for the append kernel's per-channel PSAC accumulation.
// With the full metric the Key constants expand (k - mu_j)^T Mn (k - mu_j)
// instead: p_j = Mn mu_j (fp32, columns in order), a_jc = -2 p_jc and
// b_j = sum_c p_jc mu_jc; the k^T Mn k term is the same for every centroid.
//
// A block takes kDeriveRows centroids of one head (the first block of a head
// also its small fields). Latency bounds it (a serial b_j sum per centroid).
// Packing the tables and deriving these, 10 heads, 128 centroids, d = 128: 93 us
// with one block per head, 47 us with these blocks, 29 us without a branch per
// channel in the b_j sums (10 heads, 16 centroids, d = 64, fp32: 15, 18 and 9 us).
constexpr int kDeriveRows = 16;
template <typename T>
__global__ __launch_bounds__(256) void derive_kernel(uint8_t* calib, quantwm_calib_layout C, int d, int G,
                                                     int Kc, int r, int full) {
  uint8_t* slab = calib + int64_t(blockIdx.x) * C.slab_bytes;
  const int j0 = blockIdx.y * kDeriveRows, j1 = min(j0 + kDeriveRows, Kc);
  // the fields of a slab are disjoint: with the inputs marked so, the loops below
  // load ahead of their stores
  const float* __restrict__ w = reinterpret_cast<const float*>(slab + C.w);
  float* wg = reinterpret_cast<float*>(slab + C.wg);
  const T* __restrict__ mk = reinterpret_cast<const T*>(slab + C.mu_k);
  const T* __restrict__ mv = reinterpret_cast<const T*>(slab + C.mu_v);
  float* ak = reinterpret_cast<float*>(slab + C.a_k);
  float* bk = reinterpret_cast<float*>(slab + C.b_k);
  float* __restrict__ av = reinterpret_cast<float*>(slab + C.a_v);
  float* bv = reinterpret_cast<float*>(slab + C.b_v);
  const float* __restrict__ mm = reinterpret_cast<const float*>(slab + C.m);
#pragma unroll 8
  for (int i = j0 * d + threadIdx.x; i < j1 * d; i += 256) {
    const int c = i & (d - 1);  // d is 64 or 128
    const float mkv = ldf(mk + i), mvv = ldf(mv + i);
    if (full) {
      const T* mj = mk + (i - c);
      float p = 0.0f;
      for (int c2 = 0; c2 < d; ++c2) p = __builtin_fmaf(mm[c * d + c2], ldf(mj + c2), p);
      ak[i] = -2.0f * p;
    } else {
      ak[i] = -2.0f * (w[c] * mkv);
    }
    av[i] = -2.0f * mvv;
  }
  __syncthreads();  // b_k reads the a_k rows written by other threads
  if constexpr (sizeof(T) == 2) {
    // a_k as three BF16 planes with an exact sum, for the matrix-core search:
    // p0 keeps a's top 8 significant bits (truncated), p1 the top 8 of the exact
    // remainder a - p0, and p2 = a - p0 - p1, which has at most 8 significant
    // bits left and so is a BF16 value (for |a| above 2^-110 or so)
    uint16_t* __restrict__ pl = reinterpret_cast<uint16_t*>(slab + C.a_k3);
#pragma unroll 8
    for (int i = j0 * d + threadIdx.x; i < j1 * d; i += 256) {
      const float av0 = ak[i];
      const uint32_t u0 = __float_as_uint(av0) & 0xffff0000u;
      const float r1 = av0 - __uint_as_float(u0);
      const uint32_t u1 = __float_as_uint(r1) & 0xffff0000u;
      const float r2 = r1 - __uint_as_float(u1);
      pl[i] = uint16_t(u0 >> 16);
      pl[Kc * d + i] = uint16_t(u1 >> 16);
      pl[2 * Kc * d + i] = __builtin_bit_cast(uint16_t, bf16(r2));
    }
  }
  if (threadIdx.x < 2 * kDeriveRows) {
    // even threads the Keys' b_j, odd ones the Values'
    const int j = j0 + threadIdx.x / 2;
    const bool val = threadIdx.x & 1;
    if (j < j1) {
      float acc = 0.0f;
      const T* __restrict__ mu = (val ? mv : mk) + j * d;
      if (full) {
#pragma unroll 8
        for (int c = 0; c < d; ++c) {
          const float m = ldf(mu + c), p = -0.5f * ak[j * d + c];  // p_jc exactly
          acc = __builtin_fmaf(val ? m : p, m, acc);
        }
      } else {
        // every load on both sides: no branch per channel
#pragma unroll 16
        for (int c = 0; c < d; ++c) {
          const float m = ldf(mu + c), wc = w[c];
          acc = __builtin_fmaf(val ? m : wc * m, m, acc);
        }
      }
      (val ? bv : bk)[j] = acc;
    }
  }
  if (blockIdx.y == 0) {
    for (int g = threadIdx.x; g < d / G; g += 256) {
      float s = 0.0f;
      for (int c = g * G; c < (g + 1) * G; ++c) s = s + w[c];
      wg[g] = s;
    }
    const T* ut = reinterpret_cast<const T*>(slab + C.u_t);
    float* udr = reinterpret_cast<float*>(slab + C.u_dr);
    const int rs = r == 0 ? 0 : (r <= 16 ? 16 : 32);
    for (int i = threadIdx.x; i < rs * d; i += 256) {
      const int c = rs == 16 ? i >> 4 : i >> 5, k = i & (rs - 1);
      udr[i] = k < r ? ldf(ut + k * d + c) : 0.0f;
    }
  }
  if constexpr (sizeof(T) == 2) {
    // binary16 copies of the BF16 tables for the attention producers, scaled by a
    // power of two: the table's largest magnitude lands in [2^14, 2^15), so each
    // component of at least 2^-31 of it is exact in binary16 (BF16 keeps 8
    // significant bits) and none overflows. Every block scans the whole tables.
    __shared__ float s_max[2][256];
    float mx[2] = {0.0f, 0.0f};
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const uint4* p = reinterpret_cast<const uint4*>(side ? mv : mk);
#pragma unroll 4
      for (int i = threadIdx.x; i < Kc * d / 8; i += 256) {
        const uint4 u = p[i];
        const uint32_t q[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
          mx[side] = fmaxf(mx[side], fmaxf(fabsf(__uint_as_float(q[k] << 16)), fabsf(__uint_as_float(q[k] & 0xffff0000u))));
      }
    }
    s_max[0][threadIdx.x] = mx[0];
    s_max[1][threadIdx.x] = mx[1];
    __syncthreads();
    for (int st = 128; st > 0; st /= 2) {
      if (threadIdx.x < st) {
        s_max[0][threadIdx.x] = fmaxf(s_max[0][threadIdx.x], s_max[0][threadIdx.x + st]);
        s_max[1][threadIdx.x] = fmaxf(s_max[1][threadIdx.x], s_max[1][threadIdx.x + st]);
      }
      __syncthreads();
    }
    int ek = 0, ev = 0;
    if (s_max[0][0] > 0.0f) { int x; frexpf(s_max[0][0], &x); ek = x - 15; }  // max in [2^(x-1), 2^x)
    if (s_max[1][0] > 0.0f) { int x; frexpf(s_max[1][0], &x); ev = x - 15; }
    _Float16* __restrict__ hk = reinterpret_cast<_Float16*>(slab + C.mu_k16);
    _Float16* __restrict__ hv = reinterpret_cast<_Float16*>(slab + C.mu_v16);
#pragma unroll 8
    for (int i = j0 * d + threadIdx.x; i < j1 * d; i += 256) {
      hk[i] = (_Float16)ldexpf(ldf(mk + i), -ek);
      hv[i] = (_Float16)ldexpf(ldf(mv + i), -ev);
    }
    if (threadIdx.x == 0 && blockIdx.y == 0) {
      int32_t* e16 = reinterpret_cast<int32_t*>(slab + C.e16);
      e16[0] = ek;
      e16[1] = ev;
    }
  }
}

// Copy method-level tables into the slabs: mu [BH][Kc][d], w [BH][d],
// u_t [BH][r][d] (zeros if null), lam [BH][r] (zeros if null), and the full
// metric's matrix m [BH][d][d] when given.
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(uint8_t* calib, quantwm_calib_layout C, int d, int Kc, int r,
                                                   const T* mu_k, const T* mu_v, const float* w, const T* u_t,
                                                   const float* lam, const float* m) {
  const int64_t bh = blockIdx.x;
  uint8_t* slab = calib + bh * C.slab_bytes;
  T* mk = reinterpret_cast<T*>(slab + C.mu_k);
  T* mv = reinterpret_cast<T*>(slab + C.mu_v);
  T* ut = reinterpret_cast<T*>(slab + C.u_t);
  float* wo = reinterpret_cast<float*>(slab + C.w);
  float* lo = reinterpret_cast<float*>(slab + C.lam);
  for (int i = threadIdx.x; i < Kc * d; i += 256) {
    mk[i] = mu_k[bh * Kc * d + i];
    mv[i] = mu_v[bh * Kc * d + i];
  }
  for (int i = threadIdx.x; i < d; i += 256) wo[i] = w[bh * d + i];
  for (int i = threadIdx.x; i < r * d; i += 256) ut[i] = u_t ? u_t[bh * r * d + i] : T(0.0f);
  for (int i = threadIdx.x; i < r; i += 256) lo[i] = lam ? lam[bh * r + i] : 0.0f;
  if (m) {
    float* mo = reinterpret_cast<float*>(slab + C.m);
    for (int i = threadIdx.x; i < d * d; i += 256) mo[i] = m[bh * d * d + i];
  }
}

// Eight consecutive channels as doubles
__device__ inline void load8(const float* p, double (&x)[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
  x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
__device__ inline void load8(const bf16* p, double (&x)[8]) {
  const uint4 u = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[2 * k] = (double)__uint_as_float(w[k] << 16);
    x[2 * k + 1] = (double)__uint_as_float(w[k] & 0xffff0000u);
  }
}

// Eq. 6: sums of q_i q_j over the tokens in order, in fp64 (each fp32 x fp32
// product is exact in fp64). ACC continues the stored sums of a statistics
// buffer, so a sequence of updates equals one pass over all the tokens, and
// adds n to *count; otherwise the sums start at 0 and are divided by n, and the
// tiles below the diagonal mirror those above (the product commutes).
//
// A block takes a 32 x 32 tile of one head's matrix, a wave 16 x 16 of it on the
// fp64 matrix cores: v_mfma_f64_16x16x4 adds four tokens as a chain of fmas in
// token order (the tests compare bits with that chain). 64 tokens at a time are
// staged in LDS as doubles, the next 64 loading while these multiply; rows are
// padded so that a wave's operand reads are free of bank conflicts. One matrix
// instruction per four tokens and wave is the chain that bounds it, so the tiles
// are small to spread a head over many CUs. 4,680 tokens of 10 heads at d = 128
// (ACC): 1,230 us with a thread per element and no staging, 260 us with 2 x 2
// elements per thread on the vector unit (bound by LDS reads), 124 us so.
constexpr int kMomTile = 32, kMomTok = 64, kMomRow = kMomTile + 16;
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <typename T, bool ACC>
__global__ __launch_bounds__(256) void moment_kernel(const T* q, int64_t n, int heads, int d, double* m,
                                                     int64_t* count) {
  __shared__ __attribute__((aligned(16))) double s_q[2][kMomTok][kMomRow];
  const int64_t bh = blockIdx.y;
  const int b = int(bh / heads), h = int(bh % heads), tid = threadIdx.x;
  const int nt = d / kMomTile;
  int ti = 0, tj = blockIdx.x;  // tile row and column: all of them, or those with ti <= tj
  if constexpr (ACC) {
    ti = blockIdx.x / nt;
    tj = blockIdx.x % nt;
  } else {
    while (tj >= nt - ti) { tj -= nt - ti; ++ti; }
    tj += ti;
  }
  const T* base = q + (int64_t(b) * n * heads + h) * d;
  const int64_t stride = int64_t(heads) * d;
  // staging: thread -> (token, eight channels) of each side; zeros past the last token
  const int st = tid / 4, sc = (tid % 4) * 8;
  double xi[8], xj[8];
  auto fetch = [&](int64_t t0) {
    const bool in = t0 + st < n;
    const int64_t t = in ? t0 + st : n - 1;
    load8(base + t * stride + ti * kMomTile + sc, xi);
    load8(base + t * stride + tj * kMomTile + sc, xj);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      xi[k] = in ? xi[k] : 0.0;
      xj[k] = in ? xj[k] : 0.0;
    }
  };
  // wave w: 16 x 16 elements at (16 (w / 2), 16 (w % 2)) of the tile; accumulator
  // slot i of lane l is row 4 i + l / 16, column l % 16
  const int lane = tid & 63, w = tid >> 6, l16 = lane & 15, lk = lane >> 4;
  const int i0 = (w / 2) * 16, j0 = (w % 2) * 16;
  double* mh = m + bh * d * d;
  const int gi = ti * kMomTile + i0 + lk, gj = tj * kMomTile + j0 + l16;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  if constexpr (ACC)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = mh[(gi + 4 * i) * d + gj];
  fetch(0);
  for (int64_t t0 = 0; t0 < n; t0 += kMomTok) {
    __syncthreads();  // the previous tokens are used up
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
      *reinterpret_cast<double2*>(&s_q[0][st][sc + k]) = make_double2(xi[k], xi[k + 1]);
      *reinterpret_cast<double2*>(&s_q[1][st][sc + k]) = make_double2(xj[k], xj[k + 1]);
    }
    __syncthreads();
    if (t0 + kMomTok < n) fetch(t0 + kMomTok);
#pragma unroll
    for (int t = 0; t < kMomTok; t += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s_q[0][t + lk][i0 + l16], s_q[1][t + lk][j0 + l16], acc, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double x = ACC ? acc[i] : acc[i] / (double)n;
    mh[(gi + 4 * i) * d + gj] = x;
    if (!ACC && ti != tj) mh[gj * d + gi + 4 * i] = x;
  }
  if (ACC && bh == 0 && blockIdx.x == 0 && tid == 0) *count += n;
}

// K-means (Eq. 3) of the Keys (side 0) and Values (side 1) of every head, both
// sides in each launch.
struct KmArgs {
  const void* x[2];     // [B, n, H, d]
  int64_t o_mu[2];      // tables in the slab
  int64_t o_b[2];       // [Kc] f32 in the slab: |mu_j|^2 between the rounds (derive_kernel overwrites them)
  uint8_t* assign;      // [2][BH][n]
  uint8_t* calib;
  int64_t slab, n;
  int heads, d, Kc, bh;
};

// sum over the block's d threads (one or two waves), the same on each
__device__ inline float block_sum(float v, int d, float* lds) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if (d == 64) return v;
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  return lds[0] + lds[1];
}

// Initial centroids: tokens floor(j n / Kc). One block of d threads per centroid.
template <typename T>
__global__ __launch_bounds__(128) void km_init_kernel(const KmArgs a) {
  __shared__ float s_red[2];
  const int j = blockIdx.x, c = threadIdx.x, side = blockIdx.z;
  const int64_t bh = blockIdx.y;
  const int b = int(bh / a.heads), h = int(bh % a.heads);
  uint8_t* slab = a.calib + bh * a.slab;
  const int64_t t = (int64_t(j) * a.n) / a.Kc;
  const T v = reinterpret_cast<const T*>(a.x[side])[((int64_t(b) * a.n + t) * a.heads + h) * a.d + c];
  reinterpret_cast<T*>(slab + a.o_mu[side])[j * a.d + c] = v;
  const float f = ldf(&v), s = block_sum(f * f, a.d, s_red);
  if (c == 0) reinterpret_cast<float*>(slab + a.o_b[side])[j] = s;
}

// Squared Euclidean distance in channel order (fp32, no contraction): the
// literal form that decides every assignment. Rows are 16-byte aligned.
template <int D>
__device__ inline float literal_distance(const bf16* x, const uint4* mu) {
  float acc = 0.0f;
#pragma unroll 4
  for (int c = 0; c < D; c += 8) {
    const uint4 u = *reinterpret_cast<const uint4*>(x + c), m = mu[c / 8];
    const uint32_t xw[4] = {u.x, u.y, u.z, u.w}, mw[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float e0 = __uint_as_float(xw[k] << 16) - __uint_as_float(mw[k] << 16);
      acc = acc + e0 * e0;
      const float e1 = __uint_as_float(xw[k] & 0xffff0000u) - __uint_as_float(mw[k] & 0xffff0000u);
      acc = acc + e1 * e1;
    }
  }
  return acc;
}

// Lloyd assignment of fp32 tokens: nearest centroid by the literal distance,
// ties to the lower id.
template <typename T, int D>
__global__ __launch_bounds__(256) void km_assign_kernel(const KmArgs a) {
  const int64_t bh = blockIdx.y, n = a.n;
  const int side = blockIdx.z;
  const int b = int(bh / a.heads), h = int(bh % a.heads);
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= n) return;
  const T* __restrict__ mu = reinterpret_cast<const T*>(a.calib + bh * a.slab + a.o_mu[side]);
  const T* row = reinterpret_cast<const T*>(a.x[side]) + ((int64_t(b) * n + t) * a.heads + h) * D;
  float xv[D];
#pragma unroll
  for (int c = 0; c < D; ++c) xv[c] = ldf(row + c);
  int best = 0;
  float bd = 0.0f;
  for (int j = 0; j < a.Kc; ++j) {
    float acc = 0.0f;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const float e = xv[c] - ldf(mu + j * D + c);
      acc = acc + e * e;
    }
    if (j == 0 || acc < bd) { best = j; bd = acc; }
  }
  a.assign[(int64_t(side) * a.bh + bh) * n + t] = uint8_t(best);
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Lloyd assignment of BF16 tokens: the literal distance decides, but it is only
// evaluated where it can matter. The matrix cores give d'_j = |mu_j|^2 - 2 x.mu_j
// for 32 centroids x 32 tokens at a time (a wave's tokens; lanes i and i + 32
// share token i and hold 16 centroids each per block). With u = 2^-24,
// S = |x|^2 + max_j |mu_j|^2 and D_j the real squared distance:
//   - the products are exact and the fp32 sum of the d terms of x.mu_j errs by at
//     most (d + 16) u |x| |mu_j|, doubled here for a sum in any grouping; with the
//     sum of |mu_j|^2 and the last rounding d'_j is within E = 2 (d + 32) u S;
//   - the literal distance (three roundings per term, d terms) is within
//     (d + 4) u D_j of D_j;
//   - a product or a sum below the normal range may lose up to 2^-126 each time, on
//     either side: E also carries 4 (d + 32) 2^-126.
// With D_1 the distance of the smallest d', a centroid whose d' exceeds that by
// more than 2 E + 2 (d + 4) u (D_1 + E), and a little, has the larger literal
// distance. Where a second centroid is inside that bound, a second pass over the
// same products evaluates the literal distance of every centroid inside it.
// The table is staged in LDS for the workgroup's 128 tokens (rows padded by 16
// bytes: operand reads free of bank conflicts); read from global memory, a row
// per lane, the loads' cache-line lookups bounded it. Latency does now; 4,680
// tokens of 10 heads, 128 centroids, Keys and Values: 660 us for the two literal
// launches, 39 us with the rows from global memory, 22 us so.
template <int D>
struct KmAssignLds {
  uint4 mu[256 * (D / 8 + 1)];
  float b[256];
};
template <int D>
__global__ __launch_bounds__(256) void km_assign_mfma_kernel(const KmArgs a) {
  constexpr int NS = D / 16, PR = D / 8 + 1;  // 16-byte pieces of a padded row
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  uint4* s_mu = reinterpret_cast<uint4*>(smem_raw);
  float* s_b = reinterpret_cast<float*>(smem_raw + size_t(a.Kc) * PR * 16);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n32 = lane & 31, hf = lane >> 5;
  const int64_t bh = blockIdx.y, n = a.n;
  const int side = blockIdx.z, Kc = a.Kc;
  const int b = int(bh / a.heads), h = int(bh % a.heads);
  const int64_t t0 = int64_t(blockIdx.x) * 128 + wv * 32;
  const int64_t t = t0 + n32 < n ? t0 + n32 : n - 1;
  const uint8_t* slab = a.calib + bh * a.slab;
  const bf16* mu = reinterpret_cast<const bf16*>(slab + a.o_mu[side]);
  const float* bj = reinterpret_cast<const float*>(slab + a.o_b[side]);
  const bf16* row = reinterpret_cast<const bf16*>(a.x[side]) + ((int64_t(b) * n + t) * a.heads + h) * D;
#pragma unroll 8
  for (int i = threadIdx.x; i < Kc * (D / 8); i += 256)
    s_mu[i / (D / 8) * PR + i % (D / 8)] = reinterpret_cast<const uint4*>(mu)[i];
  // a NaN norm (a NaN centroid) counts as infinite, so that the bound below is too
  for (int i = threadIdx.x; i < Kc; i += 256) s_b[i] = bj[i] == bj[i] ? bj[i] : __builtin_inff();
  // k index 8 hf + i of step s is channel 16 s + 8 hf + i on both operands
  bf16x8 xf[NS];
  float xx = 0.0f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    xf[s] = *reinterpret_cast<const bf16x8*>(row + 16 * s + 8 * hf);
#pragma unroll
    for (int k = 0; k < 8; ++k) xx = __builtin_fmaf((float)xf[s][k], (float)xf[s][k], xx);
  }
  xx += __shfl_xor(xx, 32);
  __syncthreads();
  if (t0 >= n) return;  // the whole wave is past the chunk
  auto block = [&](int j0, float (&d)[16]) __attribute__((always_inline)) {
    const uint4* mrow = s_mu + min(j0 + n32, Kc - 1) * PR + hf;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, mrow[2 * s]), xf[s], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int j = j0 + (i / 4) * 8 + hf * 4 + (i % 4);
      d[i] = j < Kc ? __builtin_fmaf(-2.0f, acc[i], s_b[j]) : __builtin_inff();
    }
  };
  float d1 = __builtin_inff(), d2 = __builtin_inff(), bmax = 0.0f;
  int best = 0;
  for (int j0 = 0; j0 < Kc; j0 += 32) {
    float d[16];
    block(j0, d);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int j = j0 + (i / 4) * 8 + hf * 4 + (i % 4);
      bmax = fmaxf(bmax, j < Kc ? s_b[j] : 0.0f);
      d2 = fminf(d2, fmaxf(d1, d[i]));
      best = d[i] < d1 ? j : best;
      d1 = fminf(d1, d[i]);
    }
  }
  {
    const float p1 = __shfl_xor(d1, 32), p2 = __shfl_xor(d2, 32);
    const int pb = __shfl_xor(best, 32);
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
    d2 = fminf(fminf(d2, p2), fmaxf(d1, p1));
    best = p1 < d1 ? pb : best;  // a tie is inside the bound and decided below
    d1 = fminf(d1, p1);
  }
  const float E = 2.0f * (D + 32) * 0x1p-24f * (xx + bmax) + 4.0f * (D + 32) * 0x1p-126f;
  const float bound = 1.01f * (2.0f * E + 2.0f * (D + 4) * 0x1p-24f * (fmaxf(d1 + xx, 0.0f) + E));
  // not greater rather than less or equal: with NaN or infinite inputs the bound is NaN or
  // infinite, and the token takes the literal form over every centroid
  const bool near = !(d2 - d1 > bound);
  if (__any(near)) {
    int lb = 0x7fffffff;
    float ld = __builtin_inff();
    for (int j0 = 0; j0 < Kc; j0 += 32) {
      float d[16];
      block(j0, d);
      // every candidate of this lane in the block, in increasing order
      uint32_t cand = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) cand |= uint32_t(near && !(d[i] - d1 > bound)) << i;
      while (cand) {
        const int i = __ffs(cand) - 1, j = j0 + (i / 4) * 8 + hf * 4 + (i % 4);
        cand &= cand - 1;
        if (j < Kc) {
          const float l = literal_distance<D>(row, s_mu + j * PR);
          if (j == 0 || l < ld) { lb = j; ld = l; }  // as the serial scan: a NaN only stays as id 0
        }
      }
    }
    const float pd = __shfl_xor(ld, 32);
    const int pb = __shfl_xor(lb, 32);
    if (pb != 0x7fffffff && (lb == 0x7fffffff || pd < ld || (pd == ld && pb < lb))) lb = pb;
    if (near && lb != 0x7fffffff) best = lb;
  }
  if (hf == 0 && t0 + n32 < n) a.assign[(int64_t(side) * a.bh + bh) * n + t] = uint8_t(best);
}

// Lloyd update: sums x_tc over the tokens of cluster j in token order (fp64),
// then stores the mean rounded once to the table type; an empty cluster keeps
// its centroid. A wave per (cluster, head, side): it lists the cluster's tokens of
// a run of kKmList in order (each lane scans kKmList / 64 ids, four at a time as
// the zero bytes of ids ^ j, keeping the finds as bits; a prefix sum places them),
// then every lane adds its D / 64 channels over the list, 16 to 32 rows in flight.
// 4,680 tokens of 10 heads, 128 centroids, Keys and Values: 665 us when each
// (cluster, channel) scanned all ids, 30 us with a block of D lanes that read its
// ids again to list them, 26 us with runs of 4,096 ids, 23 us so.
constexpr int kKmList = 8192, kKmRows = 16;
template <typename T, int D>
__global__ __launch_bounds__(64) void km_update_kernel(const KmArgs a) {
  constexpr int PT = kKmList / 64, NE = D / 64;  // ids per lane and run, channels per lane
  __shared__ uint16_t s_list[kKmList];
  const int j = blockIdx.x, lane = threadIdx.x, side = blockIdx.z;
  const int64_t bh = blockIdx.y, n = a.n;
  const int b = int(bh / a.heads), h = int(bh % a.heads);
  const uint8_t* as = a.assign + (int64_t(side) * a.bh + bh) * n;
  typedef T Row __attribute__((ext_vector_type(NE)));
  const T* x = reinterpret_cast<const T*>(a.x[side]) + (int64_t(b) * n * a.heads + h) * D + lane * NE;
  const int64_t stride = int64_t(a.heads) * D;
  double sum[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) sum[e] = 0.0;
  int64_t cnt = 0;
  for (int64_t run = 0; run < n; run += kKmList) {
    const int nr = n - run < kKmList ? int(n - run) : kKmList;
    // ids of this lane: [lo, hi) of the run, shared out evenly in multiples of 4
    const int per = ((nr + 63) / 64 + 3) / 4 * 4;
    const int lo = min(nr, lane * per), hi = min(nr, lo + per);
    uint32_t hits[PT / 4];  // bit 8 k + 7: id 4 i + k of the lane's share is j
    int mine = 0;
    // every load first (a word that would pass the run's end starts earlier)
    uint32_t w[PT / 4];
    if (nr >= 4) {
#pragma unroll
      for (int i = 0; i < PT / 4; ++i) __builtin_memcpy(&w[i], as + run + min(lo + 4 * i, nr - 4), 4);
    } else {
#pragma unroll
      for (int i = 0; i < PT / 4; ++i) w[i] = 0;
      for (int k = 0; k < nr; ++k) w[0] |= uint32_t(as[run + k]) << (8 * k);
    }
#pragma unroll
    for (int i = 0; i < PT / 4; ++i) {
      const int at = lo + 4 * i, left = min(4, hi - at);  // ids of the word that are the lane's
      const int back = nr >= 4 ? max(0, at - (nr - 4)) : 0;
      uint32_t v = left > 0 ? w[i] >> (8 * min(back, 3)) : 0;
      v ^= uint32_t(j) * 0x01010101u;
      // the top bit of every byte that is zero
      hits[i] = ~(((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & (left > 0 ? 0x80808080u >> (8 * (4 - left)) : 0u);
      mine += __popc(hits[i]);
    }
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      incl += lane >= o ? y : 0;
    }
    const int total = __shfl(incl, 63);
    int at = incl - mine;
    __syncthreads();  // the previous run's list is used up
#pragma unroll
    for (int i = 0; i < PT / 4; ++i)
      for (uint32_t m = hits[i]; m; m &= m - 1) s_list[at++] = uint16_t(lo + 4 * i + (__ffs(m) - 1) / 8);
    __syncthreads();
    // the next rows load while these are added
    Row v[kKmRows], u[kKmRows];
    auto rows = [&](Row (&r)[kKmRows], int i) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < kKmRows; ++k)
        r[k] = *reinterpret_cast<const Row*>(x + (run + s_list[min(i + k, total - 1)]) * stride);
    };
    auto add = [&](const Row (&r)[kKmRows], int i) __attribute__((always_inline)) {
      const int m = total - i;
      if (m >= kKmRows) {
#pragma unroll
        for (int k = 0; k < kKmRows; ++k)
#pragma unroll
          for (int e = 0; e < NE; ++e) sum[e] += (double)(float)r[k][e];
      } else {
#pragma unroll
        for (int k = 0; k < kKmRows; ++k)
          if (k < m)
#pragma unroll
            for (int e = 0; e < NE; ++e) sum[e] += (double)(float)r[k][e];
      }
    };
    if (total > 0) rows(v, 0);
    for (int i = 0; i < total; i += 2 * kKmRows) {
      if (i + kKmRows < total) rows(u, i + kKmRows);
      add(v, i);
      if (i + 2 * kKmRows < total) rows(v, i + 2 * kKmRows);
      if (i + kKmRows < total) add(u, i + kKmRows);
    }
    cnt += total;
  }
  if (cnt == 0) return;  // block-uniform
  uint8_t* slab = a.calib + bh * a.slab;
  T* mu = reinterpret_cast<T*>(slab + a.o_mu[side]) + j * D + lane * NE;
  float s = 0.0f;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    T m;
    store_rn(&m, sum[e] / (double)cnt);
    mu[e] = m;
    s = __builtin_fmaf(ldf(&m), ldf(&m), s);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) reinterpret_cast<float*>(slab + a.o_b[side])[j] = s;
}

template <typename T, int D>
hipError_t kmeans_td(const KmArgs& a, int iters, hipStream_t s) {
  const dim3 gc((unsigned)a.Kc, (unsigned)a.bh, 2);
  const size_t lds = size_t(a.Kc) * (D / 8 + 1) * 16 + size_t(a.Kc) * 4;
  if constexpr (sizeof(T) == 2) {
    if (lds > 64 * 1024) {  // above what a launch gets unasked (160 KB per CU on MI355X)
      const hipError_t e = hipFuncSetAttribute((const void*)km_assign_mfma_kernel<D>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(sizeof(KmAssignLds<D>)));
      if (e != hipSuccess) return e;
    }
  }
  hipLaunchKernelGGL(km_init_kernel<T>, gc, dim3(D), 0, s, a);
  for (int it = 0; it < iters; ++it) {
    if constexpr (sizeof(T) == 2)
      hipLaunchKernelGGL((km_assign_mfma_kernel<D>), dim3((unsigned)((a.n + 127) / 128), (unsigned)a.bh, 2), dim3(256),
                         lds, s, a);
    else
      hipLaunchKernelGGL((km_assign_kernel<T, D>), dim3((unsigned)((a.n + 255) / 256), (unsigned)a.bh, 2), dim3(256),
                         0, s, a);
    hipLaunchKernelGGL((km_update_kernel<T, D>), gc, dim3(64), 0, s, a);
  }
  return hipGetLastError();
}

template <typename T>
void launch_moment_t(const quantwm_config& c, const T* q, int64_t n, double* m, int64_t* count, hipStream_t s) {
  const int nt = c.head_dim / kMomTile;
  const unsigned bh = unsigned(c.batch * c.heads);
  if (count)
    hipLaunchKernelGGL((moment_kernel<T, true>), dim3(unsigned(nt * nt), bh), dim3(256), 0, s, q, n, c.heads,
                       c.head_dim, m, count);
  else
    hipLaunchKernelGGL((moment_kernel<T, false>), dim3(unsigned(nt * (nt + 1) / 2), bh), dim3(256), 0, s, q, n,
                       c.heads, c.head_dim, m, count);
}

}  // namespace

hipError_t launch_derive_constants(const quantwm_config& c, uint8_t* calib, hipStream_t s) {
  const quantwm_calib_layout C = calib_layout(c);
  const dim3 grid((unsigned)(c.batch * c.heads), (unsigned)((c.n_centroids + kDeriveRows - 1) / kDeriveRows));
  const int full = c.metric == QWM_METRIC_FULL;
  if (c.dtype == QWM_BF16)
    hipLaunchKernelGGL(derive_kernel<bf16>, grid, dim3(256), 0, s, calib, C, c.head_dim, c.group_size, c.n_centroids,
                       c.rank, full);
  else
    hipLaunchKernelGGL(derive_kernel<float>, grid, dim3(256), 0, s, calib, C, c.head_dim, c.group_size, c.n_centroids,
                       c.rank, full);
  return hipGetLastError();
}

hipError_t launch_pack_tables(const quantwm_config& c, const void* mu_k, const void* mu_v, const float* w,
                              const void* u_t, const float* lam, const float* m, uint8_t* calib, hipStream_t s) {
  const quantwm_calib_layout C = calib_layout(c);
  const dim3 grid((unsigned)(c.batch * c.heads));
  if (c.dtype == QWM_BF16)
    hipLaunchKernelGGL(pack_kernel<bf16>, grid, dim3(256), 0, s, calib, C, c.head_dim, c.n_centroids, c.rank,
                       (const bf16*)mu_k, (const bf16*)mu_v, w, (const bf16*)u_t, lam, m);
  else
    hipLaunchKernelGGL(pack_kernel<float>, grid, dim3(256), 0, s, calib, C, c.head_dim, c.n_centroids, c.rank,
                       (const float*)mu_k, (const float*)mu_v, w, (const float*)u_t, lam, m);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_derive_constants(c, calib, s);
}

// Eq. 6 over n tokens: the mean of q q^T into m, or (count given) the sums continued and n added to *count.
hipError_t launch_moment(const quantwm_config& c, const void* q, int64_t n, double* m, int64_t* count, hipStream_t s) {
  if (c.dtype == QWM_BF16) launch_moment_t<bf16>(c, (const bf16*)q, n, m, count, s);
  else launch_moment_t<float>(c, (const float*)q, n, m, count, s);
  return hipGetLastError();
}

hipError_t launch_kmeans(const quantwm_config& c, const void* k, const void* v, int64_t n, int iters, uint8_t* calib,
                         uint8_t* assign, hipStream_t s) {
  const quantwm_calib_layout C = calib_layout(c);
  const KmArgs a = {{k, v}, {C.mu_k, C.mu_v}, {C.b_k, C.b_v}, assign, calib, C.slab_bytes, n,
                    c.heads, c.head_dim, c.n_centroids, c.batch * c.heads};
  if (c.dtype == QWM_BF16) return c.head_dim == 64 ? kmeans_td<bf16, 64>(a, iters, s) : kmeans_td<bf16, 128>(a, iters, s);
  return c.head_dim == 64 ? kmeans_td<float, 64>(a, iters, s) : kmeans_td<float, 128>(a, iters, s);
}

}  // namespace qwm
