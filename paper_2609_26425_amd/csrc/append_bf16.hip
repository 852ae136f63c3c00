// Quantize-on-append for BF16 Keys and Values on gfx950: QSAC centroid choice
// (Sec. 4.1, Eq. 9-12), group-wise INT2 residual (Eq. 1-4, App. D.1) and PSAC
// coefficients (Sec. 4.2, Eq. 13 and 16) for Keys; nearest centroid + INT2
// residual for Values. The outputs are those of the fp32 kernel; the two
// centroid searches run on the matrix cores.
//
// Mapping: a wave takes 32 consecutive tokens of one (b, h); a workgroup of up to
// eight waves shares the tables, staged in LDS: the Key table for the whole Key
// part, the search planes of one 32-centroid block at a time (double-buffered),
// then the Value table, loaded while the Keys are quantised. Lanes i and i + 32 share token i and split its channels: lane half
// hf owns channels [hf d/2, (hf + 1) d/2).
//
// Searches. Both are dense products of a (Kc x d) table with the wave's (d x 32)
// tokens,
//     d'_j(t) = b_j + sum_c a_jc x_c(t),
// the expanded Eq. 9 distance (a_jc = -2 w_c mu_jc, b_j = sum_c w_c mu_jc^2) minus
// the centroid-independent sum_c w_c x_c^2, one v_mfma_f32_32x32x16_bf16 per 32
// centroids and 16 channels. The instruction's k index 8 hf + i of step s maps
// to channel hf d/2 + 8 s + i on both operands, so the B operand is the lane's
// own half-row: the token rows load once, straight into operand registers. The
// Key constants a_jc are fp32; the calibration block holds them as three BF16
// planes with an exact sum, so every product is exact in fp32 and only the
// accumulation rounds. The Value table is BF16 and the Value distance uses
// w = 1: the accumulator starts at -b_j / 2, sums mu_jc v_c, and d' is -2 times
// the result, the value the -2 v_c products would give (powers of two scale
// every rounding exactly).
//
// Selection. Each lane keeps only the M smallest distances of its candidates (one
// v_med3_f32 per list position and candidate); the pair merges its two lists to
// the M-th smallest distance T of the token, and the candidates are the ids with
// d' <= T, gathered as a bit per centroid from the distances, which stay in
// registers. Carrying the ids in the lists took 17 instructions per
// candidate instead of 6. Where more than M ids qualify (equal distances at T) the
// wave redoes the selection with lists of (d', id).
//
// Score. The M candidates' ranges are taken in one pass over the token, so their
// rows load together and a token word is unpacked once for all of them; the
// chosen one's ranges are those of the residual, which then needs no range pass.
//
// Residual and PSAC. Each lane quantises its half-row. Group ranges of a group
// that spans both halves, the 8-bit scales' shared maximum and the Eq. 12 sum
// over groups (added in group order) are combined across the pair with
// v_permlane32_swap. The PSAC projection E U_r runs on the matrix cores as
// well: the errors of each 8-channel residual chunk are the B operand of one k
// step, and each lane quantises the ranks that its accumulator holds.
// Everything that turns a float into an integer follows the equations'
// operation order in fp32 with IEEE division and round-to-nearest-even, as in
// the fp32 kernel.
//
// What bounds it: vector issue (about 6,100 instructions per wave at 128
// centroids, d = 128: 60% of the SIMDs' cycles) and the latency of its chains at two
// waves per SIMD. With
// every lane reading centroid rows from global memory the cache's tag lookups
// did: 64 lines per load instruction. 40 heads x 4,680 tokens, 128 centroids,
// r = 16: 162 us so, 94 us from LDS; 120 heads x 3,120, 256 centroids, r = 32,
// 8-bit scales: 541 and 298 us; 12 heads x 880, 64 centroids: 24.8 and 19.8 us,
// 13.7 us with Keys and Values in separate workgroups.
#include "append_common.h"
#include "xcd_order.h"

#include <atomic>

namespace qwm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaveTokens = 32;

// Waves per workgroup for up to NB blocks of 32 centroids. Every Key distance stays
// in registers through the selection (16 per block and lane), which leaves two waves
// per SIMD. Up to four blocks two workgroups of four waves share a CU (80 KB of LDS
// each at 128 centroids and d = 128); with eight blocks the tables leave room for one
// workgroup, of eight waves.
template <int NB>
constexpr int kMaxWaves = NB <= 4 ? 4 : 8;

// A table of [rows][D] BF16 in LDS, in 16-byte pieces: piece p of row j sits in
// slot p ^ key(j) of the row, so that the matrix-core operand reads (32 rows at
// one piece) hit every bank once without padding, which the direct loads into
// LDS do not allow.
template <int D>
struct Pieces {
  static constexpr int PR = D / 8;  // per row
  static __device__ inline int at(int j, int p) { return j * PR + (p ^ (D == 128 ? j & 15 : (j >> 1) & 7)); }
  // pieces of a table of n rows, rounded to one load of a wave
  static __host__ __device__ constexpr int size(int n) { return (n * PR + 63) / 64 * 64; }
};
// LDS of a workgroup, in 16-byte pieces: the Key table, then two buffers of a
// block's three planes, which the Value table takes over after the Key search
template <int D>
inline int lds_pieces(int kc) {
  const int v = Pieces<D>::size(kc), planes = 2 * 3 * Pieces<D>::size(32);
  return v + (v > planes ? v : planes);
}

// Loads rows first .. first + n - 1 of a [..][D] table (the last of them, `last`,
// in place of those past it) into LDS pieces, by the whole workgroup; complete
// after a wait for the vector memory counter and a barrier. The LDS row count is
// rounded up to whole loads. Addresses are a uniform base and 32-bit offsets.
template <int D>
__device__ inline void stage_rows(const bf16* src, uint4* dst, int first, int n, int last, int waves, int wave,
                                  int lane) {
  using P = Pieces<D>;
  constexpr int RL = 64 / P::PR;  // rows per load of a wave
  const char* base = reinterpret_cast<const char*>(src);
  for (int r0 = wave * RL; r0 < n; r0 += waves * RL) {
    const int j = r0 + lane / P::PR, p = P::at(j, lane % P::PR) - j * P::PR;
    const uint32_t off = uint32_t(min(first + j, last)) * uint32_t(2 * D) + uint32_t(p) * 16;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t*)(base + off),
                                     (__attribute__((address_space(3))) uint32_t*)(dst + r0 * P::PR), 16, 0, 0);
  }
}
// every direct load of this wave has landed, then the workgroup's
__device__ inline void staged_barrier() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// centroid row (within the 32-row block) of accumulator slot i in lane half hf;
// the lane's column (token) is lane % 32
__device__ inline constexpr int acc_row(int i, int hf) { return (i / 4) * 8 + hf * 4 + (i % 4); }

// the value x holds in lane i ^ 32
__device__ inline uint32_t partner_u32(uint32_t x, int hf) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return hf ? r[0] : r[1];
}
__device__ inline float partner(float x, int hf) { return __uint_as_float(partner_u32(__float_as_uint(x), hf)); }
__device__ inline int partner(int x, int hf) { return int(partner_u32(uint32_t(x), hf)); }

__device__ inline bf16x8 as_frag(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// element E (0..7) of eight BF16 values held as one uint4 (memory order)
__device__ inline float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
template <int E>
__device__ inline float bf_el(const uint4& u) {
  constexpr int k = E / 2;
  const uint32_t w = k == 0 ? u.x : (k == 1 ? u.y : (k == 2 ? u.z : u.w));
  return (E & 1) ? bf_hi(w) : bf_lo(w);
}

// Insert (d, j) into a list sorted by d; j exceeds every id in the list, so an
// equal distance goes after its equals. med3(l[p - 1], d, l[p]) is the new l[p].
template <int MM>
__device__ inline void top_insert(float (&bd)[MM], int (&bi)[MM], float d, int j) {
  bool lt[MM];
#pragma unroll
  for (int p = 0; p < MM; ++p) lt[p] = d < bd[p];
#pragma unroll
  for (int p = MM - 1; p >= 1; --p) {
    const int jp = lt[p] ? j : bi[p];
    bi[p] = lt[p - 1] ? bi[p - 1] : jp;
    bd[p] = __builtin_amdgcn_fmed3f(bd[p - 1], d, bd[p]);
  }
  bi[0] = lt[0] ? j : bi[0];
  bd[0] = lt[0] ? d : bd[0];
}

// Insert d into the sorted list of the MM smallest distances.
template <int MM>
__device__ inline void top_value(float (&bd)[MM], float d) {
#pragma unroll
  for (int p = MM - 1; p >= 1; --p) bd[p] = __builtin_amdgcn_fmed3f(bd[p - 1], d, bd[p]);
  bd[0] = fminf(bd[0], d);
}

// The M-th smallest distance of the two lanes' lists (M <= MM, wave-uniform).
template <int MM>
__device__ inline float merged_rank(const float (&bd)[MM], int M, int hf) {
  // the MM smallest of two sorted lists of MM are the pairwise minima of one with
  // the other reversed: a bitonic sequence, which log2(MM) steps sort
  float c[MM];
#pragma unroll
  for (int p = 0; p < MM; ++p) c[p] = fminf(bd[p], partner(bd[MM - 1 - p], hf));
#pragma unroll
  for (int o = MM / 2; o > 0; o /= 2)
#pragma unroll
    for (int p = 0; p < MM; ++p)
      if (!(p & o)) {
        const float lo = fminf(c[p], c[p + o]), hi = fmaxf(c[p], c[p + o]);
        c[p] = lo;
        c[p + o] = hi;
      }
  float t = c[MM - 1];
#pragma unroll
  for (int p = MM - 2; p >= 0; --p) t = M == p + 1 ? c[p] : t;
  return t;
}

// Bit j of the result: centroid j of a 32-row block has d' <= t, over both lanes of the pair.
__device__ inline uint32_t candidate_bits(const f32x16& acc, float t, int hf) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) m |= acc[i] <= t ? 1u << acc_row(i, 0) : 0u;
  m <<= 4 * hf;
  return m | partner_u32(m, hf);
}

// Insert (d, j) into a list sorted by (d, id) with any id order.
template <int MM>
__device__ inline void top_insert_lex(float (&bd)[MM], int (&bi)[MM], float d, int j) {
#pragma unroll
  for (int p = 0; p < MM; ++p) {
    const bool lt = (d < bd[p]) | ((d == bd[p]) & (j < bi[p]));
    const float td = lt ? bd[p] : d;
    const int tj = lt ? bi[p] : j;
    bd[p] = lt ? d : bd[p];
    bi[p] = lt ? j : bi[p];
    d = td;
    j = tj;
  }
}

// Pair-merge of the two lanes' top-MM lists: both lanes end with the MM
// smallest (d, id) of the union (ids of the two halves are distinct).
template <int MM>
__device__ inline void merge_pair(float (&bd)[MM], int (&bi)[MM], int hf) {
  float pd[MM];
  int pi[MM];
#pragma unroll
  for (int p = 0; p < MM; ++p) {
    pd[p] = partner(bd[p], hf);
    pi[p] = partner(bi[p], hf);
  }
#pragma unroll
  for (int p = 0; p < MM; ++p) top_insert_lex<MM>(bd, bi, pd[p], pi[p]);
}

// One lane's share of the group structure: DH channels, GL groups of GC
// channels each (a group larger than the half-row spans both lanes: GL = 1).
template <int D, int G>
struct Halves {
  static constexpr int DH = D / 2, NG = D / G;
  static constexpr bool SPAN = G > DH;
  static constexpr int GL = SPAN ? 1 : DH / G, GC = SPAN ? DH : G;
  static __device__ inline int group(int hf, int gl) { return SPAN ? 0 : hf * GL + gl; }
};

// Makes the compiler forget what the packed words hold, so that values unpacked
// from them earlier are not kept live to be reused later (a whole unpacked
// half-row). Emits no instruction.
template <int N>
__device__ inline void forget(uint4 (&u)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(u[i].x), "+v"(u[i].y), "+v"(u[i].z), "+v"(u[i].w));
}

// Residual of the lane's BF16 half-row xh against the half-row of centroid z,
// whose 16-byte piece i is mrow(i) (Eq. 1-2 with q_min = 0, q_max = 3, the range extended to contain 0, the
// residual quantised with the stored scale). Fills the code words of the half
// (16 channels per word), the zero-points, scales (SI8: 8-bit codes and the
// secondary scale) of the lane's groups, and calls each(k, e) with
// e = x_c - (mu_c + s (q_c - z)) for channel c = c0 + k of every 8-channel
// chunk of the half (Eq. 4, Eq. 13), then chunk(c0). The centroid row is read
// (from LDS) 8 channels at a time in each pass; each
// group's range pass precedes its code pass, and with 8-bit scales every range
// pass comes first (the groups share the secondary scale). KNOWN: the groups'
// literal ranges [gmin, gmax] are given, and there is no range pass.
template <int D, int G, bool SI8, bool KNOWN, typename R, typename F, typename FC>
__device__ inline void residual_half(uint4 (&xh)[D / 16], R mrow, int hf,
                                     const float (&gmin)[Halves<D, G>::GL], const float (&gmax)[Halves<D, G>::GL],
                                     uint32_t (&cw)[D / 32], int (&zg)[Halves<D, G>::GL],
                                     float (&sg)[Halves<D, G>::GL], int (&cg)[Halves<D, G>::GL], float& sig,
                                     F each, FC chunk) {
  using H = Halves<D, G>;
  constexpr int GL = H::GL, GC = H::GC;
  forget(xh);
  float glo[GL], gabs[GL];
  auto range = [&](auto gi, float& lo, float& hi) {
    constexpr int gl = decltype(gi)::value;
    if constexpr (KNOWN) {
      lo = fminf(0.0f, gmin[gl]);
      hi = fmaxf(0.0f, gmax[gl]);
      return;
    }
    lo = 0.0f;
    hi = 0.0f;
    static_for<0, GC, 8>([&](auto ci) {
      constexpr int c0 = gl * GC + decltype(ci)::value;
      const uint4 mu = mrow(c0 / 8);
      static_for<0, 8>([&](auto ki) {
        constexpr int k = decltype(ki)::value;
        const float r = bf_el<k>(xh[c0 / 8]) - bf_el<k>(mu);
        lo = fminf(lo, r);
        hi = fmaxf(hi, r);
      });
    });
    if constexpr (H::SPAN) {
      lo = fminf(lo, partner(lo, hf));
      hi = fmaxf(hi, partner(hi, hf));
    }
  };
  auto codes = [&](auto gi) {
    constexpr int gl = decltype(gi)::value;
    // unpack the token words and re-read the centroid words here rather than keep
    // the range pass's unpacked values live
    forget(xh);
    asm volatile("" ::: "memory");
    const float s = sg[gl];
    const float sd = s != 0.0f ? s : 1.0f;
    const int z = s != 0.0f ? (int)fminf(fmaxf(rintf(0.0f - glo[gl] / sd), 0.0f), 3.0f) : 0;
    const float inv = s != 0.0f ? 1.0f / s : 0.0f;
    const bool big = gabs[gl] * inv > 4.0f;  // the group's largest |x / s|
    zg[gl] = z;
    const float zf = (float)z;
    static_for<0, GC, 8>([&](auto ci) {
      constexpr int c0 = gl * GC + decltype(ci)::value;
      float xv[8], mu[8], t[8];
      const uint4 m0 = mrow(c0 / 8);
      static_for<0, 8>([&](auto ki) {
        constexpr int k = decltype(ki)::value;
        xv[k] = bf_el<k>(xh[c0 / 8]);
        mu[k] = bf_el<k>(m0);
      });
      round_quotients<8>(xv, mu, s, inv, big, t);
      // Eq. 1 codes as floats: a zero step has t = 0 and z = 0, so its codes are 0.
      // The code word sums q 4^k (exact); mu + s (q - z) rounds once, as the
      // product is exact (at most 21 significant bits)
      float wf = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float q = fminf(fmaxf(t[k] + zf, 0.0f), 3.0f);
        wf = __builtin_fmaf(q, float(1 << (2 * k)), wf);
        each(k, xv[k] - __builtin_fmaf(s, q - zf, mu[k]));
      }
      const uint32_t w = uint32_t(wf);
      if constexpr (c0 % 16 == 0) cw[c0 / 16] = w;
      else cw[c0 / 16] |= w << 16;
      chunk(c0);
    });
  };
  if constexpr (SI8) {
    float tg[GL], mx = 0.0f;
    static_for<0, GL>([&](auto gi) {
      constexpr int gl = decltype(gi)::value;
      float lo, hi;
      range(gi, lo, hi);
      glo[gl] = lo;
      gabs[gl] = fmaxf(-lo, hi);
      tg[gl] = (hi - lo) / 3.0f;
      mx = fmaxf(mx, tg[gl]);
    });
    if constexpr (!H::SPAN) mx = fmaxf(mx, partner(mx, hf));
    sig = f16_round(mx / 255.0f);
#pragma unroll
    for (int gl = 0; gl < GL; ++gl) {
      const int c = sig != 0.0f ? (int)fminf(fmaxf(rintf(tg[gl] / sig), 0.0f), 255.0f) : 0;
      cg[gl] = c;
      sg[gl] = sig * (float)c;  // exact: 11-bit times 8-bit significands
    }
    static_for<0, GL>([&](auto gi) {
      __builtin_amdgcn_sched_barrier(0);
      codes(gi);
    });
  } else {
    static_for<0, GL>([&](auto gi) {
      constexpr int gl = decltype(gi)::value;
      __builtin_amdgcn_sched_barrier(0);
      float lo, hi;
      range(gi, lo, hi);
      glo[gl] = lo;
      gabs[gl] = fmaxf(-lo, hi);
      sg[gl] = f16_round((hi - lo) / 3.0f);
      codes(gi);
    });
  }
}

// Stores of one token's packed fields for the lane's half: code words, and the
// lane's groups' scales; lane half 0 adds the id, the zero-point bytes (all
// groups) and the SI8 secondary scale.
template <int D, int G, bool SI8>
__device__ inline void store_half(const CacheLayout& L, uint8_t* __restrict__ cache, int64_t codes_sec,
                                  int64_t ids_sec, int64_t zp_sec, int64_t scale_sec, int64_t sigma_sec,
                                  int64_t slot, int hf, bool active, int id, const uint32_t (&cw)[D / 32],
                                  const int (&zg)[Halves<D, G>::GL], const float (&sg)[Halves<D, G>::GL],
                                  const int (&cg)[Halves<D, G>::GL], float sig) {
  using H = Halves<D, G>;
  constexpr int GL = H::GL, NG = H::NG;
  uint32_t zw = 0;
#pragma unroll
  for (int gl = 0; gl < GL; ++gl) zw |= uint32_t(zg[gl]) << (2 * H::group(hf, gl));
  if constexpr (!H::SPAN) zw |= partner_u32(zw, hf);
  if (!active) return;
  uint8_t* cp = cache + codes_sec + slot * (D / 4) + hf * (D / 8);
  if constexpr (D == 128) *reinterpret_cast<uint4*>(cp) = make_uint4(cw[0], cw[1], cw[2], cw[3]);
  else *reinterpret_cast<uint2*>(cp) = make_uint2(cw[0], cw[1]);
  if (hf == 0) {
    cache[ids_sec + slot] = uint8_t(id);
    uint8_t* zp = cache + zp_sec + slot * L.zpb;
    if constexpr (NG > 4) *reinterpret_cast<uint16_t*>(zp) = uint16_t(zw);
    else zp[0] = uint8_t(zw);
    if constexpr (SI8) *reinterpret_cast<uint16_t*>(cache + sigma_sec + slot * 2) = f16_bits(sig);
  }
  if constexpr (H::SPAN) {
    if (hf == 0) {
      if constexpr (SI8) cache[scale_sec + slot] = uint8_t(cg[0]);
      else *reinterpret_cast<uint16_t*>(cache + scale_sec + slot * 2) = f16_bits(sg[0]);
    }
  } else if constexpr (SI8) {
    uint32_t v = 0;
#pragma unroll
    for (int gl = 0; gl < GL; ++gl) v |= uint32_t(cg[gl]) << (8 * gl);
    uint8_t* p = cache + scale_sec + slot * NG + hf * GL;
    if constexpr (GL == 4) *reinterpret_cast<uint32_t*>(p) = v;
    else if constexpr (GL == 2) *reinterpret_cast<uint16_t*>(p) = uint16_t(v);
    else p[0] = uint8_t(v);
  } else {
    uint8_t* p = cache + scale_sec + slot * (2 * NG) + hf * (2 * GL);
    if constexpr (GL == 4) {
      *reinterpret_cast<uint2*>(p) = make_uint2(uint32_t(f16_bits(sg[0])) | uint32_t(f16_bits(sg[1])) << 16,
                                                uint32_t(f16_bits(sg[2])) | uint32_t(f16_bits(sg[3])) << 16);
    } else if constexpr (GL == 2) {
      *reinterpret_cast<uint32_t*>(p) = uint32_t(f16_bits(sg[0])) | uint32_t(f16_bits(sg[1])) << 16;
    } else {
      *reinterpret_cast<uint16_t*>(p) = f16_bits(sg[0]);
    }
  }
}

template <int D, int G, int RP, int MM, int NB, bool SI8>
__global__ __launch_bounds__(64 * kMaxWaves<NB>) __attribute__((amdgpu_waves_per_eu(2))) void
append_bf16_kernel(const AppendArgs a) {
  using H = Halves<D, G>;
  using P = Pieces<D>;
  constexpr int DH = H::DH, NS = D / 16, GL = H::GL;
  extern __shared__ __attribute__((aligned(16))) uint4 lds[];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
  const int waves = blockDim.x >> 6;
  const int64_t wg_tokens = int64_t(waves) * kWaveTokens, ntb = (a.n_new + wg_tokens - 1) / wg_tokens;
  // the second half of a split launch quantises the Values, the first the Keys
  const uint32_t n_task = a.split_sides ? gridDim.x / 2 : gridDim.x;
  const bool keys = blockIdx.x < n_task, values = !a.split_sides || !keys;
  const uint32_t task = qwm_xcd_task(keys ? blockIdx.x : blockIdx.x - n_task, n_task);
  const int64_t tb = task % ntb, bh = task / ntb;
  const int64_t b = bh / a.heads, h = bh % a.heads;
  const uint8_t* slab = a.calib + bh * a.slab;

  const int64_t t0 = tb * wg_tokens + wv * kWaveTokens;
  const bool idle = t0 >= a.n_new;  // the whole wave is past the chunk: it stages and keeps the barriers
  const int64_t t = t0 + n;
  const bool active = t < a.n_new;
  const int64_t tt = active ? t : a.n_new - 1;  // idle lanes recompute a real token and store nothing
  const int64_t src = ((b * a.n_new + tt) * a.heads + h) * D + hf * DH;
  const int64_t slot = bh * a.L.slots + a.n_cached + tt;
  const int Kc = a.n_centroids, nb = (Kc + 31) / 32;
  const bf16* planes = reinterpret_cast<const bf16*>(slab + a.o_a_k3);
  const bf16* muk = reinterpret_cast<const bf16*>(slab + a.o_mu_k);
  const bf16* muv = reinterpret_cast<const bf16*>(slab + a.o_mu_v);
  uint4* tabK = lds;
  uint4* bufA = lds + P::size(Kc);  // two blocks' planes, then the Value table
  constexpr int kPlane = P::size(32);
  auto stage_planes = [&](int jb) {
    for (int pl = 0; pl < 3; ++pl)
      stage_rows<D>(planes + int64_t(pl) * Kc * D, bufA + ((jb & 1) * 3 + pl) * kPlane, jb * 32, 32, Kc - 1, waves, wv, lane);
  };
  auto stage_values = [&]() { stage_rows<D>(muv, bufA, 0, Kc, Kc - 1, waves, wv, lane); };
  float gmin[GL], gmax[GL];  // literal group ranges of the chosen centroid's residual
  if (keys) {
    stage_planes(0);
    stage_rows<D>(muk, tabK, 0, Kc, Kc - 1, waves, wv, lane);
  } else {
    stage_values();
  }

  if (keys) {

  // ---- QSAC candidate search (Eq. 9 expanded) on the matrix cores, top-M by (d', id)
  uint4 xk[NS];
  {
    const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const bf16*>(a.k) + src);
#pragma unroll
    for (int s = 0; s < NS; ++s) xk[s] = p[s];
  }
  const int M = a.top_m < Kc ? a.top_m : Kc;
  int bi[MM];
  {
    const float* __restrict__ bk = reinterpret_cast<const float*>(slab + a.o_b_k);
    // distances of the 32 centroids from 32 jb on (+inf past the last one), whose
    // planes are in buffer jb & 1
    auto search = [&](int jb) __attribute__((always_inline)) {
      const int j0 = jb * 32;
      f32x16 acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = bk[min(j0 + acc_row(i, hf), Kc - 1)];
      if (j0 + 32 > Kc)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = j0 + acc_row(i, hf) < Kc ? acc[i] : __builtin_inff();
      const uint4* A = bufA + (jb & 1) * 3 * kPlane;
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(A[pl * kPlane + P::at(n, hf * NS + st)]), as_frag(xk[st]),
                                                         acc, 0, 0, 0);
      return acc;
    };
    float bd[MM];
#pragma unroll
    for (int p = 0; p < MM; ++p) bd[p] = __builtin_inff();
    f32x16 kept[NB];
    static_for<0, NB>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      if (q < nb) {
        staged_barrier();  // block q is in LDS, and every wave is done with block q - 1
        if (q + 1 < nb) stage_planes(q + 1);
        if (!idle) {
          kept[q] = search(q);
#pragma unroll
          for (int i = 0; i < 16; ++i) top_value<MM>(bd, kept[q][i]);
        }
      }
    });
    __syncthreads();  // the planes are used up
    if (values) stage_values();
    if (!idle) {
    const float T = merged_rank<MM>(bd, M, hf);
    // bit j % 32 of word j / 32: centroid j is a candidate
    uint32_t cand[NB];
    int found = 0;
    static_for<0, NB>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      cand[q] = 0;
      if (q < nb) cand[q] = candidate_bits(kept[q], T, hf);
      found += __popc(cand[q]);
    });
    // the ids in increasing order: the lowest set bit of the first word that has one
#pragma unroll
    for (int m = 0; m < MM; ++m) {
      uint32_t j = ~0u;
      static_for<0, NB>([&](auto qi) {
        constexpr int q = decltype(qi)::value;
        if (q < nb) {
          const bool here = j == ~0u && cand[q] != 0;
          j = here ? uint32_t(32 * q + __ffs(cand[q]) - 1) : j;
          cand[q] = here ? cand[q] & (cand[q] - 1) : cand[q];
        }
      });
      // a valid row whatever the distances were (infinite or NaN inputs)
      bi[m] = int(min(j, uint32_t(Kc - 1)));
    }
    if (__any(found != M)) {
      // equal distances at T (or inputs out of range): lists of (d', id), lower ids
      // first among equals. Ids start at 0, a valid row.
#pragma unroll
      for (int p = 0; p < MM; ++p) { bd[p] = __builtin_inff(); bi[p] = 0; }
      static_for<0, NB>([&](auto qi) {
        constexpr int q = decltype(qi)::value;
        if (q < nb)
#pragma unroll
          for (int i = 0; i < 16; ++i) top_insert<MM>(bd, bi, kept[q][i], q * 32 + acc_row(i, hf));
      });
      merge_pair<MM>(bd, bi, hf);
    }
    }
  }

  if (!idle) {
  // ---- QSAC score (Eq. 10, 12) over the M candidates; ties to the lower id
  const float* __restrict__ wg = reinterpret_cast<const float*>(slab + a.o_wg);
  int z = 0;
  float zs = __builtin_inff();
#pragma unroll
  for (int gl = 0; gl < GL; ++gl) gmin[gl] = gmax[gl] = 0.0f;
  {
    int row[MM];
#pragma unroll
    for (int m = 0; m < MM; ++m) row[m] = bi[m];
    float mx[MM][GL], mn[MM][GL];
    static_for<0, GL>([&](auto gi) {
      constexpr int gl = decltype(gi)::value;
#pragma unroll
      for (int m = 0; m < MM; ++m) { mx[m][gl] = -__builtin_inff(); mn[m][gl] = __builtin_inff(); }
      static_for<0, H::GC / 8>([&](auto wi) {
        constexpr int c = gl * (H::GC / 8) + decltype(wi)::value;
        // at most four chunks' rows in flight (two for eight candidates): the next
        // ones' addresses wait for the ranges so far (more would spill)
        if constexpr (c > 0 && c % (MM > 4 ? 2 : 4) == 0)
#pragma unroll
          for (int m = 0; m < MM; ++m) {
            constexpr int done = (c - 1) / (H::GC / 8);
            asm volatile("" : "+v"(row[m]), "+v"(mx[m][done]), "+v"(mn[m][done]));
          }
        float x[8];
        static_for<0, 8>([&](auto ki) { x[decltype(ki)::value] = bf_el<decltype(ki)::value>(xk[c]); });
#pragma unroll
        for (int m = 0; m < MM; ++m) {
          const uint4 mu = tabK[P::at(row[m], hf * NS + c)];
          static_for<0, 8>([&](auto ki) {
            constexpr int k = decltype(ki)::value;
            const float r = x[k] - bf_el<k>(mu);
            mx[m][gl] = fmaxf(mx[m][gl], r);
            mn[m][gl] = fminf(mn[m][gl], r);
          });
        }
      });
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, MM>([&](auto mi) {
      constexpr int m = decltype(mi)::value;
      if (m >= M) return;  // entries past M repeat a row and are not scored
      float tg[GL], S = 0.0f;
#pragma unroll
      for (int gl = 0; gl < GL; ++gl) {
        if constexpr (H::SPAN) {
          mx[m][gl] = fmaxf(mx[m][gl], partner(mx[m][gl], hf));
          mn[m][gl] = fminf(mn[m][gl], partner(mn[m][gl], hf));
        }
        const float R = mx[m][gl] - mn[m][gl];
        tg[gl] = wg[H::group(hf, gl)] * (R * R);
      }
      if constexpr (H::SPAN) {
        S = S + tg[0];
      } else {
        float pt[GL];
#pragma unroll
        for (int gl = 0; gl < GL; ++gl) pt[gl] = partner(tg[gl], hf);
#pragma unroll
        for (int gl = 0; gl < GL; ++gl) S = S + (hf ? pt[gl] : tg[gl]);
#pragma unroll
        for (int gl = 0; gl < GL; ++gl) S = S + (hf ? tg[gl] : pt[gl]);
      }
      const int j = bi[m];
      const bool better = (S < zs) | ((S == zs) & (j < z));
      zs = better ? S : zs;
      z = better ? j : z;
#pragma unroll
      for (int gl = 0; gl < GL; ++gl) {
        gmin[gl] = better ? mn[m][gl] : gmin[gl];
        gmax[gl] = better ? mx[m][gl] : gmax[gl];
      }
    });
  }
  // every score overflowed (W_g R^2 past fp32: a residual of about 1.8e19 / sqrt(W_g)
  // or more): centroid 0, with its own ranges
  const bool none = !(zs < __builtin_inff());
  if (__builtin_expect(__any(none), 0)) {
    const uint4* krow = reinterpret_cast<const uint4*>(reinterpret_cast<const bf16*>(a.k) + src);
    static_for<0, GL>([&](auto gi) {
      constexpr int gl = decltype(gi)::value;
      float mx = -__builtin_inff(), mn = __builtin_inff();
#pragma unroll 1
      for (int c = gl * (H::GC / 8); c < (gl + 1) * (H::GC / 8); ++c) {
        const uint4 mu = tabK[P::at(0, hf * NS + c)];
        const uint4 x = krow[c];
        static_for<0, 8>([&](auto ki) {
          constexpr int k = decltype(ki)::value;
          const float r = bf_el<k>(x) - bf_el<k>(mu);
          mx = fmaxf(mx, r);
          mn = fminf(mn, r);
        });
      }
      if constexpr (H::SPAN) {
        mx = fmaxf(mx, partner(mx, hf));
        mn = fminf(mn, partner(mn, hf));
      }
      gmin[gl] = none ? mn : gmin[gl];
      gmax[gl] = none ? mx : gmax[gl];
    });
  }

  // ---- Keys: INT2 residual against mu_z, and PSAC (Eq. 13, 16): C = E U_r with
  // E_c = k_c - khat_0,c, on the matrix cores. Each residual chunk is the lane's
  // 8 channels of one k step, so its errors are the B operand as they are made:
  // split into three BF16 parts with an exact sum (as the Key search constants)
  // against the BF16 rows of U_r^T (rank m = lane % 32; zero rows past r), every
  // product is exact and the fp32 accumulator holds ranks acc_row(i, hf).
  // INT8 rows with one FP16 scale (App. D.1).
  {
    auto mrow = [&](int i) { return tabK[P::at(z, hf * NS + i)]; };
    const bf16* __restrict__ ut = reinterpret_cast<const bf16*>(slab + a.o_u_t);
    const int r = a.rank;
    const uint4* urow = reinterpret_cast<const uint4*>(ut + int64_t(min(n, r > 0 ? r - 1 : 0)) * D + hf * DH);
    const bool urank = n < r;
    f32x16 cacc;
#pragma unroll
    for (int i = 0; i < 16; ++i) cacc[i] = 0.0f;
    float ech[8];
    uint32_t cw[D / 32];
    int zg[GL], cg[GL];
    float sg[GL], sig = 0.0f;
    residual_half<D, G, SI8, true>(
        xk, mrow, hf, gmin, gmax, cw, zg, sg, cg, sig,
        [&](int k, float e) {
          if constexpr (RP > 0) ech[k] = e;
        },
        [&](int c0) {
          if constexpr (RP > 0) {
            uint4 uf = urow[c0 / 8];
            if (!urank) uf = make_uint4(0u, 0u, 0u, 0u);
            uint32_t p0[4], p1[4], p2[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              // the upper halves of e, e - p0 and e - p0 - p1 (whose lower half is 0)
              uint32_t e0[2], e1[2], e2[2];
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const float e = ech[2 * q + u];
                e0[u] = __float_as_uint(e);
                const float r1 = e - __uint_as_float(e0[u] & 0xffff0000u);
                e1[u] = __float_as_uint(r1);
                e2[u] = __float_as_uint(r1 - __uint_as_float(e1[u] & 0xffff0000u));
              }
              p0[q] = __builtin_amdgcn_perm(e0[1], e0[0], 0x07060302u);
              p1[q] = __builtin_amdgcn_perm(e1[1], e1[0], 0x07060302u);
              p2[q] = __builtin_amdgcn_perm(e2[1], e2[0], 0x07060302u);
            }
            cacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(uf), as_frag(make_uint4(p0[0], p0[1], p0[2], p0[3])),
                                                           cacc, 0, 0, 0);
            cacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(uf), as_frag(make_uint4(p1[0], p1[1], p1[2], p1[3])),
                                                           cacc, 0, 0, 0);
            cacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(uf), as_frag(make_uint4(p2[0], p2[1], p2[2], p2[3])),
                                                           cacc, 0, 0, 0);
          }
        });
    store_half<D, G, SI8>(a.L, a.cache, a.L.k_codes, a.L.k_ids, a.L.k_zp, a.L.k_scale, a.L.k_sigma, slot, hf,
                          active, z, cw, zg, sg, cg, sig);
    if constexpr (RP > 0) {
      // rank k sits in slot (k / 8) * 4 + k % 4 of lane half (k / 4) % 2: each lane
      // quantises its own RP / 2 ranks, four consecutive ones per code word
      float amax = 0.0f;
#pragma unroll
      for (int i = 0; i < RP / 2; ++i)
        if (acc_row(i, hf) < r) amax = fmaxf(amax, fabsf(cacc[i]));
      amax = fmaxf(amax, partner(amax, hf));
      const float s = f16_round(amax / 127.0f);
      const float sd = s != 0.0f ? s : 1.0f;
      int qc[RP / 2];
#pragma unroll
      for (int i = 0; i < RP / 2; ++i)
        qc[i] = acc_row(i, hf) < r && s != 0.0f ? (int)fminf(fmaxf(rintf(cacc[i] / sd), -127.0f), 127.0f) : 0;
      // App. D.1 retention: keep the row only if it lowers the lam-weighted
      // error on the principal subspace (ranks in order, fp32)
      bool keep = true;
      if (a.gate) {
        const float* __restrict__ lam = reinterpret_cast<const float*>(slab + a.o_lam);
        float tb[RP / 2], ta[RP / 2];
#pragma unroll
        for (int i = 0; i < RP / 2; ++i) {
          const float e = cacc[i] - (float)qc[i] * s, l = lam[min(acc_row(i, hf), r - 1)];
          tb[i] = l * (cacc[i] * cacc[i]);
          ta[i] = l * (e * e);
        }
        float before = 0.0f, after = 0.0f;
#pragma unroll
        for (int k = 0; k < RP; ++k) {
          const int i = (k / 8) * 4 + k % 4;
          const float pb = partner(tb[i], hf), pa = partner(ta[i], hf);
          if (k < r) {
            before = before + ((k / 4) % 2 == hf ? tb[i] : pb);
            after = after + ((k / 4) % 2 == hf ? ta[i] : pa);
          }
        }
        keep = after < before;
      }
      if (active) {
        // with sparse rows the chunk's rows go to the staging rows (row tt of the
        // head) and the commit kernel stores them into the pool
        const int64_t crow = a.L.sparse ? bh * a.L.stage + tt : slot;
        uint8_t* code = a.cache + (a.L.sparse ? a.L.k_st_codes : a.L.k_coef) + crow * r;
        if (r == RP) {
          // words hf, 2 + hf, ...: ranks 8 q + 4 hf .. + 3
#pragma unroll
          for (int q = 0; q < RP / 8; ++q) {
            uint32_t v = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) v |= uint32_t(uint8_t(int8_t(keep ? qc[4 * q + k] : 0))) << (8 * k);
            *reinterpret_cast<uint32_t*>(code + 8 * q + 4 * hf) = v;
          }
        } else {
#pragma unroll
          for (int i = 0; i < RP / 2; ++i)
            if (acc_row(i, hf) < r) code[acc_row(i, hf)] = uint8_t(int8_t(keep ? qc[i] : 0));
        }
        if (a.coef_out) {
          float* co = a.coef_out + (bh * a.n_new + tt) * r;
#pragma unroll
          for (int i = 0; i < RP / 2; ++i)
            if (acc_row(i, hf) < r) co[acc_row(i, hf)] = cacc[i];
        }
        if (hf == 0) {
          *reinterpret_cast<uint16_t*>(a.cache + (a.L.sparse ? a.L.k_st_scale : a.L.k_cscale) + crow * 2) =
              f16_bits(keep ? s : 0.0f);
        }
      }
    }
  }

  }
  if (!values) return;
  }
  staged_barrier();  // the Value table is in LDS
  if (idle) return;

  // ---- Values: nearest centroid (w = 1) on the matrix cores, then the same
  // residual path as Keys, no PSAC. (The barrier keeps the Value loads out of
  // the Key residual, where they would only add to its registers.)
  __builtin_amdgcn_sched_barrier(0);
  {
    uint4 xv[NS];
    const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const bf16*>(a.v) + src);
#pragma unroll
    for (int s = 0; s < NS; ++s) xv[s] = p[s];
    const float* __restrict__ bv = reinterpret_cast<const float*>(slab + a.o_b_v);
    // the largest mu.v - b/2 is the smallest distance (times -2, exactly)
    float dv = -__builtin_inff();
    int zv = 0;
    for (int jb = 0; jb < nb; ++jb) {
      const int j0 = jb * 32;
      f32x16 acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = -0.5f * bv[min(j0 + acc_row(i, hf), Kc - 1)];
      if (j0 + 32 > Kc)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = j0 + acc_row(i, hf) < Kc ? acc[i] : -__builtin_inff();
      const int jr = min(j0 + n, Kc - 1);
#pragma unroll
      for (int st = 0; st < NS; ++st)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(bufA[P::at(jr, hf * NS + st)]), as_frag(xv[st]), acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool better = acc[i] > dv;  // ids increase: ties keep the lower one
        dv = better ? acc[i] : dv;
        zv = better ? j0 + acc_row(i, hf) : zv;
      }
    }
    {
      const float pd = partner(dv, hf);
      const int pz = partner(zv, hf);
      const bool take = (pd > dv) | ((pd == dv) & (pz < zv));
      zv = take ? pz : zv;
    }
    auto mrow = [&](int i) { return bufA[P::at(zv, hf * NS + i)]; };
    uint32_t cw[D / 32];
    int zg[GL], cg[GL];
    float sg[GL], sig = 0.0f;
    residual_half<D, G, SI8, false>(xv, mrow, hf, gmin, gmax, cw, zg, sg, cg, sig, [](int, float) {}, [](int) {});
    store_half<D, G, SI8>(a.L, a.cache, a.L.v_codes, a.L.v_ids, a.L.v_zp, a.L.v_scale, a.L.v_sigma, slot, hf,
                          active, zv, cw, zg, sg, cg, sig);
  }
}

template <int D, int G, int RP, int MM, int NB, bool SI8>
hipError_t launch_one(const AppendArgs& a, int batch, hipStream_t s) {
  // the dynamic LDS limit is raised once per device for this instance
  static std::atomic<uint64_t> raised{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
  if (!bit || !(raised.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)append_bf16_kernel<D, G, RP, MM, NB, SI8>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 16 * lds_pieces<D>(32 * NB));
    if (e != hipSuccess) return e;
    raised.fetch_or(bit, std::memory_order_release);
  }
  AppendArgs args = a;
  const int64_t bh = int64_t(a.heads) * batch, tw = (a.n_new + kWaveTokens - 1) / kWaveTokens;
  args.split_sides = tw * bh <= kSplitSideWaves;
  // as many waves share the staged tables as leave no compute unit (256 on
  // MI355X) without a workgroup; fewer waves would need a second round of
  // workgroups for the LDS (12 heads x 2,640 tokens: 17.8 us with four, 23.9 us
  // with two)
  const int64_t sides = args.split_sides ? 2 : 1;
  int waves = kMaxWaves<NB>;
  while (waves > 1 && (tw + waves - 1) / waves * bh * sides < 256) waves /= 2;
  const dim3 grid((unsigned)((tw + waves - 1) / waves * bh * sides));
  hipLaunchKernelGGL((append_bf16_kernel<D, G, RP, MM, NB, SI8>), grid, dim3(64 * waves),
                     16 * lds_pieces<D>(a.n_centroids), s, args);
  return hipGetLastError();
}

template <int D, int G, int RP, bool SI8>
hipError_t launch_rank(const AppendArgs& a, int batch, hipStream_t s) {
  // four blocks of 32 centroids for up to 128 whatever the candidate count: smaller
  // workgroups (120 heads x 600 tokens, 16 centroids, M = 8, d = 64: 32.5 us with the
  // eight-block instance, 21.7 us so)
  if (a.top_m > 4) return a.n_centroids > 128 ? launch_one<D, G, RP, 8, 8, SI8>(a, batch, s) : launch_one<D, G, RP, 8, 4, SI8>(a, batch, s);
  return a.n_centroids > 128 ? launch_one<D, G, RP, 4, 8, SI8>(a, batch, s) : launch_one<D, G, RP, 4, 4, SI8>(a, batch, s);
}

template <int D, int G, bool SI8>
hipError_t launch_dgs(const AppendArgs& a, int batch, hipStream_t s) {
  if (a.rank > 16) return launch_rank<D, G, 32, SI8>(a, batch, s);
  return a.rank > 0 ? launch_rank<D, G, 16, SI8>(a, batch, s) : launch_rank<D, G, 0, SI8>(a, batch, s);
}

}  // namespace

// This file is compiled once per (head_dim, group size): QWM_APPEND_D and
// QWM_APPEND_G select the instantiations.
template <int D, int G>
hipError_t launch_append_bf16(const AppendArgs& a, int batch, hipStream_t s) {
  return a.L.i8 ? launch_dgs<D, G, true>(a, batch, s) : launch_dgs<D, G, false>(a, batch, s);
}

template hipError_t launch_append_bf16<QWM_APPEND_D, QWM_APPEND_G>(const AppendArgs&, int, hipStream_t);

}  // namespace qwm
