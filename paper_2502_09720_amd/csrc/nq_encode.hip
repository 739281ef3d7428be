// NestQuant row encoder (Sec. 4.2, Alg. 3 with the First-beta or Opt-beta strategy of
// App. F).
//
// One lane per 8-entry block.  A row is handled by a group of LANES lanes (a power of two,
// 8 <= LANES <= 1024), lane l its blocks l + i * LANES, so that consecutive lanes read
// consecutive 8-entry blocks (16 B for bf16/fp16, 32 B for fp32).  encode_wave_kernel
// (First-beta, rows of up to 2048 blocks) works on slots of 64 blocks a wave, described
// below; encode_kernel (longer rows, and Opt-beta) gives a row of up to 64 lanes a share of a
// 256-thread workgroup and a longer one a workgroup, its blocks in registers (BPT) or streamed.
//
// Row scale (Alg. 3, s / sqrt(n)): r is the fp32 number nearest to sqrt(sum x^2 / n).  The
// squares of fp32 values are exact in fp64; the fp64 sum is accepted when it cannot straddle
// an fp32 rounding boundary, otherwise the row is summed again as a double-double and the
// boundary comparison is made exactly.
#include "nq_device.hpp"
#include "nq_kernels.hpp"
#include "nq_rotate.hpp"
#include "nq_tiles.hpp"

namespace nq {

constexpr int a_max_k = 4;

__device__ __forceinline__ float pick4(const float (&c)[4], int t) {
  return t == 0 ? c[0] : (t == 1 ? c[1] : (t == 2 ? c[2] : c[3]));
}

template <typename T>
__device__ __forceinline__ void load_block(const T* __restrict__ p, float (&v)[8]);

template <>
__device__ __forceinline__ void load_block<float>(const float* __restrict__ p, float (&v)[8]) {
  const f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  const f32x4 b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p) + 1);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

template <>
__device__ __forceinline__ void load_block<uint16_t>(const uint16_t* __restrict__ p,
                                                     float (&v)[8]) {
  // bf16: the value is the upper half of an fp32 word
  const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

template <>
__device__ __forceinline__ void load_block<_Float16>(const _Float16* __restrict__ p,
                                                     float (&v)[8]) {
  const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint16_t lo = (uint16_t)(w[i] & 0xffffu), hi = (uint16_t)(w[i] >> 16);
    v[2 * i] = (float)__builtin_bit_cast(_Float16, lo);
    v[2 * i + 1] = (float)__builtin_bit_cast(_Float16, hi);
  }
}

// v of the lane whose index differs in the bits of M (1, 2), or of the mirrored lane of the
// half row or row (M = 4, 8): once the lanes of each aligned group of M hold one value, the
// mirrored lane holds that of lane ^ M.  One DPP move, where a general shuffle goes through LDS.
template <int M>
__device__ __forceinline__ uint32_t dpp_across(uint32_t v) {
  constexpr int ctrl = M == 1 ? 0xB1 : (M == 2 ? 0x4E : (M == 4 ? 0x141 : 0x140));
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xF, 0xF, true);
}
template <int M>
__device__ __forceinline__ double dpp_add(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint64_t o = (uint64_t)dpp_across<M>((uint32_t)u) |
                     (uint64_t)dpp_across<M>((uint32_t)(u >> 32)) << 32;
  return v + __builtin_bit_cast(double, o);
}
// Sum over aligned groups of LANES lanes of a wave (8 to 64), the same in each of its lanes.
template <int LANES>
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<1>(v);
  v = dpp_add<2>(v);
  v = dpp_add<4>(v);
  if constexpr (LANES > 8) v = dpp_add<8>(v);
#pragma unroll
  for (int m = 16; m < LANES; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Sum over the LANES lanes of a row group.  LANES <= 64: within the wave by xor shuffles
// (every lane ends with the same, bit-identical sum).  LANES > 64: the workgroup is exactly
// one row (LANES threads); wave sums are combined through LDS in a fixed order.
template <int LANES>
__device__ __forceinline__ double group_sum(double v, double* red) {
  v = wave_sum<(LANES < 64 ? LANES : 64)>(v);
  if constexpr (LANES > 64) {
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int i = 1; i < LANES / 64; ++i) v += red[i];
  }
  return v;
}

// Double-double version of group_sum (error-free on the hi parts).
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  const double bv = s - a;
  const double av = s - bv;
  e = (a - av) + (b - bv);
}

template <int LANES>
__device__ __forceinline__ void group_sum_dd(double& hi, double& lo, double* red) {
#pragma unroll
  for (int m = 1; m < (LANES < 64 ? LANES : 64); m <<= 1) {
    const double oh = __shfl_xor(hi, m, 64), ol = __shfl_xor(lo, m, 64);
    double s, e;
    two_sum(hi, oh, s, e);
    hi = s;
    lo = lo + ol + e;
  }
  if constexpr (LANES > 64) {
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
      red[2 * wave] = hi;
      red[2 * wave + 1] = lo;
    }
    __syncthreads();
    hi = red[0];
    lo = red[1];
#pragma unroll
    for (int i = 1; i < LANES / 64; ++i) {
      double s, e;
      two_sum(hi, red[2 * i], s, e);
      hi = s;
      lo = lo + red[2 * i + 1] + e;
    }
  }
  double s, e;
  two_sum(hi, lo, s, e);
  hi = s;
  lo = e;
}

// sign of (hi + lo) - n * m^2, exactly (m has at most 25 significant bits, so m^2 is exact
// in fp64 and n * m^2 is exact as the pair (prod, err) of a fused multiply).
__device__ __forceinline__ int cmp_sum_square(double hi, double lo, double n, double m) {
  const double m2 = m * m;
  const double prod = n * m2;
  const double err = __builtin_fma(n, m2, -prod);
  const double t[4] = {hi, lo, -prod, -err};
  return exact_sign_sum<4>(t);
}

__device__ __forceinline__ float next_up(float v) { return __uint_as_float(__float_as_uint(v) + 1u); }
__device__ __forceinline__ float next_down(float v) { return __uint_as_float(__float_as_uint(v) - 1u); }

// NestQuantM (App. D): every point its decoder reproduces lies in |P_0| <= 2q, |P_i| <= q.
// The nearest point P of y has |P_i - 2 y_i| <= 2 (covering radius 1), so a block whose
// statistic s = max(2 max_{i>0} |x_i|, |x_0|) has s c > (q + 2)(1 + 2^-12) surely overloads
// at the multiplier c (the slack covers the rounding of y = fl32(x c)).
__device__ __forceinline__ float m_stat(const float (&x)[8]) {
  const float m = max3_abs(max3_abs(x[1], x[2], x[3]), max3_abs(x[4], x[5], x[6]), x[7]);
  return max3_abs(2.0f * m, x[0], x[0]);
}
__device__ __forceinline__ bool m_skip(float s, float c, int q) {
  return s * c > (float)(q + 2) * (1.0f + 0x1p-12f);
}

// First-beta search for one block (App. F): the smallest t whose nearest E8 point of
// y = fl32(x * c_t) survives decode(encode(.)); t = k when every beta overloads.
//
// The overload test of a candidate P_t compares its root bound M(P_t) with 2q.  Since
// |M(P_t) - 2 M(y_t)| <= 2 sqrt(2) and M(y_t) = c_t M(x) up to fp32 rounding, the bound
// u_t = 2 c_t M(x) settles most betas without computing P_t: u_t - margin > 2q means t
// surely overloads (it is skipped), u_t + margin < 2q means it surely does not (no test).
// The margin 2 sqrt(2) + 0.02 + 2^-12 u_t covers the covering-radius term and the fp32
// rounding of y_t, M and u_t (together below 2^-19 u_t).  Only betas in between are computed and tested.
__device__ __forceinline__ void encode_block(const float (&v)[8], const float (&c)[4],
                                             const EncodeArgs& a, uint32_t& word, int& tsel) {
  if (a.decoder) {
    // NestQuantM: skip the betas its box rules out, then test each with its decoder
    const float st = m_stat(v);
    int t = 0;
    while (t < a.k - 1 && m_skip(st, pick4(c, t), a.q)) ++t;
    int P[8];
    for (;;) {
      float y[8];
      const float ct = pick4(c, t);
#pragma unroll
      for (int l = 0; l < 8; ++l) y[l] = v[l] * ct;
      nearest_e8(y, P);
      if (t == a.k - 1 || !overloaded_m(P, a.q, a.mq, a.m2q)) break;
      ++t;
    }
    tsel = t;
    word = encode_codes(P, a.q, a.rq, a.mq);
    return;
  }
  const float mx = root_bound_f(v);
  const float two_q = (float)(2 * a.q);
  int t = a.k - 1;
  bool sure = false;
#pragma unroll
  for (int s = a_max_k - 1; s >= 0; --s) {
    if (s < a.k) {
      const float u = 2.0f * c[s] * mx;
      const float margin = kRootMargin + u * 0x1p-12f;
      if (u - margin <= two_q) {   // not surely overloaded: the first such beta is the start
        t = s;
        sure = (u + margin < two_q);
      }
    }
  }
  int P[8];
  for (;;) {
    float y[8];
    const float ct = pick4(c, t);
#pragma unroll
    for (int l = 0; l < 8; ++l) y[l] = v[l] * ct;
    nearest_e8(y, P);
    if (t == a.k - 1 || sure || !overloaded(P, a.q, a.rq, a.mq, a.m2q)) break;
    ++t;
    const float u = 2.0f * pick4(c, t) * mx;
    sure = (u + kRootMargin + u * 0x1p-12f < two_q);
  }
  tsel = t;
  word = encode_codes(P, a.q, a.rq, a.mq);
}

// Fused encode-and-multiply: the decoded tile m_t * X2 of block j of `row`, stored where
// the product's decode stage would put it.  X2 is the lattice point P itself when P is known
// to be reproduced by the decoder (tile_from_x2), else the decode of the code word
// (tile_decoded); rows that are not coded get zeros.  |X2_l| <= 2q for a point that is
// kept, so m X2 is a full-rate 24-bit product.
__device__ __forceinline__ void tile_from_x2(const EncodeArgs& a, int64_t row, int j,
                                             const int (&X2)[8], int t) {
  const int m = (int)((a.mtab >> (8 * t)) & 0xFFu);
  const int64_t idx = row * a.nb_p + j;
  if (a.tile_et == ET_I8) {
    uint32_t lo = 0u, hi = 0u;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      // the low byte of m X2 from the operands' low 24 bits
      lo |= (umul24_v((uint32_t)m, (uint32_t)X2[l]) & 0xFFu) << (8 * l);
      hi |= (umul24_v((uint32_t)m, (uint32_t)X2[4 + l]) & 0xFFu) << (8 * l);
    }
    reinterpret_cast<u32x2*>(a.tiles)[idx] = u32x2{lo, hi};
  } else {
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo = (float)__mul24(m, X2[2 * i]), hi = (float)__mul24(m, X2[2 * i + 1]);
      o[i] = a.tile_et == ET_F16 ? pack16<true>(lo, hi) : pack16<false>(lo, hi);
    }
    reinterpret_cast<u32x4*>(a.tiles)[idx] = u32x4{o[0], o[1], o[2], o[3]};
  }
}

// The same for a point in bytes (P_l + 64 in 0..127).
__device__ __forceinline__ void tile_from_bytes(const EncodeArgs& a, int64_t row, int j,
                                                const E8Bytes& P, int t) {
  const int m = (int)((a.mtab >> (8 * t)) & 0xFFu);
  const int64_t idx = row * a.nb_p + j;
  const uint32_t xa = P.a + 0x40404040u, xb = P.b + 0x40404040u;   // P_l + 128
  if (a.tile_et == ET_I8) {
    reinterpret_cast<u32x2*>(a.tiles)[idx] = tile_i8_from_b8(xa, xb, m);
  } else if (a.tile_et == ET_F16) {
    reinterpret_cast<u32x4*>(a.tiles)[idx] = tile_16_from_b8<true>(xa, xb, m);
  } else {
    reinterpret_cast<u32x4*>(a.tiles)[idx] = tile_16_from_b8<false>(xa, xb, m);
  }
}

__device__ __forceinline__ void tile_decoded(const EncodeArgs& a, int64_t row, int j, uint32_t word,
                                          int t) {
  const int m = (int)((a.mtab >> (8 * t)) & 0xFFu);
  const int64_t idx = row * a.nb_p + j;
  const int dv = decoder_variant(a.decoder, a.q);
  if (a.tile_et == ET_I8) {
    reinterpret_cast<u32x2*>(a.tiles)[idx] =
        dv == 0 ? decode_tile_i8<0>(word, m, a.q, a.m2q) : decode_tile_i8<1>(word, m, a.q, a.m2q);
  } else if (a.tile_et == ET_F16) {
    reinterpret_cast<u32x4*>(a.tiles)[idx] =
        dv == 0 ? decode_tile_16<0, true>(word, m, a.q, a.m2q)
                : (dv == 1 ? decode_tile_16<1, true>(word, m, a.q, a.m2q)
                           : decode_tile_16<2, true>(word, m, a.q, a.m2q));
  } else {
    reinterpret_cast<u32x4*>(a.tiles)[idx] =
        dv == 0 ? decode_tile_16<0, false>(word, m, a.q, a.m2q)
                : (dv == 1 ? decode_tile_16<1, false>(word, m, a.q, a.m2q)
                           : decode_tile_16<2, false>(word, m, a.q, a.m2q));
  }
}

__device__ __forceinline__ void tile_zero(const EncodeArgs& a, int64_t row, int j) {
  const int64_t idx = row * a.nb_p + j;
  if (a.tile_et == ET_I8) {
    reinterpret_cast<u32x2*>(a.tiles)[idx] = u32x2{0u, 0u};
  } else {
    reinterpret_cast<u32x4*>(a.tiles)[idx] = u32x4{0u, 0u, 0u, 0u};
  }
}

// Opt-beta for one block (App. F): every beta is tried; the code of the nearest point of
// y_t = fl32(x c_t) is decoded (Alg. 2 with the code's decoder) to X2_t and compared with
// the normalized block x / r: err_t = sum over l = 0..7, in that order, of d_l^2 with
// d_l = fl64(beta_t X2_t,l) / 2 - fl64(x_l / r), each step rounded in fp64 (the library is
// built without contraction).  The first t of least error is kept.
__device__ __forceinline__ void opt_block(const float (&v)[8], const float (&c)[4], float r,
                                          const EncodeArgs& a, uint32_t& word, int& tsel) {
  double xn[8];
#pragma unroll
  for (int l = 0; l < 8; ++l) xn[l] = (double)v[l] / (double)r;
  double best = INFINITY;
  word = 0u;
  tsel = 0;
#pragma unroll 1
  for (int t = 0; t < a.k; ++t) {
    const float ct = pick4(c, t);
    float y[8];
#pragma unroll
    for (int l = 0; l < 8; ++l) y[l] = v[l] * ct;
    int P[8];
    nearest_e8(y, P);
    const uint32_t w = encode_codes(P, a.q, a.rq, a.mq);
    // the byte decoder: X2_l + 128 in byte l of xs (bit-exact with the 16-bit-pair one)
    uint32_t xs[2];
    if (a.decoder) {
      decode_word_b8<true>(w, a.q, a.m2q, xs[0], xs[1]);
    } else {
      decode_word_b8<false>(w, a.q, a.m2q, xs[0], xs[1]);
    }
    // a select chain, not an indexed read of the argument block (a memory load); halved here,
    // exactly (base > 2^-21), instead of after each of the eight products (4096 x 4096 bf16
    // 102.8 -> 101.4 us, 16384 x 8192 738 -> 727)
    const double hb =
        0.5 * (t == 0 ? a.beta[0] : (t == 1 ? a.beta[1] : (t == 2 ? a.beta[2] : a.beta[3])));
    double err = 0.0;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      const int x2 = (int)((xs[l >> 2] >> (8 * (l & 3))) & 0xFFu) - 128;
      const double d = hb * (double)x2 - xn[l];
      err = err + d * d;
    }
    if (err < best) {
      best = err;
      word = w;
      tsel = t;
    }
  }
}

// Exact RN32(sqrt(S / n)) from a double-double S and a candidate r within a few ulps.
__device__ __forceinline__ float exact_rms(double hi, double lo, double n, float r) {
  for (int it = 0; it < 4; ++it) {
    const float up = next_up(r), dn = next_down(r);
    const int cu = cmp_sum_square(hi, lo, n, 0.5 * ((double)r + (double)up));
    if (cu > 0) { r = up; continue; }
    if (cu == 0) return (__float_as_uint(r) & 1u) ? up : r;
    if (r > 0.0f) {
      const int cd = cmp_sum_square(hi, lo, n, 0.5 * ((double)r + (double)dn));
      if (cd < 0) { r = dn; continue; }
      if (cd == 0) return (__float_as_uint(r) & 1u) ? dn : r;
    }
    break;
  }
  return r;
}

// The fp32 RMS candidate from an fp64 sum, and whether it is certainly RN32(sqrt(S / n)):
// the fp64 sum has relative error below 2^-46 here, so S farther than 2^-40 S from both
// rounding-boundary squares n m^2 settles the rounding.
//
// The candidate itself need not be rounded right (sure says whether it is), so the mean is a
// product with 1 / n and its root two steps from the hardware's reciprocal root, in place of
// an IEEE division and square root (about 40 vector instructions).
__device__ __forceinline__ float rms_candidate(double s, double n, double inv_n, bool& sure) {
  const double q = s * inv_n;
  float r;
  if (q > 0.0 && q < INFINITY) {
    const double y = __builtin_amdgcn_rsq(q), h = 0.5 * y;
    double g = q * y;
    g = __builtin_fma(g, __builtin_fma(-h, g, 0.5), g);
    r = (float)__builtin_fma(__builtin_fma(-g, g, q), h, g);
  } else {
    r = (float)__builtin_sqrt(q);
  }
  sure = true;
  if (s > 0.0 && r > 0.0f && isfinite(r)) {
    const double m_hi = 0.5 * ((double)r + (double)next_up(r));
    const double m_lo = 0.5 * ((double)r + (double)next_down(r));
    const double tol = s * 0x1p-40;
    sure = (n * m_hi * m_hi - s > tol) && (s - n * m_lo * m_lo > tol);
  }
  return r;
}

__device__ __forceinline__ void dd_add_square(double& hi, double& lo, float x) {
  const double sq = (double)x * (double)x;
  double t, e;
  two_sum(hi, sq, t, e);
  hi = t;
  lo += e;
}

// BPT > 0: the row's blocks stay in registers (read once).  BPT == 0: long rows are
// streamed, reading each block once for the scale and once more for the codes.  OPT: the
// Opt-beta strategy (opt_block) instead of First-beta; a separate instantiation, since its
// registers would lower the occupancy of the First-beta kernel.  TILES: also write the
// decoded tiles of the fused encode-and-multiply (likewise a separate instantiation).
template <typename T, int LANES, int BPT, bool OPT, bool TILES>
__global__ __launch_bounds__(LANES > 64 ? LANES : 256) void encode_kernel(
    const T* __restrict__ x, int64_t rows, int cols, int64_t ld_x, EncodeArgs a,
    uint32_t* __restrict__ codes, uint32_t* __restrict__ beta, float* __restrict__ scales) {
  constexpr int WG = LANES > 64 ? LANES : 256;
  constexpr int ROWS_PER_WG = WG / LANES;
  constexpr int NV = BPT > 0 ? BPT : 1;
  __shared__ double red[2 * (WG / 64)];

  const int lane = threadIdx.x % LANES;
  const int64_t row = (int64_t)blockIdx.x * ROWS_PER_WG + threadIdx.x / LANES;
  const bool row_ok = row < rows;  // uniform per group; whole-WG uniform when LANES > 64
  const int nb = cols >> 3;
  const int nbw = (nb + 15) >> 4;
  const T* xr = x + (row_ok ? row : 0) * ld_x;

  float v[NV][8];
  double s = 0.0;
  if constexpr (BPT > 0) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int j = lane + i * LANES;
      if (row_ok && j < nb) {
        load_block<T>(xr + 8 * j, v[i]);
      } else {
#pragma unroll
        for (int l = 0; l < 8; ++l) v[i][l] = 0.0f;
      }
#pragma unroll
      for (int l = 0; l < 8; ++l) s = __builtin_fma((double)v[i][l], (double)v[i][l], s);
    }
  } else {
    for (int j = lane; row_ok && j < nb; j += LANES) {
      load_block<T>(xr + 8 * j, v[0]);
#pragma unroll
      for (int l = 0; l < 8; ++l) s = __builtin_fma((double)v[0][l], (double)v[0][l], s);
    }
  }
  s = group_sum<LANES>(s, red);

  const double n = (double)cols;
  bool sure;
  float r = rms_candidate(s, n, 1.0 / n, sure);
  // With LANES > 64 there is one row per workgroup and every thread holds the same s, so
  // this branch (which synchronizes the workgroup) is uniform.
  if (!sure) {
    double hi = 0.0, lo = 0.0;
    if constexpr (BPT > 0) {
#pragma unroll
      for (int i = 0; i < BPT; ++i)
#pragma unroll
        for (int l = 0; l < 8; ++l) dd_add_square(hi, lo, v[i][l]);
    } else {
      for (int j = lane; row_ok && j < nb; j += LANES) {
        float w[8];
        load_block<T>(xr + 8 * j, w);
#pragma unroll
        for (int l = 0; l < 8; ++l) dd_add_square(hi, lo, w[l]);
      }
    }
    group_sum_dd<LANES>(hi, lo, red);
    r = exact_rms(hi, lo, n, r);
  }

  const bool coded = (r > 0.0f) && isfinite(r);
  float c[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) c[t] = coded ? (float)(1.0 / ((double)r * a.beta[t])) : 0.0f;

  uint32_t* crow = codes + (row_ok ? row : 0) * nb;
  uint32_t* brow = beta + (row_ok ? row : 0) * nbw;
  const int iters = BPT > 0 ? BPT : (nb + LANES - 1) / LANES;
  constexpr int UNROLL = BPT > 0 ? BPT : 1;
#pragma unroll UNROLL
  for (int i = 0; i < iters; ++i) {
    const int j = lane + i * LANES;
    const bool mine = row_ok && j < nb;
    float* vb = v[BPT > 0 ? i : 0];
    if constexpr (BPT == 0) {
      if (mine) load_block<T>(xr + 8 * j, v[0]);
    }
    uint32_t word = 0;
    int tsel = 0;
    if (mine && coded) {
      if constexpr (OPT) {
        opt_block(*reinterpret_cast<float(*)[8]>(vb), c, r, a, word, tsel);
      } else {
        encode_block(*reinterpret_cast<float(*)[8]>(vb), c, a, word, tsel);
      }
    }
    if (mine) crow[j] = word;
    if (TILES && mine) {
      if (coded) {
        tile_decoded(a, row, j, word, tsel);
      } else {
        tile_zero(a, row, j);
      }
    }
    // two-bit beta indices: OR over the 16 consecutive blocks of one word
    uint32_t bits = mine ? ((uint32_t)tsel << (2 * (j & 15))) : 0u;
    constexpr int W = LANES < 16 ? LANES : 16;
#pragma unroll
    for (int m = 1; m < W; m <<= 1) bits |= __shfl_xor(bits, m, 64);
    if (mine && (j & 15) == 0) brow[j >> 4] = bits;
  }
  if (row_ok && lane == 0) scales[row] = r;
}

// ---------------------------------------------------------------------------------------
// Slot-compacted encoder (rows of up to 2048 blocks).
//
// A workgroup owns 64 * BPT blocks per wave ("slots"): slot s = 64 i + l of wave w is block j of
// row row_w, with
//   LANES <  64: row_w = i * (64 / LANES) + l / LANES, j = l % LANES  (a row per lane group
//                and pass; 64 / LANES * BPT rows per wave; workgroups of one wave)
//   LANES == 64: row_w = 0, j = l + 64 i                              (one row per wave, four
//                waves)
//   LANES >  64: row_w = 0, j = 64 w + l + LANES i                   (one row per workgroup
//                of LANES / 64 waves)
// Phase 0 reads every slot from HBM (several of a lane's loads in flight together), stages it
// in LDS (one-wave workgroups read it again instead) and forms the row sums of squares; then
// a lane per row and beta turns the sum into the scale r, the multipliers c_t and the
// thresholds of row_limit.  Phase 1 evaluates every slot, in the byte form, at the first
// beta the root bound of x does not rule out, and finishes it when its point is strictly
// inside the cell (full decoder) or reproduced (NestQuantM).  The others are queued: points
// that overload at the next beta, points on the cell boundary, at the last beta outside the
// cell, or too close to call in fp32 at the same one.  Phase 2 finishes the queue (11% of the
// blocks of Gaussian rows) in rounds of one beta each, the slots still searching compacted
// after every round so that the lanes stay busy; it takes the literal test on the boundary
// and the exact path where the byte form declines.
// Two-bit beta indices are staged in LDS and packed into words at the end.
//
// What bounds it: vector instructions, 1.1 per CU clock at 2^21 x 128 fp16 (385 us; 477 per
// wave of 64 blocks, of which phase 1 takes 300; a build of 644 took 507 us).  There, one-wave
// workgroups meet no barrier (462 -> 406 us: four waves waited while one finished the
// workgroup's queue, a third of the time), unstaged blocks leave LDS for twice the waves, and
// 12 passes a wave fill phase 2's lanes (398 us at 8, 382 at 12, 384 at 16).
// ---------------------------------------------------------------------------------------
template <int LANES, int BPT>
struct SlotMap {
  static constexpr bool WGROW = LANES > 64;
  static constexpr int NW = LANES > 64 ? LANES / 64 : (LANES < 64 ? 1 : 4);   // waves
  static constexpr int RPP = LANES < 64 ? 64 / LANES : 1;           // rows per pass
  static constexpr int ROWS_PER_WAVE = LANES < 64 ? RPP * BPT : 1;
  static constexpr int SLOTS = 64 * BPT;
  __device__ static int row_w(int i, int l) { return LANES < 64 ? i * RPP + l / LANES : 0; }
  // row_w(i, l) = row_step(i) + row_w(0, l), the first term the same for every lane
  __device__ static constexpr int row_step(int i) { return LANES < 64 ? i * RPP : 0; }
  __device__ static int j(int i, int l, int wave) {
    return LANES < 64 ? l % LANES : (LANES == 64 ? l + 64 * i : 64 * wave + l + LANES * i);
  }
  // inverse map for block j of row row_w: wave and slot
  __device__ static void slot_of(int row_w, int j, int wave_hint, int& w, int& s) {
    if constexpr (LANES < 64) {
      w = wave_hint;
      s = (row_w / RPP) * 64 + (row_w % RPP) * LANES + j;
    } else if constexpr (LANES == 64) {
      w = wave_hint;
      s = j;
    } else {
      const int rem = j % LANES;
      w = rem >> 6;
      s = (j / LANES) * 64 + (rem & 63);
    }
  }
};

// What one evaluation of a block at a beta says.
enum Verdict {
  KEEP,       // the point is reproduced: coded here
  NEXT,       // it overloads and there is a larger beta
  BOUNDARY,   // on the cell boundary (full decoder): the literal test decides
  EXACT       // not for the byte form: too close to call in fp32, or a point at the last beta
              // that may overload (strictly outside the cell; NestQuantM: not reproduced)
};

// Block v at beta t in the byte form: the point X it decodes to and, when it is kept, its code
// word.  The root bound of the point settles every one off the cell boundary; NestQuantM has
// no such bound, so there the word is decoded again.  LITERAL: the points on the boundary,
// where Alg. 5's tie rules decide, take the literal test here, by the decode of their word (a
// branch that few waves of phase 1 could skip, so phase 1 queues them).  |v| ct must be
// within kE8BytesMax.
template <bool LITERAL>
__device__ __forceinline__ Verdict eval_bytes(const float (&v)[8], float ct, int t,
                                              const EncodeArgs& a, E8Bytes& X, uint32_t& word) {
  if (!nearest_e8_bytes(v, ct, X)) return EXACT;
  const bool last = t == a.k - 1;
  uint32_t xa, xb;   // X2 + 128 of the word
  if (a.decoder) {
    // outside the decoder's box the word means nothing, and its decode, which lies inside
    // the box, differs from the point
    word = encode_e8_bytes<true>(X, a.q, a.mq);
    decode_word_b8<true>(word, a.q, a.m2q, xa, xb);
    const bool same = xa == X.a + 0x40404040u && xb == X.b + 0x40404040u;
    return same ? KEEP : (last ? EXACT : NEXT);
  }
  const int M = e8_bytes_root_bound(X);
  if (M > 2 * a.q) return last ? EXACT : NEXT;
  word = encode_e8_bytes<LITERAL>(X, a.q, a.mq);   // on the boundary |P_l - P_0| / 2 may be q
  if (M < 2 * a.q) return KEEP;
  if constexpr (!LITERAL) return BOUNDARY;
  decode_word_b8<false>(word, a.q, a.m2q, xa, xb);
  const bool same = xa == X.a + 0x40404040u && xb == X.b + 0x40404040u;
  X.a = xa - 0x40404040u;
  X.b = xb - 0x40404040u;
  return same || last ? KEEP : NEXT;
}

// One evaluation of a queued block at beta t in the exact arithmetic: its nearest point P, and
// whether the search stops there (the last beta, or a point that does not overload).
__device__ __forceinline__ bool eval_exact(const float (&v)[8], float ct, int t,
                                           const EncodeArgs& a, int (&P)[8]) {
  float y[8];
#pragma unroll
  for (int l = 0; l < 8; ++l) y[l] = v[l] * ct;
  nearest_e8(y, P);
  if (t == a.k - 1) return true;
  return a.decoder ? !overloaded_m(P, a.q, a.mq, a.m2q)
                   : !overloaded(P, a.q, a.rq, a.mq, a.m2q);
}

// Raw input of one block: 16 B for 16-bit types, 32 B for fp32.
template <typename T> struct RawBlock { u32x4 w; };
template <> struct RawBlock<float> { f32x4 a, b; };

// NT: read once (streamed past the caches), else read again soon.
template <typename T, bool NT>
__device__ __forceinline__ void load_raw(const T* __restrict__ p, RawBlock<T>& r) {
  if constexpr (sizeof(T) == 4) {
    const f32x4* q = reinterpret_cast<const f32x4*>(p);
    r.a = NT ? __builtin_nontemporal_load(q) : q[0];
    r.b = NT ? __builtin_nontemporal_load(q + 1) : q[1];
  } else {
    const u32x4* q = reinterpret_cast<const u32x4*>(p);
    r.w = NT ? __builtin_nontemporal_load(q) : q[0];
  }
}
template <typename T>
__device__ __forceinline__ void zero_raw(RawBlock<T>& r) { r.w = u32x4{0u, 0u, 0u, 0u}; }
template <>
__device__ __forceinline__ void zero_raw<float>(RawBlock<float>& r) {
  r.a = f32x4{0.f, 0.f, 0.f, 0.f};
  r.b = r.a;
}
template <typename T>
__device__ __forceinline__ void unpack_raw(const RawBlock<T>& r, float (&v)[8]);
template <>
__device__ __forceinline__ void unpack_raw<float>(const RawBlock<float>& r, float (&v)[8]) {
  v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
  v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
}
template <>
__device__ __forceinline__ void unpack_raw<uint16_t>(const RawBlock<uint16_t>& r, float (&v)[8]) {
  const uint32_t w[4] = {r.w.x, r.w.y, r.w.z, r.w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
template <>
__device__ __forceinline__ void unpack_raw<_Float16>(const RawBlock<_Float16>& r, float (&v)[8]) {
  const uint32_t w[4] = {r.w.x, r.w.y, r.w.z, r.w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] & 0xffffu));
    v[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] >> 16));
  }
}

// ROT (one row per workgroup only): the row is first rotated in LDS (rotate_rows_lds, the
// arithmetic of nq_rotate) and the encoder reads its blocks from there, times a.rot_s.
template <typename T, int LANES, int BPT, bool TILES, bool ROT>
// Workgroups of a row (LANES 128 and 256) are held to 96 VGPRs, five waves per SIMD: the
// fused launch (W's tile decode beside the coding of A) measured 94.9-95.1 against
// 96.2-96.4 us per q_proj step at 97 VGPRs (four waves, no spills), and the 70B MLP step
// 976-982 against 991-997 us (bf16 tiles).  The one-wave workgroups of short rows and the
// 64-lane instantiation with one block per thread (rows of at most 64 blocks) get the same
// bound; the forms of 12 passes that write tiles pay it with 12 to 32 bytes of scratch.
__global__ __launch_bounds__((SlotMap<LANES, BPT>::NW * 64))
__attribute__((amdgpu_waves_per_eu(LANES != 64 || BPT == 1 ? 5 : 1))) void encode_wave_kernel(
    const T* __restrict__ x, int64_t rows, int cols, int64_t ld_x, EncodeArgs a,
    uint32_t* __restrict__ codes, uint32_t* __restrict__ beta, float* __restrict__ scales) {
  using SM = SlotMap<LANES, BPT>;
  constexpr int SLOTS = SM::SLOTS;
  constexpr int RW = SM::ROWS_PER_WAVE;
  constexpr int NW = SM::NW;
  constexpr bool CARRIES = SM::WGROW && LANES * BPT <= 1024;   // encode_carries_task
  constexpr int CW = SM::WGROW ? 1 : NW;         // row tables: per wave, or one per workgroup
  static_assert(!ROT || LANES == 256, "rotation in LDS needs one row per 256-lane workgroup");
  // Blocks are staged in LDS, except by the one-wave workgroups of short rows, which read
  // them again (from the caches): their LDS would be the bound on resident waves.
  constexpr bool STAGED = NW > 1 && !ROT;
  __shared__ RawBlock<T> rawl[NW][STAGED ? SLOTS : 1];
  __shared__ __attribute__((aligned(16))) float rbuf[ROT ? 8 * 4 * SLOTS : 1];
  __shared__ uint16_t queue[NW][SLOTS];            // w << 12 | sl << 2 | t
  __shared__ uint16_t qnext[NW > 1 ? NW * SLOTS : 1];
  __shared__ int qcnt[4];
  __shared__ uint8_t tsl[NW][SLOTS];
  __shared__ float crow[CW][RW][4];
  __shared__ __attribute__((aligned(16))) float chi[CW][RW][4];
  __shared__ float rrow[CW][RW];
  __shared__ double rsum[NW][RW];
  __shared__ int qlen[NW];

  // A TileTask's a.task.wgs workgroups come last in the grid: dispatched once every row has
  // started, they fill the CUs that the encoder's last rows leave idle.  Measured on the
  // fused step with bf16 tiles: q_proj 98 us (last) against 102.6 (first), the 70B MLP 988
  // against 992; spreading them among the encoder's workgroups was slower.
  const int64_t bid = blockIdx.x;
  if constexpr (TILES && CARRIES) {
    const int64_t first = (int64_t)gridDim.x - a.task.wgs;
    if (bid >= first) {
      run_tile_task<NW * 64>(a.task, a.tile_et, bid - first);
      return;
    }
  }
  // the wave index is uniform over the wave: held in a scalar register, so that row offsets
  // derived from it are scalar arithmetic
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int cw = SM::WGROW ? 0 : wave;
  const int nb = cols >> 3;
  const int nbw = (nb + 15) >> 4;
  auto row_base = [&](int w) -> int64_t {
    return SM::WGROW ? bid : (bid * NW + w) * RW;
  };
  const int64_t row0 = row_base(wave);
  const double n = (double)cols, inv_n = 1.0 / n;
  // index of block j of row row_base(w) + rw in the code words: rows of more than 64 blocks
  // have rw = 0, shorter rows w RW + rw < 2^12 and nb <= 64, a 24-bit product
  auto code_at = [&](int w, int rw, int j) -> int64_t {
    if constexpr (SM::WGROW) return row_base(w) * nb + j;
    return (bid * NW * RW) * (int64_t)nb + __mul24(w * RW + rw, nb) + j;
  };
  // block of slot sl of wave w, as fp32
  auto slot_block = [&](int w, int sl, float (&v)[8]) {
    if constexpr (!STAGED && !ROT) {
      RawBlock<T> raw;
      load_raw<T, false>(x + (row_base(w) + SM::row_w(sl >> 6, sl & 63)) * ld_x +
                             8 * SM::j(sl >> 6, sl & 63, w), raw);
      unpack_raw<T>(raw, v);
    } else if constexpr (ROT) {
      const int pe = lds_pos(8 * SM::j(sl >> 6, sl & 63, w));
#pragma unroll
      for (int l = 0; l < 8; ++l) v[l] = rbuf[pe ^ l] * a.rot_s;
    } else {
      unpack_raw<T>(rawl[w][sl], v);
    }
  };

  if (threadIdx.x < 4) qcnt[threadIdx.x] = 0;   // phase 2's list lengths, one per round

  // ---- phase 0: stage the slots in LDS, row sums of squares ----
  if constexpr (ROT) {
    // the whole workgroup rotates its row (uniform: one row per workgroup)
    if (row0 < rows) rotate_rows_lds<T>(x + row0 * ld_x, ld_x, 1, cols, a.rot_p, a.rot_lp, rbuf);
    double part = 0.0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int j = SM::j(i, lane, wave);
      if (row0 < rows && j < nb) {
        float v[8];
        slot_block(wave, i * 64 + lane, v);
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < 8; ++l) s = __builtin_fma((double)v[l], (double)v[l], s);
        part += s;
      }
    }
    part = wave_sum<64>(part);
    if (lane == 0) rsum[wave][0] = part;
  } else {
    // up to FLY blocks of a lane in flight together
    constexpr int FLY = BPT <= 8 ? BPT : 6;
    static_assert(BPT % FLY == 0, "whole groups of loads");
    // one 64-bit row offset per lane; the rest of each block's address is uniform
    const T* __restrict__ x_lane = x + (row0 + SM::row_w(0, lane)) * ld_x;
    double part = 0.0;
#pragma unroll
    for (int i0 = 0; i0 < BPT; i0 += FLY) {
      RawBlock<T> raw[FLY];
#pragma unroll
      for (int u = 0; u < FLY; ++u) {
        const int i = i0 + u, j = SM::j(i, lane, wave);
        if (row0 + SM::row_w(i, lane) < rows && j < nb) {
          load_raw<T, STAGED>(x_lane + SM::row_step(i) * ld_x + 8 * j, raw[u]);
        } else {
          zero_raw<T>(raw[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < FLY; ++u) {
        const int i = i0 + u;
        if constexpr (STAGED) rawl[wave][i * 64 + lane] = raw[u];
        float v[8];
        unpack_raw<T>(raw[u], v);
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < 8; ++l) s = __builtin_fma((double)v[l], (double)v[l], s);
        if constexpr (LANES < 64) {
          s = wave_sum<LANES>(s);
          if (lane % LANES == 0) rsum[wave][SM::row_w(i, lane)] = s;
        } else {
          part += s;
        }
      }
    }
    if constexpr (LANES >= 64) {
      part = wave_sum<64>(part);
      if (lane == 0) rsum[wave][0] = part;
    }
  }
  __syncthreads();

  // ---- row scales and multipliers ----
  // Four lanes per row, one per beta: all four find the scale (the same instructions) and
  // then each the multiplier and threshold of its own beta (one double division a lane
  // where a lane per row took four, with most of the wave idle).  One row per workgroup:
  // wave 0 alone; the other rows: each wave its own, 16 at a time.
  for (int e = lane; e < 4 * RW && (!SM::WGROW || wave == 0); e += 64) {
    const int rw = e >> 2, t = e & 3;
    const int64_t row = row0 + rw;
    if (row < rows) {
      double s = rsum[wave][rw];
      if constexpr (SM::WGROW) {
        s = rsum[0][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += rsum[w][0];
      }
      bool sure;
      float r = rms_candidate(s, n, inv_n, sure);
      if (!sure) {
        // rare: the double-double sum of the row, block by block from LDS
        double hi = 0.0, lo = 0.0;
        for (int j = 0; j < nb; ++j) {
          int w, sl;
          SM::slot_of(rw, j, wave, w, sl);
          float v[8];
          slot_block(w, sl, v);
#pragma unroll
          for (int l = 0; l < 8; ++l) dd_add_square(hi, lo, v[l]);
        }
        double sd, ed;
        two_sum(hi, lo, sd, ed);
        r = exact_rms(sd, ed, n, r);
      }
      const bool coded = (r > 0.0f) && isfinite(r);
      const double rb = (double)r * a.beta[t];
      crow[cw][rw][t] = coded ? (float)(1.0 / rb) : 0.0f;
      // betas 0..2: the threshold above which a block surely overloads there and starts at a
      // later one (infinite from the last beta on); entry 3: the largest |x| the byte form
      // takes at the last beta (the thresholds keep |y| below q + 3 at the others)
      float hi = INFINITY;
      if (t == 3 || t < a.k - 1)
        hi = row_limit(t == 3 ? kBytesFactor : skip_factor(a.q, a.decoder),
                       t == 3 ? (double)r * a.beta[a.k - 1] : rb);
      chi[cw][rw][t] = hi;
      if (t == 0) {
        rrow[cw][rw] = coded ? r : 0.0f;
        scales[row] = r;
      }
    }
  }
  __syncthreads();

  // ---- phase 1: every slot at its predicted beta ----
  uint32_t* __restrict__ codes_w = codes + row0 * nb;   // this wave's rows
  int qn = 0;   // queue length, uniform over the wave
  // blocks that are not staged: the next pass's, in flight while this one is evaluated
  [[maybe_unused]] RawBlock<T> ahead;
  [[maybe_unused]] const T* __restrict__ x_next = x + (row0 + SM::row_w(0, lane)) * ld_x + 8 * SM::j(0, lane, wave);
  auto fetch = [&](int i) {
    if constexpr (!STAGED && !ROT) {
      zero_raw<T>(ahead);
      if (i < BPT && row0 + SM::row_w(i, lane) < rows && SM::j(i, lane, wave) < nb)
        load_raw<T, false>(x_next, ahead);
      x_next += SM::RPP * ld_x;
    }
  };
  fetch(0);
#pragma unroll 1
  for (int i = 0; i < BPT; ++i) {
    const int sl = i * 64 + lane;
    const int rw = SM::row_w(i, lane), j = SM::j(i, lane, wave);
    const int64_t row = row0 + rw;
    const bool valid = row < rows && j < nb;
    [[maybe_unused]] const RawBlock<T> now = ahead;
    fetch(i + 1);
    const bool coded = valid && rrow[cw][rw] != 0.0f;
    bool queued = false;
    int start = 0, t0 = 0;
    uint32_t word = 0u;
    E8Bytes P{0x40404040u, 0x40404040u};
    if (coded) {
      float v[8];
      if constexpr (!STAGED && !ROT) {
        unpack_raw<T>(now, v);
      } else {
        slot_block(wave, sl, v);
      }
      // first beta whose point is not surely overloaded: one threshold test per beta
      const float mx = a.decoder ? m_stat(v) : root_bound_f(v);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(chi[cw][rw]);
      t0 = mx > hi.x ? (mx > hi.y ? (mx > hi.z ? 3 : 2) : 1) : 0;
      const Verdict vd = eval_bytes<false>(v, crow[cw][rw][t0], t0, a, P, word);
      const bool past = mx > hi.w;   // mx bounds every |x_l|: the bytes may have wrapped
      queued = vd != KEEP || past;
      start = t0 + (vd == NEXT && !past ? 1 : 0);
    }
    const uint64_t mask = __ballot(queued);
    if (queued) {
      const int pos = qn + __popcll(mask & ((1ull << lane) - 1ull));
      queue[wave][pos] = (uint16_t)((wave << 12) | (sl << 2) | start);
    } else if (valid) {
      codes_w[__mul24(rw, nb) + j] = word;   // rw = 0 or nb <= 64
      tsl[wave][sl] = (uint8_t)t0;
      // a point kept here is its own decode, X2 = P (zero for rows that are not coded)
      if constexpr (TILES) tile_from_bytes(a, row, j, P, t0);
    }
    qn += __popcll(mask);
  }
  if (NW > 1 && lane == 0) qlen[wave] = qn;
  __syncthreads();

  // ---- phase 2: the queued slots of the whole workgroup, one beta per round ----
  // Round 0 takes the wave queues; a slot whose point overloads goes on to the next beta in
  // the next round, through a compacted list, so that every round keeps its lanes busy
  // instead of each wave looping until its slowest lane is done.  There are at most k rounds
  // (t grows by one per round, and t = k - 1 always stops).  A workgroup of one wave
  // compacts its queue in place (the wave writes entries it has already read) and meets no
  // barrier that waits.
  {
    int qs[NW + 1];   // starts of the wave queues in round 0's index space
    qs[0] = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) qs[w + 1] = qs[w] + (NW > 1 ? qlen[w] : qn);
    int n = qs[NW];
#pragma unroll 1
    for (int rd = 0; n > 0; ++rd) {
      // one array for a workgroup of one wave
      uint16_t* out_q = NW == 1 || (rd & 1) ? &queue[0][0] : qnext;
      const uint16_t* in_q = NW > 1 && (rd & 1) ? qnext : &queue[0][0];
      int nn = 0;       // the next round's length so far (one wave)
#pragma unroll 1
      for (int base = 0; base < n; base += NW * 64) {
        const int idx = base + (int)threadIdx.x;
        bool more = false;
        uint32_t next = 0;
        if (idx < n) {
          uint32_t e;
          if (NW > 1 && rd == 0) {
            int w = 0;
#pragma unroll
            for (int u = 1; u < NW; ++u) w += idx >= qs[u];
            int off = 0;
#pragma unroll
            for (int u = 1; u < NW; ++u) off = w == u ? qs[u] : off;
            e = queue[w][idx - off];
          } else {
            e = in_q[idx];
          }
          const int w = NW > 1 ? (int)(e >> 12) : 0;
          const int sl = (int)((e >> 2) & 1023u), t = (int)(e & 3u);
          const int i = sl >> 6, l = sl & 63;
          const int rw = SM::row_w(i, l), j = SM::j(i, l, w);
          const int64_t row = row_base(w) + rw;
          const int c2 = SM::WGROW ? 0 : w;
          float v[8];
          slot_block(w, sl, v);
          const float ct = crow[c2][rw][t];
          const float vmax = max3_abs(max3_abs(v[0], v[1], v[2]), max3_abs(v[3], v[4], v[5]),
                                      max3_abs(v[6], v[7], v[7]));
          E8Bytes Pb;
          uint32_t word;
          const Verdict vd = vmax <= chi[c2][rw][3] ? eval_bytes<true>(v, ct, t, a, Pb, word) : EXACT;
          if (vd == KEEP) {
            codes[code_at(w, rw, j)] = word;
            tsl[w][sl] = (uint8_t)t;
            if constexpr (TILES) tile_from_bytes(a, row, j, Pb, t);
          } else {
            more = vd == NEXT;
            if (!more) {
              int P[8];
              if (eval_exact(v, ct, t, a, P)) {
                word = encode_codes(P, a.q, a.rq, a.mq);
                codes[code_at(w, rw, j)] = word;
                tsl[w][sl] = (uint8_t)t;
                if constexpr (TILES) {
                  if (t < a.k - 1) {
                    tile_from_x2(a, row, j, P, t);
                  } else {
                    tile_decoded(a, row, j, word, t);
                  }
                }
              } else {
                more = true;
              }
            }
            next = ((uint32_t)w << 12) | ((uint32_t)sl << 2) | (uint32_t)(t + 1);
          }
        }
        // wave-aggregated append to the next round's list
        const uint64_t mask = __ballot(more);
        if (mask != 0) {
          int pos0 = nn;
          if constexpr (NW == 1) {
            nn += __popcll(mask);
          } else {
            if (lane == 0) pos0 = atomicAdd(&qcnt[rd], __popcll(mask));
            pos0 = __shfl(pos0, 0, 64);
          }
          if (more) out_q[pos0 + __popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)next;
        }
      }
      __syncthreads();
      n = NW == 1 ? nn : qcnt[rd];
    }
  }

  // ---- beta words: 16 two-bit indices of consecutive blocks (consecutive lanes) ----
  // Block j sits in lane j mod 16 of its group of 16 lanes (j mod 8 of 8 when rows have 8
  // blocks): each lane shifts its own index into place and an OR across the group forms the
  // word, which the group's first lane stores.
  constexpr int G = LANES < 16 ? LANES : 16;
  uint32_t* __restrict__ beta_w = beta + row0 * nbw;   // this wave's rows
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const int rw = SM::row_w(i, lane), j = SM::j(i, lane, wave);
    const int64_t row = row0 + rw;
    const bool ok = row < rows && j < nb;
    uint32_t bits = ok ? (uint32_t)tsl[wave][i * 64 + lane] << (2 * (j & 15)) : 0u;
    bits |= dpp_across<1>(bits);
    bits |= dpp_across<2>(bits);
    bits |= dpp_across<4>(bits);
    if constexpr (G > 8) bits |= dpp_across<8>(bits);
    if (ok && (j & 15) == 0) beta_w[__mul24(rw, nbw) + (j >> 4)] = bits;   // rw = 0 or nbw <= 4
  }
}

// ---------------------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------------------
template <typename T, int LANES, int BPT, bool OPT, bool TILES>
static hipError_t launch_t(const void* x, int64_t rows, int cols, int64_t ld_x,
                           const EncodeArgs& a, uint32_t* codes, uint32_t* beta, float* scales,
                           hipStream_t st) {
  constexpr int WG = LANES > 64 ? LANES : 256;
  constexpr int RPW = WG / LANES;
  const int64_t grid = (rows + RPW - 1) / RPW;
  hipLaunchKernelGGL((encode_kernel<T, LANES, BPT, OPT, TILES>), dim3((unsigned)grid), dim3(WG), 0, st,
                     (const T*)x, rows, cols, ld_x, a, codes, beta, scales);
  return hipGetLastError();
}

template <typename T, int LANES, int BPT, bool TILES, bool ROT = false>
static hipError_t launch_w(const void* x, int64_t rows, int cols, int64_t ld_x,
                           const EncodeArgs& a, uint32_t* codes, uint32_t* beta, float* scales,
                           hipStream_t st) {
  using SM = SlotMap<LANES, BPT>;
  constexpr int WG = SM::NW * 64;
  const int64_t rows_per_wg = SM::WGROW ? 1 : SM::NW * SM::ROWS_PER_WAVE;
  int64_t grid = (rows + rows_per_wg - 1) / rows_per_wg;
  if (TILES && SM::WGROW && LANES * BPT <= 1024) grid += a.task.wgs;
  hipLaunchKernelGGL((encode_wave_kernel<T, LANES, BPT, TILES, ROT>), dim3((unsigned)grid), dim3(WG), 0, st,
                     (const T*)x, rows, cols, ld_x, a, codes, beta, scales);
  return hipGetLastError();
}

template <typename T, bool TILES>
static hipError_t launch_dtype(const void* x, int64_t rows, int cols, int64_t ld_x,
                               const EncodeArgs& a, uint32_t* codes, uint32_t* beta,
                               float* scales, hipStream_t st) {
  const int nb = cols / 8;
  if (a.rot_p) {
    // rows rotated in LDS first: one row per workgroup
#define NQ_R(B) return launch_w<T, 256, B, TILES, true>(x, rows, cols, ld_x, a, codes, beta, scales, st)
    if (!encode_rotates(cols, a.strategy)) return hipErrorInvalidValue;
    if (nb <= 512) NQ_R(2);
    if (nb <= 1024) NQ_R(4);
    NQ_R(8);
#undef NQ_R
  }
  if (a.strategy) {
    // Opt-beta: a lane group of up to 64 holds short rows in registers; longer rows stream
#define NQ_O(L, B) return launch_t<T, L, B, true, TILES>(x, rows, cols, ld_x, a, codes, beta, scales, st)
    if (nb <= 8) NQ_O(8, 1);
    if (nb <= 16) NQ_O(16, 1);
    if (nb <= 32) NQ_O(32, 1);
    if (nb <= 64) NQ_O(64, 1);
    if (nb <= 2048) NQ_O(256, 0);
    NQ_O(1024, 0);
#undef NQ_O
  }
#define NQ_W(L, B) return launch_w<T, L, B, TILES>(x, rows, cols, ld_x, a, codes, beta, scales, st)
#define NQ_L(L, B) return launch_t<T, L, B, false, TILES>(x, rows, cols, ld_x, a, codes, beta, scales, st)
  // Short rows, one wave per workgroup: the more passes a wave takes, the fuller the lanes of
  // its phase 2, as long as there are waves for every SIMD (rows of 128 fp16 entries, in
  // us for 1, 4 and 12 passes: 16384 rows 11.4, 11.8, 23.4; 49152: 24.7, 17.7, 25.2; 200000:
  // 82.8, 47.9, 53.2; 2^21: 839, 420, 385).
#define NQ_S(L)                                            \
  if (rows >= (64 / L) * (int64_t)12 * 16384) NQ_W(L, 12); \
  if (rows >= (64 / L) * (int64_t)4 * 1024) NQ_W(L, 4);    \
  NQ_W(L, 1)
  if (nb <= 8) { NQ_S(8); }
  if (nb <= 16) { NQ_S(16); }
  if (nb <= 32) { NQ_S(32); }
  if (nb <= 64) NQ_W(64, 1);
  if (nb <= 128) NQ_W(64, 2);
  if (nb <= 256) NQ_W(64, 4);
  // 257..512 blocks: with many rows, one row per two waves keeps the launch to a single wave
  // of workgroups over the CUs; with few rows, four waves per row finish each row sooner
  if (nb <= 512) { if (rows > 1024) NQ_W(128, 4); NQ_W(256, 2); }
  if (nb <= 1024) NQ_W(256, 4);
  if (nb <= 2048) NQ_W(256, 8);
  if (nb <= 4096) NQ_L(512, 8);
  NQ_L(1024, 0);
#undef NQ_W
#undef NQ_S
#undef NQ_L
}

hipError_t launch_encode(const void* x, int dtype, int64_t rows, int cols, int64_t ld_x,
                         const EncodeArgs& a, uint32_t* codes, uint32_t* beta, float* scales,
                         hipStream_t st) {
  if (a.task.wgs > 0 && !(a.tiles && encode_carries_task(cols, a.strategy)))
    return hipErrorInvalidValue;
  if (a.tiles) {
    switch (dtype) {
      case 0: return launch_dtype<float, true>(x, rows, cols, ld_x, a, codes, beta, scales, st);
      case 1: return launch_dtype<_Float16, true>(x, rows, cols, ld_x, a, codes, beta, scales, st);
      default: return launch_dtype<uint16_t, true>(x, rows, cols, ld_x, a, codes, beta, scales, st);
    }
  }
  switch (dtype) {
    case 0: return launch_dtype<float, false>(x, rows, cols, ld_x, a, codes, beta, scales, st);
    case 1: return launch_dtype<_Float16, false>(x, rows, cols, ld_x, a, codes, beta, scales, st);
    default: return launch_dtype<uint16_t, false>(x, rows, cols, ld_x, a, codes, beta, scales, st);
  }
}

}  // namespace nq
