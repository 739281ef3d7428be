// Nearest E8 point, root bound and Voronoi code with the point's coordinates as bytes.
// Included by nq_device.hpp inside namespace nq (it needs max3_abs, min3_abs, bcnt_add,
// umul24_v and the amdgcn byte builtins).
//
// The encoder is bound by its count of vector instructions (about one wave instruction per
// CU clock), so the point P of 2E8 is kept as eight biased bytes, byte l = P_l + 64, in two
// registers, and everything after the fp32 residuals works on four coordinates per
// instruction.  Instructions per block, against the arithmetic on one coordinate per
// register that the exact path keeps: nearest point about 110 (200), root bound 42 (55),
// code 35 (70).
//
// Where it applies: |y_l| <= kE8BytesMax for the nearest point (the bytes cannot wrap then),
// M(P) < 2q for the code.  What it cannot decide it says (false), and the caller redoes the
// block with nearest_e8.
#pragma once

// |y| up to which every byte P_l + 64 stays in [4, 124] (|P_l| <= 2 (29 + 1/2) + 1).
constexpr float kE8BytesMax = 29.0f;

constexpr float kRootMargin = 2.8284272f + 0.02f;  // 2 sqrt(2), rounded up, + slack

// The limits of a row on its blocks' entries, k rb with rb = fl64(r beta_t): products only (no
// division), since for c = fl32(fl64(1 / rb)), 1 / c <= rb (1 + 2^-23).  In fp32 while the factors
// are normal there, else in fp64 and one step up, so that the limits hold at every scale: a
// block starts at the first beta whose threshold it does not pass, and at the betas below the
// last it is that threshold which keeps |y| within kE8BytesMax.  (Limits a step too high are
// harmless: that moves |x| c by less than 2^-20.)
__device__ __forceinline__ float row_limit(float k, double rb) {
  if (rb > 1e-30) return k * (float)rb;
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, (float)((double)k * rb)) + 1u);
}

// Factor of the threshold on the root bound M(x) of a block above which beta t surely
// overloads: for the nearest point P of y = fl32(c x), M(P) >= 2 M(y) - 2 sqrt(2) (covering
// radius 1, roots of norm sqrt(2)) and M(y) = c M(x) up to relative rounding errors below
// 2^-19 (y, and the fp32 evaluation of M), so M(x) > (2q + 2 sqrt(2) + 0.02) / (2 c (1 - 2^-12))
// implies M(P) > 2q.  The 2^-19 covers the threshold's own roundings (each below 2^-24) and
// 1 / (1 - 2^-12) - 1 - 2^-12.  A threshold a little above the exact one only lets a block try a
// beta that overloads; the search still ends at the same beta.
// The NestQuantM counterpart for the statistic m_stat: (q + 2)(1 + 2^-12) / c.
__device__ __forceinline__ float skip_factor(int q, int decoder) {
  return (decoder ? (float)(q + 2) : (float)q + 0.5f * kRootMargin) *
         (1.0f + 0x1p-12f + 0x1p-19f);
}

// Factor of the largest |x| whose products x c the byte form takes.
constexpr float kBytesFactor = kE8BytesMax * (1.0f - 0x1p-16f);

struct E8Bytes {
  uint32_t a, b;   // coordinates 0-3 and 4-7, byte l = P_l + 64
};

// P = the nearest point of 2E8 / 2 to y = fl32(x * c), in 2E8 units (Alg. 5 with the tie rules
// of nearest_e8); false, and P unset, when fp32 cannot tell (the gap of the two candidates
// within its rounding error, or a coordinate exactly halfway between integers, where rounding
// half to even differs from Alg. 5's half down).  Needs |y_l| <= kE8BytesMax.
//
// With n = rint(y) and s = y - n (both exact): e = |s|, g = [s < 0], d = n - g, so that
// nearest_e8's D8 candidate is 2n and its D8+1/2 candidate 2n + sgn(s) = 2 (n - g) + 1, its
// parities are those of sum n and sum n - #g, and the fix (max e or min e, lowest index)
// moves the coordinate by 2 towards s (D8) or against it (D8+1/2).  y is formed by a fused
// multiply with +0, which turns a product -0 into +0 (so s = +0 there, g = 0) and rounds as
// the product does; n comes out of the low byte of y + 1.5 * 2^23 + 32.
__device__ __forceinline__ bool nearest_e8_bytes(const float (&x)[8], float c, E8Bytes& P) {
  constexpr float kMagic = 12582912.0f + 32.0f;
  uint32_t t[8];
  float s[8];
#pragma unroll
  for (int l = 0; l < 8; ++l) {
    const float y = __builtin_fmaf(x[l], c, 0.0f);
    const float tf = y + kMagic;
    t[l] = __builtin_bit_cast(uint32_t, tf);
    s[l] = y - (tf - kMagic);
  }
  const float ep = max3_abs(max3_abs(s[0], s[1], s[2]), max3_abs(s[3], s[4], s[5]),
                            max3_abs(s[6], s[7], s[7]));
  const float er = min3_abs(min3_abs(s[0], s[1], s[2]), min3_abs(s[3], s[4], s[5]),
                            min3_abs(s[6], s[7], s[7]));
  const float se = ((__builtin_fabsf(s[0]) + __builtin_fabsf(s[1])) +
                    (__builtin_fabsf(s[2]) + __builtin_fabsf(s[3]))) +
                   ((__builtin_fabsf(s[4]) + __builtin_fabsf(s[5])) +
                    (__builtin_fabsf(s[6]) + __builtin_fabsf(s[7])));
  // bytes n + 32, and bytes whose bit 7 is g (the top bytes of s)
  const uint32_t nA = __builtin_amdgcn_perm(t[1], t[0], 0x0C0C0400u) |
                      __builtin_amdgcn_perm(t[3], t[2], 0x04000C0Cu);
  const uint32_t nB = __builtin_amdgcn_perm(t[5], t[4], 0x0C0C0400u) |
                      __builtin_amdgcn_perm(t[7], t[6], 0x04000C0Cu);
  auto top = [&](int l) { return __builtin_bit_cast(uint32_t, s[l]); };
  const uint32_t gA = __builtin_amdgcn_perm(top(1), top(0), 0x0C0C0703u) |
                      __builtin_amdgcn_perm(top(3), top(2), 0x07030C0Cu);
  const uint32_t gB = __builtin_amdgcn_perm(top(5), top(4), 0x0C0C0703u) |
                      __builtin_amdgcn_perm(top(7), top(6), 0x07030C0Cu);
  // parities of sum n (8 * 32 is even) and of sum n - #g, as masks
  const uint32_t pn = __builtin_amdgcn_sad_u8(nA, 0u, __builtin_amdgcn_sad_u8(nB, 0u, 0u));
  const uint32_t pd = bcnt_add((gA ^ gB) & 0x80808080u, pn);
  const uint32_t odd1 = 0u - (pn & 1u), odd2 = 0u - (pd & 1u);
  // the gap of nearest_e8, in fp32: below 1e-5 off in all
  const float f1 = __builtin_bit_cast(
      float, odd1 & __builtin_bit_cast(uint32_t, __builtin_fmaf(-2.0f, ep, 1.0f)));
  const float f2 = __builtin_bit_cast(float, odd2 & __builtin_bit_cast(uint32_t, er));
  const float gap = __builtin_fmaf(-2.0f, f2, (se - 2.0f) + f1);
  const bool d8 = gap < 0.0f;

  // 2 (n - g) + 1 + 64 (D8+1/2) or 2 n + 64 (D8) in each byte
  const uint32_t half = d8 ? 0u : 0x01010101u;
  const uint32_t pA = ((nA - ((gA >> 7) & half)) << 1) | half;
  const uint32_t pB = ((nB - ((gB >> 7) & half)) << 1) | half;
  // the fix: 2 at the byte of the lowest coordinate that holds max e / min e, added where
  // g is not the D8 decision (D8: s >= 0 moves up; D8+1/2: g moves up), else subtracted
  const float target = d8 ? ep : er;
  int sh = 56;
#pragma unroll
  for (int l = 6; l >= 0; --l) sh = __builtin_fabsf(s[l]) == target ? 8 * l : sh;
  const uint32_t fd = (d8 ? odd1 : odd2) & 2u;
  const uint64_t dl = (uint64_t)fd << sh;
  const uint32_t dlA = (uint32_t)dl, dlB = (uint32_t)(dl >> 32);
  const uint32_t dm = 0u - (uint32_t)d8;
  P.a = pA - dlA + 2u * (dlA & ((gA >> 6) ^ dm));
  P.b = pB - dlB + 2u * (dlB & ((gB >> 6) ^ dm));
  return __builtin_fabsf(gap) >= 1.0e-5f && ep < 0.5f;
}

// The root bound M(P) of e8_root_bound, for bytes in [1, 127]: |P| + 64 = max(P + 64, 64 - P)
// in 16-bit lanes (coordinates l and l + 1 of a word together), the two largest of each lane,
// then of both.
__device__ __forceinline__ int e8_bytes_root_bound(const E8Bytes& P) {
  auto pair = [](uint32_t w, uint32_t sel) {
    const u16x2 v = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(0u, w, sel));
    const u16x2 n = (u16x2){128, 128} - v;
    return __builtin_elementwise_max(v, n);
  };
  const u16x2 a0 = pair(P.a, 0x0C010C00u), a1 = pair(P.a, 0x0C030C02u);
  const u16x2 a2 = pair(P.b, 0x0C010C00u), a3 = pair(P.b, 0x0C030C02u);
  u16x2 m1 = __builtin_elementwise_max(a0, a1), m2 = __builtin_elementwise_min(a0, a1);
  u16x2 mn = m2;
  m2 = __builtin_elementwise_max(m2, __builtin_elementwise_min(m1, a2));
  m1 = __builtin_elementwise_max(m1, a2);
  m2 = __builtin_elementwise_max(m2, __builtin_elementwise_min(m1, a3));
  m1 = __builtin_elementwise_max(m1, a3);
  mn = __builtin_elementwise_min(mn, __builtin_elementwise_min(a2, a3));
  const u16x2 m1s = __builtin_shufflevector(m1, m1, 1, 0);
  const u16x2 m2s = __builtin_shufflevector(m2, m2, 1, 0);
  const u16x2 mns = __builtin_shufflevector(mn, mn, 1, 0);
  const u16x2 top = __builtin_elementwise_max(m1, m1s);
  const u16x2 sec = __builtin_elementwise_max(__builtin_elementwise_min(m1, m1s),
                                              __builtin_elementwise_max(m2, m2s));
  const u16x2 low = __builtin_elementwise_min(mn, mns);
  const int pairs = (int)top.x + (int)sec.x - 128;
  const uint32_t sum = __builtin_amdgcn_sad_u8(
      P.a, 0x40404040u, __builtin_amdgcn_sad_u8(P.b, 0x40404040u, 0u));   // sum |P_l|
  // bit 6 of a byte says P_l >= 0; the count of either sign has the same parity
  const uint32_t odd = 0u - (bcnt_add((P.a ^ P.b) & 0x40404040u, 0u) & 1u);
  const int halves = ((int)sum - (int)(odd & (((uint32_t)low.x - 64u) << 1))) >> 1;
  return pairs > halves ? pairs : halves;
}

// The codes G^-1 P mod q (Alg. 1), packed as nibbles.  c_l = (P_m - P_0) / 2 mod q for six of
// them, on bytes: those differences are roots' products with P, so |P_m - P_0| / 2 < q when
// M(P) < 2q, and one conditional addition of q reduces them.  WIDE (NestQuantM's box,
// |P_0| <= 2q and |P_l| <= q): they are at most 3q / 2, reduced modulo 2q and then q.
// c0 = P_0 and c1 = (5 P_0 - P_1 - P_2 - P_3 + P_4 - P_5 - P_6 - P_7) / 4 by the 24-bit division
// of encode_codes; the biases cancel in c1 (its weights sum to zero).
template <bool WIDE = false>
__device__ __forceinline__ uint32_t encode_e8_bytes(const E8Bytes& P, int q, uint32_t mq) {
  const uint32_t p0 = __builtin_amdgcn_perm(0u, P.a, 0x00000000u);   // P_0 + 64 in every byte
  const uint32_t q1 = (uint32_t)q * 0x01010101u;
  auto reduce = [&](uint32_t p) {
    // (P_m - P_0) / 2 + 64; bit 6 says it is not negative
    const uint32_t v = (((p | 0x80808080u) - p0) >> 1) & 0x7F7F7F7Fu;
    const uint32_t m = v & 0x40404040u, k = m - (m >> 6);            // 0x3F where v >= 64
    if constexpr (!WIDE) return v - (64u * 0x01010101u - q1) - (k & q1);
    const uint32_t w = v - (64u * 0x01010101u - 2u * q1) - (k & (2u * q1));   // in [0, 2q)
    const uint32_t n = (w + (64u * 0x01010101u - q1)) & 0x40404040u;
    return w - ((n - (n >> 6)) & q1);
  };
  const int bias = q << 10;
  auto mod_q = [&](uint32_t u) { return u - umul24_v(umul24_v(u, mq) >> 20, (uint32_t)q); };
  const uint32_t c0 = mod_q((P.a & 0xFFu) + (uint32_t)(bias - 64));
  const int s = dot4_i8(P.a, 0xFFFFFF05u, dot4_i8(P.b, 0xFFFFFF01u, 4 * bias));
  const uint32_t c1 = mod_q((uint32_t)(s >> 2));
  const uint32_t even = (reduce(P.a) & 0xFFFFFF00u) | c0;   // c0 c2 c4 c6
  const uint32_t odd = (reduce(P.b) & 0xFFFFFF00u) | c1;    // c1 c3 c5 c7
  return even | (odd << 4);
}
