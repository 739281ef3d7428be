// The byte form of the encoder's nearest point, root bound and code (nq_e8b.hpp) compiled for
// the host, its AMDGCN instructions replaced by plain C++ written from their definitions in
// the CDNA3 ISA reference.  Test infrastructure; built by tests/test_encoder_host.py.
#include <cmath>
#include <cstdint>

#define __device__
#define __forceinline__ inline __attribute__((always_inline))
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// v_perm_b32: byte i of the result is byte sel_i of {s0, s1} (s1 the low word), 12 zero
static inline uint32_t host_perm(uint32_t s0, uint32_t s1, uint32_t sel) {
  const uint64_t v = ((uint64_t)s0 << 32) | s1;
  uint32_t d = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t k = (sel >> (8 * i)) & 0xFFu;
    d |= (k < 8 ? (uint32_t)(v >> (8 * k)) & 0xFFu : (k == 12 ? 0u : 0xFFu)) << (8 * i);
  }
  return d;
}
static inline uint32_t host_sad_u8(uint32_t a, uint32_t b, uint32_t c) {
  for (int i = 0; i < 4; ++i) {
    const int x = (int)((a >> (8 * i)) & 0xFFu), y = (int)((b >> (8 * i)) & 0xFFu);
    c += (uint32_t)(x > y ? x - y : y - x);
  }
  return c;
}
#define __builtin_amdgcn_perm host_perm
#define __builtin_amdgcn_sad_u8 host_sad_u8

namespace nq {
static inline uint32_t umul24_v(uint32_t a, uint32_t b) {
  return (uint32_t)((uint64_t)(a & 0xFFFFFFu) * (b & 0xFFFFFFu));
}
static inline uint32_t bcnt_add(uint32_t x, uint32_t acc) {
  return acc + (uint32_t)__builtin_popcount(x);
}
static inline float max3_abs(float a, float b, float c) {
  return std::fmax(std::fmax(std::fabs(a), std::fabs(b)), std::fabs(c));
}
static inline float min3_abs(float a, float b, float c) {
  return std::fmin(std::fmin(std::fabs(a), std::fabs(b)), std::fabs(c));
}
static inline int dot4_i8(uint32_t a, uint32_t b, int acc) {
  for (int i = 0; i < 4; ++i) acc += (int)(int8_t)(a >> (8 * i)) * (int)(int8_t)(b >> (8 * i));
  return acc;
}
#include "nq_e8b.hpp"
}  // namespace nq

static nq::E8Bytes pack(const int32_t* p) {
  nq::E8Bytes P{0, 0};
  for (int l = 0; l < 4; ++l) {
    P.a |= (uint32_t)(p[l] + 64) << (8 * l);
    P.b |= (uint32_t)(p[4 + l] + 64) << (8 * l);
  }
  return P;
}

// nearest points of n vectors x, times c; ok[i] = 0 where fp32 cannot decide
extern "C" void nq_e8b_nearest(const float* x, int64_t n, float c, int32_t* p, uint8_t* ok) {
  for (int64_t i = 0; i < n; ++i) {
    float v[8];
    for (int l = 0; l < 8; ++l) v[l] = x[8 * i + l];
    nq::E8Bytes P{0, 0};
    ok[i] = nq::nearest_e8_bytes(v, c, P);
    for (int l = 0; l < 4; ++l) {
      p[8 * i + l] = (int32_t)((P.a >> (8 * l)) & 0xFFu) - 64;
      p[8 * i + 4 + l] = (int32_t)((P.b >> (8 * l)) & 0xFFu) - 64;
    }
  }
}

// root bounds and code words of n points
extern "C" void nq_e8b_code(const int32_t* p, int64_t n, int q, int wide, int32_t* bound,
                            uint32_t* words) {
  const uint32_t mq = ((1u << 20) + (uint32_t)q - 1u) / (uint32_t)q;
  for (int64_t i = 0; i < n; ++i) {
    const nq::E8Bytes P = pack(p + 8 * i);
    bound[i] = nq::e8_bytes_root_bound(P);
    words[i] = wide ? nq::encode_e8_bytes<true>(P, q, mq) : nq::encode_e8_bytes<false>(P, q, mq);
  }
}

// The encoder's first evaluation of n blocks of a row of scale r: the beta it starts at (mx:
// the statistic its thresholds bound, one per block) and the point there; ok[i] = 0 where the
// block is left to the exact path.
extern "C" void nq_e8b_first(const float* x, const float* mx, int64_t n, float r,
                             const double* beta, int k, int q, int decoder, int32_t* t0,
                             int32_t* p, uint8_t* ok) {
  float hi[4];
  const float skip = nq::skip_factor(q, decoder);
  for (int t = 0; t < 3; ++t)
    hi[t] = t < k - 1 ? nq::row_limit(skip, (double)r * beta[t]) : INFINITY;
  hi[3] = nq::row_limit(nq::kBytesFactor, (double)r * beta[k - 1]);
  for (int64_t i = 0; i < n; ++i) {
    t0[i] = mx[i] > hi[0] ? (mx[i] > hi[1] ? (mx[i] > hi[2] ? 3 : 2) : 1) : 0;
    const float c = (float)(1.0 / ((double)r * beta[t0[i]]));
    nq_e8b_nearest(x + 8 * i, 1, c, p + 8 * i, ok + i);
    if (mx[i] > hi[3]) ok[i] = 0;
  }
}
