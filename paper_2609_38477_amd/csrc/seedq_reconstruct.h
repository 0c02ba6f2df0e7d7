// Exact reconstruction of one block from its code (section 3.1 eq. (codec),
// Algorithm 2): regenerate the 8P LFSR states of seed s, form the integer
// products acc_i = sum_j U_int[i][j] q_j (|acc| < 2^29) and scale by
// 2^-(K-1+e) after one rounding to fp32. Shared by the decoders.
#pragma once

#include "seedq_internal.h"

namespace seedq {

// Stores past the caches' replacement order (past = true) or ordinary ones. A call
// stores past them when what it reads and writes exceeds the 256 MiB memory-side
// cache (stores_past_caches): its output could not stay there whole, and ordinary
// stores only push out what the call or the next one reads. Below that the output
// stays for its reader, which pays for memory otherwise. Measured with the caches
// flushed before, past them against ordinary, in us:
//   stream to weights, then a matrix-vector product: 64 MiB of weights 69/61, 172 MiB
//     155/115, 256 MiB 195/194, 896 MiB 538/560; then the inverse permutation: 64 MiB
//     114/84, 128 MiB 282/191, 256 MiB 810/799, 896 MiB 3521/3578;
//   codes to weights, then a product: 64 MiB 64/54, 224 MiB 172/167, 896 MiB 536/544;
//   the call alone is the same either way (stream to weights, 64 MiB 39/41, 224 MiB
//     83/84, 896 MiB 266/269), and faster past the caches only where the same call on
//     the same inputs went before (224 MiB 60/70, 896 MiB 186/266).
constexpr int64_t kMemorySideCache = int64_t(256) << 20;
inline bool stores_past_caches(int64_t bytes_read, int64_t bytes_written) {
  return bytes_read + bytes_written > kMemorySideCache;
}
// (a template argument: with a run-time one the compiler makes one ordinary store of both)
template <bool kPast, typename T>
__device__ __forceinline__ void store_result(T* dst, T v) {
  if constexpr (kPast) __builtin_nontemporal_store(v, dst);
  else *dst = v;
}
template <bool kPast>
__device__ __forceinline__ void store_result(float4* dst, const float4& v) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  store_result<kPast>(reinterpret_cast<f4*>(dst), f4{v.x, v.y, v.z, v.w});
}
template <bool kPast>
__device__ __forceinline__ void store_result(uint2* dst, uint32_t x, uint32_t y) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  store_result<kPast>(reinterpret_cast<u2*>(dst), u2{x, y});
}

// Rung constants for per-lane lookups, kept in LDS: entry r = (K, P, LFSR
// feedback mask, code length l = K + 4 + 4P) of rung r < n, and entry n (n =
// rt.n <= SEEDQ_MAX_RUNGS) stands for every rung byte >= n: an invalid code of
// length 0 (K = SEEDQ_MIN_K, P = 1 keep its arithmetic in range). Threads
// 0..SEEDQ_MAX_RUNGS fill it; the caller synchronises before reading.
constexpr int kRungTable = SEEDQ_MAX_RUNGS + 1;

__device__ __forceinline__ void fill_rung_table(uint4* tab, const RungTable& rt) {
  if (threadIdx.x < kRungTable) {
    const int t = int(threadIdx.x);
    const bool v = t < rt.n;
    const int K = v ? rt.K[t] : SEEDQ_MIN_K;
    const int P = v ? rt.P[t] : 1;
    tab[t] = make_uint4(uint32_t(K), uint32_t(P), lfsr_mask(K), v ? uint32_t(K + 4 + 4 * P) : 0u);
  }
}

__device__ __forceinline__ uint32_t table_index(uint32_t r, uint32_t n) { return r < n ? r : n; }

// acc_i = sum_j (x_{8j+i} - 2^(K-1)) q_j, with q_j = qat(j) in [-8, 7], P >= 1
// and the LFSR feedback mask of K. It is formed as sum_j x q_j - 2^(K-1)
// sum_j q_j: for K <= 23 every state fits a signed 24-bit operand, so each
// product is one full-rate 24-bit multiply-add (|x q| < 2^26, every partial
// sum < 2^29). The first coefficient is peeled so that acc needs no clearing.
template <typename QAt>
__device__ __forceinline__ void block_acc_q(uint32_t s, int K, int P, uint32_t mask, QAt qat,
                                            int32_t (&acc)[kC]) {
  const int32_t half = int32_t(1) << (K - 1);
  uint32_t x = s;
  if (__builtin_expect(K <= 23, 1)) {
    const int32_t q0 = qat(0);
    int32_t qsum = q0;
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      acc[i] = __mul24(int32_t(x), q0);
      x = lfsr_step(x, mask);
    }
    for (int j = 1; j < P; ++j) {
      const int32_t qj = qat(j);
      qsum += qj;
#pragma unroll
      for (int i = 0; i < kC; ++i) {
        acc[i] += __mul24(int32_t(x), qj);
        x = lfsr_step(x, mask);
      }
    }
    const int32_t c = half * qsum;
#pragma unroll
    for (int i = 0; i < kC; ++i) acc[i] -= c;
  } else {
    const int32_t q0 = qat(0);
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      acc[i] = __mul24(int32_t(x) - half, q0);   // x - 2^23 fits 24 bits
      x = lfsr_step(x, mask);
    }
    for (int j = 1; j < P; ++j) {
      const int32_t qj = qat(j);
#pragma unroll
      for (int i = 0; i < kC; ++i) {
        acc[i] += __mul24(int32_t(x) - half, qj);
        x = lfsr_step(x, mask);
      }
    }
  }
}

// a.i16[kHi] * b.i16[0] + c (one instruction, either half of a register).
template <int kHi>
__device__ __forceinline__ int32_t mad_i16(uint32_t a, int32_t b, int32_t c) {
  int32_t d;
  if constexpr (kHi)
    asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  else
    asm("v_mad_i32_i16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// The integers of two blocks of one rung with K <= 16, their registers packed in
// one: a step of both takes four instructions (shift, low bits, their product
// with the feedback mask, and-xor) where each alone takes three, and a state's
// product with a mantissa reads its half in place (6.1 ns a state and SIMD for
// one register, 4.6 packed: shifts and bitwise operations issue in two cycles,
// products and three-operand forms in four). q0, q1: mantissa j in bits 4j..4j+3.
// K < 16 starts the sums at -2^(K-1) sum_j q_j; at K = 16 a state does not fit a
// signed half, so the registers hold x - 2^15 (x with its top bit flipped), whose
// step flips its two top bits more: the feedback term is then 0xC000 or 0xC000 ^
// mask, base + bit * delta either way.
__device__ __forceinline__ void block_acc_pair(uint32_t s0, uint32_t s1, uint32_t q0, uint32_t q1,
                                               int K, int P, uint32_t mask, int32_t (&a0)[kC],
                                               int32_t (&a1)[kC]) {
  typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
  const bool top = K == 16;
  const uint32_t b1 = top ? 0xC000u : 0u, d1 = ((mask ^ b1) - b1) & 0xFFFFu;
  const ushort2v base = __builtin_bit_cast(ushort2v, b1 | b1 << 16);
  const ushort2v delta = __builtin_bit_cast(ushort2v, d1 | d1 << 16);
  uint32_t x = (s0 | s1 << 16) ^ (top ? 0x80008000u : 0u);
  const uint32_t used = (1u << (4 * P)) - 1u;
  const int32_t c = top ? 0 : -(int32_t(1) << (K - 1));
  const int32_t c0 = __mul24(c, __builtin_amdgcn_sdot8(int32_t(q0 & used), 0x11111111, 0, false));
  const int32_t c1 = __mul24(c, __builtin_amdgcn_sdot8(int32_t(q1 & used), 0x11111111, 0, false));
  auto step = [&]() __attribute__((always_inline)) {
    const ushort2v t = __builtin_bit_cast(ushort2v, x & 0x00010001u) * delta + base;
    // 0x6A: (a and b) xor c; the mask drops the bit that crosses into the low half
    x = uint32_t(__builtin_amdgcn_bitop3_b32(int(x >> 1), 0x7FFF7FFF, __builtin_bit_cast(int, t),
                                             0x6A));
  };
  // the first coefficient is peeled so that the sums need no set-up
  {
    const int32_t m0 = __builtin_amdgcn_sbfe(int32_t(q0), 0, 4);
    const int32_t m1 = __builtin_amdgcn_sbfe(int32_t(q1), 0, 4);
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      a0[i] = mad_i16<0>(x, m0, c0);
      a1[i] = mad_i16<1>(x, m1, c1);
      step();
    }
  }
  for (int j = 1; j < P; ++j) {
    const int32_t m0 = __builtin_amdgcn_sbfe(int32_t(q0), 4 * j, 4);
    const int32_t m1 = __builtin_amdgcn_sbfe(int32_t(q1), 4 * j, 4);
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      a0[i] = mad_i16<0>(x, m0, a0[i]);
      a1[i] = mad_i16<1>(x, m1, a1[i]);
      step();
    }
  }
}

// q_j is the signed byte j of qw (bytes 0-3 in qw.x, 4-7 in qw.y).
__device__ __forceinline__ void block_acc(uint32_t s, int K, int P, uint2 qw, int32_t (&acc)[kC]) {
  block_acc_q(s, K, P, lfsr_mask(K), [&](int j) {
    const uint32_t word = (j < 4) ? qw.x : qw.y;
    return int32_t(int8_t(uint8_t(word >> (8 * (j & 3)))));
  }, acc);
}

// w_hat_i = acc_i 2^-(K-1+e), NaN for an invalid code.
__device__ __forceinline__ void block_weights(const int32_t (&acc)[kC], int K, int e, bool ok,
                                              float (&o)[kC]) {
  const int sh = -(K - 1 + e);
#pragma unroll
  for (int i = 0; i < kC; ++i)
    o[i] = ok ? ldexpf(__int2float_rn(acc[i]), sh) : __int_as_float(0x7fc00000);
}

}  // namespace seedq
