// Matrix-core engine of the per-block exhaustive seed search (section 3.1;
// the appendix on cost names this search, one least-squares fit per block and
// seed, as what the encoder spends its time on).
//
// Screen. For block w and seed s the least-squares residual
//     r_LS(s) = ||w||^2 - w^T Pi_s w,        Pi_s = projector onto range(U(s)),
// is a lower bound on every quantised error of that seed. w^T Pi_s w is linear
// in the 36 products z_ij = c_ij w_i w_j (i <= j), so the bounds of 32 seeds x
// 32 blocks are one [32 x 48] x [48 x 32] product: three
// v_mfma_f32_32x32x16_f16 with fp16 operands (2^12-scaled projector entries
// from the basis stack, 2^12-scaled pair products of the block) and fp32
// accumulation. A candidate passes when its bound can be at most the block's
// best error so far. The fp16 rounding of the operands is covered by a margin
// that is computed, not assumed: each seed carries a bound on what the rounding
// of its own projector can take off the form (in one of the padding pairs, so
// the matrix core adds it), each block one for the rounding of its own pair
// products (threshold_base). No candidate that could win is ever skipped, and
// against the worst case of both, sqrt(P) 2^-10 ||w||^2, the margin is about a
// third: where best errors are near it, the survivors fall by as much (4096 x
// 14336 at three rungs 167.5 -> 161.5 ms, (16,4) on 524 288 blocks 3.47 -> 3.32
// ms), and P = 5 can use the form too ((16,5) on 523 776 blocks 5.4 -> 4.3 ms
// against the complement screen below, whose squares take 48 vector operations a
// tile). At P = 6, where the best errors are a tenth of the margin's size, the
// screen computes r_LS directly as the squared projections of w on 2 orthonormal
// vectors orthogonal to range(U(s)) (complement_screen), whose rounding margin is
// relative to r_LS.
//
// Survivors. Each wave queues its passing (seed, block) pairs in LDS and
// evaluates them 64 at a time, one per lane, with the exact fp64 evaluation
// (seedq_exact.h). A lane whose fold passes first stores its 16 bounds as a
// record; records are turned into queued seeds a round at a time against the
// thresholds of that moment. Every block's best is its exact fp64 error (an
// atomic minimum on the bit pattern in LDS) and the smallest seed of that error
// (record_best), so the result is the exhaustive search's, ties to the smallest
// seed, whatever the order in which survivors are evaluated. A pilot pass over
// the first seed tile finds, per lane, the seed with the smallest bound; their
// exact errors start every block's best, so that the walk does not begin with
// an infinite threshold.
//
// Work split. The rung's seed tiles are cut into ranges, its blocks into units
// of one workgroup; a workgroup takes one unit through one range (seed_range),
// starting from the best that other ranges have left in the block's key, and
// offers its own best to the key at its end (merge_best). One more kernel
// emits the codes from the keys (emit_codes_kernel). A workgroup is 4
// independent waves; a wave owns 4 tiles of 32 blocks (128 blocks; 1 or 2 tiles
// where that measured faster, see launch_mfma_p), reusing each A fragment for
// all of them; its B fragments stay in registers for the whole walk.
// Block tiles go to the matrix core in pairs (six products) before the vector
// ALU folds them, with one branch per pair; the fold waits on its own
// products, so it is occupancy (several waves per SIMD) that keeps the matrix
// core busy. At P = 4 with many seeds the fp64 evaluation needs more registers
// than the walk over 128 blocks leaves free, so a second kernel rebuilds the
// block data and reloads the seed-tile fragments after every evaluation batch
// instead of keeping them live across it, and runs at four waves per SIMD.
// (At P >= 5, with many survivors, the evaluations decide from an fp32 copy of
// the pseudo-inverse, whose registers fit beside the walk of two block tiles.)
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "seedq_exact.h"
#include "seedq_internal.h"

namespace seedq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4;
constexpr int kNB = 4;               // 32-block tiles per wave
constexpr int kSlots = kNB * 32;     // blocks per wave
// The rebuilding kernel (P = 4): 16 records waiting after a pair of block
// tiles, rounds of 24 records (at most 384 queued seeds each).
constexpr int kRecFlushR = 16;
constexpr int kRecCapR = kRecFlushR + 64;
constexpr int kRecRound = 24;
constexpr int kRecQueueR = 64 + kRecRound * 16;
constexpr int kBlocksPerWG = kWaves * kSlots;

// Row and column of pair k (i <= j, row-major over the upper triangle) for
// k < 36; -1 for the padding pairs 36..47. A compile-time table, so that the
// unrolled prologue indexes it with constants.
struct PairTable {
  int i[kPairsPadded];
  int j[kPairsPadded];
};
constexpr PairTable make_pair_table() {
  PairTable t{};
  int k = 0;
  for (int i = 0; i < kC; ++i)
    for (int j = i; j < kC; ++j) {
      t.i[k] = i;
      t.j[k] = j;
      ++k;
    }
  for (; k < kPairsPadded; ++k) {
    t.i[k] = -1;
    t.j[k] = -1;
  }
  return t;
}
constexpr PairTable kPairTable = make_pair_table();
static_assert(kPairTable.i[35] == 7 && kPairTable.j[35] == 7, "36 pairs");
static_assert(pair_index(2, 5) == 18 && kPairTable.i[18] == 2 && kPairTable.j[18] == 5,
              "pair numbering agrees with the basis builder");

template <int K0>
__device__ __forceinline__ float pair_value(const float (&ws)[kC]) {
  constexpr int i = kPairTable.i[K0], j = kPairTable.j[K0];
  if constexpr (i < 0) {
    return 0.f;
  } else {
    return (i == j ? 1.f : 2.f) * ws[i] * ws[j] * kOperandScale;
  }
}

// What a block's fp16 operand differs from its pair products, as a symmetric
// matrix D (its off-diagonal entries are half a pair's difference): the squared
// Frobenius norm and the trace of the part that this lane rounds, in operand
// units.
struct Rounding {
  float f2 = 0.f, tr = 0.f;
};

template <int T, int E>
__device__ __forceinline__ _Float16 b_element(const float (&ws)[kC], float ww, int h, Rounding& rd) {
  constexpr int k0 = 16 * T + E, k1 = k0 + 8;
  if constexpr (k0 == kMarginPair) {
    static_assert(kPairTable.i[k1] < 0, "padding in the other half");
    return _Float16(h ? 0.f : ww * kMarginScale);
  } else {
    const float z0 = pair_value<k0>(ws);
    const float z1 = pair_value<k1>(ws);
    const float z = h ? z1 : z0;
    const _Float16 v = _Float16(z);
    const float d = float(v) - z;
    constexpr bool g0 = kPairTable.i[k0] == kPairTable.j[k0], g1 = kPairTable.i[k1] == kPairTable.j[k1];
    const bool g = h ? g1 : g0;
    rd.f2 = fmaf(d * d, g ? 1.f : 0.5f, rd.f2);
    if constexpr (g0 || g1) rd.tr += g ? d : 0.f;
    return v;
  }
}

template <int T>
__device__ __forceinline__ half8 b_fragment(const float (&ws)[kC], float ww, int h, Rounding& rd) {
  half8 v;
  v[0] = b_element<T, 0>(ws, ww, h, rd);
  v[1] = b_element<T, 1>(ws, ww, h, rd);
  v[2] = b_element<T, 2>(ws, ww, h, rd);
  v[3] = b_element<T, 3>(ws, ww, h, rd);
  v[4] = b_element<T, 4>(ws, ww, h, rd);
  v[5] = b_element<T, 5>(ws, ww, h, rd);
  v[6] = b_element<T, 6>(ws, ww, h, rd);
  v[7] = b_element<T, 7>(ws, ww, h, rd);
  return v;
}

// ||w||^2 less the block's share of the screen's margin, in accumulator units:
// what a seed's form must reach with the block's best error subtracted. The
// rounding D of the block's operand changes the form of a projector Pi of rank
// r <= P by <Pi, D> = (r/8) tr D + <Pi - (r/8) I, D>, at least
// min(0, P/8 tr D) - c ||D||_F with c = max over r <= P of sqrt(r - r^2/8) (the
// Frobenius norm of Pi - (r/8) I). (1 - 2^-15) covers the rest: the fp32 sum of
// the 48 products, the fp32 roundings of ww, of the pair products (2^-24
// each), of the threshold itself, and the product of both operands' roundings
// (2^-20 ||w||^2). Both halves of the wave hold half of the block's pairs.
template <int P>
__device__ __forceinline__ float threshold_base(float ww, Rounding rd) {
  constexpr float c = P == 1 ? 0.9355f : P == 2 ? 1.2248f : P == 3 ? 1.3694f : 1.4143f;
  rd.f2 += __shfl_xor(rd.f2, 32, 64);
  rd.tr += __shfl_xor(rd.tr, 32, 64);
  const float m = fmaf(c * (1.f + 0x1p-10f), sqrtf(rd.f2), fmaxf(0.f, -float(P) / 8.f * rd.tr));
  return ww * (1.f - 0x1p-15f) * (kOperandScale * kOperandScale) - m * kOperandScale;
}

#define SEEDQ_INLINE __device__ __attribute__((always_inline)) inline

// The seed ranges of a rung, decided here from the rung's count of blocks, which
// the host of a multi-rung call does not know: every unit of blocks_per_wg blocks
// goes through nranges ranges of seed tiles, one workgroup each, range by range,
// so that the resident workgroups of a large matrix walk one range at about the
// same time and a later range starts from the earlier ones' best.
struct RangeRule {
  int32_t rmin;             // at least so many ranges
  int32_t rlong, target;    // up to rlong of them for `target` workgroups
  int32_t rshort, fill;     // up to rshort of them for `fill` workgroups
  int32_t first, span;  // ranges of this launch
};
struct SeedRange {
  int range, nranges;
  int64_t unit;
};
__host__ __device__ inline int range_count(const RangeRule& rule, uint32_t units) {
  if (units == 0u) return 1;
  const int t = int(uint32_t(rule.target) / units), f = int(uint32_t(rule.fill) / units);
  const int a = t < rule.rlong ? t : rule.rlong, b = f < rule.rshort ? f : rule.rshort;
  const int nr = a > b ? a : b;
  return nr > rule.rmin ? nr : rule.rmin;
}
SEEDQ_INLINE SeedRange seed_range(const RangeRule& rule, int64_t count, int blocks_per_wg) {
  const uint32_t units = uint32_t((count + blocks_per_wg - 1) / blocks_per_wg);
  if (units == 0u) return {1, 1, 0};
  // wave-uniform (the divisions are done in vector registers)
  const int nr = __builtin_amdgcn_readfirstlane(range_count(rule, units));
  const uint32_t r = uint32_t(__builtin_amdgcn_readfirstlane(int(blockIdx.x / units)));
  if (r >= uint32_t(rule.span)) return {nr, nr, 0};
  return {int(r) + rule.first, nr, int64_t(blockIdx.x - r * units)};
}

// First seed tile of range r of nr (wave-uniform; ntiles <= 2^19, r <= nr <= 2^16).
SEEDQ_INLINE int range_tile(int r, int64_t ntiles, int nr) {
  return __builtin_amdgcn_readfirstlane(int(uint64_t(r) * uint64_t(ntiles) / uint32_t(nr)));
}

SEEDQ_INLINE void load_block(const float* __restrict__ W, int64_t b, bool ok, float (&w)[kC]) {
  float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
  if (ok) {
    const float4* src = reinterpret_cast<const float4*>(W + b * kC);
    lo = src[0];
    hi = src[1];
  }
  w[0] = lo.x; w[1] = lo.y; w[2] = lo.z; w[3] = lo.w;
  w[4] = hi.x; w[5] = hi.y; w[6] = hi.z; w[7] = hi.w;
}

// Largest of the 16 bounds of a lane. The bounds are finite (products of
// finite fp16 values), so the NaN-propagating maximum equals the IEEE maxNum
// here; it needs no operand canonicalisation and folds as v_maximum3_f32. The
// compiler inserts the wait states between the matrix-core write and the reads.
SEEDQ_INLINE float fold_max(const floatx16& acc) {
  float m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(acc[0], acc[1]), acc[2]);
#pragma unroll
  for (int j = 3; j < 15; j += 2)
    m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, acc[j]), acc[j + 1]);
  return __builtin_elementwise_maximum(m, acc[15]);
}

// Wave-wide vote (a bit per lane whose p is set).
SEEDQ_INLINE uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

SEEDQ_INLINE floatx16 bounds(const half8& a0, const half8& a1, const half8& a2, const half8 (&b)[3]) {
  floatx16 acc = {};
  acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b[2], acc, 0, 0, 0);
  return acc;
}

// Complement screen (P >= kComplementMinP = 6): the projections d_c = 2^4 n_c^T w
// of a block on the M complement vectors of 32 seeds are M products with K =
// 16 (the hi and lo parts of 2^4 n_c against the block's fp16 weights, given
// twice), and -sum_c d_c^2 is returned so that the max-fold, the records and
// the pilot treat it like the quadratic form's bound: larger passes.
template <int M>
SEEDQ_INLINE floatx16 complement_screen(const half8 (&a)[M], const half8& b) {
  floatx16 d[M];
#pragma unroll
  for (int c = 0; c < M; ++c) d[c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[c], b, floatx16{}, 0, 0, 0);
  floatx16 v;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    float r = -(d[0][j] * d[0][j]);
#pragma unroll
    for (int c = 1; c < M; ++c) r = fmaf(-d[c][j], d[c][j], r);
    v[j] = r;
  }
  return v;
}

// Seed of accumulator j of a lane in half h of the wave, for tile seedbase.
SEEDQ_INLINE uint32_t seed_of(uint32_t seedbase, int j, int h) {
  return seedbase + 8u * uint32_t(j / 4) + 4u * uint32_t(h) + uint32_t(j % 4);
}

// Per-block best of one wave's walk, in LDS: the exact fp64 error of the best
// code so far as its bit pattern (errors are >= 0, so the bits order like the
// values) and the smallest seed among the codes of exactly that error. The
// slots belong to the wave, so one evaluation batch (a candidate per lane,
// `mine`) updates both in four steps: every lane lowers the error; if any lane
// tied or improved, every lane reads the minimum the batch left; a lane that
// holds that minimum while its slot held a larger one before resets the seed;
// then every lane that holds the minimum lowers the seed to its own. LDS
// operations of one wave take effect in program order; the fence waits for the
// reset before the minimum. Ties in the exact error go to the smallest seed,
// and the result does not depend on the order in which candidates are
// evaluated.
SEEDQ_INLINE void record_best(unsigned long long* best, uint32_t* sbest, int slot, double err,
                              uint32_t seed, bool mine) {
  const unsigned long long eb = mine ? (unsigned long long)__double_as_longlong(err) : 0ull;
  unsigned long long old = 0ull;
  if (mine) old = atomicMin(&best[slot], eb);
  const bool cand = mine && eb <= old;
  if (__builtin_amdgcn_ballot_w64(cand) == 0ull) return;
  __threadfence_block();
  const unsigned long long now = cand ? best[slot] : ~0ull;
  const bool holds = cand && eb == now;
  const bool reset = holds && old != now;
  if (__builtin_amdgcn_ballot_w64(reset) != 0ull) {
    if (reset) atomicExch(&sbest[slot], seed);
    __threadfence_block();
  }
  if (holds) atomicMin(&sbest[slot], seed);
}

// Per-block best over all seed ranges: one 64-bit key per block in the caller's
// mantissa output, the exact error's bit pattern cut to its upper 40 bits (sign,
// exponent and 28 mantissa bits) above the 24-bit seed; ~0 before the first.
// The order of two keys is that of (exact error, seed); where their upper 40
// bits agree, the exact error of the seed already there is computed again
// (merge_best), so the cut loses nothing. Waves of different XCDs meet here,
// hence the agent scope of every access.
constexpr unsigned long long kKeySeed = 0xFFFFFFull;
constexpr uint32_t kNoSeed = ~0u;

SEEDQ_INLINE unsigned long long load_key(unsigned long long* keys, int64_t b) {
  return __hip_atomic_load(&keys[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// An upper bound on the error behind a key, as its bit pattern (~0 stays ~0).
SEEDQ_INLINE unsigned long long key_bound(unsigned long long key) { return key | kKeySeed; }

// Offers the code (error bits eb, seed s) of block b to its key, one block per
// lane where `mine`; exact(seed) is the exact error of a seed for that block.
// Every turn of the loop either settles a lane or follows another wave's
// successful exchange on its key, so it ends.
template <typename Exact>
SEEDQ_INLINE void merge_best(unsigned long long* keys, int64_t b, unsigned long long eb, uint32_t s,
                             bool mine, Exact&& exact) {
  const unsigned long long key = (eb & ~kKeySeed) | s;
  unsigned long long cur = mine ? load_key(keys, b) : 0ull;
  bool open = mine;
  while (ballot(open) != 0ull) {
    const bool tie = open && (cur >> 24) == (key >> 24);
    open = open && (key >> 24) <= (cur >> 24);
    if (ballot(tie) != 0ull) {
      if (tie) {
        const uint32_t s2 = uint32_t(cur & kKeySeed);
        const unsigned long long e2 = (unsigned long long)__double_as_longlong(exact(s2));
        open = eb < e2 || (eb == e2 && s < s2);
      }
    }
    if (open)
      open = !__hip_atomic_compare_exchange_strong(&keys[b], &cur, key, __ATOMIC_RELAXED,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Writes the code of block b: seed's, evaluated once more, or, where no seed was ever
// a candidate (kNoSeed: the weights are all zero), the smallest seed with e = 15,
// q = 0 and error 0. q_out holds a block's mantissas, q_0 first.
template <int P>
SEEDQ_INLINE void emit_code(int64_t b, uint32_t seed, const float (&w)[kC], int K, uint32_t mask,
                            const uint32_t* __restrict__ ub, const float* __restrict__ pinv32,
                            const double* __restrict__ pinv64, uint32_t* __restrict__ seed_out,
                            uint8_t* __restrict__ exp_out, unsigned long long* __restrict__ q_out,
                            float* __restrict__ err_out) {
  int qe = 15, q[P] = {};
  double err = 0.0;
  if (seed != kNoSeed) {
    const double* A = pinv64 + int64_t(seed - 1) * (P * kC);
    const uint32_t* Ub = ub + int64_t(seed - 1) * basis_words(K, P);
    if constexpr (many_survivors(P))
      err = exact_eval_f32<P>(w, pinv32 + int64_t(seed - 1) * (P * kC), A, Ub, seed, K, mask, qe, q);
    else
      err = exact_eval<P, false>(w, A, Ub, seed, K, mask, qe, q);
  }
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t byte = uint32_t(uint8_t(int8_t(q[p])));
    if (p < 4) lo |= byte << (8 * p);
    else hi |= byte << (8 * (p - 4));
  }
  seed_out[b] = seed != kNoSeed ? seed : 1u;
  exp_out[b] = uint8_t(qe);
  q_out[b] = uint64_t(lo) | uint64_t(hi) << 32;
  if (err_out) err_out[b] = float(err);
}

// Number of lanes below this one whose bit is set in mask.
SEEDQ_INLINE int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u));
}

// This lane's index, recomputed where it is used (volatile, so that it is not
// hoisted and kept live through the walk, where registers are short).
SEEDQ_INLINE uint32_t lane_now() {
  uint32_t l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// Queue entries: seed << 8 | slot (slot < 128). Seed 0 = no-op.
static_assert(kSlots <= 128, "slot must fit 7 bits");

// Walk survivors are first kept as records: a lane whose fold
// passes stores its 16 bounds with the seed tile, its half and the block slot
// (one row and one meta word in LDS; meta = tile << 8 | half << 7 | slot).
// Records become candidates 64 at a time, each compared with its block's
// threshold of that moment, so the per-seed ballots run once per 64 records
// instead of once per passing block tile, and records whose block has
// meanwhile found a better code drop out before the exact evaluation.
// At P >= 5, where tens to hundreds of seeds per block survive the screen, the
// records wait until they fill a round (kRecRoundMin; the rest wait for the next
// call) and a round's passing bounds are compacted by a prefix sum over the
// lanes instead of one ballot and branch per seed row (measured on 2.1 M blocks
// with the complement screen: (16,6) 9-10 % and (13..16,5) 6-10 % faster than
// per-row ballots over rounds of 32-64).
template <int P>
constexpr int kRecFlush = complement_dims(P) > 0 ? 64 : 32;   // records waiting after a pair
template <int P>
constexpr int kRecCap = kRecFlush<P> + 64;   // one block tile adds at most 64
template <int P>
constexpr int kRecRoundMin = complement_dims(P) > 0 ? 64 : many_survivors(P) ? 32 : 1;
// Records per round: 64 lanes' worth, or fewer where fp32 records, and at P = 5
// the blocks' weights, leave the queue less LDS (three workgroups per CU need
// their 13 KB per wave).
template <int P>
constexpr int kRecTake = complement_dims(P) > 0 ? 64 : many_survivors(P) ? 48 : 56;
template <int P>
constexpr int kQCapRec = 64 + kRecTake<P> * 16;   // < 64 waiting + one round of records
// With the complement screen (P = 6) records hold their bounds as fp16 (16 x 2
// bytes: two float4 of storage instead of four). The values
// -sum d^2 lie in fp16's range (sum d^2 <= 2^8 ||w||^2 < 2^13: the complement
// operand carries 2^4 and the block's power-of-two scaling leaves every |w_i|
// below 2) and are rounded toward zero, i.e. up, so that a stored bound is
// never below the computed one.
__host__ __device__ constexpr bool half_records(int P) { return complement_dims(P) > 0; }
template <int P>
constexpr int kRecVecs = half_records(P) ? 2 : 4;
typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));

// kOne: a walk known to be of one range, which emits its codes itself; otherwise the keys
// hold the best and emit_codes_kernel follows. (As a run-time choice its code made the
// walks of several ranges slower: (12,3) on 8192 blocks 32.5 -> 34.0 us.)
template <int P, int NT, bool kOne>
__global__ void __launch_bounds__(kWaves * 64)
__attribute__((amdgpu_waves_per_eu(3)))
search_mfma_kernel(const float* __restrict__ W, int64_t nblocks, const int32_t* __restrict__ list,
                   const int32_t* __restrict__ off, int rung, int K, uint32_t mask,
                   const uint32_t* __restrict__ ub, const float* __restrict__ pinv32,
                   const double* __restrict__ pinv64, const half8* __restrict__ pi16,
                   int64_t ntiles, RangeRule rule,
                   unsigned long long* __restrict__ keys, uint32_t* __restrict__ seed_out,
                   uint8_t* __restrict__ exp_out, float* __restrict__ err_out) {
  constexpr int kS = NT * 32;   // blocks per wave
  __shared__ unsigned long long best_all[kWaves][kS];
  __shared__ uint32_t sbest_all[kWaves][kS];
  __shared__ int32_t blk_all[kWaves][kS];
  __shared__ float thr_base_all[kWaves][kS];   // threshold_base, in accumulator units
  // power-of-two scaling of the block: ilogb of its largest |w_i|, down to -149
  // for fp32 subnormals, so 16 bits
  __shared__ int16_t ex_all[kWaves][kS];
  // 16 bounds per record: fp32, or fp16 at P = 6 (see half_records)
  __shared__ float4 rec_all[kWaves][kRecCap<P>][kRecVecs<P>];
  __shared__ uint32_t meta_all[kWaves][kRecCap<P>];
  __shared__ uint32_t queue_all[kWaves][kQCapRec<P>];
  // the weights of the blocks, where evaluations are many: a gather of 32 bytes
  // a candidate less (rungs of P = 6 2-10 % faster, P = 5 1 %)
  __shared__ float4 w_all[kWaves][many_survivors(P) ? kS : 1][2];

  const int lane = threadIdx.x & 63;
  // wave-uniform, so that the per-wave LDS addresses are scalar
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int n = lane & 31;   // block column of the MFMA tile
  const int h = lane >> 5;   // which half of the rows / reduction this lane holds
  unsigned long long* best = best_all[wave];
  int32_t* blk = blk_all[wave];
  float* slot_thr = thr_base_all[wave];
  int16_t* slot_ex = ex_all[wave];
  float4 (*rec)[kRecVecs<P>] = rec_all[wave];
  uint32_t* meta = meta_all[wave];
  uint32_t* queue = queue_all[wave];
  uint32_t* sbest = sbest_all[wave];

  int64_t begin = 0, count = nblocks;
  if (list) {
    begin = off[rung];
    count = int64_t(off[rung + 1]) - begin;
  }
  const SeedRange rg = seed_range(rule, count, kWaves * kS);
  const int64_t wave_base = (rg.unit * kWaves + wave) * kS;
  if (rg.range >= rg.nranges || wave_base >= count) return;  // wave-uniform; waves never synchronise
  const uint32_t nseeds = uint32_t((int64_t(1) << K) - 1);
  // quadratic form: 3 A and 3 B fragments per tile; complement screen: M A
  // fragments (one per complement vector) and one B fragment (the weights)
  constexpr int M = complement_dims(P);
  constexpr int NA = M > 0 ? M : 3;
  constexpr int NB = M > 0 ? 1 : 3;
  constexpr int64_t kTileFrags = NA * 64;   // half8 per seed tile of A fragments
  auto screen = [&](const half8 (&a)[NA], const half8 (&b)[NB]) __attribute__((always_inline)) {
    if constexpr (M > 0) return complement_screen<M>(a, b[0]);
    else return bounds(a[0], a[1], a[2], b);
  };

  // ---------------------------------------------------------------- prologue
  half8 bop[NT][NB];
  float thr[NT];
  bool active[NT], valid[NT];
  bool fresh = false;   // a block of this lane has no error yet
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int64_t idx = wave_base + nt * 32 + n;
    valid[nt] = idx < count;
    const int64_t b = valid[nt] ? (list ? int64_t(list[begin + idx]) : idx) : 0;
    float w[kC];
    load_block(W, b, valid[nt], w);
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < kC; ++i) amax = fmaxf(amax, fabsf(w[i]));
    const int ex = valid[nt] && amax > 0.f ? ilogbf(amax) : 0;
    float ws[kC], ww = 0.f;
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      ws[i] = ldexpf(w[i], -ex);
      ww = fmaf(ws[i], ws[i], ww);
    }
    // a block with a weight that is not finite has no bound that passes, only the
    // pilot's errors: the first range's, so that its code does not depend on which
    // range runs first
    active[nt] = valid[nt] && amax > 0.f && (ww < INFINITY || rg.range == 0);
    thr[nt] = active[nt] ? -INFINITY : INFINITY;
    float base = 0.f;
    if constexpr (M > 0) {
#pragma unroll
      for (int e = 0; e < kC; ++e) bop[nt][0][e] = _Float16(ws[e]);
    } else {
      Rounding rd;
      bop[nt][0] = b_fragment<0>(ws, ww, h, rd);
      bop[nt][1] = b_fragment<1>(ws, ww, h, rd);
      bop[nt][2] = b_fragment<2>(ws, ww, h, rd);
      base = threshold_base<P>(ww, rd);
    }
    // a range starts from the best that the others have left so far
    const unsigned long long bound =
        !kOne && valid[nt] ? key_bound(load_key(keys, b)) : ~0ull;
    fresh |= active[nt] && bound == ~0ull;
    if (h == 0) {
      best[nt * 32 + n] = bound;
      sbest[nt * 32 + n] = kNoSeed;
      blk[nt * 32 + n] = int32_t(b);
      if constexpr (many_survivors(P)) {
        w_all[wave][nt * 32 + n][0] = make_float4(w[0], w[1], w[2], w[3]);
        w_all[wave][nt * 32 + n][1] = make_float4(w[4], w[5], w[6], w[7]);
      }
      if constexpr (M > 0) {
        // sqrt(M) times the bound on the error of each computed projection,
        // in accumulator units (kComplementScale): fp16 rounding of the
        // weights (2^-11 relative each, Cauchy-Schwarz with |n_c| = 1) plus
        // that of the hi/lo complement vector (2^-22 relative; below fp16's
        // normal range 2^-25 absolute in the 2^4-scaled entries, 2^-29 of
        // n_c) and the fp32 accumulation of 16 exact products,
        // all under 2^-11 (1 + 2^-7) |w| + 2^-20; |w| <= sqrt(ww) (1 + 2^-20)
        const float norm = sqrtf(ww) * (1.0f + 0x1p-20f);
        slot_thr[nt * 32 + n] = sqrtf(float(M)) * (1.0f + 0x1p-20f) * kComplementScale *
                                (0x1p-11f * (1.0f + 0x1p-7f) * norm + 0x1p-20f);
      } else {
        // thresholds live in accumulator units (both operands carry 2^12)
        slot_thr[nt * 32 + n] = base;
      }
      slot_ex[nt * 32 + n] = int16_t(ex);
    }
  }
  __threadfence_block();

  // Screening threshold of slot s from its best: a bound passes when it can
  // reach the block's best exact error so far (-inf before the first one).
  auto slot_threshold = [&](int s) __attribute__((always_inline)) {
    const unsigned long long key = best[s];
    if (key == ~0ull) return -INFINITY;
    if constexpr (M > 0) {
      // a seed whose residual r_LS(w) is at most the best error b has computed
      // projections of norm <= 2^4 sqrt(b 2^-2ex) + slot_thr (triangle
      // inequality over the M of them), so their fp32 sum of squares (within
      // 2^-20 of its value) is at most T = (2^4 sqrt(b 2^-2ex) + slot_thr)^2
      // (1 + 2^-19). Evaluated in fp32 and rounded up by the factors below:
      // the nearest-rounded conversion (2^-24 relative, 2^-150 absolute below
      // the normal range), sqrtf (1 ulp) and each later rounding (2^-24).
      const float bs = float(ldexp(__longlong_as_double((long long)key), -2 * int(slot_ex[s])));
      const float rb = fmaf(sqrtf(bs), 1.0f + 0x1p-21f, 0x1p-62f);
      const float t = fmaf(rb, kComplementScale, slot_thr[s]) * (1.0f + 0x1p-22f);
      return -(t * t * (1.0f + 0x1p-18f));
    } else {
      return slot_thr[s] - __double2float_ru(ldexp(__longlong_as_double((long long)key),
                                                   24 - 2 * int(slot_ex[s])));
    }
  };
  auto refresh = [&]() __attribute__((always_inline)) {
    __threadfence_block();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      if (active[nt]) thr[nt] = slot_threshold(nt * 32 + n);
  };

  // Exact error of a seed for the block of a slot.
  auto exact_error = [&](int slot, uint32_t seed) __attribute__((always_inline)) {
    float w[kC];
    if constexpr (many_survivors(P)) {
      const float4 lo = w_all[wave][slot][0], hi = w_all[wave][slot][1];
      w[0] = lo.x; w[1] = lo.y; w[2] = lo.z; w[3] = lo.w;
      w[4] = hi.x; w[5] = hi.y; w[6] = hi.z; w[7] = hi.w;
    } else {
      load_block(W, blk[slot], true, w);
    }
    int qe, q[P];
    if constexpr (many_survivors(P))
      return exact_eval_f32<P>(w, pinv32 + int64_t(seed - 1) * (P * kC),
                               pinv64 + int64_t(seed - 1) * (P * kC),
                               ub + int64_t(seed - 1) * basis_words(K, P), seed, K, mask, qe, q);
    else
      return exact_eval<P, false>(w, pinv64 + int64_t(seed - 1) * (P * kC),
                                  ub + int64_t(seed - 1) * basis_words(K, P), seed, K, mask, qe,
                                  q);
  };
  int qcount = 0;  // wave-uniform
  // Evaluate the top min(64, qcount) candidates, one per lane, until fewer
  // than min_batch remain.
  auto evaluate = [&](int min_batch) __attribute__((always_inline)) {
    __threadfence_block();
    while (qcount >= min_batch && qcount > 0) {
      const int e = qcount < 64 ? qcount : 64;
      const int base = qcount - e;
      bool mine = false;
      uint32_t seed = 0u;
      int slot = 0;
      double err = 0.0;
      if (lane < e) {
        const uint32_t ent = queue[base + lane];
        seed = ent >> 8;
        slot = int(ent & 0x7Fu);
        if (seed != 0u) {
          err = exact_error(slot, seed);
          mine = true;
        }
      }
      record_best(best, sbest, slot, err, seed, mine);
      qcount = base;
    }
    __threadfence_block();
  };

  int nrec = 0;  // wave-uniform
  // Records -> candidates: lane l takes record base + l of the top kRecTake and
  // compares its 16 bounds with the block's current threshold; the passing
  // seeds are queued. Rounds run while at least min_round records wait. Full
  // batches are evaluated after each round of records; the walk's thresholds
  // are refreshed at the end.
  auto process = [&](int min_round) __attribute__((always_inline)) {
    __threadfence_block();
    while (nrec >= min_round && nrec > 0) {
      const int e = nrec < kRecTake<P> ? nrec : kRecTake<P>;
      const int base = nrec - e;
      const bool live = lane < e;
      uint32_t m = 0u;
      float t = INFINITY;
      float bnd[16];
      if constexpr (half_records(P)) {
        float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0;
        if (live) {
          m = meta[base + lane];
          t = slot_threshold(int(m & 0x7Fu));
          r0 = rec[base + lane][0];
          r1 = rec[base + lane][1];
        }
        const float r[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const fp16x2 v = __builtin_bit_cast(fp16x2, r[k]);
          bnd[2 * k] = float(v[0]);
          bnd[2 * k + 1] = float(v[1]);
        }
      } else {
        float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0, r3 = r0;
        if (live) {
          m = meta[base + lane];
          t = slot_threshold(int(m & 0x7Fu));
          r0 = rec[base + lane][0];
          r1 = rec[base + lane][1];
          r2 = rec[base + lane][2];
          r3 = rec[base + lane][3];
        }
        const float r[16] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w,
                             r2.x, r2.y, r2.z, r2.w, r3.x, r3.y, r3.z, r3.w};
#pragma unroll
        for (int k = 0; k < 16; ++k) bnd[k] = r[k];
      }
      const uint32_t seedbase = (m >> 8) * 32u + 1u;
      const int hh = int((m >> 7) & 1u);
      const uint32_t slot = m & 0x7Fu;
      if constexpr (many_survivors(P)) {
        // the lane's passing bounds as a mask (t = +inf on lanes without a
        // record), the exclusive prefix sum of their counts over the wave (by
        // the counts' five bit planes), then one queued seed per lane and step
        uint32_t pm = 0u;
#pragma unroll
        for (int j = 0; j < 16; ++j) pm |= (bnd[j] >= t ? 1u : 0u) << j;
        const uint32_t cnt = uint32_t(__builtin_popcount(pm));
        uint32_t off = uint32_t(qcount);
        int total = 0;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          const uint64_t mk = ballot(((cnt >> k) & 1u) != 0u);
          off += uint32_t(lanes_below(mk)) << k;
          total += __popcll(mk) << k;
        }
        while (ballot(pm != 0u) != 0ull) {
          if (pm != 0u) {
            // seed_of for the lowest set row j
            const uint32_t j = uint32_t(__builtin_ctz(pm));
            const uint32_t seed = seedbase + 8u * (j >> 2) + 4u * uint32_t(hh) + (j & 3u);
            queue[off] = ((seed <= nseeds ? seed : 0u) << 8) | slot;
            ++off;
            pm &= pm - 1u;
          }
        }
        qcount += total;
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const bool pass = bnd[j] >= t;   // t = +inf on lanes without a record
          const uint64_t mk = ballot(pass);
          if (mk != 0ull) {
            if (pass) {
              const uint32_t seed = seed_of(seedbase, j, hh);
              queue[qcount + lanes_below(mk)] = ((seed <= nseeds ? seed : 0u) << 8) | slot;
            }
            qcount += __popcll(mk);
          }
        }
      }
      nrec = base;
      if (qcount >= 64) evaluate(64);
    }
    refresh();
  };

  const half8* A = pi16;

  // The walk of this range: seed tiles [T0, T1), at least 8 of them.
  const int64_t T0 = range_tile(rg.range, ntiles, rg.nranges);
  const int64_t T1 = range_tile(rg.range + 1, ntiles, rg.nranges);

  // ---------------------------------------------------------------- pilot
  // Over the range's first tile each lane tracks its seed of smallest bound;
  // their exact errors start the best of every block that has none yet. (Longer
  // pilots cost more matrix time than the survivors they save.)
  if (ballot(fresh) == 0ull) {
    refresh();
  } else {
    half8 a[NA];
#pragma unroll
    for (int t = 0; t < NA; ++t) a[t] = A[T0 * kTileFrags + 64 * t + lane];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const floatx16 acc = screen(a, bop[nt]);
      const float mx = fold_max(acc);
      int jb = 15;
#pragma unroll
      for (int j = 14; j >= 0; --j)
        if (acc[j] == mx) jb = j;
      // every seed of the tile exists: only the last tile of the rung is short,
      // and no range starts there (K >= 8)
      const uint32_t sd = seed_of(uint32_t(T0) * 32u + 1u, jb, h);
      const bool put = active[nt];
      const uint64_t mk = ballot(put);
      if (put) queue[qcount + lanes_below(mk)] = (sd << 8) | uint32_t(nt * 32 + n);
      qcount += __popcll(mk);
      if (qcount >= 64) evaluate(64);
    }
    evaluate(1);
    refresh();
  }

  // ---------------------------------------------------------------- seed walk
  // Lanes of block tile nt whose fold passed store their 16 bounds as records.
  // mk = ballot(pass), taken once by the caller.
  auto record = [&](int nt, const floatx16& acc, bool pass, uint64_t mk, uint32_t T)
                    __attribute__((always_inline)) {
    if (mk == 0ull) return;
    if (pass) {
      const int r = nrec + lanes_below(mk);
      if constexpr (half_records(P)) {
        float pk[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          pk[k] = __builtin_bit_cast(float, __builtin_amdgcn_cvt_pkrtz(acc[2 * k], acc[2 * k + 1]));
        rec[r][0] = make_float4(pk[0], pk[1], pk[2], pk[3]);
        rec[r][1] = make_float4(pk[4], pk[5], pk[6], pk[7]);
      } else {
        rec[r][0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        rec[r][1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
        rec[r][2] = make_float4(acc[8], acc[9], acc[10], acc[11]);
        rec[r][3] = make_float4(acc[12], acc[13], acc[14], acc[15]);
      }
      meta[r] = (T << 8) | (uint32_t(h) << 7) | uint32_t(nt * 32 + n);
    }
    nrec += __popcll(mk);
  };
  static_assert(NT == 1 || NT == 2 || NT == 4, "one block tile or pairs of them");

  // One seed tile against the block tiles: two block tiles at a time, six
  // products to the matrix core, then the folds, one branch per pair. Before
  // each block tile's records at most kRecCap - 64 are waiting.
  auto tile = [&](const half8 (&a)[NA], int64_t T) __attribute__((always_inline)) {
    const uint32_t t32 = uint32_t(T);
    if constexpr (NT == 1) {
      const floatx16 acc = screen(a, bop[0]);
      const bool p = fold_max(acc) >= thr[0];
      const uint64_t m = ballot(p);
      if (m != 0ull) {
        record(0, acc, p, m, t32);
        if (nrec >= kRecFlush<P>) process(kRecRoundMin<P>);
      }
      return;
    }
#pragma unroll
    for (int pr = 0; pr < NT / 2; ++pr) {
      // raised issue priority while this wave feeds the matrix core, so that
      // its products start ahead of the other waves' folds (measured +0.5 to
      // +1.1 % at (16,3); the rebuilding kernel measured slower with it)
      __builtin_amdgcn_s_setprio(1);
      const floatx16 acc0 = screen(a, bop[2 * pr]);
      const floatx16 acc1 = screen(a, bop[2 * pr + 1]);
      __builtin_amdgcn_s_setprio(0);
      const bool p0 = fold_max(acc0) >= thr[2 * pr];
      const bool p1 = fold_max(acc1) >= thr[2 * pr + 1];
      const uint64_t m0 = ballot(p0), m1 = ballot(p1);
      if ((m0 | m1) != 0ull) {
        record(2 * pr, acc0, p0, m0, t32);
        if (nrec > kRecCap<P> - 64) process(kRecRoundMin<P>);
        record(2 * pr + 1, acc1, p1, m1, t32);
        if (nrec >= kRecFlush<P>) process(kRecRoundMin<P>);
      }
    }
  };
  // Two register sets of seed-tile fragments in turn: the set of one tile is
  // loaded while the other tile is screened. The loads are unconditional (the
  // index is clamped to the last tile) so that the wait before each tile
  // covers only that tile's own loads.
  const int64_t last = T1 - 1;
  half8 x[NA], y[NA];
#pragma unroll
  for (int t = 0; t < NA; ++t) x[t] = A[T0 * kTileFrags + 64 * t + lane];
  for (int64_t T = T0; T < T1; T += 2) {
    {
      const half8* An = A + (T + 1 < last ? T + 1 : last) * kTileFrags;
#pragma unroll
      for (int t = 0; t < NA; ++t) y[t] = An[64 * t + lane];
    }
    tile(x, T);
    {
      const half8* An = A + (T + 2 < last ? T + 2 : last) * kTileFrags;
#pragma unroll
      for (int t = 0; t < NA; ++t) x[t] = An[64 * t + lane];
    }
    if (T + 1 < T1) tile(y, T + 1);
  }
  process(1);
  evaluate(1);

  // ---------------------------------------------------------------- results
  if constexpr (kOne) {
    for (int slot = lane; slot < kS && wave_base + slot < count; slot += 64) {
      float w[kC];
      load_block(W, blk[slot], true, w);
      emit_code<P>(blk[slot], sbest[slot], w, K, mask, ub, pinv32, pinv64, seed_out, exp_out, keys,
                   err_out);
    }
    return;
  }
  for (int i = 0; !kOne && i < kS; i += 64) {
    const bool mine = i + lane < kS && sbest[i + lane] != kNoSeed;
    const int slot = mine ? i + lane : 0;
    merge_best(keys, blk[slot], best[slot], sbest[slot], mine,
               [&](uint32_t s2) __attribute__((always_inline)) { return exact_error(slot, s2); });
  }
}

// The same search at P = 4 and many seeds, where the fp64 evaluation needs more
// registers than the walk of four block tiles leaves:
// the block data (B fragments and thresholds) and the seed-tile fragments are
// rebuilt from W, the keys and the projector stack after every evaluation
// batch, so none of it is live across that code and the kernel fits four waves
// per SIMD.
template <int P>
__global__ void __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
search_mfma_remat_kernel(const float* __restrict__ W, int64_t nblocks, const int32_t* __restrict__ list,
                   const int32_t* __restrict__ off, int rung, int K, uint32_t mask,
                   const uint32_t* __restrict__ ub, const float* __restrict__,
                   const double* __restrict__ pinv64, const half8* __restrict__ pi16,
                   int64_t ntiles, RangeRule rule,
                   unsigned long long* __restrict__ keys, uint32_t* __restrict__,
                   uint8_t* __restrict__, float* __restrict__) {
  // 40 KB in all: four workgroups per CU
  __shared__ unsigned long long best_all[kWaves][kSlots];
  __shared__ uint32_t sbest_all[kWaves][kSlots];
  __shared__ int32_t blk_all[kWaves][kSlots];
  __shared__ float thr_base_all[kWaves][kSlots];
  __shared__ int16_t ex_all[kWaves][kSlots];   // ilogb, down to -149
  __shared__ float4 rec_all[kWaves][kRecCapR][4];
  __shared__ uint32_t meta_all[kWaves][kRecCapR];
  __shared__ uint32_t queue_all[kWaves][kRecQueueR];

  const int lane = threadIdx.x & 63;
  // wave-uniform, so that the per-wave LDS addresses are scalar
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int n = lane & 31;   // block column of the MFMA tile
  const int h = lane >> 5;   // which half of the rows / reduction this lane holds
  unsigned long long* best = best_all[wave];
  uint32_t* sbest = sbest_all[wave];
  int32_t* blk = blk_all[wave];
  float* slot_thr = thr_base_all[wave];
  int16_t* slot_ex = ex_all[wave];
  float4 (*rec)[4] = rec_all[wave];
  uint32_t* meta = meta_all[wave];
  uint32_t* queue = queue_all[wave];

  int64_t begin = 0, count = nblocks;
  if (list) {
    begin = off[rung];
    count = int64_t(off[rung + 1]) - begin;
  }
  const SeedRange rg = seed_range(rule, count, kBlocksPerWG);
  const int64_t wave_base = (rg.unit * kWaves + wave) * kSlots;
  if (rg.range >= rg.nranges || wave_base >= count) return;  // wave-uniform; waves never synchronise
  const uint32_t nseeds = uint32_t((int64_t(1) << K) - 1);

  // ---------------------------------------------------------------- prologue
#pragma unroll
  for (int nt = 0; nt < kNB; ++nt) {
    const int64_t idx = wave_base + nt * 32 + n;
    const int64_t b = idx < count ? (list ? int64_t(list[begin + idx]) : idx) : 0;
    if (h == 0) {
      // a range starts from the best that the others have left so far
      best[nt * 32 + n] = idx < count ? key_bound(load_key(keys, b)) : ~0ull;
      sbest[nt * 32 + n] = kNoSeed;
      blk[nt * 32 + n] = int32_t(b);
    }
    const bool valid = idx < count;
    float w[kC];
    load_block(W, b, valid, w);
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < kC; ++i) amax = fmaxf(amax, fabsf(w[i]));
    const int ex = valid && amax > 0.f ? ilogbf(amax) : 0;
    float ws[kC], ww = 0.f;
#pragma unroll
    for (int i = 0; i < kC; ++i) {
      ws[i] = ldexpf(w[i], -ex);
      ww = fmaf(ws[i], ws[i], ww);
    }
    Rounding rd;
    b_fragment<0>(ws, ww, h, rd);
    b_fragment<1>(ws, ww, h, rd);
    b_fragment<2>(ws, ww, h, rd);
    float base = threshold_base<P>(ww, rd);
    // a block with a weight that is not finite: searched in the first range only, as
    // in search_mfma_kernel (elsewhere the threshold +inf over an error of 0)
    const bool skip = valid && !(ww < INFINITY) && rg.range > 0;
    if (skip) base = INFINITY;
    if (h == 0) {
      if (skip) best[nt * 32 + n] = 0ull;
      slot_thr[nt * 32 + n] = base;
      slot_ex[nt * 32 + n] = int16_t(ex);
    }
  }
  __threadfence_block();

  // Per-lane block data: the B fragments (2^12-scaled pair products of the
  // block scaled by a power of two so that max |w_i| lies in [1, 2)) and the
  // screening threshold in accumulator units. Rebuilt from W and the keys after
  // every exact evaluation, so that none of it is live across that code.
  half8 bop[kNB][3];
  float thr[kNB];
  auto setup = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < kNB; ++nt) {
      const bool valid = wave_base + nt * 32 + n < count;
      float w[kC];
      load_block(W, blk[nt * 32 + n], valid, w);
      float amax = 0.f;
#pragma unroll
      for (int i = 0; i < kC; ++i) amax = fmaxf(amax, fabsf(w[i]));
      const bool active = valid && amax > 0.f;
      const int ex = active ? ilogbf(amax) : 0;
      float ws[kC], ww = 0.f;
#pragma unroll
      for (int i = 0; i < kC; ++i) {
        ws[i] = ldexpf(w[i], -ex);
        ww = fmaf(ws[i], ws[i], ww);
      }
      Rounding rd;   // (its threshold is in LDS)
      bop[nt][0] = b_fragment<0>(ws, ww, h, rd);
      bop[nt][1] = b_fragment<1>(ws, ww, h, rd);
      bop[nt][2] = b_fragment<2>(ws, ww, h, rd);
      // -inf before a block's first exact error, +inf for blocks not searched
      const unsigned long long key = best[nt * 32 + n];
      thr[nt] = !active ? INFINITY
                : key == ~0ull ? -INFINITY
                : slot_thr[nt * 32 + n] -
                      __double2float_ru(ldexp(__longlong_as_double((long long)key), 24 - 2 * ex));
    }
  };

  // Exact error of a seed for block b.
  auto exact_error = [&](int64_t b, uint32_t seed) __attribute__((always_inline)) {
    float w[kC];
    load_block(W, b, true, w);
    int qe, q[P];
    return exact_eval<P, false>(w, pinv64 + int64_t(seed - 1) * (P * kC),
                                    ub + int64_t(seed - 1) * basis_words(K, P), seed, K, mask, qe,
                                    q);
  };
  int qcount = 0;  // wave-uniform
  // Evaluate the top min(64, qcount) queued entries, one per lane, until fewer
  // than min_batch remain; after any evaluation rebuild what is needed of the
  // block data, the thresholds and the fragments.
  auto exact_with = [&](int min_batch, auto&& rebuild) __attribute__((always_inline)) {
    bool ran = false;
    while (qcount >= min_batch && qcount > 0) {
      const int e = qcount < 64 ? qcount : 64;
      const int base = qcount - e;
      bool mine = false;
      uint32_t seed = 0u;
      int slot = 0;
      double err = 0.0;
      if (lane < e) {
        const uint32_t ent = queue[base + lane];
        seed = ent >> 8;
        slot = int(ent & 0x7Fu);
        if (seed != 0u) {
          err = exact_error(blk[slot], seed);
          mine = true;
        }
      }
      record_best(best, sbest, slot, err, seed, mine);
      qcount = base;
      ran = true;
    }
    if (ran) {
      __threadfence_block();
      rebuild();
    }
  };

  // Records -> queued seeds (P = 4): lane l < kRecRound takes record base + l of the
  // top kRecRound and compares its 16 bounds with the block's current threshold; one
  // ballot per seed row queues the passing seeds, and full batches are
  // evaluated after each round, each evaluation followed at once by rebuild()
  // (block data and the fragments the walk still needs), so that none of the
  // walk's state is live across the evaluation.
  int nrec = 0;  // wave-uniform
  auto process = [&](auto&& rebuild) __attribute__((always_inline)) {
    __threadfence_block();
    while (nrec > 0) {
      const int e = nrec < kRecRound ? nrec : kRecRound;
      const int base = nrec - e;
      uint32_t m = 0u;
      float t = INFINITY;
      float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0, r3 = r0;
      if (lane < e) {
        m = meta[base + lane];
        const int sl = int(m & 0x7Fu);
        const unsigned long long key = best[sl];
        t = -INFINITY;
        if (key != ~0ull)
          t = slot_thr[sl] - __double2float_ru(ldexp(__longlong_as_double((long long)key),
                                                     24 - 2 * int(slot_ex[sl])));
        r0 = rec[base + lane][0];
        r1 = rec[base + lane][1];
        r2 = rec[base + lane][2];
        r3 = rec[base + lane][3];
      }
      const float bnd[16] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w,
                             r2.x, r2.y, r2.z, r2.w, r3.x, r3.y, r3.z, r3.w};
      const uint32_t seedbase = (m >> 8) * 32u + 1u;
      const int hh = int((m >> 7) & 1u);
      const uint32_t slot = m & 0x7Fu;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const bool pass = bnd[j] >= t;   // t = +inf on lanes without a record
        const uint64_t mk = ballot(pass);
        if (mk != 0ull) {
          if (pass) {
            const uint32_t seed = seed_of(seedbase, j, hh);
            queue[qcount + lanes_below(mk)] = ((seed <= nseeds ? seed : 0u) << 8) | slot;
          }
          qcount += __popcll(mk);
        }
      }
      nrec = base;
      if (qcount >= 64) exact_with(64, rebuild);
    }
  };
  // Lanes of block tile nt whose fold passed store their 16 bounds as records.
  // mk = ballot(pass), taken once by the caller.
  auto record = [&](int nt, const floatx16& acc, bool pass, uint64_t mk, uint32_t T)
                    __attribute__((always_inline)) {
    if (mk == 0ull) return;
    if (pass) {
      const int r = nrec + lanes_below(mk);
      rec[r][0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
      rec[r][1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
      rec[r][2] = make_float4(acc[8], acc[9], acc[10], acc[11]);
      rec[r][3] = make_float4(acc[12], acc[13], acc[14], acc[15]);
      const uint32_t l = lane_now();   // = lane
      meta[r] = (T << 8) | ((l >> 5) << 7) | (uint32_t(nt * 32) + (l & 31u));
    }
    nrec += __popcll(mk);
  };

  const half8* A = pi16;
  setup();

  // The walk of this range: seed tiles [T0, T1), at least 8 of them (32-bit
  // tile indices, ntiles < 2^19, kept scalar).
  const int T0 = range_tile(rg.range, ntiles, rg.nranges);
  const int T1 = range_tile(rg.range + 1, ntiles, rg.nranges);
  const int last = T1 - 1;

  // ---------------------------------------------------------------- pilot
  // Over the range's first tile each lane takes its seed of smallest bound;
  // their exact errors start the best of every block that has none yet (setup()
  // has given those the threshold -inf). (Longer pilots cost more matrix time
  // than the survivors they save.)
  bool fresh = false;
#pragma unroll
  for (int nt = 0; nt < kNB; ++nt) fresh |= thr[nt] == -INFINITY;
  if (ballot(fresh) != 0ull) {
    const half8* At = A + T0 * 192;
    const half8 a0 = At[lane], a1 = At[64 + lane], a2 = At[128 + lane];
#pragma unroll
    for (int nt = 0; nt < kNB; ++nt) {
      const floatx16 acc = bounds(a0, a1, a2, bop[nt]);
      const float m = fold_max(acc);
      int jb = 15;
#pragma unroll
      for (int j = 14; j >= 0; --j)
        if (acc[j] == m) jb = j;
      // every seed of the tile exists: only the last tile of the rung is short,
      // and no range starts there (K >= 8)
      const uint32_t sd = seed_of(uint32_t(T0) * 32u + 1u, jb, h);
      const bool put = thr[nt] != INFINITY;
      const uint64_t mk = ballot(put);
      if (put) queue[qcount + lanes_below(mk)] = (sd << 8) | uint32_t(nt * 32 + n);
      qcount += __popcll(mk);
    }
    exact_with(1, setup);
  }

  // ---------------------------------------------------------------- seed walk
  static_assert(kNB == 4, "the walk below unrolls four block tiles");

  // Seed-tile fragments; the index is clamped to the last tile so that every
  // load is unconditional and each wait covers only the tile it is for.
  auto load_tile = [&](int T, half8 (&f)[3]) __attribute__((always_inline)) {
    // the lane's offset is recomputed here, so that no 64-bit per-lane address
    // stays live (or spilled) across the walk
    const half8* At = A + (T < last ? T : last) * 192;
    const uint32_t l = lane_now();
    f[0] = At[l];
    f[1] = At[64 + l];
    f[2] = At[128 + l];
  };

  // Seed tile T (fragments c) against the four block tiles, two block tiles
  // at a time: six products to the matrix core, then the folds, one branch per
  // pair. An exact evaluation rebuilds the block data and reloads both this
  // tile's fragments and those of the other set (tile To, in o).
  auto tile = [&](half8 (&c)[3], int T, half8 (&o)[3], int To)
                  __attribute__((always_inline)) {
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
      const floatx16 acc0 = bounds(c[0], c[1], c[2], bop[2 * pr]);
      const floatx16 acc1 = bounds(c[0], c[1], c[2], bop[2 * pr + 1]);
      const bool p0 = fold_max(acc0) >= thr[2 * pr];
      const bool p1 = fold_max(acc1) >= thr[2 * pr + 1];
      const uint64_t m0 = ballot(p0), m1 = ballot(p1);
      if ((m0 | m1) != 0ull) {
        auto rebuild = [&]() __attribute__((always_inline)) {
          setup();
          if (pr == 0) load_tile(T, c);
          load_tile(To, o);
        };
        record(2 * pr, acc0, p0, m0, uint32_t(T));
        if (nrec > kRecCapR - 64) process(rebuild);
        record(2 * pr + 1, acc1, p1, m1, uint32_t(T));
        if (nrec >= kRecFlushR) process(rebuild);
      }
    }
  };

  // Two fragment sets in turn: one tile is loaded while the other is screened.
  half8 x[3], y[3];
  load_tile(T0, x);
  for (int T = T0; T < T1; T += 2) {
    load_tile(T + 1, y);
    tile(x, T, y, T + 1);
    load_tile(T + 2, x);
    if (T + 1 < T1) tile(y, T + 1, x, T + 2);
  }
  process(setup);
  exact_with(1, [] {});

  // ---------------------------------------------------------------- results
  for (int i = 0; i < kSlots; i += 64) {
    const int slot = i + int(lane_now());
    const uint32_t seed = sbest[slot];
    merge_best(keys, blk[slot], best[slot], seed, seed != kNoSeed, [&](uint32_t s2)
                   __attribute__((always_inline)) { return exact_error(blk[slot], s2); });
  }
}

// ---------------------------------------------------------------- codes
// Keys of a single-rung search before its walk (a multi-rung call's keys are
// cleared by its compaction).
__global__ void __launch_bounds__(kWaves * 64)
clear_keys_kernel(unsigned long long* __restrict__ keys, int64_t nblocks) {
  const int64_t b = int64_t(blockIdx.x) * (kWaves * 64) + threadIdx.x;
  if (b < nblocks) keys[b] = ~0ull;
}

// The codes of the rung's blocks from their keys, one block per thread, unless the
// walk was known to be of one range and has written them.
template <int P>
__global__ void __launch_bounds__(kWaves * 64)
emit_codes_kernel(const float* __restrict__ W, int64_t nblocks, const int32_t* __restrict__ list,
                  const int32_t* __restrict__ off, int rung, int K, uint32_t mask,
                  const uint32_t* __restrict__ ub, const float* __restrict__ pinv32,
                  const double* __restrict__ pinv64,
                  unsigned long long* __restrict__ keys, uint32_t* __restrict__ seed_out,
                  uint8_t* __restrict__ exp_out, float* __restrict__ err_out) {
  int64_t begin = 0, count = nblocks;
  if (list) {
    begin = off[rung];
    count = int64_t(off[rung + 1]) - begin;
  }
  const int64_t i = int64_t(blockIdx.x) * (kWaves * 64) + threadIdx.x;
  if (i >= count) return;
  const int64_t b = list ? int64_t(list[begin + i]) : i;
  const unsigned long long key = keys[b];
  float w[kC];
  load_block(W, b, true, w);
  emit_code<P>(b, key == ~0ull ? kNoSeed : uint32_t(key & kKeySeed), w, K, mask, ub, pinv32, pinv64,
               seed_out, exp_out, keys, err_out);
}

// ---------------------------------------------------------------- launch
// The number of seed ranges of a rung (per unit of blocks; see RangeRule).
// Bound: a small tensor leaves the chip idle, not the matrix core busy. With one
// range per block, 1024 x 4096 weights at (12,2)/(16,3)/(20,4) put 250
// workgroups of the (20,4) rung on 1024 places and took 18.9 ms; 16 016 blocks of
// that rung took one wave's walk, 18 ms, whatever else the chip could have done.
// - rmin: never a range longer than kRangeTiles (K >= 17). 2048 tiles are the
//   6 MB of fragments that a K = 16 walk covers; the workgroups of one range run
//   together and their L2s keep it, where one walk over the 101 MB of (20,4)
//   missed on 59 % of its requests. 512 to 4096 tiles measure within 0.2 % on
//   4096 x 14336 (171.0-171.3 ms).
// - up to kTargetWorkgroups, ranges of kLongTiles or more: about 12 rounds of
//   the 1024 places even out the last round. 1024 x 4096, three rungs: 14.0,
//   13.5, 13.0, 12.8 ms at targets of 1024, 4096, 8192, 12288 (18.9 ms with one
//   launch per 2048 tiles before).
//   Ranges of 32 or 128 tiles instead of 64 are 0-4 % slower ((12,2) on 2.1 M
//   blocks 1.19 -> 1.21 ms at 32: every range has its own prologue, pilot and
//   first survivors).
// - up to kFillWorkgroups, ranges of 8 or more: with fewer workgroups than
//   places even a short range pays (256 to 1536 measure within 15 %).
constexpr int64_t kRangeTiles = 2048;
constexpr int64_t kLongTiles = 64;
constexpr int kTargetWorkgroups = 12288;
constexpr int kFillWorkgroups = 768;
// Up to so many seed tiles (K <= 13) units of 4 block tiles go through one range where
// they put two or three workgroups on nearly every CU: a second range then costs its
// prologue, pilot and first survivors for nothing ((13,2) on 262 144 blocks 317 us with
// 4 ranges, 300 with one, 301 before there were ranges; (13,3) 344, 318; at K = 14 and
// above 2 % either way). Decided on the host, for calls with one rung: as a part of
// range_count it cost every workgroup, 32.5 -> 33.5 us for (12,3) on 8192 blocks.
constexpr int64_t kEvenTiles = 256;
// Launches above this many workgroups are cut (HIP grids hold 2^32 threads).
constexpr int64_t kMaxGrid = int64_t(1) << 23;

// Block tiles per wave: 4 share each seed-tile fragment and its load. Fewer:
// - 1, when units of 512 blocks times all the ranges of 8 tiles would not make
//   kFewWorkgroups, for calls of up to kFewBlocks: smaller units then even out the
//   workgroups that do not fill the places twice. One tile against 4, each with its
//   ranges: (12,2) on 200 000 blocks 159 and 247 us, on 350 000 266 and 310; (13,2) on
//   140 000 186 and 265, on 230 000 297 and 298; (14,2) on 66 000 167 and 213, on
//   140 000 310 and 298; (15,3) on 33 000 176 and 293, on 66 000 306 and 316; (16,3) on
//   16 000 163 and 193, on 50 000 401 and 370; (8,2) on 400 000 98 and 115, on 2.1 M
//   434 and 367. Against 2: (12,4) on 140 000 182 and 214, on 262 144 287 and 300;
//   (11,4) on 300 000 237 and 216; (12,5) on 262 144 322 and 349; (14,6) on 140 000 910
//   and 971, on 600 000 3682 and 3583; (10,6) on 600 000 569 and 598.
// - 2, at P = 4 below K = 15 ((11,4) on 524 288 blocks 415 -> 335 us, (12,4) on
//   1 M 1122 -> 950 us, (14,4) 2382 -> 2293 us; (15,4) 3943 -> 3962 us, (16,4)
//   +2 %, (20,4) +5 % against the rebuilding kernel) and at P >= 5 ((14,6) 3393
//   -> 3218 us, (16,6) 8450 -> 8316 us on 524 288 blocks; 4 tiles spill at
//   P = 5, (16,5) a third slower): there the survivors' registers
//   and not the fragments' loads bound the walk. At P <= 3 two tiles are 4-14 %
//   slower.
constexpr int64_t kFewWorkgroups = 12288;
template <int P>
constexpr int64_t kFewBlocks = P == 4 ? 262144 : P == 6 ? INT64_MAX : 393216;
constexpr bool two_tiles(int K, int P) {
  return P >= 5 || (P == 4 && K < 15);
}

int64_t env_int(const char* name, int64_t fallback) {
  if (const char* env = std::getenv(name)) {
    char* end = nullptr;
    const long long v = std::strtoll(env, &end, 10);
    if (end != env && v >= 0) return v;
  }
  return fallback;
}

template <int P>
hipError_t launch_mfma_p(const float* d_W, int64_t nblocks, const int32_t* d_list,
                         const int32_t* d_off, int rung, int K, const void* d_bases,
                         uint32_t* d_seed, uint8_t* d_exp, int8_t* d_q, float* d_err,
                         hipStream_t stream) {
  const BasesLayout L = bases_layout(K, P);
  const char* base = static_cast<const char*>(d_bases);
  if (nblocks == 0) return hipSuccess;
  const uint32_t mask = lfsr_mask(K);
  const uint32_t* ub = reinterpret_cast<const uint32_t*>(base + L.off_ub);
  const double* pinv64 = reinterpret_cast<const double*>(base + L.off_pinv64);
  const float* pinv32 =
      many_survivors(P) ? reinterpret_cast<const float*>(base + L.off_pinv32) : nullptr;
  const half8* pi16 =
      reinterpret_cast<const half8*>(base + (complement_dims(P) > 0 ? L.off_nc16 : L.off_pi16));
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(d_q);
  const unsigned threads = kWaves * 64;
  const unsigned per_block = unsigned((nblocks + threads - 1) / threads);
  // SEEDQ_SEED_CHUNK_TILES fixes the range length (0 = one range; at least 8
  // tiles per range) for testing: the codes are the same for every length.
  const int64_t tiles = env_int("SEEDQ_SEED_CHUNK_TILES", -1);
  const int64_t most = std::max<int64_t>(1, L.ntiles / 8);
  const bool few = (nblocks + kBlocksPerWG - 1) / kBlocksPerWG * most < kFewWorkgroups &&
                   nblocks <= kFewBlocks<P>;
  const int nt = few ? 1 : two_tiles(K, P) ? 2 : kNB;
  const int64_t units = (nblocks + kWaves * 32 * nt - 1) / (kWaves * 32 * nt);
  RangeRule rule;
  rule.first = 0;
  rule.target = rule.fill = 0;
  rule.rlong = rule.rshort = 1;
  if (tiles >= 0) {
    rule.rmin = int32_t(tiles > 0 ? std::max<int64_t>(1, std::min(most, L.ntiles / tiles)) : 1);
  } else {
    rule.rmin = int32_t(std::max<int64_t>(1, L.ntiles / kRangeTiles));
    rule.rlong = int32_t(std::max<int64_t>(1, L.ntiles / kLongTiles));
    rule.target = kTargetWorkgroups;
    rule.rshort = int32_t(most);
    rule.fill = kFillWorkgroups;
    // (the count of blocks of a call with one rung is known here)
    const bool even = (units > 460 && units <= 512) || (units > 690 && units <= 768);
    if (!d_list && nt == kNB && L.ntiles <= kEvenTiles && even) rule.target = rule.fill = 0;
  }
  // a multi-rung call does not know its counts of blocks here: the grid holds
  // every choice that the rule can make, and the workgroups past it return
  int64_t grid = std::max<int64_t>({units * rule.rmin, rule.target, rule.fill});
  int64_t step = rule.rmin;
  rule.span = INT32_MAX;
  if (grid > kMaxGrid) {   // too many workgroups for one launch: ranges in turn
    rule.target = rule.fill = 0;
    step = std::max<int64_t>(1, kMaxGrid / units);
    rule.span = int32_t(step);
    grid = units * step;
  }
  // one range, known here: a single-rung call's count of blocks is, and of 8 seed tiles
  // every count makes one. The walk then emits (the rebuilding kernel does not), there
  // are no keys to clear and nothing is left to do after it.
  const bool one = !(P == 4 && nt == kNB) &&
                   (d_list ? std::max({rule.rmin, rule.rlong, rule.rshort}) == 1
                           : range_count(rule, uint32_t(units)) == 1);
  if (!d_list && !one)
    hipLaunchKernelGGL(clear_keys_kernel, dim3(per_block), dim3(threads), 0, stream, keys, nblocks);
  auto walk = [&](auto kern) {
    for (; rule.first < rule.rmin; rule.first += int32_t(step))
      hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(threads), 0, stream, d_W, nblocks, d_list,
                         d_off, rung, K, mask, ub, pinv32, pinv64, pi16, L.ntiles,
                         rule, keys, d_seed, d_exp, d_err);
  };
  if (nt == 1) {
    one ? walk(search_mfma_kernel<P, 1, true>) : walk(search_mfma_kernel<P, 1, false>);
  } else if (nt == 2) {
    if constexpr (P >= 4)
      one ? walk(search_mfma_kernel<P, 2, true>) : walk(search_mfma_kernel<P, 2, false>);
  } else if constexpr (P == 4) {
    walk(search_mfma_remat_kernel<P>);
  } else {
    if constexpr (P < 4)
      one ? walk(search_mfma_kernel<P, kNB, true>) : walk(search_mfma_kernel<P, kNB, false>);
  }
  if (!one)
    hipLaunchKernelGGL(emit_codes_kernel<P>, dim3(per_block), dim3(threads), 0, stream, d_W, nblocks,
                       d_list, d_off, rung, K, mask, ub, pinv32, pinv64, keys, d_seed, d_exp, d_err);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_search(const float* d_W, int64_t nblocks, const int32_t* d_list,
                         const int32_t* d_off, int rung_index, int K, int P, const void* d_bases,
                         uint32_t* d_seed, uint8_t* d_exp, int8_t* d_q, float* d_err,
                         hipStream_t stream) {
  switch (P) {
#define SEEDQ_CASE(PP)                                                                    \
  case PP:                                                                                \
    return launch_mfma_p<PP>(d_W, nblocks, d_list, d_off, rung_index, K, d_bases, d_seed, \
                             d_exp, d_q, d_err, stream);
    SEEDQ_CASE(1)
    SEEDQ_CASE(2)
    SEEDQ_CASE(3)
    SEEDQ_CASE(4)
    SEEDQ_CASE(5)
    SEEDQ_CASE(6)
#undef SEEDQ_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace seedq
