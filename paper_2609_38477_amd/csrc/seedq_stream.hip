// The headerless variable-length code stream of one tensor (Algorithm 1, the
// emit step: every block contributes exactly l(g_b) = K + 4P + 4 bits of
// eq. (rate), with no header; Algorithm 2 and the appendix on encoding and
// decoding: a decoder reads a tensor's blocks in order from its start, the
// length of each known from the allocation alone).
//
// Layout: blocks in row-major order; inside a block the seed (K bits), the
// exponent (4 bits) and the mantissas q_0 .. q_{P-1} (4 bits each, two's
// complement), every field least-significant bit first at increasing stream bit
// positions; stream bit n is bit n % 32 of 32-bit word n / 32; the payload is
// padded with zero bits to a whole word.
//
// Offsets. The blocks are cut into units (2048 blocks for the packer and the
// parsers, one row for the decode-GEMV). With one rung a unit's bit offset is a
// product. Otherwise a first pass writes the bits of every unit and of every
// group of 16 units, and the workgroup that needs an offset adds up the groups
// and units before it itself (at most 1024 group sums, 4 loads a thread, from
// L2), which replaced a one-workgroup scan between the passes (4.3-12.7 us of a
// 23-290 us decode-GEMV). Above kMaxGroups groups that sum would grow with the
// square of the tensor, and the scan runs.
//
// Decoding (fetch_step, use_step). A wave decodes 128 consecutive blocks a step, two per
// lane. Neighbouring blocks mostly share a rung (an encoder sorts the channels
// by importance): when all 128 do, offsets are products, the rung's constants
// are wave-uniform, and for K <= 16 the lane's two LFSRs run packed in one
// register (block_acc_pair). Otherwise a prefix sum over the lanes gives the
// offsets and every lane steps its own register. The packer assembles a chunk
// in LDS; the workgroup in whose chunk a word begins writes that word, so
// every word is stored once, whole.
#include <algorithm>

#include "seedq_reconstruct.h"

namespace seedq {
namespace {

constexpr int kThreads = 256;
constexpr int kWaveBlocks = 512;                 // blocks of a chunk per wave
constexpr int kChunk = 4 * kWaveBlocks;          // blocks per workgroup
constexpr int kMaxBlockBits = SEEDQ_MAX_K + 4 + 4 * SEEDQ_MAX_P;
constexpr int kGroup = 16;                       // units per group
constexpr int64_t kMaxGroups = 1024;
constexpr int64_t kMaxUnitBlocks = int64_t(1) << 26;   // a unit's bits fit 32 bits

// The rungs of a stream, with the code lengths of rungs 0..7 as bytes (0 for
// rungs >= n) for four lookups in one byte permutation.
struct StreamRungs {
  RungTable rt;
  uint32_t len_lo, len_hi;
};

// Where the bit offset of a unit comes from.
enum OffsetMode : int32_t { kProduct, kGroups, kScanned };
struct Offsets {
  int32_t mode;
  int64_t unit_bits;          // kProduct: bits of every unit
  const uint32_t* bits;       // kGroups: bits of every unit
  const int64_t* sums;        // kGroups: bits of every group; kScanned: offset of every unit
};

__device__ __forceinline__ int64_t wave_sum(int64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__device__ __forceinline__ uint32_t wave_sum32(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// Sum of a value over the workgroup (every thread takes part).
template <int kWavesOfGroup>
__device__ __forceinline__ int64_t wg_sum(int64_t v) {
  __shared__ int64_t part[kWavesOfGroup];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t t = 0;
#pragma unroll
  for (int w = 0; w < kWavesOfGroup; ++w) t += part[w];
  return t;
}

// This thread's share of the bits before unit u (kGroups).
__device__ __forceinline__ int64_t groups_share(const Offsets& o, int64_t u) {
  const int64_t g = u / kGroup;
  int64_t s = 0;
  for (int64_t k = threadIdx.x; k < g; k += blockDim.x) s += o.sums[k];
  const int64_t v = g * kGroup + threadIdx.x;
  if (threadIdx.x < kGroup && v < u) s += o.bits[v];
  return s;
}

// Bits of 8 consecutive blocks from their rung bytes: four lengths per byte
// permutation (8-byte loads where the run is whole and aligned and every byte
// below 8, byte loads otherwise).
__device__ __forceinline__ uint32_t bits_of_8(const uint8_t* __restrict__ rung,
                                              const StreamRungs& sr, int64_t b0, int64_t b1) {
  uint32_t sum = 0;
  if (b0 + 8 <= b1 && (reinterpret_cast<uintptr_t>(rung + b0) & 7u) == 0) {
    const uint2 v = *reinterpret_cast<const uint2*>(rung + b0);
    if (((v.x | v.y) & 0xF8F8F8F8u) == 0u) {
      sum = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(sr.len_hi, sr.len_lo, v.x), 0u, 0u);
      return __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(sr.len_hi, sr.len_lo, v.y), 0u, sum);
    }
  }
  for (int64_t b = b0; b < min(b0 + 8, b1); ++b) {
    const uint32_t r = rung[b];
    if (r < 8u) sum += ((r < 4u ? sr.len_lo : sr.len_hi) >> (8u * (r & 3u))) & 0xFFu;
  }
  return sum;
}

// Bits of blocks [b0, b1) over one wave, in every lane.
__device__ __forceinline__ int64_t wave_bits(const uint8_t* __restrict__ rung,
                                             const StreamRungs& sr, int64_t b0, int64_t b1) {
  int64_t sum = 0;
  for (int64_t b = b0 + 8 * int64_t(threadIdx.x & 63); b < b1; b += 512)
    sum += bits_of_8(rung, sr, b, b1);
  return wave_sum(sum);
}

// One workgroup of 16 waves per group: the bits of its 16 units (unit_blocks
// blocks each), one per wave, and their sum.
__global__ void __launch_bounds__(64 * kGroup)
unit_bits_kernel(const uint8_t* __restrict__ rung, StreamRungs sr, int64_t nblocks,
                 int64_t unit_blocks, uint32_t* __restrict__ bits, int64_t* __restrict__ sums) {
  const int64_t u = int64_t(blockIdx.x) * kGroup + (threadIdx.x >> 6);
  const int64_t b0 = u * unit_blocks;
  const int64_t n = b0 < nblocks ? wave_bits(rung, sr, b0, min(nblocks, b0 + unit_blocks)) : 0;
  if (b0 < nblocks && (threadIdx.x & 63) == 0) bits[u] = uint32_t(n);
  const int64_t total = wg_sum<kGroup>((threadIdx.x & 63) == 0 ? n : 0);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// kScanned, one wave per unit: off[u] = bits of unit u.
__global__ void __launch_bounds__(kThreads)
unit_bits64_kernel(const uint8_t* __restrict__ rung, StreamRungs sr, int64_t nblocks,
                   int64_t unit_blocks, int64_t nunits, int64_t* __restrict__ off) {
  const int64_t u = int64_t(blockIdx.x) * (kThreads / 64) + (threadIdx.x >> 6);
  if (u >= nunits) return;
  const int64_t b0 = u * unit_blocks;
  const int64_t n = wave_bits(rung, sr, b0, min(nblocks, b0 + unit_blocks));
  if ((threadIdx.x & 63) == 0) off[u] = n;
}

// One workgroup: off[u] (bits of unit u) -> bit offset of unit u, in place. Each
// of the 1024 threads owns a contiguous run of units and reads it 8 values at a
// time with independent loads, so the pass is not one load latency per unit.
constexpr int kScanThreads = 1024;
constexpr int kScanBatch = 8;

__global__ void __launch_bounds__(kScanThreads)
unit_offsets_kernel(int64_t* __restrict__ off, int64_t nunits) {
  __shared__ int64_t part[kScanThreads / 64];
  const int64_t per = (nunits + kScanThreads - 1) / kScanThreads;
  const int64_t c0 = min(nunits, int64_t(threadIdx.x) * per);
  const int64_t c1 = min(nunits, c0 + per);
  int64_t s = 0;
  for (int64_t c = c0; c < c1; c += kScanBatch) {
    int64_t v[kScanBatch];
#pragma unroll
    for (int k = 0; k < kScanBatch; ++k) v[k] = c + k < c1 ? off[c + k] : 0;
#pragma unroll
    for (int k = 0; k < kScanBatch; ++k) s += v[k];
  }
  // exclusive scan of the per-thread sums: within each wave by shuffles, then
  // across the waves
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) part[wave] = x;
  __syncthreads();
  int64_t run = x - s;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) run += w < wave ? part[w] : 0;
  for (int64_t c = c0; c < c1; c += kScanBatch) {
    int64_t v[kScanBatch];
#pragma unroll
    for (int k = 0; k < kScanBatch; ++k) v[k] = c + k < c1 ? off[c + k] : 0;
#pragma unroll
    for (int k = 0; k < kScanBatch; ++k) {
      if (c + k < c1) {
        off[c + k] = run;
        run += v[k];
      }
    }
  }
}

// Bit offset of this wave's first block in a chunk of the packer and the
// parsers (every thread of the 256 takes part; one barrier), and of the chunk.
__device__ __forceinline__ int64_t chunk_wave_offset(const Offsets& o, const uint8_t* rung,
                                                     const StreamRungs& sr, int64_t base,
                                                     int64_t nblocks, int64_t* chunk_off) {
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  if (o.mode == kProduct) {
    const int64_t len = sr.len_lo & 0xFFu;   // one rung
    *chunk_off = int64_t(blockIdx.x) * o.unit_bits;
    return *chunk_off + wave * (kWaveBlocks * len);
  }
  // bits of this wave's blocks, and its share of the bits before the chunk
  const int64_t b0 = base + wave * kWaveBlocks;
  const uint32_t mine = b0 < nblocks ? uint32_t(wave_bits(rung, sr, b0, min(nblocks, b0 + kWaveBlocks)))
                                     : 0u;
  __shared__ uint32_t bits[kThreads / 64];
  __shared__ int64_t part[kThreads / 64];
  const int64_t share = o.mode == kGroups ? wave_sum(groups_share(o, blockIdx.x)) : 0;
  if ((threadIdx.x & 63) == 0) {
    bits[wave] = mine;
    part[wave] = share;
  }
  __syncthreads();
  int64_t off = o.mode == kScanned ? o.sums[blockIdx.x] : 0, before = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    off += part[w];
    before += w < wave ? bits[w] : 0u;
  }
  *chunk_off = off;
  return off + before;
}

// The first chunk from u on that has bits (or the number of chunks), 64 a step:
// the packer's way across blocks without bits, which block by block and from every
// chunk took a time that grew with the square of their number (4096 x 14336 with
// bits in the first half only: 53 us, 47 with bits everywhere). Wave-uniform.
__device__ __forceinline__ int64_t next_unit_with_bits(const Offsets& o, int64_t u, int64_t nblocks) {
  const int64_t nunits = (nblocks + kChunk - 1) / kChunk;
  for (; u < nunits; u += 64) {
    const int64_t v = u + int64_t(threadIdx.x & 63);
    bool has = v < nunits;
    if (has && o.mode == kGroups) has = o.bits[v] != 0u;
    if (has && o.mode == kScanned) has = v + 1 == nunits || o.sums[v + 1] != o.sums[v];
    const uint64_t m = __builtin_amdgcn_ballot_w64(has);
    if (m != 0ull) return u + __builtin_ctzll(m);
  }
  return nunits;
}

// Exclusive prefix sum over the wave and its total, of 32-bit values: shifts
// within rows of 16 lanes, then the rows' last lanes broadcast to the rows after
// them (data-parallel primitives: no LDS).
__device__ __forceinline__ uint32_t wave_exclusive_scan(uint32_t v, uint32_t* total) {
  uint32_t x = v;
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x111, 0xF, 0xF, true));   // row_shr:1
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x112, 0xF, 0xF, true));   // row_shr:2
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x114, 0xF, 0xF, true));   // row_shr:4
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x118, 0xF, 0xF, true));   // row_shr:8
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x142, 0xA, 0xF, false));  // row_bcast:15
  x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x143, 0xC, 0xF, false));  // row_bcast:31
  *total = uint32_t(__builtin_amdgcn_readlane(int(x), 63));
  return x - v;
}

// A code, parsed.
struct Code {
  uint32_t seed, q;   // q: mantissa j in bits 4j..4j+3
  int e;
  bool ok;            // inside the stream, of a rung of the table
};

__device__ __forceinline__ Code parse_code(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t bit, int K,
                                           bool ok) {
  const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, bit);
  const uint32_t hi = __builtin_amdgcn_alignbit(w2, w1, bit);
  Code c;
  c.seed = lo & ((1u << K) - 1u);
  c.e = int((lo >> K) & 15u);
  c.q = __builtin_amdgcn_alignbit(hi, lo, uint32_t(K + 4));
  c.ok = ok;
  return c;
}

// A wave step: blocks lane and 64 + lane from a place on, two per lane, the three
// stream words that hold each code and the bit it starts at in them.
struct Step {
  uint32_t w[2][3];
  uint32_t bit[2];
  uint32_t r[2];      // table index
  bool ok[2];
  bool one;           // wave-uniform: all 128 blocks share rung r0, inside the stream
  uint32_t r0;
};

// A wave-uniform value that the compiler does not see to be one.
__device__ __forceinline__ int64_t uniform(int64_t v) {
  return int64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(v)))) |
         int64_t(__builtin_amdgcn_readfirstlane(int(v >> 32))) << 32;
}

// Fetches a step: rp = rung bytes from its first block on (null for one rung),
// left = blocks of the run from there on, run = its first bit, which moves past
// the step.
__device__ __forceinline__ Step fetch_step(const uint32_t* __restrict__ stream, int64_t nwords,
                                           const uint4* tab, uint32_t nr,
                                           const uint8_t* __restrict__ rp, int64_t left,
                                           int64_t& run) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n = uint32_t(left < 128 ? left : 128);
  Step s;
#pragma unroll
  for (int i = 0; i < 2; ++i)
    s.r[i] = 64 * i + lane < n ? (rp ? table_index(uint32_t(rp[64 * i + lane]), nr) : 0u) : nr;
  s.r0 = uint32_t(__builtin_amdgcn_readfirstlane(int(s.r[0])));
  const uint32_t len = uint32_t(__builtin_amdgcn_readfirstlane(int(tab[s.r0].w)));
  s.one = __builtin_amdgcn_ballot_w64(s.r[0] != s.r0 || s.r[1] != s.r0) == 0ull && len != 0u &&
          run + int64_t(128 * len) + 96 <= (nwords << 5);
  if (s.one) {
    const uint32_t at = uint32_t(run) & 31u;
    const uint32_t* base = stream + (run >> 5);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      s.bit[i] = at + uint32_t(64 * i + lane) * len;
      const uint32_t* sp = base + (s.bit[i] >> 5);
      s.w[i][0] = sp[0];
      s.w[i][1] = sp[1];
      s.w[i][2] = sp[2];
      s.ok[i] = true;
    }
    run += int64_t(128 * len);
    return s;
  }
  const uint32_t l0 = tab[s.r[0]].w, l1 = tab[s.r[1]].w;
  // 64 codes of at most kMaxBlockBits bits fit 16 bits: both sums in one scan
  static_assert(64 * kMaxBlockBits < 65536, "16 bits hold 64 codes");
  uint32_t tot;
  const uint32_t ex = wave_exclusive_scan(l0 | l1 << 16, &tot);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t l = i ? l1 : l0;
    const int64_t pos = run + int64_t((ex >> (16 * i)) & 0xFFFFu);
    run += int64_t((tot >> (16 * i)) & 0xFFFFu);
    s.bit[i] = uint32_t(pos) & 31u;
    s.ok[i] = l != 0u && pos + int64_t(l) <= (nwords << 5);
    s.w[i][0] = s.w[i][1] = s.w[i][2] = 0u;
    if (s.ok[i]) {
      // words past the stream's end hold no bit of the code
      const int64_t wi = pos >> 5;
      const uint32_t* sp = stream + wi;
      s.w[i][0] = sp[0];
      if (wi + 1 < nwords) s.w[i][1] = sp[1];
      if (wi + 2 < nwords) s.w[i][2] = sp[2];
    }
  }
  return s;
}

// Decodes a fetched step. pair(a, b, K, P, mask) gets both codes of the lane when
// all 128 blocks share one rung with K <= 16; single(i, c, info) gets block i of
// the lane otherwise (info = its table entry; c.ok false for a code that is not
// there).
template <typename Pair, typename Single>
__device__ __forceinline__ void use_step(const Step& s, const uint4* tab, Pair&& pair,
                                         Single&& single) {
  if (s.one) {
    const uint4 t0 = tab[s.r0];
    const int K = __builtin_amdgcn_readfirstlane(int(t0.x)), P = __builtin_amdgcn_readfirstlane(int(t0.y));
    const uint32_t mask = uint32_t(__builtin_amdgcn_readfirstlane(int(t0.z)));
    const Code a = parse_code(s.w[0][0], s.w[0][1], s.w[0][2], s.bit[0] & 31u, K, true);
    const Code b = parse_code(s.w[1][0], s.w[1][1], s.w[1][2], s.bit[1] & 31u, K, true);
    if (K <= kPackedMaxK) {
      pair(a, b, K, P, mask);
    } else {
      const uint4 info = make_uint4(uint32_t(K), uint32_t(P), mask, 0u);
      single(0, a, info);
      single(1, b, info);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint4 info = tab[s.r[i]];
    single(i, parse_code(s.w[i][0], s.w[i][1], s.w[i][2], s.bit[i], int(info.x), s.ok[i]), info);
  }
}

// 2^-(K-1+e), the factor of a block's integers (exact: between 2^-38 and 2^-7),
// or NaN for a code that is not valid.
__device__ __forceinline__ float code_scale(int K, int e, bool ok) {
  return ok ? __builtin_amdgcn_ldexpf(1.0f, 1 - K - e) : __int_as_float(0x7fc00000);
}

// The integers of both blocks of a lane, unscaled and converted, and their
// factors. A seed 0 is never emitted: NaN.
__device__ __forceinline__ void pair_values(const Code& a, const Code& b, int K, int P,
                                            uint32_t mask, float (&fa)[kC], float& sa,
                                            float (&fb)[kC], float& sb) {
  int32_t xa[kC], xb[kC];
  block_acc_pair(a.seed, b.seed, a.q, b.q, K, P, mask, xa, xb);
#pragma unroll
  for (int i = 0; i < kC; ++i) {
    fa[i] = __int2float_rn(xa[i]);
    fb[i] = __int2float_rn(xb[i]);
  }
  sa = code_scale(K, a.e, a.seed != 0u);
  sb = code_scale(K, b.e, b.seed != 0u);
}

__device__ __forceinline__ void one_value(const Code& c, const uint4& info, float (&f)[kC],
                                          float& s) {
  const bool ok = c.ok && c.seed != 0u;
  int32_t x[kC];
  block_acc_q(ok ? c.seed : 1u, int(info.x), int(info.y), info.z,
              [&](int j) { return __builtin_amdgcn_sbfe(int32_t(c.q), 4 * j, 4); }, x);
#pragma unroll
  for (int i = 0; i < kC; ++i) f[i] = __int2float_rn(x[i]);
  s = code_scale(int(info.x), c.e, ok);
}

// The code bits of a block: seed, exponent, the P mantissas (bytes of qw) as
// nibbles.
__device__ __forceinline__ uint64_t code_bits(uint32_t seed, uint32_t e, uint2 qw, int K, int P) {
  auto nibbles = [](uint32_t x) {
    x &= 0x0F0F0F0Fu;
    x = (x | x >> 4) & 0x00FF00FFu;
    return (x | x >> 8) & 0xFFFFu;
  };
  const uint32_t q = (nibbles(qw.x) | nibbles(qw.y) << 16) & ((1u << (4 * P)) - 1u);
  return uint64_t(seed & ((1u << K) - 1u)) | uint64_t((e & 15u) | q << 4) << K;
}

// ORs a code into the words staged in LDS, from bit pos.
__device__ __forceinline__ void stage_code(uint32_t* stage, uint32_t pos, uint64_t code) {
  const int wi = int(pos >> 5), sh = int(pos & 31);
  const uint64_t lo = code << sh;
  const uint32_t hi = sh ? uint32_t(code >> (64 - sh)) : 0u;
  atomicOr(&stage[wi], uint32_t(lo));
  if (uint32_t(lo >> 32)) atomicOr(&stage[wi + 1], uint32_t(lo >> 32));
  if (hi) atomicOr(&stage[wi + 2], hi);
}

// bit 31 + every bit of a chunk, the words that a code may spill into, and the
// codes that complete the last word (at most 64 blocks past it at a time)
constexpr int kStageWords = (31 + (kChunk + 64) * kMaxBlockBits) / 32 + 3;

__global__ void __launch_bounds__(kThreads)
pack_kernel(const uint32_t* __restrict__ seed, const uint8_t* __restrict__ expo,
            const int8_t* __restrict__ q, const uint8_t* __restrict__ rung, StreamRungs sr,
            int64_t nblocks, Offsets o, uint32_t* __restrict__ stream, int64_t nwords) {
  __shared__ uint32_t stage[kStageWords];
  __shared__ uint4 tab[kRungTable];
  __shared__ int64_t end_s;
  fill_rung_table(tab, sr.rt);
  const int64_t base = int64_t(blockIdx.x) * kChunk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < kStageWords; i += kThreads) stage[i] = 0u;
  int64_t off0;
  int64_t run = chunk_wave_offset(o, rung, sr, base, nblocks, &off0);
  __syncthreads();
  const int64_t w0 = off0 >> 5;
  const uint32_t nr = uint32_t(sr.rt.n);
  // 64 blocks from b0 on, of which those below b1 exist; returns their bits
  auto put = [&](int64_t b0, int64_t b1, int64_t from) __attribute__((always_inline)) {
    const int64_t b = b0 + lane;
    const uint32_t r = b < b1 ? (rung ? table_index(uint32_t(rung[b]), nr) : 0u) : nr;
    const uint4 in = tab[r];
    const uint32_t r0 = __builtin_amdgcn_readfirstlane(r);
    uint32_t ex, tot;
    if (__builtin_amdgcn_ballot_w64(r != r0) == 0ull) {
      ex = uint32_t(lane) * in.w;
      tot = 64u * __builtin_amdgcn_readfirstlane(in.w);
    } else {
      ex = wave_exclusive_scan(in.w, &tot);
    }
    if (in.w)
      stage_code(stage, uint32_t(from - (w0 << 5)) + ex,
                 code_bits(seed[b], expo[b], reinterpret_cast<const uint2*>(q)[b], int(in.x),
                           int(in.y)));
    return tot;
  };
  const int64_t b1 = min(nblocks, base + kChunk);
  for (int64_t b = base + wave * kWaveBlocks; b < min(b1, base + (wave + 1) * kWaveBlocks); b += 64)
    run += put(b, b1, run);
  // the last wave that has blocks completes the chunk's last word, if that begins in
  // the chunk, from the blocks that follow (two codes, unless blocks without bits
  // come between)
  if (wave == int((b1 - base - 1) / kWaveBlocks)) {
    if (lane == 0) end_s = run;
    const int64_t word_end = (run + 31) & ~int64_t(31);
    if (((off0 + 31) >> 5) < (word_end >> 5))
      for (int64_t b = b1; b < nblocks && run < word_end; b += 64) {
        if (b > b1 && b % kChunk == 0) b = next_unit_with_bits(o, b / kChunk, nblocks) * kChunk;
        if (b < nblocks) run += put(b, nblocks, run);
      }
  }
  __syncthreads();
  // the words that begin inside the chunk, past the caches' replacement order: an
  // eighth of what the call reads, so that its reader pays little for it (a
  // decode-GEMV of 4096 x 11008 right after 101 us, 99 with ordinary stores), and a
  // call among others finds more of its inputs (30 us, 37)
  const int64_t off1 = end_s, g0 = (off0 + 31) >> 5, g1 = min(nwords, (off1 + 31) >> 5);
  for (int64_t gw = g0 + threadIdx.x; gw < g1; gw += kThreads)
    __builtin_nontemporal_store(stage[gw - w0], &stream[gw]);
}

// Four mantissa nibbles as sign-extended bytes.
__device__ __forceinline__ uint32_t nibbles_to_bytes(uint32_t n) {
  uint32_t t = (n | n << 8) & 0x00FF00FFu;
  t = (t | t << 4) & 0x0F0F0F0Fu;
  const uint32_t s = t & 0x08080808u;
  return t | ((s << 5) - (s << 1));   // 0xF0 where the nibble is negative
}

// One-pass parse of a chunk: MODE 0 writes the codes (seed, exponent, the P
// mantissas as bytes), MODE 1 the reconstructed weights. A block whose bits
// are not all inside the stream, or whose rung byte is out of range, decodes
// to seed 0 (MODE 1: NaN weights).
template <int MODE, bool kPast>
__global__ void __launch_bounds__(kThreads)
parse_kernel(const uint32_t* __restrict__ stream, int64_t nwords, const uint8_t* __restrict__ rung,
             StreamRungs sr, int64_t nblocks, Offsets o, uint32_t* __restrict__ seed_out,
             uint8_t* __restrict__ exp_out, int8_t* __restrict__ q_out, float* __restrict__ W_hat) {
  __shared__ uint4 tab[kRungTable];
  fill_rung_table(tab, sr.rt);
  const int64_t base = int64_t(blockIdx.x) * kChunk;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  int64_t chunk_off;
  int64_t run = uniform(chunk_wave_offset(o, rung, sr, base, nblocks, &chunk_off));
  __syncthreads();
  const int64_t b0 = base + wave * kWaveBlocks, b1 = min(nblocks, b0 + kWaveBlocks);
  // MODE 1: 64 blocks are 2 KB of contiguous weights, staged in LDS (one region
  // per wave, no barrier) and stored so that every store instruction of the wave
  // writes 1 KB without gaps.
  __shared__ float4 stage_all[kThreads / 64][MODE == 1 ? 128 : 1];
  float4* stage = stage_all[wave];
  auto store = [&](int64_t g0, const float (&f)[kC], float s) __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    stage[2 * lane] = make_float4(f[0] * s, f[1] * s, f[2] * s, f[3] * s);
    stage[2 * lane + 1] = make_float4(f[4] * s, f[5] * s, f[6] * s, f[7] * s);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float4* dst = reinterpret_cast<float4*>(W_hat + g0 * kC);
    const int n = 2 * int(min(int64_t(64), b1 - g0));
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (64 * k + lane < n) store_result<kPast>(&dst[64 * k + lane], stage[64 * k + lane]);
    __builtin_amdgcn_wave_barrier();
  };
  auto code = [&](int64_t g, const Code& c, int P) __attribute__((always_inline)) {
    const uint32_t q = c.ok ? c.q & ((1u << (4 * P)) - 1u) : 0u;
    store_result<kPast>(&seed_out[g], c.ok ? c.seed : 0u);
    store_result<kPast>(&exp_out[g], uint8_t(c.ok ? c.e : 0));
    store_result<kPast>(reinterpret_cast<uint2*>(q_out) + g, nibbles_to_bytes(q & 0xFFFFu),
                        nibbles_to_bytes(q >> 16));
  };
  auto fetch = [&](int64_t g0) __attribute__((always_inline)) {
    return fetch_step(stream, nwords, tab, uint32_t(sr.rt.n), rung ? rung + g0 : nullptr, b1 - g0,
                      run);
  };
  if (b0 >= b1) return;
  // MODE 1: a step's words are loaded one step before they are used
  Step s = fetch(b0);
  for (int64_t g0 = b0; g0 < b1; g0 += 128) {
    Step next;
    if (MODE == 1 && g0 + 128 < b1) next = fetch(g0 + 128);
    use_step(
        s, tab,
        [&](const Code& a, const Code& b, int K, int P, uint32_t mask)
            __attribute__((always_inline)) {
          if constexpr (MODE == 0) {
            code(g0 + lane, a, P);
            code(g0 + 64 + lane, b, P);
          } else {
            float fa[kC], fb[kC], sa, sb;
            pair_values(a, b, K, P, mask, fa, sa, fb, sb);
            store(g0, fa, sa);
            store(g0 + 64, fb, sb);
          }
        },
        [&](int i, const Code& c, const uint4& info) __attribute__((always_inline)) {
          const int64_t g = g0 + 64 * i;
          if constexpr (MODE == 0) {
            if (g + lane < b1) code(g + lane, c, int(info.y));
          } else {
            if (g >= b1) return;   // wave-uniform
            float f[kC], f2;
            one_value(c, info, f, f2);
            store(g, f, f2);
          }
        });
    if (MODE == 1) s = next;
    else if (g0 + 128 < b1) s = fetch(g0 + 128);
  }
}

// ---------------------------------------------------------------- decode-GEMV
// y_v = W_hat x_v for nv right-hand sides, W_hat decoded from the stream on the
// fly and never stored (the bandwidth motivation of the codec: a GEMV reads
// l(g)/8 bytes per block instead of 16 for fp16). One wave per row, 128 blocks
// per wave step (fetch_step, use_step), so the loads of x stay coalesced. The lane
// rebuilds a block's integers exactly as seedq_decompress does and forms
// d_v = sum_i fp32(acc_i) x_v[8g + i]; since w_hat_i = fp32(acc_i) 2^-(K-1+e)
// exactly, d_v 2^-(K-1+e) is the block's partial product up to fp32 rounding. A
// wave reduction gives y_v[r], with `segs` waves a row each over a run of whole
// steps and their sums added in order. Bound: the vector ALU regenerating the
// basis (8P LFSR states a block), not the bytes; 8192 x 28672 at three rungs and
// 4.0 bits a weight 160 -> 125 us with one vector, 217 -> 159 with four (one
// block a lane and register, rung constants per lane, one prefix sum a step
// before).
template <int NV>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(8)))
gemv_stream_kernel(const uint32_t* __restrict__ stream, int64_t nwords,
                   const uint8_t* __restrict__ rung, StreamRungs sr, int64_t nrows, int64_t G,
                   Offsets o, int segs, const float* __restrict__ x, int64_t ldx,
                   float* __restrict__ y, int64_t ldy) {
  __shared__ uint4 tab[kRungTable];
  fill_rung_table(tab, sr.rt);
  constexpr int kWavesPerWG = kThreads / 64;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  // wave = row-in-workgroup * segs + segment of the row
  const int64_t r0 = int64_t(blockIdx.x) * (kWavesPerWG / segs), r = r0 + wave / segs;
  const int seg = wave % segs;
  const int64_t per = ((G + 127) / 128 + segs - 1) / segs * 128;   // blocks per segment
  const int64_t ga = min(G, seg * per), gb = r < nrows ? min(G, ga + per) : ga;
  const uint8_t* row = rung && r < nrows ? rung + r * G : nullptr;
  int64_t run = 0;
  __shared__ uint32_t seg_bits[kWavesPerWG];
  __shared__ float seg_sum[NV][kWavesPerWG];
  if (o.mode == kGroups) {
    if (segs > 1) {
      const uint32_t n = row ? uint32_t(wave_bits(row, sr, ga, gb)) : 0u;
      if (lane == 0) seg_bits[wave] = n;
    }
    run = wg_sum<kWavesPerWG>(groups_share(o, r0));
  }
  __syncthreads();
  if (r < nrows) {
    if (o.mode == kProduct) {
      run = r * o.unit_bits + ga * int64_t(sr.len_lo & 0xFFu);
    } else if (o.mode == kGroups) {
      for (int64_t k = r0; k < r; ++k) run += o.bits[k];
      for (int k = 0; k < seg; ++k) run += seg_bits[wave - seg + k];
    } else {
      run = o.sums[r];   // one segment
    }
  }
  run = uniform(run);
  float acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.f;
  // the blocks from g0 (wave-uniform) on
  auto add = [&](int64_t g0, const float (&f)[kC], float s) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const float4* xv = reinterpret_cast<const float4*>(x + v * ldx + g0 * kC);
      const float4 x0 = xv[2u * uint32_t(lane)], x1 = xv[2u * uint32_t(lane) + 1u];
      float d = f[0] * x0.x;
      d = fmaf(f[1], x0.y, d);
      d = fmaf(f[2], x0.z, d);
      d = fmaf(f[3], x0.w, d);
      d = fmaf(f[4], x1.x, d);
      d = fmaf(f[5], x1.y, d);
      d = fmaf(f[6], x1.z, d);
      d = fmaf(f[7], x1.w, d);
      acc[v] = fmaf(d, s, acc[v]);   // d s is exact: one rounding
    }
  };
  for (int64_t g0 = ga; g0 < gb; g0 += 128) {
    const Step s = fetch_step(stream, nwords, tab, uint32_t(sr.rt.n), row ? row + g0 : nullptr,
                              gb - g0, run);
    use_step(
        s, tab,
        [&](const Code& a, const Code& b, int K, int P, uint32_t mask)
            __attribute__((always_inline)) {
          float fa[kC], fb[kC], sa, sb;
          pair_values(a, b, K, P, mask, fa, sa, fb, sb);
          add(g0, fa, sa);
          add(g0 + 64, fb, sb);
        },
        [&](int i, const Code& c, const uint4& info) __attribute__((always_inline)) {
          const int64_t g = g0 + 64 * i;
          if (g + lane < gb) {
            float f[kC], f2;
            one_value(c, info, f, f2);
            add(g, f, f2);
          }
        });
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    float t = acc[v];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
    if (segs == 1) {
      if (lane == 0 && r < nrows) y[v * ldy + r] = t;
    } else if (lane == 0) {
      seg_sum[v][wave] = t;
    }
  }
  if (segs > 1) {
    __syncthreads();
    if (seg == 0 && lane < NV && r < nrows) {
      float t = seg_sum[lane][wave];
      for (int k = 1; k < segs; ++k) t += seg_sum[lane][wave + k];
      y[lane * ldy + r] = t;
    }
  }
}

// Decode-GEMV for eight vectors with the products on the matrix core
// (v_mfma_f32_16x16x4_f32). A workgroup of 16 waves takes 16 rows, one wave
// per row decoding 128 consecutive blocks per step exactly as the one-vector
// kernel does, into a 16-row tile of weights in LDS (64 KB: two workgroups per
// CU). Then wave w multiplies the tile's blocks 4w .. 4w + 3 of either half by
// the vectors: product m takes A[i][k] = weight m of block 4w + k of row i and
// B[k][n] = x_n at the same column, so that lane (i, k) reads 8 consecutive
// weights of the tile and lane (k, n) 8 consecutive entries of x_n. The 16
// waves' partial products are summed in a fixed order at the end. Rounding: a
// product passes through at most 8 matrix-core accumulations of its 64 blocks
// (5 + 7 x 4 roundings), one addition per 64 blocks and the 16-way sum (15). 258
// -> 204 us on 8192 x 28672; the next step's words are loaded before the products.
constexpr int kTlRows = 16;
constexpr int kTlBlocks = 128;                 // blocks per row and step
constexpr int kTlStride = kTlBlocks * kC + 4;  // floats per tile row (padded)
typedef float tl_floatx4 __attribute__((ext_vector_type(4)));

template <int NV>
__global__ void __launch_bounds__(64 * kTlRows)
gemv_stream_tile_kernel(const uint32_t* __restrict__ stream, int64_t nwords,
                        const uint8_t* __restrict__ rung, StreamRungs sr, int64_t nrows, int64_t G,
                        Offsets o, const float* __restrict__ x, int64_t ldx, float* __restrict__ y,
                        int64_t ldy) {
  static_assert(NV >= 1 && NV <= 16, "one B column per vector");
  static_assert(kTlRows * 8 == kTlBlocks, "each wave multiplies 4 blocks of either half of the tile");
  static_assert(kTlRows == kGroup, "a workgroup's rows are one group of units");
  __shared__ uint4 tab[kRungTable];
  __shared__ __attribute__((aligned(16))) float tile[kTlRows][kTlStride];
  fill_rung_table(tab, sr.rt);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = int(threadIdx.x & 63);
  const int i = lane & 15, k = lane >> 4;
  const int64_t r0 = int64_t(blockIdx.x) * kTlRows, r = r0 + wave;   // the row this wave decodes
  const bool row_ok = r < nrows;
  const uint8_t* row = rung && row_ok ? rung + r * G : nullptr;
  int64_t run = o.mode == kGroups ? wg_sum<kTlRows>(groups_share(o, r0)) : 0;
  __syncthreads();
  if (row_ok) {
    if (o.mode == kGroups) run += wave_sum32(lane < wave ? o.bits[r0 + lane] : 0u);
    else run = o.mode == kProduct ? r * o.unit_bits : o.sums[r];
  }
  tl_floatx4 sum = {0.f, 0.f, 0.f, 0.f};
  auto put = [&](int half, const float (&f)[kC], float s) __attribute__((always_inline)) {
    float4* dst = reinterpret_cast<float4*>(&tile[wave][(64 * half + lane) * kC]);
    dst[0] = make_float4(f[0] * s, f[1] * s, f[2] * s, f[3] * s);
    dst[1] = make_float4(f[4] * s, f[5] * s, f[6] * s, f[7] * s);
  };
  const float zero[kC] = {};
  run = uniform(run);
  auto fetch = [&](int64_t g0) __attribute__((always_inline)) {
    return fetch_step(stream, nwords, tab, uint32_t(sr.rt.n), row ? row + g0 : nullptr, G - g0,
                      run);
  };
  Step s;
  if (row_ok) s = fetch(0);
  for (int64_t g0 = 0; g0 < G; g0 += kTlBlocks) {   // the same trip count in every wave
    if (row_ok) {
      use_step(
          s, tab,
          [&](const Code& a, const Code& b, int K, int P, uint32_t mask)
              __attribute__((always_inline)) {
            float fa[kC], fb[kC], sa, sb;
            pair_values(a, b, K, P, mask, fa, sa, fb, sb);
            put(0, fa, sa);
            put(1, fb, sb);
          },
          [&](int half, const Code& c, const uint4& info) __attribute__((always_inline)) {
            if (g0 + 64 * half + lane < G) {
              float f[kC], f2;
              one_value(c, info, f, f2);
              put(half, f, f2);
            } else {
              put(half, zero, 0.f);
            }
          });
      // the next step's words are on their way during the products
      if (g0 + kTlBlocks < G) s = fetch(g0 + kTlBlocks);
    } else {
      put(0, zero, 0.f);
      put(1, zero, 0.f);
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      // blocks gb = g0 + 64 half + 4 wave + k of the 16 rows against the vectors
      const int64_t gb = g0 + 64 * half + 4 * wave + k;
      const float4* src = reinterpret_cast<const float4*>(&tile[i][(64 * half + 4 * wave + k) * kC]);
      const float4 a0 = src[0], a1 = src[1];
      float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f), b1 = b0;
      if (i < NV && gb < G) {
        const float4* xv = reinterpret_cast<const float4*>(x + i * ldx + gb * kC);
        b0 = xv[0];
        b1 = xv[1];
      }
      tl_floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.x, b0.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.y, b0.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.z, b0.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.w, b0.w, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.x, b1.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.y, b1.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.z, b1.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.w, b1.w, acc, 0, 0, 0);
      sum += acc;
    }
    __syncthreads();   // the tile is read before the next step writes it
  }
  // lane l of wave w holds rows 4 (l / 16) + v, vector l % 16; the 16 waves'
  // sums go through the tile
  float* part = &tile[0][0];
#pragma unroll
  for (int v = 0; v < 4; ++v) part[(wave * 4 + v) * 64 + lane] = sum[v];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float t = part[v * 64 + lane];
      for (int w = 1; w < kTlRows; ++w) t += part[(w * 4 + v) * 64 + lane];
      const int64_t rr = int64_t(blockIdx.x) * kTlRows + 4 * k + v;
      if (i < NV && rr < nrows) y[i * ldy + rr] = t;
    }
  }
}

}  // namespace

static int64_t stream_chunks(int64_t nblocks) { return (nblocks + kChunk - 1) / kChunk; }

// One int64 per unit and one more: the sums of kGroups and its 32-bit bits of
// units, or the offsets of kScanned.
size_t stream_workspace_bytes(int64_t nblocks, int64_t nrows) {
  const int64_t n = std::max(stream_chunks(nblocks), nrows) + 1;
  return align256(sizeof(int64_t) * size_t(n));
}

static StreamRungs stream_rungs(const RungTable& rt) {
  StreamRungs sr;
  sr.rt = rt;
  sr.len_lo = sr.len_hi = 0;
  for (int r = 0; r < rt.n; ++r)
    (r < 4 ? sr.len_lo : sr.len_hi) |= uint32_t(rt.K[r] + 4 + 4 * rt.P[r]) << (8 * (r & 3));
  return sr;
}

static hipError_t launch_offsets(const uint8_t* d_rung, const StreamRungs& sr, int64_t nblocks,
                                 int64_t unit_blocks, int64_t nunits, void* d_ws, Offsets* o,
                                 hipStream_t stream) {
  o->unit_bits = unit_blocks * int64_t(sr.len_lo & 0xFFu);
  o->bits = nullptr;
  o->sums = nullptr;
  o->mode = kProduct;
  if (!d_rung || nunits == 0) return hipSuccess;
  int64_t* sums = static_cast<int64_t*>(d_ws);
  o->sums = sums;
  const int64_t ngroups = (nunits + kGroup - 1) / kGroup;
  if (ngroups <= kMaxGroups && unit_blocks <= kMaxUnitBlocks) {
    uint32_t* bits = reinterpret_cast<uint32_t*>(sums + ngroups);
    o->bits = bits;
    o->mode = kGroups;
    hipLaunchKernelGGL(unit_bits_kernel, dim3(unsigned(ngroups)), dim3(64 * kGroup), 0, stream, d_rung,
                       sr, nblocks, unit_blocks, bits, sums);
  } else {
    o->mode = kScanned;
    hipLaunchKernelGGL(unit_bits64_kernel, dim3(unsigned((nunits + 3) / 4)), dim3(kThreads), 0,
                       stream, d_rung, sr, nblocks, unit_blocks, nunits, sums);
    hipLaunchKernelGGL(unit_offsets_kernel, dim3(1), dim3(kScanThreads), 0, stream, sums, nunits);
  }
  return hipGetLastError();
}

hipError_t launch_pack(const uint32_t* d_seed, const uint8_t* d_exp, const int8_t* d_q,
                       const uint8_t* d_rung, const RungTable& rt, int64_t nblocks,
                       uint32_t* d_stream, int64_t nwords, void* d_ws, hipStream_t stream) {
  const int64_t nchunks = stream_chunks(nblocks);
  if (nchunks == 0) return hipSuccess;
  const StreamRungs sr = stream_rungs(rt);
  Offsets o;
  const hipError_t err = launch_offsets(d_rung, sr, nblocks, kChunk, nchunks, d_ws, &o, stream);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(pack_kernel, dim3(unsigned(nchunks)), dim3(kThreads), 0, stream, d_seed, d_exp,
                     d_q, d_rung, sr, nblocks, o, d_stream, nwords);
  return hipGetLastError();
}

hipError_t launch_parse(const uint32_t* d_stream, int64_t nwords, const uint8_t* d_rung,
                        const RungTable& rt, int64_t nblocks, void* d_ws, uint32_t* d_seed,
                        uint8_t* d_exp, int8_t* d_q, float* d_W_hat, hipStream_t stream) {
  const int64_t nchunks = stream_chunks(nblocks);
  if (nchunks == 0) return hipSuccess;
  const StreamRungs sr = stream_rungs(rt);
  Offsets o;
  const hipError_t err = launch_offsets(d_rung, sr, nblocks, kChunk, nchunks, d_ws, &o, stream);
  if (err != hipSuccess) return err;
  const int64_t bytes_in = 4 * nwords + (d_rung ? nblocks : 0);
  const bool past = stores_past_caches(bytes_in, (d_W_hat ? 32 : 13) * nblocks);
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(unsigned(nchunks)), dim3(kThreads), 0, stream, d_stream, nwords, d_rung,
                       sr, nblocks, o, d_seed, d_exp, d_q, d_W_hat);
  };
  if (d_W_hat) past ? launch(parse_kernel<1, true>) : launch(parse_kernel<1, false>);
  else past ? launch(parse_kernel<0, true>) : launch(parse_kernel<0, false>);
  return hipGetLastError();
}

hipError_t launch_gemv_stream(const uint32_t* d_stream, int64_t nwords, const uint8_t* d_rung,
                              const RungTable& rt, int64_t nrows, int64_t ncols, void* d_ws,
                              const float* d_x, int64_t ldx, float* d_y, int64_t ldy, int nv,
                              hipStream_t stream) {
  const int64_t G = ncols / kC;
  const StreamRungs sr = stream_rungs(rt);
  Offsets o;
  const hipError_t err = launch_offsets(d_rung, sr, nrows * G, G, nrows, d_ws, &o, stream);
  if (err != hipSuccess) return err;
  // Waves per row: the most of 4, 2 and 1 with a step of 128 blocks for each and, over
  // all rows, no more than the 8192 that the chip holds at a time and 2048 for every
  // step of a row. A row's wave goes through its steps one after the other, so few rows
  // leave the chip waiting, above all for words not yet in the caches; each wave more
  // has its own prologue and sum. Kernel times in us at 1, 2 and 4 waves a row, one
  // vector and three rungs in runs, repeated and with the caches flushed before:
  //   512 x 1024 (1 step) 5.2/5.7/5.8, 6.5/6.7/6.9; 1500 x 2048 (2) 7.4/7.0/8.0,
  //   9.9/8.5/9.5; 4096 x 2048 10.2/12.6/16.1, 12.8/12.9/18.6; 1500 x 4096 (4)
  //   10.4/9.3/9.2, 14.8/11.5/11.0; 4096 x 4096 15.2/15.8/18.6, 19.6/18.4/21.5; 6000
  //   rows 19.8/21.8/25.4, 24.1/26.7/30.0; 2047 x 8192 (8) 16.4/15.3/15.0,
  //   24.6/19.4/17.8; 4096 rows 24.0/23.1/25.8, 31.6/28.2/31.2; 8192 rows
  //   41.4/43.1/48.9, 45.8/50.6/56.7.
  // With 1, 2 and 4 vectors, rungs in runs, mixed and one, 512 to 12000 rows of 512 to
  // 28672 columns the choice is within 13 % of the best in the sum of both.
  const int64_t steps = (G + 127) / 128;
  auto fits = [&](int64_t w) {
    return w <= steps && nrows * w <= std::min<int64_t>(8192, 2048 * steps);
  };
  const int segs = o.mode == kScanned ? 1 : fits(4) ? 4 : fits(2) ? 2 : 1;
  const unsigned grid = unsigned((nrows * segs + kThreads / 64 - 1) / (kThreads / 64));
  switch (nv) {
    case 1:
      hipLaunchKernelGGL(gemv_stream_kernel<1>, dim3(grid), dim3(kThreads), 0, stream, d_stream,
                         nwords, d_rung, sr, nrows, G, o, segs, d_x, ldx, d_y, ldy);
      break;
    case 2:
      hipLaunchKernelGGL(gemv_stream_kernel<2>, dim3(grid), dim3(kThreads), 0, stream, d_stream,
                         nwords, d_rung, sr, nrows, G, o, segs, d_x, ldx, d_y, ldy);
      break;
    case 4:
      hipLaunchKernelGGL(gemv_stream_kernel<4>, dim3(grid), dim3(kThreads), 0, stream, d_stream,
                         nwords, d_rung, sr, nrows, G, o, segs, d_x, ldx, d_y, ldy);
      break;
    case 8:
      hipLaunchKernelGGL(gemv_stream_tile_kernel<8>, dim3(unsigned((nrows + kTlRows - 1) / kTlRows)),
                         dim3(64 * kTlRows), 0, stream, d_stream, nwords, d_rung, sr, nrows, G, o,
                         d_x, ldx, d_y, ldy);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace seedq
