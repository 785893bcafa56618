// qsl_dense.h -- An operator that keeps every coordinate (k = size in every segment: the error-feedback schemes
// without sparsification that Section 5 compares with, as this operator) with the index-free message format: two
// streaming passes and nothing per entry in between.
//   k_dense_norm    v = m + Delta (Algorithm 1, first worker line) written over the error memory, 12 bytes per
//                   coordinate, with the exact digits of every segment's norm added up on the way
//   k_dense_sum     the digit sums that the blocks of k_dense_norm stored, into their units' counters
//   k_dense_scales  one wave per unit: digits -> fp32 scale (||v||_2 for QSGD, ||v||_1 / k or ||v||_2 / k for Sign)
//   k_dense_norm_one, k_dense_scale_one   in place of those for one segment: a wave's sum formed in registers
//   k_dense_encode  reads v, writes m' = v - g (second worker line) and the packed codes, 8 bytes per coordinate:
//                   a wave owns 1024 consecutive coordinates and with them whole 32-bit words of the code stream
// Part of the single translation unit qsl.hip (included after qsl_encode.h); not a public header.
#pragma once

#include "qsl_device.h"
#include "qsl_layout.h"
#include "qsl_select.h"
#include "qsl_encode.h"

namespace {

constexpr uint32_t DTILE = 4096;             // coordinates per tile: 256 threads x 4 x dwordx4
// Blocks per worker of the first pass, each a contiguous range of tiles.  The pass wants many: without the digits
// (fp32 values, 2 x 25.6 M coordinates) 1024 blocks per worker take 127 us, 2048 121 us, 4096 112 us, 16384 100 us.  With
// that many, adding every block's digits to its unit's counters by atomics costs more than it saves (292 us: additions
// to one address queue up), so a block stores the sums of its first unit as a row of its own and k_dense_sum adds the
// rows up; only what a block meets beyond its first unit (few blocks, if any) goes to the counters directly.
constexpr uint32_t MAX_DENSE_BLOCKS = 16384;
constexpr uint32_t NO_UNIT = 0xFFFFFFFFu;

// digits of |v| (or v^2) straight into a unit's counters in memory (for the few tiles that span several segments)
__device__ __forceinline__ void add_digits_global(uint64_t* acc, uint32_t bits, uint32_t power) {
  const uint32_t ab = bits & 0x7FFFFFFFu;
  const uint32_t ex = ab >> 23, frac = ab & 0x7FFFFFu;
  const uint32_t M = ex ? (frac | 0x800000u) : frac;
  const uint32_t e1 = ex ? ex : 1u;
  if (M == 0) return;
  auto add = [&](uint32_t q, uint64_t x) { if (x) atomicAdd(reinterpret_cast<unsigned long long*>(acc + q), static_cast<unsigned long long>(x)); };
  uint64_t lo, hi;                                         // M^power < 2^96
  power_of_mantissa(M, power, &lo, &hi);
  const uint32_t p = power * (e1 - 1u), q = p >> 5, r = p & 31u;
  const uint64_t a0 = lo << r;
  const uint64_t a1 = (hi << r) | (r ? lo >> (64 - r) : 0);
  add(q, a0 & 0xFFFFFFFFu); add(q + 1, a0 >> 32); add(q + 2, a1 & 0xFFFFFFFFu); add(q + 3, a1 >> 32);
}

// the tiles [t_lo, t_hi) of block b out of nb
__device__ __forceinline__ void dense_range(uint64_t d, uint32_t b, uint32_t nb, uint64_t* t_lo, uint64_t* t_hi) {
  const uint64_t ntiles = (d + DTILE - 1) / DTILE;
  *t_lo = ntiles * b / nb; *t_hi = ntiles * (b + 1) / nb;
}

// With `xm` given, `delta` holds the local models and Delta = xm - delta is formed on the fly (as in k_stream).
template <bool DIFF>
__global__ __launch_bounds__(BLOCK) void k_dense_norm(DevCtx c, const float* m, const float* delta, const float* xm,
                                                      float* m_out) {
  __shared__ uint64_t acc[ACC_ROWS * (ACC_SLOTS + 1)];
  const uint32_t w = blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t power = norm_power(c.quantizer);
  const bool need_norm = c.quantizer != QSL_FP32;
  uint64_t* mine = acc + (wave * 8 + (lane & 7u)) * acc_stride(c.quantizer);
  for (uint32_t i = threadIdx.x; i < ACC_ROWS * acc_stride(c.quantizer); i += BLOCK) acc[i] = 0;
  __syncthreads();
  const uint64_t row = static_cast<uint64_t>(w) * c.d;
  uint64_t t_lo, t_hi;
  dense_range(c.d, blockIdx.x, gridDim.x, &t_lo, &t_hi);
  uint32_t cur = NO_UNIT;                           // the segment whose digits the block's rows hold
  bool nonfinite = false;
  bool own_row = true;                              // nothing stored yet: the next sums go to the block's own row
  const uint64_t nb = gridDim.x;
  // the rows added up: into the block's own row the first time, into the segment's counters after that; then zero again
  // (uniform over the block)
  auto flush = [&]() {
    __syncthreads();
    if (cur != NO_UNIT) {
      uint64_t* ga = c.norm_acc + (static_cast<uint64_t>(w) * c.L + cur) * ACC_SLOTS;
      for (uint32_t s = wave; s < acc_slots(c.quantizer); s += BLOCK / 64) {
        uint64_t x = lane < ACC_ROWS ? acc[lane * acc_stride(c.quantizer) + s] : 0;
        x = wave_sum64(x);
        if (lane == 0) {
          if (own_row) c.dense_part[(static_cast<uint64_t>(w) * ACC_SLOTS + s) * nb + blockIdx.x] = x;
          else if (x) atomicAdd(reinterpret_cast<unsigned long long*>(ga + s), static_cast<unsigned long long>(x));
        }
      }
      if (own_row && threadIdx.x == 0) c.dense_tag[static_cast<uint64_t>(w) * nb + blockIdx.x] = cur;
      own_row = false;
      __syncthreads();
      for (uint32_t i = threadIdx.x; i < ACC_ROWS * acc_stride(c.quantizer); i += BLOCK) acc[i] = 0;
      __syncthreads();
    }
  };
  for (uint64_t tile = t_lo; tile < t_hi; ++tile) {
    const uint64_t base = tile * DTILE;
    f4u v[4];
    // the tile's loads first, then its stores (146 us against 159 us one group of four at a time, 2 x 25.6 M coordinates in
    // 1024 blocks per worker; the next tile's loads issued before this tile's digits are added: no change)
    if (base + DTILE <= c.d) {
      f4u a[4], b[4], x[4];
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint64_t e = base + q * 1024 + threadIdx.x * 4;
        a[q] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(m + row + e));
        b[q] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(delta + row + e));
        if (DIFF) x[q] = *reinterpret_cast<const f4u*>(xm + e);
      }
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint64_t e = base + q * 1024 + threadIdx.x * 4;
        if (DIFF) b[q] = x[q] - b[q];
        v[q] = a[q] + b[q];
        __builtin_nontemporal_store(v[q], reinterpret_cast<f4u*>(m_out + row + e));
      }
    } else {                                        // the row's last, ragged tile
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint64_t e = base + q * 1024 + threadIdx.x * 4;
        v[q] = f4u{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
          if (e + j < c.d) {
            const float dl = DIFF ? xm[e + j] - delta[row + e + j] : delta[row + e + j];
            v[q][j] = m[row + e + j] + dl;
            m_out[row + e + j] = v[q][j];
          }
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) nonfinite |= (__float_as_uint(v[q][j]) & 0x7FFFFFFFu) >= 0x7F800000u;
    }
    if (!need_norm) continue;
    const uint64_t last = min(base + DTILE, c.d) - 1;
    const uint32_t seg_first = c.L == 1 ? 0u : seg_of_coord(c, static_cast<uint32_t>(base));
    const uint32_t seg_last = c.L == 1 ? 0u : seg_of_coord(c, static_cast<uint32_t>(last));
    if (seg_first == seg_last) {
      if (seg_first != cur) { flush(); cur = seg_first; }
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint64_t e = base + q * 1024 + threadIdx.x * 4;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) if (e + j < c.d) add_digits(mine, __float_as_uint(v[q][j]), power);
      }
    } else {                                          // several segments in one tile: each coordinate to its own unit's counters
      flush(); cur = NO_UNIT;
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint64_t e = base + q * 1024 + threadIdx.x * 4;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
          if (e + j < c.d) {
            const uint32_t seg = seg_of_coord(c, static_cast<uint32_t>(e + j));
            add_digits_global(c.norm_acc + (static_cast<uint64_t>(w) * c.L + seg) * ACC_SLOTS, __float_as_uint(v[q][j]), power);
          }
      }
    }
  }
  flush();
  if (own_row && threadIdx.x == 0) c.dense_tag[static_cast<uint64_t>(w) * nb + blockIdx.x] = NO_UNIT;   // no row from this block
  if (__ballot(nonfinite) != 0 && lane == 0) atomicOr(c.status, 1u);
}

// The rows of k_dense_norm's blocks into the counters of their units.  A block takes 512 rows, each of its waves one digit
// (or two, or three): a lane adds up its eight rows' sums of that digit, the wave its lanes', and one lane adds the result
// to the unit's counter -- if the 512 rows belong to one unit, as they nearly always do; else every row goes to its own
// unit's counters.  (A thread per row and a wave-wide sum per digit: 14 us for 2 x 6240 rows; this way 4.5 us.)
constexpr uint32_t SUM_BLOCK = 1024, SUM_ROWS = 512;
__global__ __launch_bounds__(SUM_BLOCK) void k_dense_sum(DevCtx c, uint32_t nb) {
  constexpr uint32_t G = SUM_ROWS / 64;
  const uint32_t w = blockIdx.y, lane = lane_id(), wave = threadIdx.x >> 6;
  const uint32_t r0 = blockIdx.x * SUM_ROWS;
  uint32_t tags[G];
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
    const uint32_t b = r0 + g * 64 + lane;
    tags[g] = b < nb ? c.dense_tag[static_cast<uint64_t>(w) * nb + b] : NO_UNIT;
  }
  uint32_t tag0 = NO_UNIT;                           // the unit of the first row that has one (every wave finds the same)
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
    const uint64_t bal = __ballot(tags[g] != NO_UNIT);
    if (tag0 == NO_UNIT && bal != 0) tag0 = __shfl(tags[g], __ffsll(static_cast<long long>(bal)) - 1, WAVE);
  }
  if (tag0 == NO_UNIT) return;
  bool mixed = false;
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) mixed = mixed || __ballot(tags[g] != NO_UNIT && tags[g] != tag0) != 0;
  for (uint32_t s = wave; s < acc_slots(c.quantizer); s += SUM_BLOCK / 64) {
    uint64_t x[G];
#pragma unroll
    for (uint32_t g = 0; g < G; ++g)
      x[g] = tags[g] != NO_UNIT ? c.dense_part[(static_cast<uint64_t>(w) * ACC_SLOTS + s) * nb + r0 + g * 64 + lane] : 0;
    if (!mixed) {
      uint64_t sum = 0;
#pragma unroll
      for (uint32_t g = 0; g < G; ++g) sum += x[g];
      sum = wave_sum64(sum);
      if (lane == 0 && sum)
        atomicAdd(reinterpret_cast<unsigned long long*>(c.norm_acc + (static_cast<uint64_t>(w) * c.L + tag0) * ACC_SLOTS + s),
                  static_cast<unsigned long long>(sum));
    } else {
#pragma unroll
      for (uint32_t g = 0; g < G; ++g)
        if (x[g]) atomicAdd(reinterpret_cast<unsigned long long*>(c.norm_acc + (static_cast<uint64_t>(w) * c.L + tags[g]) * ACC_SLOTS + s),
                            static_cast<unsigned long long>(x[g]));
    }
  }
}

// The same first pass for one segment, by the streaming pass's recipe: a wave per 1024 coordinates, no LDS and no barrier.  The
// exact sum of a wave's magnitudes (or squares) is formed in registers: every lane adds its 16 as integers counted from
// the lowest exponent of a window of 30 (squares: 32) octaves that ends at the wave's largest, DPP adds the lanes, and five
// lanes add the total's 32-bit digits to one of DENSE_COPIES rows of counters, each counter in a cache line of its own.
// Bits: 24 + 29 + 4 (16 values) + 6 (lanes) = 63; squares 48 + 62 + 4 + 6 = 120 of 128.  Magnitudes below the window, if there
// are any, have a window of their own after it.  2 x 25.6 M coordinates, by LDS digits, barriers and rows per block (k_dense_norm, for
// several segments and for cubes and fourth powers) / this way: magnitudes 108 / 97 us, squares 118 / 99; the sums after it, two
// launches of 4.7 us / one of 5.  3 to 6 waves per SIMD: 98, 97, 98, 98 us.
constexpr uint32_t DENSE_COPIES = 64, DENSE_PITCH = 16;      // rows; 64-bit words from counter to counter

template <uint32_t POWER>
__device__ __forceinline__ void add_wave_digits(uint64_t* row, const f4u (&v)[4]) {
  const uint32_t lane = lane_id();
  uint32_t ab[16], top = 0;
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i) { ab[i] = __float_as_uint(v[i >> 2][i & 3]) & 0x7FFFFFFFu; top = max(top, ab[i]); }
  top = wave_max(top);
  while (top != 0) {                                         // (uniform) a window; at most 10 of them (squares: 9)
    const bool last = top < 2u << 23;                        // exponents 0 and 1: the bits are the mantissa, the unit is the same
    const uint32_t e0 = last ? 1u : max(2u, (top >> 23) - min(top >> 23, POWER == 1 ? 29u : 31u)), low = last ? 1u : e0 << 23;
    uint64_t lo = 0, hi = 0;                                 // the lane's sum is hi * 2^64 + lo
    uint32_t rest = 0;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
      const bool in = ab[i] >= low;
      const uint32_t M = in ? (last ? ab[i] : (ab[i] & 0x7FFFFFu) | 0x800000u) : 0u, e = last ? 0u : (ab[i] >> 23) - e0;
      ab[i] = in ? 0u : ab[i];
      rest = max(rest, ab[i]);
      if (POWER == 1) lo += static_cast<uint64_t>(M) << (e & 63u);
      else {
        const uint64_t sq = static_cast<uint64_t>(M) * M;
        const uint32_t sh = 2u * e & 63u;
        const uint64_t x = sq << sh;
        lo += x;
        hi += (sq >> 1 >> (63u - sh)) + (lo < x ? 1u : 0u);
      }
    }
    if (POWER == 1) lo = wave_sum64(lo);
    else {                                                   // limbs none of which overflows
      const uint64_t s0 = wave_sum64(lo & 0xFFFFFFFFu), s1 = wave_sum64(lo >> 32), s2 = wave_sum64(hi);
      lo = s0 + (s1 << 32);
      hi = s2 + (s1 >> 32) + (lo < s0 ? 1u : 0u);
    }
    const uint32_t p = POWER * (e0 - 1u), q = p >> 5, r = p & 31u;      // bit 0 of the sum is bit p of the digits
    const uint64_t a0 = lo << r, a1 = (hi << r) | (lo >> 1 >> (63u - r));
    const uint32_t digit = lane == 0 ? static_cast<uint32_t>(a0) : lane == 1 ? static_cast<uint32_t>(a0 >> 32) : lane == 2 ? static_cast<uint32_t>(a1)
                         : lane == 3 ? static_cast<uint32_t>(a1 >> 32) : static_cast<uint32_t>(hi >> 1 >> (63u - r));
    if (lane < 5 && digit) atomicAdd(reinterpret_cast<unsigned long long*>(row + (q + lane) * DENSE_PITCH), static_cast<unsigned long long>(digit));
    top = wave_max(rest);
  }
}

template <uint32_t POWER, bool DIFF>      // POWER 0: no norm wanted
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_dense_norm_one(
    DevCtx c, const float* m, const float* delta, const float* xm, float* m_out) {
  const uint32_t w = blockIdx.y, lane = lane_id();
  const uint64_t chunk = static_cast<uint64_t>(blockIdx.x) * (BLOCK / 64) + (threadIdx.x >> 6), base = chunk * CHUNK;
  if (base >= c.d) return;
  const uint32_t valid = static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), c.d - base));
  const uint64_t row = static_cast<uint64_t>(w) * c.d + base;
  const float* mp = m + row;
  const float* dp = delta + row;
  const float* xp = DIFF ? xm + base : nullptr;
  float* op = m_out + row;
  f4u v[4];
  if (valid == CHUNK) {
    f4u a[4], b[4], x[4];
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
      const uint32_t e = t * 256 + lane * 4;
      a[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(mp + e));
      b[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(dp + e));
      if (DIFF) x[t] = *reinterpret_cast<const f4u*>(xp + e);
    }
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
      if (DIFF) b[t] = x[t] - b[t];
      v[t] = a[t] + b[t];
      __builtin_nontemporal_store(v[t], reinterpret_cast<f4u*>(op + t * 256 + lane * 4));
    }
  } else {
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t e = t * 256 + lane * 4 + j;
        float x = 0.0f;
        if (e < valid) {
          const float dl = DIFF ? xp[e] - dp[e] : dp[e];
          x = mp[e] + dl; op[e] = x;
        }
        v[t][j] = x;
      }
    }
  }
  bool nonfinite = false;
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) nonfinite |= (__float_as_uint(v[t][j]) & 0x7FFFFFFFu) >= 0x7F800000u;
  }
  if (__ballot(nonfinite) != 0 && lane == 0) atomicOr(c.status, 1u);
  if (POWER != 0)
    add_wave_digits<POWER>(c.dense_part + (static_cast<uint64_t>(w) * DENSE_COPIES + (static_cast<uint32_t>(chunk) & (DENSE_COPIES - 1))) * (20 * DENSE_PITCH), v);
}

// ... and its rows added up, one block per worker: the scales; the rows back to zero.
__global__ __launch_bounds__(SUM_BLOCK) void k_dense_scale_one(DevCtx c) {
  __shared__ uint64_t acc[20];
  static_assert(DENSE_COPIES == 64, "a row per lane");
  const uint32_t w = blockIdx.x, lane = lane_id(), wave = threadIdx.x >> 6;
  const uint32_t ns = c.quantizer == QSL_FP32 ? 0u : 20u;
  for (uint32_t s = wave; s < ns; s += SUM_BLOCK / 64) {
    uint64_t* p = c.dense_part + ((static_cast<uint64_t>(w) * DENSE_COPIES + lane) * 20 + s) * DENSE_PITCH;
    uint64_t x = *p;
    if (x) *p = 0;
    x = wave_sum64(x);
    if (lane == 0) acc[s] = x;
  }
  __syncthreads();
  if (wave != 0) return;
  const uint32_t k = static_cast<uint32_t>(c.d);
  const UnitScale us = unit_scale(c, ns ? finalize_scale(acc, c.quantizer, k) : 0.0f, k);
  if (lane == 0) {
    UnitState* u = &c.units[w];
    u->scale_code = __float_as_uint(us.scale);
    u->scale_bits = __float_as_uint(us.sent);
    u->cand = 0; u->fell_back = 0; u->tau = 0; u->need = 0; u->n_gt = k; u->nnz = k;
  }
}

// one wave per unit: the scale the codes are computed with and the scale the message carries; the digit counters
// are returned to zero for the next call
__global__ __launch_bounds__(BLOCK) void k_dense_scales(DevCtx c, uint32_t U) {
  const uint32_t u = blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
  if (u >= U) return;
  const uint32_t seg = u % c.L, lane = lane_id();
  const uint32_t kl = c.segs[seg].k;
  const float sc = finalize_scale(c.norm_acc + static_cast<uint64_t>(u) * ACC_SLOTS, c.quantizer, kl);
  if (lane < ACC_SLOTS) c.norm_acc[static_cast<uint64_t>(u) * ACC_SLOTS + lane] = 0;
  if (lane == 0) {
    const UnitScale us = unit_scale(c, sc, kl);
    c.units[u].scale_code = __float_as_uint(us.scale);
    c.units[u].scale_bits = __float_as_uint(us.sent);
    c.units[u].cand = 0; c.units[u].fell_back = 0; c.units[u].tau = 0; c.units[u].need = 0; c.units[u].n_gt = kl; c.units[u].nnz = kl;
  }
}

// The second pass, a wave per 1024 coordinates as in the streaming pass: v is read once more, m' = v - g and the packed codes
// written.  The coordinates of a wave fill whole words of the code stream: sign bits are put together by shuffles, wider
// codes in an LDS line of the wave.  Workers and chunks go from the last to the first: what the first pass wrote last
// may still be in the last-level cache.  2 x 25.6 M coordinates: sign 75 us with 6 waves per SIMD (3: 88, 4: 76, 8: 78; blocks
// of 4096 coordinates with barriers around a shared bit buffer: 94), no quantiser 3; QSGD 92 us with 8 (4: 125, 6: 103; IEEE divisions in
// blocks of 4096: 127), where the vector ALU is the bound: Philox and a quotient per coordinate.  Without the second quotient where no lane
// has a level to send, and with four codes of up to 8 bits put together in 32 bits, a round of 2 x 25.6 M went from 244 to 237 us.
enum { DENSE_SIGN, DENSE_QSGD, DENSE_FP32 };
template <int KIND>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(KIND == DENSE_QSGD ? 8 : KIND == DENSE_SIGN ? 6 : 3, KIND == DENSE_QSGD ? 8 : KIND == DENSE_SIGN ? 6 : 3)))
void k_dense_encode(DevCtx c, float* m_out, uint32_t worker0, uint64_t round, uint8_t* msg, uint64_t* msg_bits, uint32_t* dbg_idx,
                    uint16_t* dbg_level) {
  __shared__ uint32_t s_bits[KIND == DENSE_QSGD ? BLOCK / 64 : 1][KIND == DENSE_QSGD ? 32 * 17 : 1];      // at most 17 bits per code
  const uint32_t w = gridDim.y - 1 - blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t wv = c.w_val;
  uint32_t* words = reinterpret_cast<uint32_t*>(msg + static_cast<uint64_t>(w) * c.cap_words * 4);
  const uint64_t hdr = 1 + static_cast<uint64_t>(c.L);
  const uint64_t code_words = (c.d * wv + 31) / 32;
  if (blockIdx.x == 0) {                               // header: the length word, the scales; the payload bit count; padding
    for (uint64_t i = threadIdx.x; i < hdr; i += BLOCK)
      words[i] = i == 0 ? static_cast<uint32_t>(c.d) : c.units[static_cast<uint64_t>(w) * c.L + (i - 1)].scale_bits;
    for (uint64_t i = hdr + code_words + threadIdx.x; i < c.cap_words; i += BLOCK) words[i] = 0;
    if (threadIdx.x == 0 && msg_bits) msg_bits[w] = hdr * 32 + c.d * wv;
  }
  const uint64_t nchunk = (c.d + CHUNK - 1) / CHUNK, at = static_cast<uint64_t>(blockIdx.x) * (BLOCK / 64) + wave;
  if (at >= nchunk) return;                            // (no barrier follows)
  const uint64_t chunk = nchunk - 1 - at, base = chunk * CHUNK;
  const uint32_t valid = static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), c.d - base));
  const uint32_t seg = c.L == 1 ? 0u : seg_of_coord(c, static_cast<uint32_t>(base));
  const bool one_seg = c.L == 1 || seg == seg_of_coord(c, static_cast<uint32_t>(base + valid - 1));
  const UnitState& us = c.units[static_cast<uint64_t>(w) * c.L + seg];
  const float scale = __uint_as_float(us.scale_code), sent = __uint_as_float(us.scale_bits);      // of the whole chunk, if it is one segment
  float* vp = m_out + static_cast<uint64_t>(w) * c.d + base;
  f4u v[4];
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    v[t] = f4u{0.f, 0.f, 0.f, 0.f};
    if (valid == CHUNK) v[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(vp + e));
    else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) v[t][j] = vp[e + j];
    }
  }
  const float s = static_cast<float>(c.s);
  const RandKey rk1 = make_rand_key(c.seed, worker0 + w, round, 1);
  SharedDivisor by_norm = {}, by_s = {};
  bool quick = false;                                  // divisions by the chunk's norm and by s may take the short way
  if (KIND == DENSE_QSGD) {
    by_norm = shared_divisor(scale); by_s = shared_divisor(s);
    quick = one_seg && by_norm.ok && sent >= 0x1p-40f && sent <= 0x1p60f;
    for (uint32_t i = lane; i < 32 * wv; i += WAVE) s_bits[wave][i] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");      // the line is private to the wave
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  uint32_t sign_word = 0;                              // KIND == DENSE_SIGN: lane l = 8 g + t (t < 4) holds word t * 8 + g of the chunk
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    Words4 rw = {{0u, 0u, 0u, 0u}};
    if (KIND == DENSE_QSGD) rw = rand_words4(rk1, static_cast<uint32_t>(base) + e);             // a multiple of 4: one block
    f4u res = v[t];
    uint32_t code[4], level[4] = {1u, 1u, 1u, 1u};
    bool plain = true;                                 // no coordinate of the wave's that the short division is not made for
    if (KIND == DENSE_QSGD) {
      bool odd = !quick;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) { const float x = fabsf(v[t][j]); odd = odd || (x < by_norm.lo && x > 0.0f) || x > 0x1p100f; }
      plain = __ballot(odd) == 0;
    }
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const float x = v[t][j];
      const bool neg = x < 0.0f;
      float sc = scale, se = sent;
      if (!one_seg && e + j < valid) {
        const UnitState& u = c.units[static_cast<uint64_t>(w) * c.L + seg_of_coord(c, static_cast<uint32_t>(base) + e + j)];
        sc = __uint_as_float(u.scale_code); se = __uint_as_float(u.scale_bits);
      }
      if (KIND == DENSE_QSGD) {                        // Definition 1, example 1: the same single IEEE operations as encode_entry
        float lf = 0.0f;
        if (sc > 0.0f) {
          const float a = plain ? shared_div(fabsf(x), by_norm) : fabsf(x) / sc;
          float tt = a * s;
          if (tt > s) tt = s;
          const float fl = floorf(tt);
          const float frac = tt - fl;
          const float r01 = static_cast<float>(rw.w[j] >> 8) * 0x1p-24f;
          lf = fl + (r01 < frac ? 1.0f : 0.0f);
        }
        level[j] = static_cast<uint32_t>(lf);
        if (__ballot(level[j] != 0) != 0) {            // (uniform) with few levels most of a wave's coordinates send none
          const float prod = se * lf;
          const float mag = plain ? shared_div(prod, by_s) : prod / s;
          const float g = neg ? -mag : mag;
          if (level[j] != 0) res[j] = x - g;           // Algorithm 1, second worker line
        }
        code[j] = level[j] | (static_cast<uint32_t>(neg) << c.w_lev);
      } else if (KIND == DENSE_FP32) {
        res[j] = x - x;
        code[j] = __float_as_uint(x);
      } else {                                         // Definition 2
        res[j] = x - (neg ? -sc : sc);
        code[j] = neg;
      }
      if (e + j < valid) {
        const uint64_t slot = static_cast<uint64_t>(w) * c.K + base + e + j;
        if (dbg_idx) dbg_idx[slot] = static_cast<uint32_t>(base) + e + j;
        if (dbg_level) dbg_level[slot] = static_cast<uint16_t>(level[j]);
      } else code[j] = 0;
    }
    if (valid == CHUNK) __builtin_nontemporal_store(res, reinterpret_cast<f4u*>(vp + e));
    else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) vp[e + j] = res[j];
    }
    if (KIND == DENSE_FP32) {
      if (valid == CHUNK) __builtin_nontemporal_store(u4u{code[0], code[1], code[2], code[3]}, reinterpret_cast<u4u*>(words + hdr + base + e));
      else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) words[hdr + base + e + j] = code[j];
      }
    } else if (KIND == DENSE_SIGN) {
      uint32_t x = (code[0] | code[1] << 1 | code[2] << 2 | code[3] << 3) << (lane & 7u) * 4;
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) x |= __shfl_xor(x, o, WAVE);
      if ((lane & 7u) == t) sign_word = x;
    } else if (wv <= 8) {                              // the lane's four codes in one word, in one or two words of the line
      const uint32_t val = code[0] | code[1] << wv | code[2] << (2 * wv) | code[3] << (3 * wv);
      const uint32_t o = e * wv, word = o >> 5, sh = o & 31u, over = val >> 1 >> (31u - sh);
      if (val << sh) atomicOr(&s_bits[wave][word], val << sh);
      if (over) atomicOr(&s_bits[wave][word + 1], over);
    } else if (wv <= 16) {
      const uint64_t val = static_cast<uint64_t>(code[0]) | (static_cast<uint64_t>(code[1]) << wv) |
                           (static_cast<uint64_t>(code[2]) << (2 * wv)) | (static_cast<uint64_t>(code[3]) << (3 * wv));
      const uint32_t o = e * wv, word = o >> 5, sh = o & 31u;
      const uint64_t lo = val << sh;
      if (static_cast<uint32_t>(lo)) atomicOr(&s_bits[wave][word], static_cast<uint32_t>(lo));
      if (lo >> 32) atomicOr(&s_bits[wave][word + 1], static_cast<uint32_t>(lo >> 32));
      if (sh && (val >> (64 - sh))) atomicOr(&s_bits[wave][word + 2], static_cast<uint32_t>(val >> (64 - sh)));
    } else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t o = (e + j) * wv, word = o >> 5, sh = o & 31u;
        const uint64_t lo = static_cast<uint64_t>(code[j]) << sh;
        if (static_cast<uint32_t>(lo)) atomicOr(&s_bits[wave][word], static_cast<uint32_t>(lo));
        if (lo >> 32) atomicOr(&s_bits[wave][word + 1], static_cast<uint32_t>(lo >> 32));
      }
    }
  }
  const uint64_t w0 = chunk * (CHUNK / 32) * wv;       // the chunk's first word of the code stream
  if (KIND == DENSE_SIGN) {
    const uint64_t q = w0 + (lane & 7u) * 8 + (lane >> 3);
    if ((lane & 7u) < 4 && q < code_words) words[hdr + q] = sign_word;
  } else if (KIND == DENSE_QSGD) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t i = lane; i < 32 * wv; i += WAVE) if (w0 + i < code_words) words[hdr + w0 + i] = s_bits[wave][i];
  }
}

}  // namespace
