// qsl_whole.h -- A short vector that is one segment: the whole of qsl_compress in one launch, a block of 1024 threads per worker.
// v = m + Delta (Algorithm 1, first worker line) stays in registers; exact selection (Section 2.2), norm, QSGD levels or signs
// (Definitions 1 and 2), error update (second worker line) and the packed message follow behind barriers.
// Part of the single translation unit qsl.hip (included after qsl_lean.h); not a public header.
#pragma once

#include "qsl_device.h"
#include "qsl_layout.h"
#include "qsl_select.h"
#include "qsl_encode.h"
#include "qsl_lean.h"

namespace {

constexpr uint32_t WHOLE_MAX = 16384;      // coordinates: 16 per thread (32: the compiler spills)
constexpr uint32_t WHOLE_K = 4096;         // selected ones: their list lies in LDS
constexpr uint32_t WHOLE_GROUPS_K = 512;   // k up to which 1024 groups' maxima give a guess
constexpr uint32_t WHOLE_LIST = 256;       // candidates that are ranked one against the other instead of going through (further) digits

// fields [0, n) of `width` bits each, from LDS, into the words that hold them (all of them the block's)
__device__ __forceinline__ void write_fields(uint32_t* words, const uint32_t* s_val, uint32_t n, uint32_t width) {
  const uint32_t total = n * width, nw = (total + 31) / 32;               // < 2^32: at most 4096 fields of 32 bits
  for (uint32_t q = threadIdx.x; q < nw; q += BIG) {
    uint32_t e = q * 32 / width, out = 0;
    int32_t sh = static_cast<int32_t>(e * width) - static_cast<int32_t>(q * 32);      // <= 0
    for (; sh < 32 && e < n; ++e, sh += static_cast<int32_t>(width)) out |= sh >= 0 ? s_val[e] << sh : s_val[e] >> -sh;
    words[q] = out;
  }
}

// PER: groups of four coordinates per thread.  Wave w owns the coordinates [w * 256 * PER, (w + 1) * 256 * PER), lane l of it those from
// t * 256 + l * 4 on, t < PER.
// Top_k with k at most half the number of threads (of groups of four coordinates): the k-th largest of the groups' maxima can't lie
// above the k-th largest key, so what is below the histogram bin it falls in is left out; if that leaves more than WHOLE_K
// candidates (ties), nothing is.
// What bounds it is the chain of memory and LDS round trips between some twenty barriers.  15 workers of 7,850 coordinates, k = 40, QSGD:
// 26,500 cycles (reading v 4,900, the guess 5,600, ranking 3,700, list and norm 7,000, codes 2,200, message 3,000), 11 us, where
// the kernels for longer vectors took 28 in three launches; a call by itself 27.0 -> 14.6 us; 8 x 4,000, k = 1,000: 49 -> 12 us; 8 x
// 16,001, k = 1,000: 59 -> 22 us; 8 x 12,011, k = 60, sign: 23.4 -> 19.8 us.
template <int SPARS, uint32_t PER>
__global__ __launch_bounds__(BIG) void k_whole(DevCtx c, SegInfo sg, const float* m, const float* delta, const float* xm, float* m_out,
                                               uint32_t worker0, uint64_t round, uint8_t* msg, uint64_t* msg_bits, uint32_t* dbg_idx,
                                               uint16_t* dbg_level) {
  __shared__ uint32_t lh[HBINS];
  __shared__ uint64_t acc[LEAN_ROWS * (ACC_SLOTS + 1)];
  __shared__ uint64_t scratch[17];
  __shared__ uint32_t s_idx[WHOLE_K], s_code[WHOLE_K];
  __shared__ uint64_t s_list[WHOLE_LIST];               // key << 32 | ~coordinate: a larger one ranks before
  __shared__ uint32_t result[6], s_wt[16 * PER], s_nlist, s_tau, s_tie, s_need;
  __shared__ float s_scale;
  const uint32_t w = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  const uint32_t n = static_cast<uint32_t>(sg.size), k = sg.k, e0 = wave * (256 * PER) + lane * 4;
  const uint64_t row = static_cast<uint64_t>(w) * c.d;
  const uint32_t st = acc_stride(c.quantizer), ns = acc_slots(c.quantizer), power = norm_power(c.quantizer);
  const bool need_norm = c.quantizer != QSL_FP32;
  f4u v[PER];
  {
    f4u a[PER], b[PER], x[PER];
    const float* mp = m + row;
    const float* dp = delta + row;
#pragma unroll
    for (uint32_t t = 0; t < PER; ++t) {
      const uint32_t e = e0 + t * 256;
      a[t] = b[t] = x[t] = f4u{0.f, 0.f, 0.f, 0.f};
      if (e + 4 <= n) {
        a[t] = *reinterpret_cast<const f4u*>(mp + e);
        b[t] = *reinterpret_cast<const f4u*>(dp + e);
        if (xm != nullptr) x[t] = *reinterpret_cast<const f4u*>(xm + e);
      } else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) if (e + j < n) { a[t][j] = mp[e + j]; b[t][j] = dp[e + j]; if (xm != nullptr) x[t][j] = xm[e + j]; }
      }
    }
    for (uint32_t i = threadIdx.x; i < HBINS; i += BIG) lh[i] = 0;
    for (uint32_t i = threadIdx.x; i < LEAN_ROWS * st; i += BIG) acc[i] = 0;
    if (threadIdx.x == 0) { s_nlist = 0; s_tau = 0; s_tie = 0; s_need = 0; s_scale = 0.0f; }
    float* op = m_out + row;
    bool nonfinite = false;
#pragma unroll
    for (uint32_t t = 0; t < PER; ++t) {
      const uint32_t e = e0 + t * 256;
      if (xm != nullptr) b[t] = x[t] - b[t];
      v[t] = a[t] + b[t];
      if (e + 4 <= n) *reinterpret_cast<f4u*>(op + e) = v[t];
      else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) { if (e + j < n) op[e + j] = v[t][j]; else v[t][j] = 0.0f; }
      }
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) nonfinite |= (__float_as_uint(v[t][j]) & 0x7FFFFFFFu) >= 0x7F800000u;
    }
    if (__ballot(nonfinite) != 0 && lane == 0) atomicOr(c.status, 1u);
  }
  // the rank keys; a place behind the vector's end is no coordinate
  const RandKey rk = make_rand_key(c.seed, worker0 + w, round, 0), rk1 = make_rand_key(c.seed, worker0 + w, round, 1);
  uint32_t key[4 * PER], inside = 0, top[PER];
#pragma unroll
  for (uint32_t t = 0; t < PER; ++t) {
    Words4 rw = {{0u, 0u, 0u, 0u}};
    if (SPARS == QSL_RANDK && e0 + t * 256 < n) rw = rand_words4(rk, e0 + t * 256);
    top[t] = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const bool in = e0 + t * 256 + j < n;
      key[t * 4 + j] = SPARS == QSL_TOPK ? key_of_value(__float_as_uint(v[t][j])) : rw.w[j];
      inside |= (in ? 1u : 0u) << (t * 4 + j);
      if (in) top[t] = max(top[t], key[t * 4 + j]);
    }
  }
  // the coordinates with a key in [T, end): how many, and as many of them as there is room for in the list
  auto collect = [&](uint32_t T, uint64_t end) {
    uint32_t mask = 0, total;
#pragma unroll
    for (uint32_t i = 0; i < 4 * PER; ++i) mask |= (((inside >> i) & 1u) && key[i] >= T && key[i] < end ? 1u : 0u) << i;
    const uint32_t before = wave_exclusive_scan32(__popc(mask), &total);
    uint32_t at = 0;
    if (total) {                                             // (uniform over the wave)
      if (lane == 0) at = atomicAdd(&s_nlist, total);
      at = lane_value(at, 0) + before;
#pragma unroll
      for (uint32_t i = 0; i < 4 * PER; ++i)
        if ((mask >> i) & 1u) {
          if (at < WHOLE_LIST) s_list[at] = static_cast<uint64_t>(key[i]) << 32 | (0xFFFFFFFFu - (e0 + (i >> 2) * 256 + (i & 3u)));
          ++at;
        }
    }
    __syncthreads();
  };
  __syncthreads();
  const bool all = k == n;                                   // (uniform)
  const bool guess = SPARS == QSL_TOPK && !all && k <= WHOLE_GROUPS_K * PER;
  uint32_t T = 0, cand = n, above, failed = 0;
  if (guess) {
    if (k <= WHOLE_GROUPS_K) {                               // a group per thread, else one per four coordinates
#pragma unroll
      for (uint32_t t = 1; t < PER; ++t) top[0] = max(top[0], top[t]);
      if (inside) atomicAdd(&lh[top[0] >> 20], 1u);
    } else {
#pragma unroll
      for (uint32_t t = 0; t < PER; ++t) if ((inside >> (t * 4)) & 1u) atomicAdd(&lh[top[t] >> 20], 1u);
    }
    __syncthreads();
    T = find_from_top<BIG>(lh, k, &above, scratch, result, true) << 20;     // fewer than k groups: bin 0
    collect(T, 1ull << 32);
    cand = s_nlist;
    if (cand > WHOLE_K) { failed = 1; T = 0; }
  }
  uint32_t tau = 0, tie = 0xFFFFFFFFu;                       // selected: key > tau, or key == tau and coordinate <= tie
  bool ranked = false;
  if (!all) {
    uint32_t prefix = 0, k_rem = k;
    auto count = [&](auto&& bin_of) {
#pragma unroll
      for (uint32_t i = 0; i < 4 * PER; ++i) {
        uint32_t bin;
        if (((inside >> i) & 1u) && key[i] >= T && bin_of(key[i], &bin)) atomicAdd(&lh[bin], 1u);
      }
      __syncthreads();
    };
    ranked = guess && cand <= WHOLE_LIST;                    // few candidates: ranked by (key descending, coordinate ascending)
    if (!ranked) {
      if (guess) { __syncthreads(); if (threadIdx.x == 0) s_nlist = 0; }      // (everyone has read it)
      count([&](uint32_t x, uint32_t* bin) { return level_bin<0>(x, 0, bin); });
      find2_from_top<BIG>(lh, k, k, scratch, result, true);
      prefix = result[0] << 20; k_rem = k - result[1];
      ranked = result[4] <= WHOLE_LIST;                      // ... or few in the threshold's bin
      if (ranked) {
        collect(prefix, static_cast<uint64_t>(prefix) + (1u << 20));
      }
    }
    if (ranked) {
      constexpr uint32_t SUB = BIG / WHOLE_LIST;             // lanes per entry
      const uint32_t nl = s_nlist, sub = threadIdx.x % SUB, me = threadIdx.x / SUB;
      if (wave * (64 / SUB) < nl) {                          // (uniform over the wave)
        const uint64_t x = s_list[min(me, nl - 1)];
        uint32_t rank = 0;
        for (uint32_t j = 0; j < nl; j += 4 * SUB) {         // four reads in flight
          uint64_t o[4];
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) o[i] = s_list[min(j + i * SUB + sub, WHOLE_LIST - 1)];
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) rank += j + i * SUB + sub < nl && o[i] > x ? 1u : 0u;
        }
#pragma unroll
        for (int o = SUB / 2; o > 0; o >>= 1) rank += __shfl_xor(rank, o, WAVE);
        if (sub == 0 && me < nl && rank == k_rem - 1) { s_tau = static_cast<uint32_t>(x >> 32); s_tie = 0xFFFFFFFFu - static_cast<uint32_t>(x); }
      }
      __syncthreads();
      tau = s_tau; tie = s_tie;
    } else {
      count([&](uint32_t x, uint32_t* bin) { return level_bin<1>(x, prefix, bin); });
      uint32_t bin = find_from_top<BIG>(lh, k_rem, &above, scratch, result, true);
      prefix |= bin << 8; k_rem -= above;
      count([&](uint32_t x, uint32_t* bin2) { return level_bin<2>(x, prefix, bin2); });
      bin = find_from_top<BIG, 1024>(lh, k_rem, &above, scratch, result, false);      // bins 256 .. 1023 are empty
      tau = prefix | bin; k_rem -= above;                    // k_rem ties are kept, the first ones
      // the last of them: ties counted in coordinate order, wave after wave
      uint32_t qn = 0;
#pragma unroll
      for (uint32_t i = 0; i < 4 * PER; ++i) qn += ((inside >> i) & 1u) && key[i] == tau ? 1u : 0u;
      const uint32_t tot = wave_sum(qn);
      if (lane == 0) s_wt[wave] = tot;
      __syncthreads();
      uint32_t run = 0;
      for (uint32_t i = 0; i < wave; ++i) run += s_wt[i];
#pragma unroll
      for (uint32_t t = 0; t < PER; ++t) {
        uint32_t q = 0, total;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) q += ((inside >> (t * 4 + j)) & 1u) && key[t * 4 + j] == tau ? 1u : 0u;
        uint32_t r = run + wave_exclusive_scan32(q, &total);
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
          if (((inside >> (t * 4 + j)) & 1u) && key[t * 4 + j] == tau && ++r == k_rem) s_tie = e0 + t * 256 + j;
        run += total;
      }
      __syncthreads();
      tie = s_tie;
    }
  }
  // the selected ones in coordinate order (wave, t, lane, j)
  uint32_t gm = 0, nt = 0;
#pragma unroll
  for (uint32_t i = 0; i < 4 * PER; ++i) {
    const bool eq = key[i] == tau;
    const bool take = ((inside >> i) & 1u) && (all || key[i] > tau || (eq && e0 + (i >> 2) * 256 + (i & 3u) <= tie));
    gm |= (take ? 1u : 0u) << i;
    nt += take && !all && eq ? 1u : 0u;
  }
  uint32_t pre[PER];
#pragma unroll
  for (uint32_t t = 0; t < PER; ++t) {
    uint32_t tot;
    pre[t] = wave_exclusive_scan32(__popc((gm >> (t * 4)) & 0xFu), &tot);
    if (lane == 0) s_wt[wave * PER + t] = tot;
  }
  if (__ballot(nt != 0) != 0) { nt = wave_sum(nt); if (lane == 0) atomicAdd(&s_need, nt); }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // v is in m_out: the transmitted coordinates are written again below
  __syncthreads();
  uint32_t base = 0;                                         // selected ones before the wave's
  {
    uint32_t x = 0;
    for (uint32_t i = lane; i < wave * PER; i += WAVE) x += s_wt[i];
    base = wave_sum(x);
  }
#pragma unroll
  for (uint32_t t = 0; t < PER; ++t) {
    uint32_t pos = base + pre[t];
    const uint32_t nib = (gm >> (t * 4)) & 0xFu;
    if (nib) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if ((nib >> j) & 1u) {
          if (pos < k) { s_idx[pos] = e0 + t * 256 + j; s_code[pos] = __float_as_uint(v[t][j]); }
          ++pos;
        }
    }
    base += s_wt[wave * PER + t];
  }
  __syncthreads();
  if (need_norm) {                                           // the digits, their rows added up (a row per lane), then the scale
    uint64_t* mine = acc + ((wave & 7u) * 8 + (lane & 7u)) * st;
    for (uint32_t j = threadIdx.x; j < k; j += BIG) add_digits(mine, s_code[j], power);
    __syncthreads();
    constexpr uint32_t PW = (ACC_SLOTS + 15) / 16;
    uint64_t x[PW];
#pragma unroll
    for (uint32_t i = 0; i < PW; ++i) {
      const uint32_t s = wave + i * 16;
      x[i] = 0;
      if (s < ns) x[i] = wave_sum64(acc[lane * st + s]);
    }
    __syncthreads();
    if (lane == 0) {
#pragma unroll
      for (uint32_t i = 0; i < PW; ++i) if (wave + i * 16 < ns) acc[wave + i * 16] = x[i];
    }
    __syncthreads();
    if (wave == 0) {
      const float sc = finalize_scale(acc, c.quantizer, k);
      if (lane == 0) s_scale = sc;
    }
    __syncthreads();
  }
  const UnitScale usc = unit_scale(c, s_scale, k);
  // codes, error update; QSGD: the transmitted entries move up to where they stand in the message
  const bool qsgd = is_qsgd(c.quantizer);
  uint32_t nnz = 0;
  for (uint32_t j0 = 0; j0 < k; j0 += BIG) {
    const uint32_t j = j0 + threadIdx.x;
    uint32_t idx = 0, code = 0;
    bool sent = false;
    if (j < k) {
      idx = s_idx[j];
      sent = encode_value(c, static_cast<uint64_t>(w) * c.K + j, idx, s_code[j], usc, rk1, dbg_idx, dbg_level, m_out + row, &code);
    }
    if (!qsgd) { if (j < k) s_code[j] = code; continue; }
    const uint64_t bal = __ballot(sent);
    if (lane == 0) s_wt[wave] = static_cast<uint32_t>(__popcll(bal));
    __syncthreads();                                         // ... and every entry of this step has been read
    const uint32_t cnt = lane < 16 ? s_wt[lane] : 0u;
    const uint32_t inc = wave_inclusive_scan32(cnt);
    const uint32_t at = nnz + (wave ? lane_value(inc, wave - 1) : 0u) + popc_below(bal);
    if (sent) { s_idx[at] = idx; s_code[at] = code; }
    nnz += lane_value(inc, 15);
    __syncthreads();
  }
  if (!qsgd) { nnz = k; __syncthreads(); }
  uint32_t* words = reinterpret_cast<uint32_t*>(msg + static_cast<uint64_t>(w) * c.cap_words * 4);
  const uint32_t idx_words = (nnz * c.w_idx + 31) / 32, code_words = (nnz * c.w_val + 31) / 32;
  write_fields(words + 2, s_idx, nnz, c.w_idx);
  write_fields(words + 2 + idx_words, s_code, nnz, c.w_val);
  for (uint32_t q = 2 + idx_words + code_words + threadIdx.x; q < c.cap_words; q += BIG) words[q] = 0;
  if (threadIdx.x == 0) {
    words[0] = nnz; words[1] = __float_as_uint(usc.sent);
    if (msg_bits) msg_bits[w] = 64 + static_cast<uint64_t>(nnz) * (c.w_idx + c.w_val);
    UnitState* us = &c.units[w];
    us->cand = cand; us->fell_back = failed; us->tau = tau; us->need = s_need; us->n_gt = k - s_need; us->scale_bits = __float_as_uint(usc.sent);
    us->nnz = nnz; us->T_used = T;
  }
}

}  // namespace
