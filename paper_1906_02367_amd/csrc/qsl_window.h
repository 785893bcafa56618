// qsl_window.h -- A dense k on the whole vector (one segment, more than 40,960 coordinates, too many selected ones for the
// guessing path): a window of rank keys that holds the k-th largest one.  Coordinates above the window are selected for
// certain, those below it are not, and only the window's -- a per cent or two -- are looked at more than once:
//   k_win_sample, k_win_scan  Top_k: the window, as two quantiles of a sample of m + Delta (Rand_k: analytic)
//   k_win_stream  v = m + Delta; per chunk the number of coordinates above the window, the window's coordinates into the
//                 chunk's slot, the exact digits of the norm of those above (a row of sums per block)
//   k_win_hist    histogram of the window's keys
//   k_win_mark    the bin of the k-th largest key; digits and numbers of the selected ones above it; those inside to a list
//   k_win_mid     the exact threshold and the last tie that is kept, the scale, where every chunk's entries begin
//   k_win_apply   reads v once more: selected entries in order to the message's arrays, m' = v - g (Algorithm 1, second
//                 worker line) written chunk by chunk
// v is read twice in all (20 bytes per coordinate with the streaming pass), where the multi-pass kernels read it six times
// and update it by scattered words.  If the window did not hold the threshold, held too much (ties, zeros) or its bin holds
// more than the list takes, the unit is left to the multi-pass kernels, whose launches stand by (they end at once otherwise);
// the host hears of it and leaves the window out of the next calls (WindowPolicy in qsl_policy.h).
// Part of the single translation unit qsl.hip (included after qsl_lean.h); not a public header.
#pragma once

#include "qsl_device.h"
#include "qsl_layout.h"
#include "qsl_select.h"
#include "qsl_encode.h"
#include "qsl_lean.h"

namespace {

constexpr uint32_t WBINS = 16384;          // bins of the sample: 1/64 of a binade each
constexpr uint32_t WSHIFT = 18;            // key bits below a bin
constexpr uint32_t WCOPIES = 4;            // copies of the sample's histogram that a worker's blocks spread over
constexpr uint32_t WRUN = 16;              // consecutive coordinates per sample run (64 bytes)

// Of one worker, and what the window's kernels have for scratch (apart from DevCtx, which goes into every launch).
struct WinState {
  uint32_t lo, hi, sh;       // the window [lo, hi) of rank keys and the width 2^sh of its bins (k_win_scan; Rand_k: static)
  uint32_t above;            // coordinates above the window (k_win_hist)
  uint32_t tie;              // the last coordinate of the threshold's key that is selected (k_win_mid)
};
struct WinCtx {
  WinState* state;           // [R]
  uint32_t* sample;          // [R][WCOPIES][WBINS] histogram of the sample, in copies; all zero between calls
  uint32_t* hist;            // [R][HBINS] histogram of the window's keys; all zero between calls
  uint64_t* part;            // [R][blocks of k_win_stream][acc_slots] digit sums of the coordinates above the window
  uint4* list;               // [R][WLIST] (coordinate, value bits, key, -) of the window's candidates in the threshold's bin
  uint32_t* off;             // [R][NWT] selected coordinates before every chunk
};

// ------------------------------------------------------------------------------------------------
// the window of Top_k
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(BIG) void k_win_sample(DevCtx c, WinCtx wc, SegInfo sg, const float* m, const float* delta, const float* xm,
                                                    uint32_t R) {
  __shared__ uint32_t lh[WBINS];
  const uint32_t j = blockIdx.x / R, w = blockIdx.x % R;
  const uint64_t row = static_cast<uint64_t>(w) * c.d;
  const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t nwaves = sg.nsamp * (BIG / 64), gw = j * (BIG / 64) + wave;
  constexpr uint32_t UN = 8, PER = WAVE / WRUN;            // steps in flight, runs per step of a wave
  for (uint32_t i = threadIdx.x; i < WBINS; i += BIG) lh[i] = 0;
  __syncthreads();
  for (uint32_t q0 = gw * PER; q0 < sg.n_runs; q0 += UN * nwaves * PER) {
    float a[UN], b[UN]; bool ok[UN];
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      const uint32_t q = q0 + u * nwaves * PER + lane / WRUN;
      const uint64_t pos = static_cast<uint64_t>(q) * sg.samp_stride + lane % WRUN;
      ok[u] = q < sg.n_runs && pos < sg.size;
      a[u] = ok[u] ? m[row + pos] : 0.f;
      b[u] = ok[u] ? delta[row + pos] : 0.f;
      if (xm != nullptr && ok[u]) b[u] = xm[pos] - b[u];
    }
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u)
      if (ok[u]) atomicAdd(&lh[key_of_value(__float_as_uint(a[u] + b[u])) >> WSHIFT], 1u);
  }
  __syncthreads();
  uint32_t* gh = wc.sample + (static_cast<uint64_t>(w) * WCOPIES + j % WCOPIES) * WBINS;
  for (uint32_t i = threadIdx.x; i < WBINS; i += BIG) { const uint32_t x = lh[i]; if (x) atomicAdd(&gh[i], x); }
}

// the window from the sample's ranks r_tau (above the threshold) and r_s (below it); the histogram back to zero
__global__ __launch_bounds__(BIG) void k_win_scan(WinCtx wc, SegInfo sg) {
  __shared__ uint64_t scratch[17];
  __shared__ uint32_t s_bin[2], s_cum[2];
  constexpr uint32_t PER = WBINS / BIG;
  const uint32_t w = blockIdx.x, t = threadIdx.x;
  uint32_t* gh = wc.sample + static_cast<uint64_t>(w) * WCOPIES * WBINS;
  uint32_t h[PER], sum = 0;
  const uint32_t low = WBINS - PER * (t + 1);              // thread t's bins: PER below those of the threads before it
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) h[i] = 0;
#pragma unroll
  for (uint32_t i = 0; i < PER; i += 4) {
#pragma unroll
    for (uint32_t cp = 0; cp < WCOPIES; ++cp) {
      const uint4 x = *reinterpret_cast<const uint4*>(gh + cp * WBINS + low + i);
      h[i] += x.x; h[i + 1] += x.y; h[i + 2] += x.z; h[i + 3] += x.w;
    }
    sum += h[i] + h[i + 1] + h[i + 2] + h[i + 3];
  }
  if (t == 0) { s_bin[0] = 0; s_bin[1] = 0; s_cum[0] = 0; s_cum[1] = 0xFFFFFFFFu; }
  uint64_t total;
  const uint64_t before = block_exclusive_scan64(sum, scratch, &total);
#pragma unroll
  for (uint32_t which = 0; which < 2; ++which) {
    const uint32_t target = which ? sg.r_s : sg.r_tau;
    if (before < target && before + sum >= target) {
      uint64_t cum = before;
#pragma unroll
      for (uint32_t i = PER; i-- > 0;) {
        // s_cum: the sample's coordinates above the window, and those above its lower end
        if (cum + h[i] >= target) { s_bin[which] = low + i; s_cum[which] = static_cast<uint32_t>(which ? cum + h[i] : cum); break; }
        cum += h[i];
      }
    }
  }
  if (sum) {
#pragma unroll
    for (uint32_t i = 0; i < PER; i += 4) {
#pragma unroll
      for (uint32_t cp = 0; cp < WCOPIES; ++cp) *reinterpret_cast<uint4*>(gh + cp * WBINS + low + i) = make_uint4(0, 0, 0, 0);
    }
  }
  __syncthreads();
  if (t == 0) {
    WinState* ws = &wc.state[w];
    const uint32_t lo = s_bin[1] << WSHIFT;
    const uint32_t hi = sg.r_tau == 0 || s_bin[0] == WBINS - 1 ? 0xFFFFFFFFu : (s_bin[0] + 1) << WSHIFT;
    // An eighth of the sample or more inside: ties, or more places than there are non-zero coordinates.  No pool would take
    // what such a window holds; it is closed, so that the streaming pass lists nothing (k_win_hist sees that it failed).
    const uint32_t inside = static_cast<uint32_t>(min<uint64_t>(s_cum[1], total)) - s_cum[0];
    const bool closed = static_cast<uint64_t>(inside) * 8 >= total;
    uint32_t sh = 0;
    while (((hi - 1 - lo) >> sh) >= HBINS) ++sh;
    ws->lo = closed ? 0xFFFFFFFFu : lo; ws->hi = closed ? 0xFFFFFFFFu : hi; ws->sh = sh;
  }
}

// ------------------------------------------------------------------------------------------------
// the streaming pass (k_stream's recipe; slots as there, the header's upper half holding the number above the window)
// A block waits for its slowest wave twice (zeroed digit rows, finished rows) and works a while between its loads and its
// end, so it wants more waves in flight than k_stream does: 3 waves per SIMD 273 us, 4: 226, 5: 212, 6: 206, 8: 207 on 4 x
// 25.6 M coordinates with k = d / 10.
// ------------------------------------------------------------------------------------------------
template <int SPARS, bool DIFF>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(6, 6))) void k_win_stream(
    DevCtx c, WinCtx wc, StreamSeg sg, const float* m, const float* delta, const float* xm, float* m_out, uint32_t worker0, uint64_t round,
    uint32_t R, uint32_t* msg_zero) {
  __shared__ uint2 s_stage[BLOCK / 64][64];
  __shared__ uint32_t s_stage_key[SPARS == QSL_RANDK ? BLOCK / 64 : 1][64];
  __shared__ uint64_t acc[ACC_ROWS * (ACC_SLOTS + 1)];
  const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
  uint32_t blk = blockIdx.x, w = blockIdx.y;
  if (DIFF) {
    const uint32_t slot = blockIdx.x >> 3;
    w = slot % R;
    blk = (slot / R) * 8 + (blockIdx.x & 7u);
    if (blk * 4 >= c.NWT) return;                           // (uniform over the block)
  }
  const uint32_t chunk = blk * 4 + wave;
  const bool here = chunk < c.NWT;                          // a wave past the end only takes part in the barriers
  const uint32_t lo = wc.state[w].lo, hi = wc.state[w].hi;
  const uint64_t first = static_cast<uint64_t>(chunk) * CHUNK;
  const uint32_t valid = here ? static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), sg.size - first)) : 0u;
  const uint64_t row = static_cast<uint64_t>(w) * c.d + first;
  const float* mp = m + row;
  const float* dp = delta + row;
  const float* xp = DIFF ? xm + first : nullptr;
  float* op = m_out + row;
  f4u v[4];
  if (valid == CHUNK) {
    f4u a[4], b[4], x[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t e = t * 256 + lane * 4;
      a[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(mp + e));
      b[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(dp + e));
      if (DIFF) x[t] = *reinterpret_cast<const f4u*>(xp + e);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (DIFF) b[t] = x[t] - b[t];
      v[t] = a[t] + b[t];
      __builtin_nontemporal_store(v[t], reinterpret_cast<f4u*>(op + t * 256 + lane * 4));
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
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
  const uint32_t power = norm_power(c.quantizer), st = acc_stride(c.quantizer);
  const bool need_norm = c.quantizer != QSL_FP32;
  for (uint32_t i = threadIdx.x; i < ACC_ROWS * st; i += BLOCK) acc[i] = 0;
  __syncthreads();
  bool nonfinite = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) nonfinite |= (__float_as_uint(v[t][j]) & 0x7FFFFFFFu) >= 0x7F800000u;
  }
  if (__ballot(nonfinite) != 0 && lane == 0) atomicOr(c.status, 1u);
  if (msg_zero != nullptr && here && chunk < (c.cap_words + 63u) / 64u)
    for (uint64_t q = static_cast<uint64_t>(chunk) * 64 + lane; q < c.cap_words; q += static_cast<uint64_t>(c.NWT) * 64)
      msg_zero[static_cast<uint64_t>(w) * c.cap_words + q] = 0;

  const RandKey rk = make_rand_key(c.seed, worker0 + w, round, 0);
  uint64_t* mine = acc + (wave * 8 + (lane & 7u)) * st;
  uint32_t pm = 0, n_above = 0;                             // bit t*4+j: coordinate (t, j) lies in the window; how many lie above
  Words4 rws[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    Words4 rw;
    if (SPARS == QSL_RANDK) { rw = rand_words4(rk, static_cast<uint32_t>(first + t * 256 + lane * 4)); rws[t] = rw; }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t bits = __float_as_uint(v[t][j]);
      const uint32_t key = SPARS == QSL_TOPK ? key_of_value(bits) : rw.w[j];
      const bool inside = static_cast<uint32_t>(t * 256 + lane * 4 + j) < valid;
      const bool above = inside && key >= hi;
      pm |= (inside && key >= lo && !above ? 1u : 0u) << (t * 4 + j);
      n_above += above;
      if (above && need_norm) add_digits(mine, bits, power);
    }
  }
  n_above = wave_sum(n_above);
  const uint32_t cap = sg.lpc * 2 - 1;
  uint2* stage = s_stage[wave];
  uint32_t total = 0, ovf_at = 0;
  uint32_t* ctr = c.ctr + static_cast<uint64_t>(w) * (CTR_LINES * PAD);
  if (__ballot(pm != 0) != 0) {
    uint32_t before[4], tot[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      before[t] = 0; tot[t] = 0;
      const uint32_t nib = (pm >> (t * 4)) & 0xFu;
      if (__ballot(nib != 0) == 0) continue;                // wave-uniform
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t bal = __ballot((nib >> j) & 1u);
        before[t] += popc_below(bal);
        tot[t] += __popcll(bal);
      }
    }
    total = tot[0] + tot[1] + tot[2] + tot[3];
    uint2* dst = stage + 1;
    uint32_t* dst_key = SPARS == QSL_RANDK ? s_stage_key[wave] + 1 : nullptr;
    bool write = true;
    if (total > cap) {                                      // wave-uniform: the slot cannot hold this chunk
      if (lane == 0) {
        ovf_at = atomicAdd(&ctr[CTR_OVF * PAD], total);
        if (ovf_at > sg.ovf_cap || total > sg.ovf_cap - ovf_at) { atomicOr(&ctr[CTR_FAIL * PAD], 1u); ovf_at = 0xFFFFFFFFu; }
      }
      ovf_at = __shfl(ovf_at, 0, WAVE);
      write = ovf_at != 0xFFFFFFFFu;
      dst = c.ovf + static_cast<uint64_t>(w) * c.ovf_stride + ovf_at;
      if (SPARS == QSL_RANDK) dst_key = c.ovf_key + static_cast<uint64_t>(w) * c.ovf_stride + ovf_at;
    }
    if (write) {
      uint32_t base = 0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint32_t nib = (pm >> (t * 4)) & 0xFu;
        uint32_t pos = base + before[t];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if ((nib >> j) & 1u) {
            if (SPARS == QSL_RANDK) dst_key[pos] = rws[t].w[j];
            dst[pos++] = make_uint2(static_cast<uint32_t>(first + t * 256 + lane * 4 + j), __float_as_uint(v[t][j]));
          }
        }
        base += tot[t];
      }
    }
  }
  if (lane == 0) {
    stage[0] = make_uint2(total | n_above << 16, ovf_at);
    if (total | n_above)                                     // window in the low half, above it in the high half; nobody waits
      atomicAdd(reinterpret_cast<unsigned long long*>(&ctr[(chunk & (NSUB - 1)) * PAD]),
                static_cast<unsigned long long>(n_above) << 32 | total);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the staging line is private to the wave
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (here && lane < sg.lpc * 2) {
    const uint2 e = stage[lane];
    const u2v ev = {e.x, e.y};
    const uint64_t at = static_cast<uint64_t>(w) * c.slot_stride + static_cast<uint64_t>(chunk) * (sg.lpc * 2);
    __builtin_nontemporal_store(ev, reinterpret_cast<u2v*>(c.slots + at + lane));
    if (SPARS == QSL_RANDK) __builtin_nontemporal_store(s_stage_key[wave][lane], c.slot_key + at + lane);
  }
  if (!need_norm) return;                                    // (uniform)
  __syncthreads();
  const uint32_t ns = acc_slots(c.quantizer);
  uint64_t* part = wc.part + (static_cast<uint64_t>(w) * ((c.NWT + 3) / 4) + blk) * ns;
  for (uint32_t s = wave; s < ns; s += BLOCK / 64) {
    const uint64_t x = wave_sum64(lane < ACC_ROWS ? acc[lane * st + s] : 0);
    if (lane == 0) part[s] = x;
  }
}

// ------------------------------------------------------------------------------------------------
// the window's candidates
// ------------------------------------------------------------------------------------------------
// element e of the row that this lane holds: f(idx, bits, key), for the lane's candidates of its own slot
template <int SPARS, typename F>
__device__ __forceinline__ void win_own(const SlotRow& r, F&& f) {
  if (r.spill) return;
  if (r.has0) f(r.idx0, r.bits0, SPARS == QSL_TOPK ? key_of_value(r.bits0) : r.key0);
  if (r.has1) f(r.idx1, r.bits1, SPARS == QSL_TOPK ? key_of_value(r.bits1) : r.key1);
}

template <int SPARS>
__global__ __launch_bounds__(BIG) void k_win_hist(DevCtx c, WinCtx wc, SegInfo one, uint32_t R) {
  __shared__ uint32_t lh[HBINS];
  __shared__ unsigned long long s_ctr[CTR_LINES];
  LeanUnit lu;
  lean_unit<SPARS>(c, one, R, lu);
  const SegInfo& sg = lu.sg;
  UnitState* usp = &c.units[lu.u];
  const uint32_t T = wc.state[lu.w].lo, sh = wc.state[lu.w].sh;
  RawRow rr[ROWS_IN_FLIGHT];
#pragma unroll
  for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, lu.r_lo + b, lu.r_hi);
  for (uint32_t i = threadIdx.x; i < HBINS; i += BIG) lh[i] = 0;
  if (threadIdx.x < CTR_LINES) s_ctr[threadIdx.x] = *reinterpret_cast<const unsigned long long*>(&c.ctr[(lu.u * CTR_LINES + threadIdx.x) * PAD]);
  __syncthreads();
  unsigned long long sum = 0;                                // no carry between the halves: at most 2^32 - 1 coordinates
  for (uint32_t i = 0; i < NSUB; ++i) sum += s_ctr[i];
  const uint32_t cand = static_cast<uint32_t>(sum), above = static_cast<uint32_t>(sum >> 32);
  const bool failed = s_ctr[CTR_FAIL] != 0 || above >= sg.k || static_cast<uint64_t>(above) + cand < sg.k;
  if (threadIdx.x == 0 && lu.j == 0) {
    usp->cand = cand; wc.state[lu.w].above = above; usp->fell_back = failed; usp->crowded = 0; usp->nnz = 0;
    if (failed) c.host_flag[FLAG_WINDOW] = 1u;
  }
  if (failed) return;
  const uint32_t lane = lane_id();
  for (uint64_t row0 = lu.r_lo; row0 < lu.r_hi; row0 += ROWS_IN_FLIGHT) {
    if (row0 != lu.r_lo) {
#pragma unroll
      for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, row0 + b, lu.r_hi);
    }
#pragma unroll
    for (int b = 0; b < ROWS_IN_FLIGHT; ++b) {
      if (row0 + b >= lu.r_hi) break;
      const SlotRow r = parse_slot_row<true>(rr[b], sg.lpc);
      win_own<SPARS>(r, [&](uint32_t, uint32_t, uint32_t key) { atomicAdd(&lh[lean_bin(key, T, sh)], 1u); });
      for (uint64_t spilled = __ballot(r.spill); spilled; spilled &= spilled - 1) {
        const int holder = __ffsll(static_cast<unsigned long long>(spilled)) - 1;
        const uint32_t cnt = __shfl(r.count, holder, WAVE), at = __shfl(r.ovf_at, holder, WAVE);
        for (uint32_t e = lane; e < cnt; e += WAVE)
          atomicAdd(&lh[lean_bin(SPARS == QSL_TOPK ? key_of_value(lu.ovf[at + e].y) : lu.ovf_key[at + e], T, sh)], 1u);
      }
    }
  }
  __syncthreads();
  flush_hist(lh, wc.hist + lu.u * HBINS);
}

template <int SPARS>
__global__ __launch_bounds__(BIG) void k_win_mark(DevCtx c, WinCtx wc, SegInfo one, uint32_t R) {
  __shared__ uint64_t acc[LEAN_ROWS * (ACC_SLOTS + 1)];
  __shared__ uint64_t scratch[17];
  __shared__ uint32_t result[6];
  LeanUnit lu;
  lean_unit<SPARS>(c, one, R, lu);
  const SegInfo& sg = lu.sg;
  UnitState* usp = &c.units[lu.u];
  const UnitState us = *usp;
  if (us.fell_back) return;
  const uint32_t T = wc.state[lu.w].lo, sh = wc.state[lu.w].sh;
  RawRow rr[ROWS_IN_FLIGHT];
#pragma unroll
  for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, lu.r_lo + b, lu.r_hi);
  const uint32_t st = acc_stride(c.quantizer), ns = acc_slots(c.quantizer);
  for (uint32_t i = threadIdx.x; i < LEAN_ROWS * st; i += BIG) acc[i] = 0;
  const uint32_t target = sg.k - wc.state[lu.w].above;                 // >= 1
  find2_from_top<BIG>(wc.hist + lu.u * HBINS, target, target, scratch, result, false);
  const uint32_t taubin = result[0], above = result[1];
  // Four times what a bin holds on average is as much as smooth values put into one; a longer list (ties) is worth ranking where
  // the multi-pass kernels would have much to read, for large vectors and for many workers, whose lists are ranked side by side
  // (3.2 M values on a grid of 0.001, 660 of them at the threshold: one worker 137 us by the list, 88 by the multi-pass kernels;
  // 64 workers 1110 and 1900).
  const bool crowded = result[4] > max(256u, static_cast<uint32_t>(min<uint64_t>(WLIST, (static_cast<uint64_t>(us.cand) * R) >> 10)));
  if (threadIdx.x == 0 && lu.j == 0) {
    usp->taubin = taubin; usp->above = above; usp->crowded = crowded;
    if (crowded) c.host_flag[FLAG_WINDOW] = 1u;
  }
  if (crowded) return;                                       // (uniform) the multi-pass kernels take the unit
  const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t power = norm_power(c.quantizer);
  const bool need_norm = c.quantizer != QSL_FP32;
  uint64_t* mine = acc + ((wave & 7u) * 8 + (lane & 7u)) * st;
  if (need_norm) {                                           // this block's share of the rows that k_win_stream left
    const uint64_t nrow = (c.NWT + 3) / 4;
    const uint64_t a = nrow * lu.j / sg.nsel, b = nrow * (lu.j + 1) / sg.nsel;
    const uint64_t* part = wc.part + lu.u * nrow * ns;
    const uint32_t per = BIG / ns, s = threadIdx.x % ns, r0 = threadIdx.x / ns;       // thread: digit s of rows r0, r0 + per, ...
    uint64_t x = 0;
    if (r0 < per) for (uint64_t r = a + r0; r < b; r += per) x += part[r * ns + s];
    if (x) lds_add(&mine[s], x);
  }
  uint32_t* cursor = c.ctr + (lu.u * CTR_LINES + CTR_LIST) * PAD;
  uint4* list = wc.list + lu.u * WLIST;
  uint32_t n_sel = 0;
  auto visit = [&](bool has, uint32_t idx, uint32_t bits, uint32_t key) {              // all lanes of the wave together
    bool inside = false;
    if (has) {
      const uint32_t b = lean_bin(key, T, sh);
      if (b > taubin) { ++n_sel; if (need_norm) add_digits(mine, bits, power); }
      else inside = b == taubin;
    }
    const uint64_t ib = __ballot(inside);
    if (ib != 0) {
      const int first = __ffsll(static_cast<unsigned long long>(ib)) - 1;
      uint32_t base = 0;
      if (static_cast<int>(lane) == first) base = atomicAdd(cursor, static_cast<uint32_t>(__popcll(ib)));
      base = lane_value(base, first);
      const uint32_t q = base + popc_below(ib);
      if (inside && q < WLIST) list[q] = make_uint4(idx, bits, key, 0u);
    }
  };
  for (uint64_t row0 = lu.r_lo; row0 < lu.r_hi; row0 += ROWS_IN_FLIGHT) {
    if (row0 != lu.r_lo) {
#pragma unroll
      for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, row0 + b, lu.r_hi);
    }
#pragma unroll
    for (int b = 0; b < ROWS_IN_FLIGHT; ++b) {
      if (row0 + b >= lu.r_hi) break;
      const SlotRow r = parse_slot_row<true>(rr[b], sg.lpc);
      n_sel += r.above;                                      // the chunk's coordinates above the window (its header's lane)
      const bool h0 = !r.spill && r.has0, h1 = !r.spill && r.has1;
      if (__ballot(h0 || h1) != 0) {
        visit(h0, r.idx0, r.bits0, SPARS == QSL_TOPK ? key_of_value(r.bits0) : r.key0);
        visit(h1, r.idx1, r.bits1, SPARS == QSL_TOPK ? key_of_value(r.bits1) : r.key1);
      }
      for (uint64_t spilled = __ballot(r.spill); spilled; spilled &= spilled - 1) {
        const int holder = __ffsll(static_cast<unsigned long long>(spilled)) - 1;
        const uint32_t cnt = __shfl(r.count, holder, WAVE), at = __shfl(r.ovf_at, holder, WAVE);
        for (uint32_t e0 = 0; e0 < cnt; e0 += WAVE) {
          const uint32_t e = e0 + lane;
          uint2 ent = make_uint2(0, 0); uint32_t key = 0;
          if (e < cnt) { ent = lu.ovf[at + e]; key = SPARS == QSL_TOPK ? key_of_value(ent.y) : lu.ovf_key[at + e]; }
          visit(e < cnt, ent.x, ent.y, key);
        }
      }
    }
  }
  n_sel = wave_sum(n_sel);
  if (lane == 0) lu.wsel[lu.gw] = n_sel;
  if (!need_norm) return;
  __syncthreads();
  uint64_t* ga = c.norm_acc + lu.u * ACC_SLOTS;
  for (uint32_t s = wave; s < ns; s += BIG / 64) {
    const uint64_t x = wave_sum64(acc[lane * st + s]);
    if (lane == 0 && x) atomicAdd(reinterpret_cast<unsigned long long*>(ga + s), static_cast<unsigned long long>(x));
  }
}

template <int SPARS>
__global__ __launch_bounds__(BIG) void k_win_mid(DevCtx c, WinCtx wc, SegInfo one, uint32_t R) {
  __shared__ uint64_t acc[ACC_SLOTS + 1];
  __shared__ uint4 s_list[WLIST];
  __shared__ uint32_t s_tau, s_tie, s_need;
  LeanUnit lu;
  lean_unit<SPARS>(c, one, R, lu);
  const SegInfo& sg = lu.sg;
  for (uint32_t i = lu.j * BIG + threadIdx.x; i < HBINS; i += sg.nsel * BIG) wc.hist[lu.u * HBINS + i] = 0;      // k_win_mark was its last reader
  UnitState* usp = &c.units[lu.u];
  const UnitState us = *usp;
  if (us.fell_back || us.crowded) return;
  const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
  const uint32_t power = norm_power(c.quantizer);
  RawRow rr[ROWS_IN_FLIGHT];
#pragma unroll
  for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, lu.r_lo + b, lu.r_hi);
  static_assert(WLIST <= BIG, "a thread per list entry");
  const uint32_t n_list = min(c.ctr[(lu.u * CTR_LINES + CTR_LIST) * PAD], WLIST);
  uint4 me = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < WLIST) me = wc.list[lu.u * WLIST + threadIdx.x];
  const uint64_t my_digit = threadIdx.x < acc_slots(c.quantizer) ? c.norm_acc[lu.u * ACC_SLOTS + threadIdx.x] : 0;
  uint32_t s_off = waves_before(lu.wsel, lu.gw);
  if (threadIdx.x == 0) { s_need = 0; s_tau = 0; s_tie = 0; }
  if (threadIdx.x < ACC_SLOTS + 1) acc[threadIdx.x] = 0;
  if (threadIdx.x < n_list) s_list[threadIdx.x] = me;
  __syncthreads();
  // the list ranked by (key descending, coordinate ascending): the last one selected gives threshold and last kept tie
  const uint32_t k_rem = sg.k - wc.state[lu.w].above - us.above;
  // (eight lanes per entry: with one each, the walk through a list of a hundred entries alone took 8 us)
  const uint32_t sub = threadIdx.x & 7u;
  for (uint32_t i = threadIdx.x >> 3; i < n_list; i += BIG / 8) {
    const uint4 e = s_list[i];
    uint32_t rank = 0;
    for (uint32_t j = sub; j < n_list; j += 8) {
      const uint4 o = s_list[j];
      rank += (o.z > e.z || (o.z == e.z && o.x < e.x)) ? 1u : 0u;
    }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) rank += __shfl_xor(rank, o, WAVE);
    if (sub == 0) {
      if (rank == k_rem - 1) { s_tau = e.z; s_tie = e.x; }
      if (rank < k_rem) add_digits(acc, e.y, power);
    }
  }
  __syncthreads();
  const uint32_t tau = s_tau, tie = s_tie;
  if (threadIdx.x < n_list && me.z == tau && me.x <= tie) atomicAdd(&s_need, 1u);
  if (threadIdx.x < acc_slots(c.quantizer)) acc[threadIdx.x] += my_digit;
  __syncthreads();
  if (lu.j == 0 && wave == 0) {
    const UnitScale usc = unit_scale(c, finalize_scale(acc, c.quantizer, sg.k), sg.k);
    if (lane == 0) {
      usp->tau = tau; wc.state[lu.w].tie = tie; usp->need = s_need; usp->n_gt = sg.k - s_need;
      usp->scale_code = __float_as_uint(usc.scale); usp->scale_bits = __float_as_uint(usc.sent);
    }
  }
  // where every chunk's entries begin: selected coordinates before it
  const uint32_t cpr = 64 / sg.lpc;                          // chunks per slot row
  const uint64_t first = lu.r_lo * cpr * CHUNK;              // the wave's first coordinate
  {
    uint32_t x = 0;
    for (uint32_t j = lane; j < n_list; j += WAVE) {
      const uint4 o = s_list[j];
      x += (o.z > tau || (o.z == tau && o.x <= tie)) && o.x < first ? 1u : 0u;
    }
    s_off += wave_sum(x);
  }
  auto taken = [&](uint32_t idx, uint32_t key) { return key > tau || (key == tau && idx <= tie); };
  uint32_t* off = wc.off + lu.u * c.NWT;
  for (uint64_t row0 = lu.r_lo; row0 < lu.r_hi; row0 += ROWS_IN_FLIGHT) {
    if (row0 != lu.r_lo) {
#pragma unroll
      for (int b = 0; b < ROWS_IN_FLIGHT; ++b) rr[b] = load_slot_row(lu.slots, lu.slot_key, sg.lpc, sg.nwt, row0 + b, lu.r_hi);
    }
#pragma unroll
    for (int b = 0; b < ROWS_IN_FLIGHT; ++b) {
      if (row0 + b >= lu.r_hi) break;
      const SlotRow r = parse_slot_row<true>(rr[b], sg.lpc);
      uint32_t n = r.above;
      win_own<SPARS>(r, [&](uint32_t idx, uint32_t, uint32_t key) { n += taken(idx, key) ? 1u : 0u; });
      for (uint64_t spilled = __ballot(r.spill); spilled; spilled &= spilled - 1) {
        const int holder = __ffsll(static_cast<unsigned long long>(spilled)) - 1;
        const uint32_t cnt = __shfl(r.count, holder, WAVE), at = __shfl(r.ovf_at, holder, WAVE);
        uint32_t x = 0;
        for (uint32_t e = lane; e < cnt; e += WAVE) {
          const uint2 ent = lu.ovf[at + e];
          x += taken(ent.x, SPARS == QSL_TOPK ? key_of_value(ent.y) : lu.ovf_key[at + e]) ? 1u : 0u;
        }
        x = wave_sum(x);
        if (static_cast<int>(lane) == holder) n += x;
      }
      uint32_t tot;
      const uint32_t pos = s_off + wave_exclusive_scan32(n, &tot);
      s_off += tot;
      const uint64_t chunk = (row0 + b) * cpr + lane / sg.lpc;
      if ((lane & (sg.lpc - 1)) == 0 && chunk < sg.nwt) off[chunk] = pos;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// the second pass over v: a wave per chunk.  The selected coordinates are lined up in LDS, quantised 64 at a time and
// written in order to the arrays that the message is packed from; the chunk goes back whole (a tenth of the coordinates
// touches four of five 64-byte sectors).  (The wave could write its fields into the message itself; the words that two
// chunks share then cost an atomicOr each, 0.5 ns of the whole GPU: 336 us for 4 x 25.6 M coordinates with k = d / 10, against
// 165 us and k_pack's 30.)
// ------------------------------------------------------------------------------------------------
template <int SPARS>
__global__ __launch_bounds__(BLOCK) void k_win_apply(DevCtx c, WinCtx wc, SegInfo sg, float* m_out, uint32_t worker0, uint64_t round,
                                                     uint32_t* dbg_idx, uint16_t* dbg_level) {
  __shared__ uint16_t s_loc[BLOCK / 64][CHUNK];              // selected coordinates of the chunk ...
  __shared__ f4u s_v[BLOCK / 64][CHUNK / 4];                 // ... and the chunk itself
  const uint32_t w = blockIdx.y, wave = threadIdx.x >> 6, lane = lane_id();
  if (blockIdx.x == 0 && threadIdx.x < CTR_LINES)            // the counters of this call have served
    *reinterpret_cast<unsigned long long*>(&c.ctr[(static_cast<uint64_t>(w) * CTR_LINES + threadIdx.x) * PAD]) = 0;
  const uint32_t chunk = blockIdx.x * (BLOCK / 64) + wave;
  if (chunk >= c.NWT) return;                                // (no barrier follows)
  const UnitState& us = c.units[w];
  if (us.fell_back || us.crowded) return;
  const uint32_t tau = us.tau, tie = wc.state[w].tie;
  UnitScale usc; usc.scale = __uint_as_float(us.scale_code); usc.sent = __uint_as_float(us.scale_bits);
  const uint32_t pos = wc.off[static_cast<uint64_t>(w) * c.NWT + chunk];
  const uint64_t first = static_cast<uint64_t>(chunk) * CHUNK;
  const uint32_t valid = static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), sg.size - first));
  float* vp = m_out + static_cast<uint64_t>(w) * c.d + first;
  const RandKey rk = make_rand_key(c.seed, worker0 + w, round, 0), rk1 = make_rand_key(c.seed, worker0 + w, round, 1);
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
  uint32_t n = 0;
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    s_v[wave][e / 4] = v[t];
    Words4 rw = {{0u, 0u, 0u, 0u}};
    if (SPARS == QSL_RANDK) rw = rand_words4(rk, static_cast<uint32_t>(first + e));
    uint32_t nib = 0, below = 0, tot = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t key = SPARS == QSL_TOPK ? key_of_value(__float_as_uint(v[t][j])) : rw.w[j];
      const bool take = e + j < valid && (key > tau || (key == tau && static_cast<uint32_t>(first) + e + j <= tie));
      const uint64_t bal = __ballot(take);
      nib |= (take ? 1u : 0u) << j;
      below += popc_below(bal); tot += static_cast<uint32_t>(__popcll(bal));
    }
    uint32_t at = n + below;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) if ((nib >> j) & 1u) s_loc[wave][at++] = static_cast<uint16_t>(e + j);
    n += tot;
  }
  if (n == 0 || pos >= sg.k) return;                         // (uniform over the wave)
  n = min(n, sg.k - pos);
  float* img = reinterpret_cast<float*>(s_v[wave]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (uint32_t i0 = 0; i0 < n; i0 += WAVE) {
    const uint32_t i = i0 + lane;
    bool sent = false;
    if (i < n) {
      const uint32_t loc = s_loc[wave][i], idx = static_cast<uint32_t>(first) + loc;
      const float x = img[loc];
      float g;
      sent = encode_entry_at(c, static_cast<uint64_t>(w) * c.K + pos + i, idx, __float_as_uint(x), usc, rk1, dbg_idx, dbg_level, &g);
      if (sent) img[loc] = x - g;
    }
    if (is_qsgd(c.quantizer)) {                              // survivors per block of 256 slots: 64 slots touch at most two
      const uint64_t sb = __ballot(sent);
      if (sb != 0) {
        const uint32_t b_first = (pos + i0) >> 8;
        const uint32_t n0 = static_cast<uint32_t>(__popcll(__ballot(sent && ((pos + i) >> 8) == b_first)));
        const uint32_t n1 = static_cast<uint32_t>(__popcll(sb)) - n0;
        if (lane == 0) {
          uint32_t* bc = c.blk_cnt + static_cast<uint64_t>(w) * c.QB;
          if (n0) atomicAdd(&bc[b_first], n0);
          if (n1) atomicAdd(&bc[b_first + 1], n1);
        }
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    const f4u x = s_v[wave][e / 4];
    if (valid == CHUNK) __builtin_nontemporal_store(x, reinterpret_cast<f4u*>(vp + e));
    else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) vp[e + j] = x[j];
    }
  }
}

}  // namespace
