// qsl_decode.h -- Reading messages: the stand-alone error update (k_add_rows, k_subtract_msg, k_update_rows) and the master's
// aggregation (k_fill_zero, k_msg_directory, k_aggregate, k_aggregate_small, k_aggregate_entries, k_aggregate_cells,
// k_aggregate_dense, k_aggregate_dense_one), k_read_nnz.
// Part of the single translation unit qsl.hip (included there, in this order: device, layout, select,
// encode, stream, lean, window, dense, decode); not a public header.
#pragma once

#include "qsl_device.h"
#include "qsl_layout.h"
#include "qsl_select.h"
#include "qsl_encode.h"

namespace {

// ------------------------------------------------------------------------------------------------
// reading messages: stand-alone error update, aggregation
// ------------------------------------------------------------------------------------------------
struct MsgView {
  const uint32_t* words; uint32_t nnz; uint64_t idx_bit0, code_bit0;
};
__device__ __forceinline__ MsgView view_msg(const DevCtx& c, const uint8_t* msg, uint32_t row) {
  MsgView v;
  v.words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(row) * c.cap_words * 4);
  v.nnz = min(v.words[0], c.K);                         // a well-formed message never holds more than K entries
  const bool counts = is_qsgd(c.quantizer) && c.L > 1 && !c.dense;
  const uint64_t hdr = 1 + static_cast<uint64_t>(c.L) + (counts ? c.L : 0);
  v.idx_bit0 = hdr * 32;
  v.code_bit0 = (hdr + (static_cast<uint64_t>(v.nnz) * c.w_idx + 31) / 32) * 32;
  return v;
}
__device__ __forceinline__ uint32_t msg_index(const DevCtx& c, const MsgView& v, uint32_t j) {
  if (c.dense) return j;                                 // the index-free format: entry j is coordinate j
  return get_bits(v.words, v.idx_bit0 + static_cast<uint64_t>(j) * c.w_idx, c.w_idx);
}
// the value a code field stands for, given the scale its segment transmitted
__device__ __forceinline__ float value_of_code(const DevCtx& c, uint32_t code, float scale) {
  if (is_qsgd(c.quantizer)) {
    // with indices only the levels 1..s are transmitted, as level - 1; the index-free format writes 0..s as they are
    const uint32_t level = (code & ((1u << c.w_lev) - 1u)) + (c.dense ? 0u : 1u);
    if (level == 0) return 0.0f;
    return qsgd_value(scale, level, c.s, (code >> c.w_lev) & 1u);
  }
  if (c.quantizer == QSL_FP32) return __uint_as_float(code);
  return code ? -scale : scale;
}
__device__ __forceinline__ float msg_value(const DevCtx& c, const MsgView& v, uint32_t j, uint32_t idx) {
  const uint32_t code = get_bits(v.words, v.code_bit0 + static_cast<uint64_t>(j) * c.w_val, c.w_val);
  const uint32_t seg = c.L == 1 ? 0u : seg_of_coord(c, idx);
  return value_of_code(c, code, __uint_as_float(v.words[1 + seg]));
}
// position of coordinate idx in the message, or -1
__device__ __forceinline__ int64_t msg_find(const DevCtx& c, const MsgView& v, uint32_t idx) {
  if (v.nnz == c.d) return idx;                          // every coordinate is there (k = d): entry j is coordinate j
  uint32_t lo = 0, hi = v.nnz;
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    const uint32_t x = msg_index(c, v, mid);
    if (x == idx) return mid;
    if (x < idx) lo = mid + 1; else hi = mid;
  }
  return -1;
}

typedef uint32_t u2u __attribute__((ext_vector_type(2), aligned(4)));
// `width` (1 .. 32) bits from bit `bit` of a message on, by one 8-byte read that stays inside its cap_words words
struct FieldRead { u2u w; uint32_t sh; };
__device__ __forceinline__ FieldRead read_field(const uint32_t* words, uint64_t bit, uint32_t cap_words) {
  const uint64_t q = min(bit >> 5, static_cast<uint64_t>(cap_words) - 2);
  FieldRead f;
  f.w = *reinterpret_cast<const u2u*>(words + q);
  f.sh = static_cast<uint32_t>(bit - q * 32) & 63u;
  return f;
}
__device__ __forceinline__ uint32_t field_of(const FieldRead& f, uint32_t width) {
  const uint64_t v = (static_cast<uint64_t>(f.w.y) << 32 | f.w.x) >> f.sh;
  return width == 32 ? static_cast<uint32_t>(v) : static_cast<uint32_t>(v) & ((1u << width) - 1u);
}

// m <- m + delta over the flat [R * d] arrays: the streaming recipe of k_stream (a wave per 1024 elements,
// non-temporal dwordx4 accesses, 3 waves per SIMD)
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_add_rows(float* m, const float* delta,
                                                                                              uint64_t n) {
  const uint64_t chunk = static_cast<uint64_t>(blockIdx.x) * (BLOCK / 64) + (threadIdx.x >> 6);
  const uint64_t cb = chunk * CHUNK;
  if (cb >= n) return;
  const uint32_t lane = lane_id();
  if (n - cb >= CHUNK) {
    f4u a[4], b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      a[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(m + cb + t * 256 + lane * 4));
      b[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(delta + cb + t * 256 + lane * 4));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) __builtin_nontemporal_store(a[t] + b[t], reinterpret_cast<f4u*>(m + cb + t * 256 + lane * 4));
  } else {
    for (uint64_t i = cb + lane; i < n; i += 64) m[i] = m[i] + delta[i];
  }
}

__global__ __launch_bounds__(BLOCK) void k_subtract_msg(DevCtx c, float* m, const uint8_t* msg) {
  const uint32_t w = blockIdx.y;
  const MsgView v = view_msg(c, msg, w);
  const uint32_t j = blockIdx.x * BLOCK + threadIdx.x;
  if (j >= v.nnz) return;
  const uint32_t idx = msg_index(c, v, j);
  if (idx >= c.d) { atomicOr(c.status, 4u); return; }   // malformed message
  float* p = m + static_cast<uint64_t>(w) * c.d + idx;
  *p = *p - msg_value(c, v, j, idx);
}

// Both in one launch, for vectors so short that a launch counts: a wave per 1024 coordinates of a row finds the message's entries among
// them itself -- half of its lanes the first, half the last, 32 parts of the message a step -- while its reads of m and delta
// are under way.  Where there are entries, the sums take the way through LDS to meet them, UPDATE_STEPS times 64 entries' reads in flight.
// What bounds it is the chain of reads, so registers are kept to what eight waves per SIMD allow, and an entry's segment comes from bits
// in two lane moves.  With four waves per SIMD (126 registers), 64 entries a step and a search in memory for every entry's segment it lost to the
// two launches above where small tensors fill a chunk (176 tensors, 7 x 119,847, k = 1000: 11.5 by two launches, 18.3 that way, 11.4 us
// now) and beyond 4.2 M coordinates (4 x 2.09 M, 0.1 %: 18.9, 20.6, 17.2).
constexpr uint32_t UPDATE_STEPS = 2;      // (4: 80 registers, and slower from 6 M coordinates on)
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_update_rows(DevCtx c, float* m, const float* delta, const uint8_t* msg) {
  __shared__ f4u s_image[BLOCK / 64][CHUNK / 4];
  __shared__ uint32_t s_starts[BLOCK / 64][CHUNK / 32];
  const uint32_t w = blockIdx.y, lane = lane_id(), wave = threadIdx.x >> 6;
  const uint64_t first = (static_cast<uint64_t>(blockIdx.x) * (BLOCK / 64) + wave) * CHUNK;
  if (first >= c.d) return;                              // (no barrier follows)
  const uint32_t valid = static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), c.d - first));
  // the segments of the chunk, a bit per coordinate where one begins: lane l < 32 holds those of 32 coordinates and how many lie before
  // them.  Their reads come first: a wave's loads return in order.
  uint32_t seg_lo = 0, n_seg = 1, my_start = 0, starts = 0, starts_before = 0;
  if (c.L > 1) {
    seg_lo = __builtin_amdgcn_readfirstlane(c.seg_dir[first >> 10]);
    n_seg = __builtin_amdgcn_readfirstlane(c.seg_dir[(first >> 10) + 1]) + 1 - seg_lo;
    my_start = c.seg_start[seg_lo + min(lane, n_seg - 1)];
  }
  const MsgView v = view_msg(c, msg, w);
  const bool few = n_seg <= WAVE;                        // then lane l holds the message's scale of the l-th
  const float my_scale = __uint_as_float(v.words[1 + seg_lo + min(lane, n_seg - 1)]);
  float* mp = m + static_cast<uint64_t>(w) * c.d + first;
  const float* dp = delta + static_cast<uint64_t>(w) * c.d + first;
  f4u a[4], b[4];
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    a[t] = b[t] = f4u{0.f, 0.f, 0.f, 0.f};
    if (valid == CHUNK) {
      a[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(mp + e));
      b[t] = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(dp + e));
    } else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) { a[t][j] = mp[e + j]; b[t][j] = dp[e + j]; }
    }
  }
  if (n_seg > 1) {
    if (lane < CHUNK / 32) s_starts[wave][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t l = lane; l < n_seg; l += WAVE) {
      const uint32_t at = (l < WAVE ? my_start : c.seg_start[seg_lo + l]) - static_cast<uint32_t>(first);
      if (l != 0 && at < CHUNK) atomicOr(&s_starts[wave][at >> 5], 1u << (at & 31u));      // (the last one may begin with the next chunk)
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < CHUNK / 32) starts = s_starts[wave][lane];
    uint32_t all;
    starts_before = wave_exclusive_scan32(static_cast<uint32_t>(__popc(starts)), &all);
  }
  // lanes 0 .. 31: the first entry at or behind `first`; 32 .. 63: at or behind the chunk's end (the last chunk takes what is left, and
  // neighbouring chunks find the same end between them, so that every entry of the message is looked at)
  const bool tail = lane >= 32;
  const uint32_t d = static_cast<uint32_t>(c.d), target = static_cast<uint32_t>(first) + (tail ? CHUNK : 0u);      // (< d where there is a search)
  uint32_t lo = tail && first + CHUNK >= c.d ? v.nnz : 0u, hi = first == 0 && !tail ? 0u : v.nnz;
  bool bad = false;                                      // a step met an index >= d (a malformed message), which says nothing about where to go on
  while (__ballot(lo < hi) != 0) {                       // (each half of the wave agrees on its lo and hi)
    const uint32_t width = hi - lo, part = lane & 31u;
    const uint32_t at = lo + static_cast<uint32_t>(static_cast<uint64_t>(width) * (part + 1) / 33);
    const uint32_t x = field_of(read_field(v.words, v.idx_bit0 + static_cast<uint64_t>(min(at, v.nnz - 1)) * c.w_idx, c.cap_words), c.w_idx);
    const bool open = lo < hi;
    bad |= open & (x >= d);
    const uint64_t bal = __ballot(open & (x < target));
    const uint32_t n = static_cast<uint32_t>(__popcll(tail ? bal >> 32 : bal & 0xFFFFFFFFull));
    if (lo < hi) {
      const uint32_t base = lo;
      if (n) lo = base + static_cast<uint32_t>(static_cast<uint64_t>(width) * n / 33) + 1;
      if (n < 32) hi = base + static_cast<uint32_t>(static_cast<uint64_t>(width) * (n + 1) / 33);
    }
  }
  // (then the wave goes through the whole message; where no step met such an index, what the steps found holds for all the others)
  const bool lost = __ballot(bad) != 0;
  const uint32_t j_lo = lost ? 0u : lane_value(lo, 0), j_hi = lost ? v.nnz : lane_value(lo, 32);
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) a[t] = a[t] + b[t];
  if (j_lo < j_hi) {                                     // (uniform)
    float* image = reinterpret_cast<float*>(s_image[wave]);
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) s_image[wave][t * 64 + lane] = a[t];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");      // the image is private to the wave
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t j0 = j_lo; j0 < j_hi; j0 += UPDATE_STEPS * WAVE) {
      FieldRead fi[UPDATE_STEPS], fc[UPDATE_STEPS];
#pragma unroll
      for (uint32_t u = 0; u < UPDATE_STEPS; ++u) {
        const uint32_t j = min(j0 + u * WAVE + lane, v.nnz - 1);
        fi[u] = read_field(v.words, v.idx_bit0 + static_cast<uint64_t>(j) * c.w_idx, c.cap_words);
        fc[u] = read_field(v.words, v.code_bit0 + static_cast<uint64_t>(j) * c.w_val, c.cap_words);
      }
#pragma unroll
      for (uint32_t u = 0; u < UPDATE_STEPS; ++u) {
        const uint32_t idx = field_of(fi[u], c.w_idx);
        const bool in = j0 + u * WAVE + lane < j_hi, ok = in && idx >= first && idx - first < valid;
        if (in && !ok && (!lost || idx >= d)) atomicOr(c.status, 4u);      // malformed message
        uint32_t seg = 0;                                // the entry's segment, of the chunk's
        if (n_seg > 1) {
          const uint32_t r = idx - static_cast<uint32_t>(first), word = __shfl(starts, r >> 5 & 31u, WAVE), before = __shfl(starts_before, r >> 5 & 31u, WAVE);
          seg = before + static_cast<uint32_t>(__popc(word & ((2u << (r & 31u)) - 1u)));
        }
        const float scale = few ? __shfl(my_scale, seg, WAVE) : __uint_as_float(v.words[1 + seg_lo + seg]);
        if (ok) image[idx - first] = image[idx - first] - value_of_code(c, field_of(fc[u], c.w_val), scale);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) a[t] = s_image[wave][t * 64 + lane];
  }
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    if (valid == CHUNK) __builtin_nontemporal_store(a[t], reinterpret_cast<f4u*>(mp + e));
    else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) mp[e + j] = a[t][j];
    }
  }
}

__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_fill_zero(float* out, uint64_t n) {
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * BLOCK * 4;
  const f4u z = {0.f, 0.f, 0.f, 0.f};
  for (uint64_t i = (static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x) * 4; i < n; i += stride) {
    if (i + 4 <= n) __builtin_nontemporal_store(z, reinterpret_cast<f4u*>(out + i));
    else for (uint64_t j = i; j < n; ++j) out[j] = 0.f;
  }
}

struct RowList { uint32_t row[64]; };
constexpr uint32_t AGG_ENTRIES = 32;     // message entries per block; 8 threads look one entry up in parallel
constexpr uint32_t AGG_DIR_SHIFT = 10;   // a directory entry per 1024 coordinates
constexpr uint32_t AGG_DIR_MIN = 4096;   // messages expected to be at least this long are searched through their directories
constexpr uint32_t AGG_CELLS_MIN_R = 36; // short messages go to k_aggregate_cells from this many on

// Cells in which the listed messages' entries pile up, found while the directories are made (k_aggregate_cells gives them to many
// waves).  count[0], count[1] and bits are zero between calls.  list == nullptr: they are not listed.
struct AggPile {
  uint32_t* count; uint32_t* bits; uint32_t* list;
  const uint32_t* planned;   // a bit per cell that the plan already gives to several waves (or null)
  uint32_t* flag;            // pinned host memory: set when a cell is piled up (or null)
};

// Directory of a long message: dir[t] = number of entries whose coordinate lies below t * 1024, for
// t = 0 .. ndir - 1 (ndir = ceil(d / 1024) + 1, so dir[ndir - 1] = nnz).  Entry j fills the slots between
// its predecessor's 1024-block and its own; the last entry also fills the rest.  A lookup then needs
// dir[t], dir[t + 1] and a binary search over the few entries of one 1024-block instead of log2(nnz)
// dependent probes of the whole message.
// UN: entries per thread and step, their reads in flight together (1 while the grid covers the messages).
// `pile`: the cells in which a message has 64 entries side by side in one wave's hands are listed, once each (the first such wave
// of a message looks whether the cell's bit is set already).
template <uint32_t UN>
__global__ __launch_bounds__(BLOCK) void k_msg_directory(DevCtx c, const uint8_t* msg, RowList rows, uint32_t* dir,
                                                         uint32_t ndir, AggPile pile) {
  const uint32_t q = blockIdx.y, lane = lane_id();
  const MsgView v = view_msg(c, msg, rows.row[q]);
  uint32_t* mine = dir + static_cast<uint64_t>(q) * ndir;
  const uint32_t nth = gridDim.x * BLOCK, tid = blockIdx.x * BLOCK + threadIdx.x;
  if (v.nnz == 0) { for (uint32_t t = tid; t < ndir; t += nth) mine[t] = 0; return; }
  for (uint64_t j0 = tid; j0 - lane < v.nnz; j0 += static_cast<uint64_t>(nth) * UN) {      // (uniform over the wave)
    uint32_t cell[UN], prev[UN];
    bool bad = false;
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      const uint64_t j = j0 + static_cast<uint64_t>(u) * nth;
      cell[u] = 0; prev[u] = 0;
      if (j < v.nnz) {
        const uint32_t idx = msg_index(c, v, static_cast<uint32_t>(j));
        bad = bad || idx >= c.d;                           // malformed message: here every index is seen, whoever decodes the entry
        cell[u] = min(idx >> AGG_DIR_SHIFT, ndir - 2);
        if (lane == 0 && j) prev[u] = min(msg_index(c, v, static_cast<uint32_t>(j) - 1) >> AGG_DIR_SHIFT, ndir - 2);
      }
    }
    if (bad) atomicOr(c.status, 4u);
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      const uint64_t j = j0 + static_cast<uint64_t>(u) * nth;
      const uint32_t below = __shfl_up(cell[u], 1, WAVE);                                  // the entry before stands in the lane before
      if (j < v.nnz) {
        const uint32_t first = j == 0 ? 0u : (lane ? below : prev[u]) + 1;
        for (uint32_t t = first; t <= cell[u]; ++t) mine[t] = static_cast<uint32_t>(j);   // empty when the predecessor shares the block
        if (j == v.nnz - 1) for (uint32_t t = cell[u] + 1; t < ndir; ++t) mine[t] = v.nnz;
      }
      if (pile.list != nullptr) {
        const uint32_t t0 = __builtin_amdgcn_readfirstlane(cell[u]);
        if (j - lane + 63 < v.nnz && t0 == static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(cell[u]), 63)) && lane == 0 &&
            (j < 64 || (msg_index(c, v, static_cast<uint32_t>(j) - 64) >> AGG_DIR_SHIFT) != t0)) {
          uint32_t* word = pile.bits + (t0 >> 5);
          const uint32_t bit = 1u << (t0 & 31u);
          const bool planned = pile.planned != nullptr && (pile.planned[t0 >> 5] & bit);
          if (!planned && !(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) && !(atomicOr(word, bit) & bit)) {
            const uint32_t at = atomicAdd(&pile.count[0], 1u);
            if (at < ndir) pile.list[at] = t0;               // (a cell once: there is room)
          }
        }
      }
    }
  }
}

// The same directories where there are many entries to a cell (directory_by_search): a thread per slot
// finds its entry by bisection, from where it would stand if the entries lay evenly, instead of every entry being read.  Whatever
// the message holds, slot 0 is 0 and the last one its length, so that every entry, also one with an index >= d, lies between two
// neighbouring slots and is met by whoever decodes that cell -- but for the last cell, where it may fall to a part behind d that has
// no coordinates: that cell's entries are looked through here.  Bound by the chain of reads, two and then half the logarithm of the
// window.  4 messages of 2.6 M entries, d = 25.6 M: 25.7 us
// by reading every entry, 16.8 this way.
constexpr uint32_t DIR_WINDOW = 2048;
__global__ __launch_bounds__(BLOCK) void k_msg_directory_search(DevCtx c, const uint8_t* msg, RowList rows, uint32_t* dir, uint32_t ndir) {
  __shared__ uint32_t s_last;
  const uint32_t q = blockIdx.y, t = blockIdx.x * BLOCK + threadIdx.x;
  const MsgView v = view_msg(c, msg, rows.row[q]);
  uint32_t lo = 0, hi = t == 0 ? 0u : v.nnz;
  if (t >= ndir - 1) lo = hi;
  const uint64_t target = static_cast<uint64_t>(t) << AGG_DIR_SHIFT;
  if (lo < hi) {
    const uint32_t at = static_cast<uint32_t>(static_cast<uint64_t>(v.nnz) * t / (ndir - 1));
    const uint32_t a = at > DIR_WINDOW ? at - DIR_WINDOW : 0u, z = min(v.nnz - 1, at + DIR_WINDOW);
    const uint32_t xa = msg_index(c, v, a), xz = msg_index(c, v, z);
    if (xa >= target) hi = a; else lo = a + 1;           // the first entry at or behind the target lies in [lo, hi]
    if (lo <= z && z < hi) { if (xz >= target) hi = z; else lo = z + 1; }
  }
  while (lo < hi) {
    uint32_t x[3];
#pragma unroll
    for (uint32_t i = 0; i < 3; ++i) x[i] = msg_index(c, v, lo + static_cast<uint32_t>(static_cast<uint64_t>(hi - lo) * (i + 1) >> 2));
    const uint32_t w = hi - lo, base = lo;
    auto part = [&](uint32_t i) { return base + static_cast<uint32_t>(static_cast<uint64_t>(w) * i >> 2); };
    if (x[0] >= target) hi = part(1);
    else if (x[1] >= target) { lo = part(1) + 1; hi = part(2); }
    else if (x[2] >= target) { lo = part(2) + 1; hi = part(3); }
    else lo = part(3) + 1;
  }
  if (t < ndir) dir[static_cast<uint64_t>(q) * ndir + t] = lo;
  if (blockIdx.x != (ndir - 2) / BLOCK) return;          // (uniform) the block with the last cell
  if (t == ndir - 2) s_last = lo;
  __syncthreads();
  bool bad = false;
  for (uint32_t j = s_last + threadIdx.x; j < v.nnz; j += BLOCK) bad = bad || msg_index(c, v, j) >= c.d;
  if (bad) atomicOr(c.status, 4u);
}

// Short messages (no directory).  Entry j of the q-th listed message is served by 8 threads, which look its
// coordinate up in the other listed messages (binary search on the packed, ascending indices).  The coordinate is
// written by the earliest listed message that holds it -- one writer per coordinate, no atomics --
// and the values are added in list order, so the result does not depend on the schedule.
__global__ __launch_bounds__(BLOCK) void k_aggregate(DevCtx c, const uint8_t* msg, RowList rows, uint32_t R,
                                                     float scale, int accumulate, float* out) {
  __shared__ float s_val[AGG_ENTRIES][65];
  __shared__ unsigned long long s_has[AGG_ENTRIES];
  const uint32_t q = blockIdx.y;
  const uint32_t e = threadIdx.x >> 3, sub = threadIdx.x & 7u;
  const MsgView mine = view_msg(c, msg, rows.row[q]);
  // the grid is sized for a moderate message; a block walks the tiles of 32 entries that exist
  for (uint32_t tile = blockIdx.x; tile * AGG_ENTRIES < mine.nnz; tile += gridDim.x) {
    const uint32_t j = tile * AGG_ENTRIES + e;
    if (sub == 0) s_has[e] = 0;
    __syncthreads();
    uint32_t idx = 0xFFFFFFFFu;
    if (j < mine.nnz) {
      idx = msg_index(c, mine, j);
      if (idx >= c.d) { if (sub == 0) atomicOr(c.status, 4u); idx = 0xFFFFFFFFu; }   // malformed message
    }
    if (idx != 0xFFFFFFFFu) {
      unsigned long long has = 0;
      for (uint32_t p = sub; p < R; p += 8) {
        if (p == q) { s_val[e][p] = msg_value(c, mine, j, idx); has |= 1ull << p; continue; }
        const MsgView other = view_msg(c, msg, rows.row[p]);
        const int64_t pos = msg_find(c, other, idx);
        if (pos >= 0) { s_val[e][p] = msg_value(c, other, static_cast<uint32_t>(pos), idx); has |= 1ull << p; }
      }
      if (has) atomicOr(&s_has[e], has);
    }
    __syncthreads();
    if (sub == 0 && idx != 0xFFFFFFFFu) {
      const unsigned long long has = s_has[e];
      if (!(has & ((1ull << q) - 1ull))) {                // no earlier listed message owns this coordinate
        float acc = 0.0f;
        bool first = true;
        for (uint32_t p = q; p < R; ++p) {
          if (!((has >> p) & 1ull)) continue;
          acc = first ? s_val[e][p] : acc + s_val[e][p];
          first = false;
        }
        const float term = scale * acc;
        out[idx] = accumulate ? out[idx] + term : term;
      }
    }
    __syncthreads();                                       // s_val and s_has are reused by the next tile
  }
}

// Few entries in all, on a short vector: the whole master line in one launch, whether `out` is added to or written.  A block owns
// SMALL_AGG_SPAN coordinates, with room in LDS for every message's value of each; its waves (wave v: messages v, v + waves, ...) put the
// entries of its range in their places; then each thread adds up a coordinate's values in list order.  A wave looks at every
// `stride`-th entry first, all in one step, and then reads only what lies between the two that enclose the block's range.  What bounds it
// is the chain of reads, four or five whatever the messages' lengths: 15 messages of 40 entries on 7,850 coordinates 4.5 us, where
// clearing and k_aggregate are two launches of 2.0 and 8.4 us.
// Whatever a message holds, the parts that neighbouring blocks read meet, so that every entry is looked at; where one of the entries
// looked at first has an index >= d, all blocks go through the whole message, and no other entry is lost.
constexpr uint32_t SMALL_AGG_THREADS = 512, SMALL_AGG_SPAN = 512;      // (the fewest coordinates that give every thread one)
constexpr uint32_t SMALL_AGG_R = AGG_CELLS_MIN_R - 1;                  // messages: more of them go to k_aggregate_cells
constexpr uint32_t SMALL_AGG_STEPS = 4;                                // entries of a lane whose reads are in flight together
constexpr uint32_t small_agg_lds(uint32_t R) { return 4 * (R + 2) * SMALL_AGG_SPAN; }
static_assert(SMALL_AGG_R <= 64 && small_agg_lds(SMALL_AGG_R) <= 160 * 1024, "a mark per message in 64 bits, the LDS of a compute unit");
template <bool SHORT>      // messages expected to hold 128 entries at most: all of them are read at once (stride is 1)
__global__ __launch_bounds__(SMALL_AGG_THREADS) void k_aggregate_small(DevCtx c, const uint8_t* msg, RowList rows, uint32_t R, float scale,
                                                                       int accumulate, float* out, uint32_t stride) {
  extern __shared__ float s_values[];                    // [R][SPAN], then the messages that hold each coordinate, [SPAN][2]
  uint32_t* s_who = reinterpret_cast<uint32_t*>(s_values + R * SMALL_AGG_SPAN);
  const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), d = static_cast<uint32_t>(c.d);
  const uint32_t base = blockIdx.x * SMALL_AGG_SPAN, n = min(SMALL_AGG_SPAN, d - base);
  // this wave's messages: their headers and the entries looked at first are read before the marks are cleared
  constexpr uint32_t NW = SMALL_AGG_THREADS / 64, PER = (SMALL_AGG_R + NW - 1) / NW;
  const bool counts = is_qsgd(c.quantizer) && c.L > 1;
  const uint32_t hdr = 1 + c.L + (counts ? c.L : 0);
  uint32_t nnz[PER], probe[PER], next[SHORT ? PER : 1];   // next: the 64 entries behind the first
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) {
    const uint32_t p = wave + i * NW;
    nnz[i] = 0; probe[i] = 0;
    if (SHORT) next[i] = 0;
    if (p >= R) continue;                                // (uniform over the wave)
    const uint32_t* words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[p]) * c.cap_words * 4);
    nnz[i] = __builtin_amdgcn_readfirstlane(min(words[0], c.K));
    probe[i] = field_of(read_field(words, static_cast<uint64_t>(hdr) * 32 + static_cast<uint64_t>(lane * stride) * c.w_idx, c.cap_words), c.w_idx);
    if (SHORT && c.K > WAVE) next[i] = field_of(read_field(words, static_cast<uint64_t>(hdr) * 32 + static_cast<uint64_t>(lane + WAVE) * c.w_idx, c.cap_words), c.w_idx);
  }
  for (uint32_t i = threadIdx.x; i < 2 * SMALL_AGG_SPAN; i += SMALL_AGG_THREADS) s_who[i] = 0;
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) {
    const uint32_t p = wave + i * NW;
    if (p >= R) break;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[p]) * c.cap_words * 4);
    const uint64_t idx_bit0 = static_cast<uint64_t>(hdr) * 32, code_bit0 = (hdr + (static_cast<uint64_t>(nnz[i]) * c.w_idx + 31) / 32) * 32;
    auto code_at = [&](uint32_t j) { return read_field(words, code_bit0 + static_cast<uint64_t>(j) * c.w_val, c.cap_words); };
    auto put = [&](uint32_t at, const FieldRead& code) {
      const uint32_t seg = c.L == 1 ? 0u : seg_of_coord(c, at);
      s_values[p * SMALL_AGG_SPAN + (at - base)] = value_of_code(c, field_of(code, c.w_val), __uint_as_float(words[1 + seg]));
      atomicOr(&s_who[2 * (at - base) + (p >> 5)], 1u << (p & 31u));
    };
    const bool there = lane * stride < nnz[i];
    if (there && probe[i] >= d) atomicOr(c.status, 4u);  // malformed message: the entry is skipped
    if (SHORT) {
      if (there && probe[i] >= base && probe[i] - base < n) put(probe[i], code_at(lane));
      for (uint32_t j = lane + WAVE; j < nnz[i]; j += WAVE) {
        const uint32_t at = j < 2 * WAVE ? next[i] : field_of(read_field(words, idx_bit0 + static_cast<uint64_t>(j) * c.w_idx, c.cap_words), c.w_idx);
        if (at >= d) atomicOr(c.status, 4u);
        if (at >= base && at - base < n) put(at, code_at(j));
      }
      continue;
    }
    const uint32_t n_there = static_cast<uint32_t>(__popcll(__ballot(there)));
    const uint32_t n_lo = static_cast<uint32_t>(__popcll(__ballot(there && probe[i] < base))), n_hi = static_cast<uint32_t>(__popcll(__ballot(there && probe[i] < base + n)));
    uint32_t j0 = n_lo ? (n_lo - 1) * stride + 1 : 0u, end = n_hi < n_there ? n_hi * stride : nnz[i];
    if (__ballot(there && probe[i] >= d) != 0) { j0 = 0; end = nnz[i]; }
    auto read = [&](auto steps) {                        // 64 entries from j0 on, or 256
      constexpr uint32_t STEPS = decltype(steps)::value;
      FieldRead fi[STEPS], fc[STEPS];
#pragma unroll
      for (uint32_t u = 0; u < STEPS; ++u) {
        const uint32_t j = min(j0 + u * WAVE + lane, nnz[i] - 1);
        fi[u] = read_field(words, idx_bit0 + static_cast<uint64_t>(j) * c.w_idx, c.cap_words);
        fc[u] = code_at(j);
      }
#pragma unroll
      for (uint32_t u = 0; u < STEPS; ++u) {
        const uint32_t at = field_of(fi[u], c.w_idx);
        if (j0 + u * WAVE + lane >= end) continue;
        if (at >= d) atomicOr(c.status, 4u);             // malformed message: the entry is skipped
        if (at >= base && at - base < n) put(at, fc[u]);
      }
      j0 += STEPS * WAVE;
    };
    while (j0 < end) {                                   // (uniform over the wave)
      if (end - j0 <= WAVE) read(std::integral_constant<uint32_t, 1>());
      else read(std::integral_constant<uint32_t, SMALL_AGG_STEPS>());
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += SMALL_AGG_THREADS) {
    uint64_t who = static_cast<uint64_t>(s_who[2 * i + 1]) << 32 | s_who[2 * i];
    if (who == 0) { if (!accumulate) out[base + i] = 0.0f; continue; }
    float sum = s_values[(__ffsll(static_cast<unsigned long long>(who)) - 1) * SMALL_AGG_SPAN + i];
    for (who &= who - 1; who; who &= who - 1) sum = sum + s_values[(__ffsll(static_cast<unsigned long long>(who)) - 1) * SMALL_AGG_SPAN + i];
    const float term = scale * sum;
    out[base + i] = accumulate ? out[base + i] + term : term;
  }
}

// Long messages (with directories).  One thread per entry: the thread that holds entry j of the q-th listed
// message looks its coordinate up in the other listed messages itself, AGG_GROUP messages at a time with the
// binary searches advancing in step (their probes are independent loads, so a step costs one memory round trip,
// not one per message); a directory narrows every search to the entries of one 1024-block.  The rule is the same -- the
// earliest listed message that holds a coordinate writes it, the values are added in list order -- but a wave
// serves 64 entries instead of 8, and kernels of this kind are bound by the number of waves they start
// (8 messages of 99,400 entries: 104 us with 8 threads per entry, 55 us this way; short messages are the
// other way round: 8 x 543 entries 8 us against 16 us).  Four searches at a time: with eight the kernel needs 83
// registers (5 waves per SIMD) and takes 56.6 us on those messages, with four 51 registers and 53 us, with two 58 us.
constexpr uint32_t AGG_GROUP = 4;

struct GroupSearch {
  MsgView v[AGG_GROUP];
  uint32_t lo[AGG_GROUP], hi[AGG_GROUP];
  int64_t pos[AGG_GROUP];       // where the coordinate is in message g, or -1
};

// positions of coordinate idx in n (<= 8) of the other listed messages: the o-th other message, o = o0 .. o0 + n - 1,
// is list entry o for o < q and o + 1 from there on.  The loads of a step are unconditional (a closed search
// reads entry 0 again, which every message buffer has room for) so that all of a group are in flight together.
// `fixed_pos` >= 0: where the coordinate stands in every message that holds all K entries (a segment kept whole under a
// quantiser that drops nothing: its entries are at the same places in every such message) -- no search then.
__device__ __forceinline__ void group_find(const DevCtx& c, const uint8_t* msg, const RowList& rows, uint32_t o0, uint32_t n,
                                           uint32_t q, uint32_t idx, const uint32_t* dir, uint32_t ndir, int64_t fixed_pos,
                                           GroupSearch& s) {
  const uint32_t t = idx >> AGG_DIR_SHIFT;
  uint32_t nnz[AGG_GROUP], dlo[AGG_GROUP], dhi[AGG_GROUP];
#pragma unroll
  for (uint32_t g = 0; g < AGG_GROUP; ++g) {                // headers and directory cells: one batch of loads
    const uint32_t o = min(o0 + g, o0 + n - 1);             // slots beyond n repeat the last message and stay closed
    const uint32_t p = o + (o >= q ? 1u : 0u);
    s.v[g].words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[p]) * c.cap_words * 4);
    nnz[g] = s.v[g].words[0];
    dlo[g] = dir ? dir[static_cast<uint64_t>(p) * ndir + t] : 0u;
    dhi[g] = dir ? dir[static_cast<uint64_t>(p) * ndir + t + 1] : 0xFFFFFFFFu;
  }
  const bool counts = is_qsgd(c.quantizer) && c.L > 1;
  const uint64_t hdr = 1 + static_cast<uint64_t>(c.L) + (counts ? c.L : 0);
#pragma unroll
  for (uint32_t g = 0; g < AGG_GROUP; ++g) {
    s.v[g].nnz = min(nnz[g], c.K);
    s.v[g].idx_bit0 = hdr * 32;
    s.v[g].code_bit0 = (hdr + (static_cast<uint64_t>(s.v[g].nnz) * c.w_idx + 31) / 32) * 32;
    s.pos[g] = -1; s.lo[g] = 0; s.hi[g] = 0;
    if (g < n) {
      if (s.v[g].nnz == c.d) s.pos[g] = idx;               // every coordinate is there (k = d): entry j is coordinate j
      else if (fixed_pos >= 0 && s.v[g].nnz == c.K) s.pos[g] = fixed_pos;
      else { s.hi[g] = min(dhi[g], s.v[g].nnz); s.lo[g] = min(dlo[g], s.hi[g]); }
    }
  }
  for (uint32_t step = 0; step < 33; ++step) {             // a window of 2^32 entries is empty after 33 halvings
    bool open = false;
    uint32_t mid[AGG_GROUP], w0[AGG_GROUP], w1[AGG_GROUP];
#pragma unroll
    for (uint32_t g = 0; g < AGG_GROUP; ++g) {
      const bool active = s.lo[g] < s.hi[g];
      open = open || active;
      mid[g] = active ? s.lo[g] + ((s.hi[g] - s.lo[g]) >> 1) : 0u;
      const uint64_t bit = s.v[g].idx_bit0 + static_cast<uint64_t>(mid[g]) * c.w_idx;
      w0[g] = s.v[g].words[bit >> 5];
      w1[g] = s.v[g].words[(bit >> 5) + 1];
    }
    if (!open) break;
#pragma unroll
    for (uint32_t g = 0; g < AGG_GROUP; ++g) {
      const uint64_t bit = s.v[g].idx_bit0 + static_cast<uint64_t>(mid[g]) * c.w_idx;
      const uint32_t x = static_cast<uint32_t>(((static_cast<uint64_t>(w1[g]) << 32) | w0[g]) >> (bit & 31)) &
                         (c.w_idx == 32 ? 0xFFFFFFFFu : (1u << c.w_idx) - 1u);
      if (s.lo[g] < s.hi[g]) {
        if (x == idx) { s.pos[g] = mid[g]; s.hi[g] = s.lo[g]; }
        else if (x < idx) s.lo[g] = mid[g] + 1;
        else s.hi[g] = mid[g];
      }
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_aggregate_entries(DevCtx c, const uint8_t* msg, RowList rows, uint32_t R,
                                                             float scale, int accumulate, float* out, const uint32_t* dir,
                                                             uint32_t ndir) {
  const uint32_t q = blockIdx.y;
  const MsgView mine = view_msg(c, msg, rows.row[q]);
  const uint32_t stride = gridDim.x * BLOCK;
  GroupSearch s;
  for (uint32_t j = blockIdx.x * BLOCK + threadIdx.x; j < mine.nnz; j += stride) {
    const uint32_t idx = msg_index(c, mine, j);
    if (idx >= c.d) { atomicOr(c.status, 4u); continue; }          // malformed message
    const uint32_t seg = c.L == 1 ? 0u : seg_of_coord(c, idx);
    // a segment that is kept whole (k = size, e.g. the small tensors under a per-tensor rule) by a quantiser that drops
    // nothing stands at the same places in every full message
    int64_t fixed_pos = -1;
    if (c.L > 1 && !is_qsgd(c.quantizer) && mine.nnz == c.K && c.seg_whole[seg])
      fixed_pos = static_cast<int64_t>(c.seg_koff[seg]) + (idx - c.seg_start[seg]);
    // ... so if the first listed message is full it owns the coordinate: nothing to look up for the others' threads
    if (fixed_pos >= 0 && q > 0 &&
        reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[0]) * c.cap_words * 4)[0] == c.K) continue;
    const uint32_t my_code = get_bits(mine.words, mine.code_bit0 + static_cast<uint64_t>(j) * c.w_val, c.w_val);
    float acc = value_of_code(c, my_code, __uint_as_float(mine.words[1 + seg]));
    bool owned = false;                                            // an earlier listed message holds the coordinate: its thread writes it
    for (uint32_t o0 = 0; o0 + 1 < R && !owned; o0 += AGG_GROUP) {
      const uint32_t n = min(AGG_GROUP, R - 1 - o0);
      group_find(c, msg, rows, o0, n, q, idx, dir, ndir, fixed_pos, s);
      uint32_t w0[AGG_GROUP], w1[AGG_GROUP]; float sc[AGG_GROUP];
#pragma unroll
      for (uint32_t g = 0; g < AGG_GROUP; ++g) {              // code fields and scales of the group, found or not: one batch
        const uint64_t bit = s.v[g].code_bit0 + static_cast<uint64_t>(s.pos[g] >= 0 ? s.pos[g] : 0) * c.w_val;
        const uint64_t w = min(bit >> 5, static_cast<uint64_t>(c.cap_words) - 2);
        w0[g] = s.v[g].words[w]; w1[g] = s.v[g].words[w + 1];
        sc[g] = __uint_as_float(s.v[g].words[1 + seg]);
        if (s.pos[g] >= 0 && o0 + g < q) owned = true;
      }
#pragma unroll
      for (uint32_t g = 0; g < AGG_GROUP; ++g) {
        if (s.pos[g] >= 0 && o0 + g >= q) {
          const uint64_t bit = s.v[g].code_bit0 + static_cast<uint64_t>(s.pos[g]) * c.w_val;
          const uint64_t w = min(bit >> 5, static_cast<uint64_t>(c.cap_words) - 2);        // the pair of words that was loaded
          const uint32_t code = static_cast<uint32_t>(((static_cast<uint64_t>(w1[g]) << 32) | w0[g]) >> (bit - w * 32)) &
                                (c.w_val == 32 ? 0xFFFFFFFFu : (1u << c.w_val) - 1u);
          acc = acc + value_of_code(c, code, sc[g]);
        }
      }
    }
    if (owned) continue;
    const float term = scale * acc;
    out[idx] = accumulate ? out[idx] + term : term;
  }
}

// Long messages, or many: work linear in the number of entries.  A wave owns the 1024 coordinates of a directory cell (or
// a part of them) and has an image of them in LDS.  Through the directories it finds the listed messages' entries of its range; they are
// decoded 64 at a time, side by side, whichever message they come from, and added into the image message after message in
// list order: a message's coordinates are distinct, so the additions of one message do not meet, and a wave's LDS accesses
// are done in order, so no barrier is needed anywhere.  A place of the image that nothing was added to holds NOBODY.  Then
// the range of the model is updated, four coordinates at a time.
// What bounds a wave is the chain of its reads (directory, entries, model: about a microsecond each), so what counts is
// how many waves are in flight (2048 or 4096 coordinates per wave: slower on every shape tried) and that none is much longer
// than the others: a cell in which the plan expects many entries (segments kept whole, or nearly) is given to several
// waves, ahead of the others in the grid (a part's ends by bisection).  Measured, directories included, d = 25.6 M: 8 / 15 /
// 32 / 64 messages of 99,400 entries in 161 tensors 42 / 46 / 82 / 169 us (by look-ups 53 / 129 / 440 / 1480 us; by ranges
// added up message after message, a block of 1024 threads per crowded one: 32 / 64 messages 279 / 490 us); 2 / 4 / 8 messages
// of 2.6 M entries 71 / 93 / 140 us (by look-ups 172 / 336 / 1109 us).
constexpr uint32_t AGG_CELL = 1u << AGG_DIR_SHIFT;       // coordinates per directory cell
constexpr uint32_t AGG_SCALES = 192;                     // scales (segments of the range x messages) and ...
constexpr uint32_t AGG_SEGS = 32;                        // ... segments that a wave has room for in LDS
constexpr uint32_t AGG_LEVELS = 3;
constexpr uint32_t AGG_LEVEL[AGG_LEVELS] = {512, 128, 32};       // lists of crowded cells: more entries of one message than this
constexpr uint32_t NOBODY = 0xFFFFFFFFu;                 // a NaN that no value and no sum is (a sum keeps the payload of its NaN)

struct AggPart { uint32_t t; uint16_t i, parts; };       // part i of the 2^parts equal parts of cell t
struct AggCrowd { const AggPart* part; const uint32_t* bits; uint32_t n; };   // the parts of a level's crowded cells; a bit per cell (null: none is crowded)

// `split`: the cells that are not crowded are given to 2^split waves each (few cells with many entries: a short vector).
// `pile`: cells that no plan could foresee, in a vector whose large coordinates stand side by side (AGG_PILE entries or more, a
// whole 64 of them from one message).  With a list of them the launch with PILE set gives each to 16 or 32 waves, and
// their own waves leave them alone; without one they are worked through as they are and the host hears of it.
// 10^6 coordinates, 10,000 entries among the first 12,000, 8 / 16 / 32 / 64 messages: 102 / 184 / 203 / 227 us without a list, 49 / 52 / 61 / 84
// with one.
constexpr uint32_t AGG_PILE = 2048;
// (uniform) whether the cell whose entries of message `lane` are [lo, hi) is such a one
__device__ __forceinline__ bool piled_up(uint32_t lo, uint32_t hi, uint32_t split) {
  const bool whole = hi > lo && ((lo + 63u) & ~63u) + 64 <= hi;
  return __ballot(whole) != 0 && wave_sum(hi > lo ? min(hi - lo, AGG_CELL) : 0u) >= AGG_PILE << split;
}

// PILE: the listed cells, AGG_PILE_BLOCKS blocks.  Else a wave per item of the grid, which it returns from as soon as it can.
template <bool PILE>
__global__ __launch_bounds__(BLOCK, PILE ? 4 : 8) void k_aggregate_cells(DevCtx c, const uint8_t* msg, RowList rows, int in_order, uint32_t R,
                                                                         float scale, int accumulate, float* out, const uint32_t* dir,
                                                                         uint32_t ndir, AggCrowd crowd, uint32_t split, AggPile pile) {
  __shared__ f4u s_image[BLOCK / 64][AGG_CELL / 4];
  __shared__ float s_scale[BLOCK / 64][AGG_SCALES];
  __shared__ uint32_t s_segat[BLOCK / 64][AGG_SEGS];
  __shared__ uint32_t s_last;
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  float* image = reinterpret_cast<float*>(s_image[wave]);
  uint32_t n_items, parts = 0;
  if (PILE) {
    const uint32_t n = min(pile.count[0], ndir);
    if (n == 0) return;                                   // (uniform over the grid)
    parts = n <= 64 ? 5u : 4u;                            // (few of them: 40 messages, 3 cells of 27,000 entries 48 us in 16 parts, 38 in 32; 300 cells 844 and 858)
    n_items = n << parts;
  } else n_items = crowd.n + ((ndir - 1) << split);       // (no barrier follows)
  for (uint32_t b = blockIdx.x * (BLOCK / 64) + wave; b < n_items; b += gridDim.x * (BLOCK / 64)) {
  if (PILE) {                                             // the LDS of the item before is used again
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // ---- the messages: lane p is listed message p
  const bool counts = is_qsgd(c.quantizer) && c.L > 1;
  const uint32_t hdr = 1 + c.L + (counts ? c.L : 0);
  uint32_t my_row = lane < R ? lane : 0u;
  if (!in_order) my_row = rows.row[lane];
  const uint32_t* my_words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(my_row) * c.cap_words * 4);
  // ---- the coordinates: a cell, or a part of a crowded one
  uint32_t t0, from, width;
  const bool crowded = !PILE && b < crowd.n, is_part = PILE || crowded || split != 0;
  if (PILE) { t0 = pile.list[b >> parts]; width = AGG_CELL >> parts; from = (b & ((1u << parts) - 1u)) * width; }
  else if (crowded) { const AggPart a = crowd.part[b]; t0 = a.t; width = AGG_CELL >> a.parts; from = a.i * width; }
  else { t0 = (b - crowd.n) >> split; width = AGG_CELL >> split; from = ((b - crowd.n) & ((1u << split) - 1u)) * width; }
  const uint32_t* my_dir = dir + static_cast<uint64_t>(lane < R ? lane : 0u) * ndir + t0;
  const uint32_t my_nnz = lane < R ? min(my_words[0], c.K) : 0u;
  uint32_t lo = lane < R ? min(my_dir[0], my_nnz) : 0u, hi = lane < R ? min(my_dir[1], my_nnz) : 0u;
  uint32_t seg0 = 0, ns = 1;
  if (c.L > 1 && !is_part) { seg0 = c.seg_dir[t0]; ns = c.seg_dir[t0 + 1] - seg0 + 1; }
  if (!crowded && crowd.bits != nullptr && ((crowd.bits[t0 >> 5] >> (t0 & 31u)) & 1u)) { if (PILE) continue; return; }      // waves of its own look after it
  if (PILE) {
    if (!piled_up(lo, hi, split)) continue;
    if (lane == 0 && from == 0 && pile.flag != nullptr) *pile.flag = 1u;
  } else if (split != 0 && !crowded && piled_up(lo, hi, split)) {
    if (pile.list != nullptr) return;
    if (lane == 0 && pile.flag != nullptr) *pile.flag = 1u;
  }
  const float nobody = __uint_as_float(NOBODY);
  uint64_t c0 = static_cast<uint64_t>(t0) << AGG_DIR_SHIFT;
  uint32_t span = AGG_CELL;
  if (is_part) {
    // the part's entries among the cell's [lo, hi): both ends by bisection in step, every step reads the quarter points
    const uint32_t la = lo, lb = max(lo, hi), f1 = from + width;
    uint32_t l0 = la, h0 = from == 0 ? la : lb, l1 = f1 >= AGG_CELL ? lb : la, h1 = lb;
    if (lb - la == AGG_CELL) { l0 = h0 = la + from; l1 = h1 = la + f1; }        // every coordinate is there
    auto at = [&](uint32_t j) { return field_of(read_field(my_words, static_cast<uint64_t>(hdr) * 32 + static_cast<uint64_t>(min(j, my_nnz - 1)) * c.w_idx, c.cap_words), c.w_idx); };
    while (l0 < h0 || l1 < h1) {
      uint32_t m0[3], m1[3], x0[3], x1[3];
#pragma unroll
      for (uint32_t q = 0; q < 3; ++q) {
        m0[q] = l0 + ((h0 - l0) * (q + 1) >> 2); m1[q] = l1 + ((h1 - l1) * (q + 1) >> 2);
        x0[q] = at(m0[q]); x1[q] = at(m1[q]);
      }
      if (l0 < h0) {
        if (!(x0[0] < c0 + from)) h0 = m0[0];
        else if (!(x0[1] < c0 + from)) { l0 = m0[0] + 1; h0 = m0[1]; }
        else if (!(x0[2] < c0 + from)) { l0 = m0[1] + 1; h0 = m0[2]; }
        else l0 = m0[2] + 1;
      }
      if (l1 < h1) {
        if (!(x1[0] < c0 + f1)) h1 = m1[0];
        else if (!(x1[1] < c0 + f1)) { l1 = m1[0] + 1; h1 = m1[1]; }
        else if (!(x1[2] < c0 + f1)) { l1 = m1[1] + 1; h1 = m1[2]; }
        else l1 = m1[2] + 1;
      }
    }
    lo = l0; hi = l1; c0 += from; span = width;
  }
  if (c0 >= c.d) { if (PILE) continue; return; }
  const uint32_t cnt = hi > lo ? min(hi - lo, span) : 0u; // a well-formed message has at most one entry per coordinate
  if (hi > lo && hi - lo > span) atomicOr(c.status, 4u);  // malformed: what is beyond that is skipped
  span = static_cast<uint32_t>(min<uint64_t>(span, c.d - c0));
  const uint32_t base = static_cast<uint32_t>(c0);
  uint32_t n;
  const uint32_t before = wave_exclusive_scan32(cnt, &n);
  if (n == 0 && accumulate) { if (PILE) continue; return; }
  if (!is_part && n >= AGG_PILE && piled_up(lo, hi, 0)) {     // (a cell in parts has been looked at as a whole above)
    if (pile.list != nullptr) return;
    if (lane == 0 && pile.flag != nullptr) *pile.flag = 1u;
  }
  if (c.L > 1 && is_part) { seg0 = seg_of_coord(c, base); ns = seg_of_coord(c, base + span - 1) - seg0 + 1; }
  // lane p, for the lanes that decode entries of message p: entry f of the item is the message's entry f + my_j
  const uint32_t my_j = lo - before;
  const uint32_t my_code = hdr + static_cast<uint32_t>((static_cast<uint64_t>(my_nnz) * c.w_idx + 31) / 32);      // first word of its codes
  constexpr uint32_t UN = 4;                              // steps of 64 entries whose reads are in flight together
  FieldRead fi[UN], fc[UN]; uint32_t pp[UN];
  auto load = [&](uint32_t f0) {
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      if (f0 + u * WAVE >= n) break;                      // (uniform)
      const uint32_t f = f0 + u * WAVE + lane;
      uint32_t a = 0;                                     // the last message whose entries begin at or before f
      for (uint32_t step = R > 32 ? 32u : R > 16 ? 16u : R > 8 ? 8u : R > 4 ? 4u : R > 2 ? 2u : 1u; step; step >>= 1) {
        const uint32_t m = a + step;
        const uint32_t x = __shfl(before, m & 63u, WAVE);
        if (m < R && x <= f) a = m;
      }
      pp[u] = a;
      const uint32_t j = f + __shfl(my_j, a, WAVE), code0 = __shfl(my_code, a, WAVE), row = __shfl(my_row, a, WAVE);
      if (f < n) {
        const uint32_t* words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(row) * c.cap_words * 4);
        fi[u] = read_field(words, static_cast<uint64_t>(hdr) * 32 + static_cast<uint64_t>(j) * c.w_idx, c.cap_words);
        fc[u] = read_field(words, static_cast<uint64_t>(code0) * 32 + static_cast<uint64_t>(j) * c.w_val, c.cap_words);
      }
    }
  };
  load(0);
  // the segments of the range and every message's scales: one segment -- lane p its message's scale; several -- in LDS
  const bool table = ns <= AGG_SEGS && ns * R <= AGG_SCALES;
  float my_scale = 0.0f;
  if (ns == 1) my_scale = lane < R ? __uint_as_float(my_words[1 + seg0]) : 0.0f;
  else if (table) {
    if (lane < ns) s_segat[wave][lane] = c.seg_start[seg0 + lane];
    for (uint32_t i = lane; i - lane < ns * R; i += WAVE) {
      const uint32_t p = i / ns, g = i - p * ns, row = __shfl(my_row, p & 63u, WAVE);
      if (p < R) s_scale[wave][i] = reinterpret_cast<const float*>(msg + static_cast<uint64_t>(row) * c.cap_words * 4)[1 + seg0 + g];
    }
  }
  for (uint32_t i = lane; i * 4 < span; i += WAVE) s_image[wave][i] = f4u{nobody, nobody, nobody, nobody};
  // ---- decode and add
  for (uint32_t f0 = 0; f0 < n; f0 += UN * WAVE) {
    if (f0) load(f0);
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      if (f0 + u * WAVE >= n) break;                      // (uniform)
      const bool mine = f0 + u * WAVE + lane < n;
      const uint32_t idx = field_of(fi[u], c.w_idx), loc = idx - base;
      const bool ok = mine && idx >= base && loc < span;
      float sc = __shfl(my_scale, pp[u], WAVE);
      if (ns > 1) {
        if (table) {
          uint32_t a = 0, z = ns;
          while (z - a > 1) { const uint32_t mid = (a + z) >> 1; if (s_segat[wave][mid] <= idx) a = mid; else z = mid; }
          sc = s_scale[wave][pp[u] * ns + a];
        } else {
          const uint32_t row = __shfl(my_row, pp[u], WAVE);
          if (ok) sc = reinterpret_cast<const float*>(msg + static_cast<uint64_t>(row) * c.cap_words * 4)[1 + seg_of_coord(c, idx)];
        }
      }
      if (mine && !ok) atomicOr(c.status, 4u);            // malformed message: the entry is skipped
      float v = value_of_code(c, field_of(fc[u], c.w_val), sc);
      if ((__float_as_uint(v) | 0x400000u) == NOBODY) v = __uint_as_float(NOBODY - 1u);      // that NaN, quiet or not: the one beside it
      uint64_t todo = __ballot(ok);
      while (todo) {                                      // the messages of this step, in order
        const uint32_t p = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(pp[u]), __ffsll(static_cast<unsigned long long>(todo)) - 1));
        const bool now = ok && pp[u] == p;
        if (now) {
          const float have = image[loc];
          image[loc] = __float_as_uint(have) == NOBODY ? v : have + v;
        }
        todo &= ~__ballot(now);
        // the next message may hold the same coordinates in other lanes: order the LDS traffic (the lanes run in lockstep)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // ---- the range of the model
  constexpr uint32_t ON = 4;
  for (uint32_t i0 = lane * 4; i0 - lane * 4 < span; i0 += ON * WAVE * 4) {
    f4u a[ON], o[ON];
    bool any[ON];
#pragma unroll
    for (uint32_t u = 0; u < ON; ++u) {
      const uint32_t i = i0 + u * WAVE * 4;
      any[u] = false;
      a[u] = f4u{nobody, nobody, nobody, nobody}; o[u] = f4u{0.f, 0.f, 0.f, 0.f};
      if (i < span) {
        a[u] = s_image[wave][i / 4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) any[u] = any[u] || __float_as_uint(a[u][j]) != NOBODY;
        any[u] = any[u] || !accumulate;                   // without `accumulate` the coordinates nobody holds are written too
        if (any[u] && accumulate) {
          if (i + 4 <= span) o[u] = *reinterpret_cast<const f4u*>(out + c0 + i);
          else for (uint32_t j = 0; j < 4; ++j) if (i + j < span) o[u][j] = out[c0 + i + j];
        }
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < ON; ++u) {
      const uint32_t i = i0 + u * WAVE * 4;
      if (!any[u]) continue;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if (__float_as_uint(a[u][j]) != NOBODY) { const float term = scale * a[u][j]; o[u][j] = accumulate ? o[u][j] + term : term; }
      if (i + 4 <= span) *reinterpret_cast<f4u*>(out + c0 + i) = o[u];
      else for (uint32_t j = 0; j < 4; ++j) if (i + j < span) out[c0 + i + j] = o[u][j];
    }
  }
  if (!PILE) return;
  }
  if (!PILE) return;                                      // (a wave beyond the last item)
  __syncthreads();                                        // the last block to be done clears the list for the next call
  if (threadIdx.x == 0) s_last = atomicAdd(&pile.count[1], 1u) + 1 == gridDim.x;
  __syncthreads();
  if (s_last == 0) return;
  for (uint32_t i = threadIdx.x; i < n_items >> parts; i += BLOCK) pile.bits[pile.list[i] >> 5] = 0;
  if (threadIdx.x == 0) { pile.count[0] = 0; pile.count[1] = 0; }
}

// The master line when every message holds every coordinate (an operator with k = d whose quantiser drops
// nothing, e.g. the sign of the whole vector): entry j of a message is coordinate j, so the sum is a plain
// pass over the coordinates, in the same list order and with the same roundings as k_aggregate.  An
// all-zero (empty) message adds nothing; any other entry count is reported as a malformed message.
// four consecutive coordinates from j0 on (nj of them exist); `o`: what `out` holds there (if accumulate)
__device__ __forceinline__ void aggregate_dense_quad(const DevCtx& c, const uint8_t* __restrict__ msg, const RowList& rows, uint32_t R,
                                                     float scale, int accumulate, float* __restrict__ out, uint64_t code_bit0,
                                                     uint64_t j0, uint32_t nj, f4u o) {
  uint32_t seg[4] = {0u, 0u, 0u, 0u};
  if (c.L > 1) {
    seg[0] = seg_of_coord(c, static_cast<uint32_t>(j0));
    seg[3] = seg_of_coord(c, static_cast<uint32_t>(j0 + nj - 1));
    seg[1] = seg[2] = seg[0];
    if (seg[3] != seg[0]) {
      seg[1] = nj > 1 ? seg_of_coord(c, static_cast<uint32_t>(j0 + 1)) : seg[0];
      seg[2] = nj > 2 ? seg_of_coord(c, static_cast<uint32_t>(j0 + 2)) : seg[0];
    }
  }
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  bool first = true;
  for (uint32_t p = 0; p < R; ++p) {
    const uint32_t* words = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[p]) * c.cap_words * 4);
    const uint32_t nnz = words[0];
    if (nnz != c.d) {
      if (nnz != 0 && j0 == 0) atomicOr(c.status, 4u);
      continue;
    }
    // the codes of the four coordinates are consecutive in the stream: up to 8 bits each come in one read
    // (77 -> 62 us for two messages of 25.6 M one-bit codes; with the value computed per code, as here, a wave per 1024
    // coordinates and the reads of several messages together were slower, 72 - 77 us: k_aggregate_dense_one looks it up)
    const bool packed = c.w_val <= 8;                      // uniform
    const uint32_t four = packed ? get_bits(words, code_bit0 + j0 * c.w_val, nj * c.w_val) : 0u;
    const float scale0 = __uint_as_float(words[1 + seg[0]]);
#pragma unroll
    for (uint32_t jj = 0; jj < 4; ++jj) {
      if (jj < nj) {
        const uint32_t code = packed ? (four >> (jj * c.w_val)) & ((1u << c.w_val) - 1u)
                                     : get_bits(words, code_bit0 + (j0 + jj) * c.w_val, c.w_val);
        const float sc = seg[jj] == seg[0] ? scale0 : __uint_as_float(words[1 + seg[jj]]);
        const float val = value_of_code(c, code, sc);
        acc[jj] = first ? val : acc[jj] + val;
      }
    }
    first = false;
  }
  if (first && accumulate) return;                       // no message had anything to add
#pragma unroll
  for (uint32_t jj = 0; jj < 4; ++jj) {
    const float term = scale * acc[jj];
    o[jj] = first ? 0.0f : accumulate ? o[jj] + term : term;
  }
  if (nj == 4) *reinterpret_cast<f4u*>(out + j0) = o;
  else for (uint32_t jj = 0; jj < nj; ++jj) out[j0 + jj] = o[jj];
}

// A thread takes two groups of four consecutive coordinates at a time, a grid's width apart; what `out` holds of both is
// read first (one group: 62 us for two messages of 25.6 M one-bit codes; its read of `out` before those of the messages
// instead of after them: 59 us; two groups: 57 us; with streaming hints on `out`, which the next round's call finds
// partly in the last-level cache otherwise: 61 us).
__global__ __launch_bounds__(BLOCK) void k_aggregate_dense(DevCtx c, const uint8_t* __restrict__ msg, RowList rows, uint32_t R,
                                                           float scale, int accumulate, float* __restrict__ out) {
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * BLOCK;
  const uint64_t n4 = (c.d + 3) / 4;
  const bool counts = is_qsgd(c.quantizer) && c.L > 1 && !c.dense;
  const uint64_t hdr = 1 + static_cast<uint64_t>(c.L) + (counts ? c.L : 0);
  const uint64_t code_bit0 = (hdr + (c.d * c.w_idx + 31) / 32) * 32;      // of a message that holds all d entries
  for (uint64_t g = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x; g < n4; g += 2 * stride) {
    const uint64_t ja = g * 4, jb = (g + stride) * 4;
    const uint32_t na = static_cast<uint32_t>(min<uint64_t>(4, c.d - ja));
    const uint32_t nb = g + stride < n4 ? static_cast<uint32_t>(min<uint64_t>(4, c.d - jb)) : 0u;
    f4u oa = {0.f, 0.f, 0.f, 0.f}, ob = {0.f, 0.f, 0.f, 0.f};
    if (accumulate) {
      if (na == 4) oa = *reinterpret_cast<const f4u*>(out + ja);
      else for (uint32_t jj = 0; jj < na; ++jj) oa[jj] = out[ja + jj];
      if (nb == 4) ob = *reinterpret_cast<const f4u*>(out + jb);
      else for (uint32_t jj = 0; jj < nb; ++jj) ob[jj] = out[jb + jj];
    }
    aggregate_dense_quad(c, msg, rows, R, scale, accumulate, out, code_bit0, ja, na, oa);
    if (nb) aggregate_dense_quad(c, msg, rows, R, scale, accumulate, out, code_bit0, jb, nb, ob);
  }
}

// The same for one segment and narrow codes.
// A wave per 1024 coordinates, four times four per lane; what `out` holds of them and the codes of several messages are read
// before anything waits.  What a code stands for is looked up: one-bit codes choose between two values that the whole wave
// shares, codes of up to eight bits index a table in LDS that the block makes first (all messages' values of all codes), if
// it has room for that; everything else is computed value by value, by k_aggregate_dense.  Measured: 2 x 25.6 M coordinates
// 46 us with one-bit codes, 47 us with five-bit ones (k_aggregate_dense: 69 and 71 us), 13 x 17.2 M four-bit codes 58 us;
// held to 6 waves per SIMD 51, 52 and 58 us, to 8: 51, 63 and 74 us.
enum { AGG_SIGN, AGG_TABLE };
constexpr uint32_t AGG_TABLE_MAX = 2048;
template <int MODE>
__global__ __launch_bounds__(BLOCK) void k_aggregate_dense_one(DevCtx c, const uint8_t* __restrict__ msg, RowList rows, uint32_t R,
                                                               float scale, int accumulate, float* __restrict__ out) {
  __shared__ float s_value[MODE == AGG_TABLE ? AGG_TABLE_MAX : 1];
  const uint32_t lane = lane_id(), wv = c.w_val;
  const uint64_t chunk = static_cast<uint64_t>(blockIdx.x) * (BLOCK / 64) + (threadIdx.x >> 6), base = chunk * CHUNK;
  const uint32_t valid = base < c.d ? static_cast<uint32_t>(min(static_cast<uint64_t>(CHUNK), c.d - base)) : 0u;
  const uint64_t code_bit0 = (2 + (c.d * c.w_idx + 31) / 32) * 32 + base * wv;      // of the chunk, in a message that holds all d entries
  auto words_of = [&](uint32_t p) { return reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(rows.row[p]) * c.cap_words * 4); };
  f4u o[4], acc[4];
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
    o[t] = acc[t] = f4u{0.f, 0.f, 0.f, 0.f};
    if (accumulate) {
      if (valid == CHUNK) o[t] = *reinterpret_cast<const f4u*>(out + base + e);
      else {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) o[t][j] = out[base + e + j];
      }
    }
  }
  if (MODE == AGG_TABLE) {
    for (uint32_t i = threadIdx.x; i < R << wv; i += BLOCK) s_value[i] = value_of_code(c, i & ((1u << wv) - 1u), __uint_as_float(words_of(i >> wv)[1]));
    __syncthreads();
  }
  if (valid == 0) return;
  bool first = true;
  constexpr uint32_t UN = 2;                           // messages whose codes are read together
  for (uint32_t p0 = 0; p0 < R; p0 += UN) {
    uint32_t four[UN][4], nnz[UN];                     // the lane's four codes of each group, at most 32 bits
    float sc[UN];
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      if (p0 + u >= R) break;
      const uint32_t* words = words_of(p0 + u);
      nnz[u] = words[0]; sc[u] = __uint_as_float(words[1]);
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t) {
        const uint32_t e = t * 256 + lane * 4;
        if (MODE == AGG_SIGN) four[u][t] = e < valid ? words[(code_bit0 >> 5) + (e >> 5)] >> (e & 31u) : 0u;      // (a chunk's bits begin with a word)
        else { const FieldRead f = read_field(words, code_bit0 + e * wv, c.cap_words); four[u][t] = static_cast<uint32_t>((static_cast<uint64_t>(f.w.y) << 32 | f.w.x) >> f.sh); }
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < UN; ++u) {
      if (p0 + u >= R) break;
      if (nnz[u] != c.d) {
        if (nnz[u] != 0 && chunk == 0 && lane == 0) atomicOr(c.status, 4u);
        continue;
      }
      const float* value = s_value + (MODE == AGG_TABLE ? (p0 + u) << wv : 0u);
      const uint32_t mask = (1u << wv) - 1u;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          float val;
          if (MODE == AGG_SIGN) val = (four[u][t] >> j) & 1u ? -sc[u] : sc[u];
          else val = value[(four[u][t] >> (j * wv)) & mask];
          acc[t][j] = first ? val : acc[t][j] + val;
        }
      }
      first = false;
    }
  }
  if (first && accumulate) return;                       // no message had anything to add
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    const uint32_t e = t * 256 + lane * 4;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const float term = scale * acc[t][j];
      o[t][j] = first ? 0.0f : accumulate ? o[t][j] + term : term;
    }
    if (valid == CHUNK) *reinterpret_cast<f4u*>(out + base + e) = o[t];
    else {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) if (e + j < valid) out[base + e + j] = o[t][j];
    }
  }
}

__global__ void k_read_nnz(DevCtx c, const uint8_t* msg, uint32_t R, uint32_t* out) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < R) out[r] = reinterpret_cast<const uint32_t*>(msg + static_cast<uint64_t>(r) * c.cap_words * 4)[0];
}

}  // namespace
