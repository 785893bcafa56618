// qsl_policy.h -- What the host makes of the failures that the kernels report through pinned words (a report may be seen a few calls
// late), and which of the master line's kernels it takes for given sizes.  Only speed depends on any of it, never the result.  Plain C++,
// no HIP.
#pragma once

#include <algorithm>
#include <cstdint>

namespace {

// Guessing units (Top_k takes its guesses from the previous call, or from a sample; Rand_k's are fixed).  Three kinds of failure:
//   mild      made good by many blocks, or by one block on a small unit.  When it happens again within 16 calls, the next 32 take
//             their guesses from samples, as a context's first call does (15 workers of 5.4 M coordinates whose thresholds jump
//             from call to call: 490 us a call that way, 1000 with failed guesses made good; 260 undisturbed).  If guesses keep
//             failing all the same, the multi-pass kernels stand by for the units whose guess fails.
//   crawl     one block walked through a large unit, for milliseconds: the next four calls take samples at once, so that a
//             second jump costs no second walk.
//   hopeless  the same, and no sample would have helped (too few non-zero values, ties): the multi-pass kernels stand by for 16
//             calls, and again at the next such failure.
struct GuessPolicy {
  uint32_t safe_left = 0;      // calls still to be made with the multi-pass kernels standing by
  uint32_t cold_left = 0;      // calls still to be made with sampled guesses
  uint32_t recent_left = 0;    // calls for which the last failure still counts as recent
  uint32_t strikes = 0;        // mild failures reported while guesses were sampled
  bool last_cold = false;      // the previous call sampled

  struct Call { bool safe, cold; };
  // `must`: the call samples in any case (its context's first one, or a flag)
  Call next(bool mild, bool crawl, bool hopeless, bool must) {
    if (mild || crawl || hopeless) {
      if (hopeless || (crawl && last_cold)) safe_left = 16;
      else {
        if (cold_left > 0 && ++strikes > 3) safe_left = 16;
        if (cold_left == 0 && recent_left > 0) { cold_left = 32; strikes = 0; }
        else if (cold_left == 0 && crawl) { cold_left = 4; strikes = 0; }
      }
      recent_left = 16;
    } else if (recent_left > 0) --recent_left;
    Call c;
    c.safe = safe_left > 0;
    if (c.safe) --safe_left;
    c.cold = must || cold_left > 0;
    if (cold_left > 0) --cold_left;
    last_cold = c.cold;
    return c;
  }
};

// The window of a dense k (qsl_window.h).  While it fails -- the threshold among ties or zeros -- its kernels are left out and the
// multi-pass kernels take every unit at once: for 2, 8, 32 and then 128 calls after a failure, then it is tried again.  16 calls
// without a report, and the next failure starts at 2 again.
struct WindowPolicy {
  uint32_t skip_left = 0, backoff = 0, held = 0;
  bool next(bool failed) {     // whether this call tries the window
    if (failed) { backoff = std::min(128u, std::max(2u, 4 * backoff)); skip_left = backoff; held = 0; }
    if (skip_left > 0) { --skip_left; return false; }
    if (backoff > 0 && ++held > 16) backoff = 0;
    return true;
  }
};

// The master line: cells in which the messages' entries pile up (qsl_decode.h).  Once they are met, the next 64 calls list them and
// give them to many waves in a launch of its own, as do the calls after those while there still are any.
struct PilePolicy {
  uint32_t left = 0;
  bool next(bool met) {        // whether this call lists them
    if (met) left = 64;
    if (left == 0) return false;
    --left;
    return true;
  }
};

// Whether the directories of `R` messages of about `entries` entries each, `cells` of 1024 coordinates, are made by search
// (k_msg_directory_search) or by reading every entry (k_msg_directory).  A search waits for some eight dependent reads whatever there is
// to find, so there have to be about 3 M entries in all; its reads are scattered, twenty to a cell and message, so there
// have to be many entries to each of them, and fewer cells in all than keep the caches busy.  Entries that lie evenly, us for the master
// line by reading / by search: 100,001 coordinates, 4 messages, 48 to a cell 11.9 / 14.5; 10^6, 8, 100: 17.3 / 19.1; 10^6, 64, 48: 42.5 / 37.4; 4 M,
// 4, 200: 29.4 / 27.8; 25.6 M, 4, 100: 75.2 / 68.5; 25.6 M, 16, 48: 125 / 179; 60 M, 2, 64: 103 / 106; 25.6 M, 10, 200: 251 / 211.
inline bool directory_by_search(uint32_t entries, uint32_t cells, uint32_t R) {
  const uint64_t all = static_cast<uint64_t>(cells) * R, per_cell = entries / cells;
  return per_cell >= 48 && static_cast<uint64_t>(entries) * R >= 2900000 && all <= (per_cell >= 200 ? 256u << 10 : 112u << 10);
}

}  // namespace
