// The host's launch rules: which kernel and which grid a call gets, from its
// sizes alone.  Plain C++ without device code, so that a test without a GPU can
// ask them.
#pragma once

#include <stddef.h>

#include <algorithm>

#include "eldr_moe.h"

namespace eldr {

// ----------------------------------------------------------------- moe_bucket

constexpr int kBucketMaxWords = 16384;  // E * ceil(T / 32) limit
constexpr int kBucketSmall = 256;       // tokens of a batch counted by one thread an expert
constexpr int kBucketPairs = 2048;      // pairs a workgroup writes: two a thread
constexpr int kBucketMaxWgs = 16;

// Words from one expert's bitmap to the next: odd, so that the lanes of a
// wave, which set bits of a few words of many experts, hit different LDS banks.
constexpr int bucket_stride(int T) { return ((T + 31) / 32) | 1; }

// Bitmaps, bits before each of their words, and four tables of E entries.
constexpr size_t bucket_lds_bytes(int T, int E) {
  const size_t EW = (size_t)E * bucket_stride(T);
  return EW * 4 + ((EW + 1) & ~(size_t)1) * 2 + (size_t)E * 4 * 4;
}

struct BucketLaunch {
  bool large;  // several threads an expert
  int wgs;
  size_t lds;
};

// One workgroup up to 2048 pairs (a decode batch of 256 tokens at top-8), then
// as many as leave each about that many to write, up to 16: past that every
// workgroup's own pass over the ids is most of its time.  With pair_pos written
// over topk_ids one workgroup at any size: it has read every id before it writes,
// and a thread reads an id again before it replaces it, while another workgroup
// might still be counting.
inline BucketLaunch bucket_launch(int T, int E, int K, bool in_place) {
  const int wgs = std::min(kBucketMaxWgs, (T * K + kBucketPairs - 1) / kBucketPairs);
  return {T > kBucketSmall, in_place ? 1 : std::max(1, wgs), bucket_lds_bytes(T, E)};
}

}  // namespace eldr
