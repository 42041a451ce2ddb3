// The expert FFN's kernel for batches of a few tokens.
#pragma once

#include <algorithm>

#include "ffn_common.hpp"

namespace eldr {

constexpr int kSlimTokens = 4;

// Whether the one-wave kernel runs a projection of a batch of T tokens.  Up to
// 4 tokens the union is small (at most T K experts) and the four-wave items of
// the other kernel leave CUs idle or unevenly loaded; measured up + down, with
// every shape tried ahead: T = 1 +12 to +44%, T = 4 +2 to +28%.  From 8 tokens
// its waves each staging the activations for themselves costs more than it
// gains where buckets fill (T = 8 in 4 experts, MXFP4: -16%; bf16 T = 8: -3%).
// The down projection keeps the four-wave items where they give each of the
// 256 CUs one and the bf16 reduction is too short to make up for a start of
// its own in every wave (768 values, T = 2 and 4: -7% and -9%).
template <int MODE, int FMT>
bool ffn_slim_pays(int T, int K, int E, int rows, int kdim) {
  if (T > kSlimTokens) return false;
  const int items = (rows + 127) / 128 * std::min(E, T * K);
  return !(MODE == kDown && FMT == kBf16 && kdim < 1024 && items >= 256);
}

// Launches it; ROUTED (up): the buckets are built from a.ids and written out.
template <int MODE, int FMT, bool ROUTED>
void launch_ffn_slim(const FfnArgs& args, int T, int K, int E, hipStream_t s);

}  // namespace eldr
