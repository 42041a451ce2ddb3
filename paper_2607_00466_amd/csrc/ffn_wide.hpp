// The expert FFN's kernel for batches whose buckets are large.
#pragma once

#include "ffn_common.hpp"

namespace eldr {

constexpr int kWideTokens = 128;  // tokens of one item

// Items an expert's rows make for one token group: 128 rows of W1 and of W3
// (up) or 256 rows of W2 (down) each.
template <int MODE>
constexpr int wide_tiles(int rows) {
  return MODE == kUp ? (rows + 127) / 128 : (rows + 255) / 256;
}

// Whether the wide kernel runs a projection of a batch of T > 64 tokens.  Its
// items are twice as long as the small-batch kernel's, so there must be enough
// of them to give every CU one: with E experts and T K / 128 further token
// groups about 300 (measured: 312 items +4%, 330 items +15%, but 280 items
// -6% and 171 items -14%).  With bf16 weights the buckets must also be large
// enough for the MFMAs to show: 20 tokens on average for the up projection (25
// tokens +6%; 16 tokens even, 18% with 64 of 128 experts active; 18.5 tokens
// -1%; 12.5 tokens of one domain -2%) and 12 for the down projection, which
// gains from staging h in whole lines (12.5 tokens +1%, of one domain +6%; 8
// tokens -2%); 32 where the reduction is short and an item's start weighs more
// (256 values: 9 and 16 tokens -6% and -7%, 62 tokens +14%).  MXFP4 streams a
// quarter of the bytes and gains earlier, from 4 tokens (gpt-oss shape: T =
// 128 +5%, 256 +3%, and +7% and +22% where 32 experts are active; at T = 80,
// 2.5 tokens, with 4 experts active -5%).
template <int MODE, int FMT>
bool ffn_wide_pays(int T, int K, int E, int rows, int kdim) {
  const long long items = (long long)wide_tiles<MODE>(rows) * (E + T * K / kWideTokens);
  return T > 64 && items >= 300 && T * K >= (FMT == kMxfp4 ? 4 : kdim < 512 ? 32 : MODE == kUp ? 20 : 12) * E;
}

// Launches the wide kernel (and sets a.tiles).
template <int MODE, int FMT>
void launch_ffn_wide(FfnArgs a, int T, int K, int E, hipStream_t s);

}  // namespace eldr
