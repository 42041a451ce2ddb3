// The host's launch rules: which kernel and which grid a call gets, from its
// sizes alone.  Plain C++ without device code, so that a test without a GPU can
// ask them.
#pragma once

#include <stddef.h>

#include <algorithm>

#include "eldr_moe.h"

namespace eldr {

constexpr int kNumXcd = 8;  // MI355X: 8 XCDs, workgroups dispatched round-robin over them

// ----------------------------------------------------------------- moe_bucket

constexpr int kBucketMaxWords = 16384;  // E * ceil(T / 32) limit (without the odd stride)
constexpr int kBucketSmall = 256;       // tokens, and
constexpr int kBucketFew = 3072;        // pairs, of a batch counted by one thread an expert
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

static_assert(bucket_lds_bytes(2048, 256) == 103936, "the most that the limits admit: 104 KB");

struct BucketLaunch {
  bool large;  // several threads an expert
  int wgs;
  size_t lds;
};

// Several threads an expert, with eight ids in flight each, pay once a thread
// has more than about three pairs and an expert more than 8 words (one thread an
// expert against several: T = 300 top-8 of 128, 2400 pairs, 4.74 us against 5.47;
// T = 512 top-4 of 128 4.91 against 5.74; T = 700 top-2 of 8 4.17 against 4.75;
// but T = 512 top-8, 4096 pairs, 7.3 against 6.0).
//
// One workgroup up to 2048 pairs (a decode batch of 256 tokens at top-8), then
// as many as leave each about that many to write, up to 16: past that every
// workgroup's own pass over the ids is most of its time.  With pair_pos written
// over topk_ids one workgroup at any size: it has read every id before it writes,
// and a thread reads an id again before it replaces it, while another workgroup
// might still be counting.
inline BucketLaunch bucket_launch(int T, int E, int K, bool in_place) {
  const int wgs = std::min(kBucketMaxWgs, (T * K + kBucketPairs - 1) / kBucketPairs);
  return {T > kBucketSmall && T * K > kBucketFew, in_place ? 1 : std::max(1, wgs), bucket_lds_bytes(T, E)};
}

// --------------------------------------------------------------- gate scores

struct GateLaunch {
  int tile;       // tokens and experts of a workgroup's tile
  bool by_token;  // an XCD takes whole token tiles, each against every expert tile
};

// Tiles of 4 tokens x 4 experts up to 128 tokens: the most workgroups for a
// reduction that is one or two loads a lane long.  Above that 8 x 8: half the
// loads of x and of the gate rows per product (16 x 8 and 8 x 16 measured even
// from T = 512 and 15% slower at 256; 16 x 16 30% slower).  The scores are the
// same bits either way.  Above 256 tokens x outweighs the gate rows, so an XCD
// takes whole token tiles and reads its share of x once, where a grid with the
// experts innermost has every XCD read all of it (E = 128, H = 2048: T = 1000
// 23.5 -> 22.2 us, T = 200 9.5 -> 9.7).  But then every XCD reads all the gate
// rows for each of its token tiles, which pays while they fit its 4 MB of L2:
// E = 256, H = 4096 (4 MiB) T = 2048 110.9 -> 105.0 us, H = 7168 (7 MiB) 173.2
// -> 250.1.
constexpr long long kGateRowBytes = 4ll << 20;
inline GateLaunch gate_launch(int T, int E, int H) {
  return {T <= 128 ? 4 : 8, T > 256 && 4ll * E * H <= kGateRowBytes};
}

// ----------------------------------------------------------------- expert FFN

// Weight formats.
//   kBf16:  packed by moe_pack_up_weights / moe_pack_down_weights; a ring
//           slot is one k-step of the wave's two 16-row tiles, two adjacent
//           1 KB loads.
//   kMxfp4: packed by moe_pack_mxfp4_up / _down; a ring slot is two k-steps
//           of the wave's two 16-row tiles: one 1 KB load of FP4 codes (a
//           lane's 16 bytes are its 8 codes of tile 0 step 0, tile 0 step 1,
//           tile 1 step 0, tile 1 step 1) and one 64-byte load of their E8M0
//           scales (a dword per row, its bytes in the same order).  For up the
//           two tiles are W1's and W3's rows of the band, for down two
//           adjacent 16-row tiles of W2.
enum WeightFmt { kBf16 = 0, kMxfp4 = 1 };

enum FfnMode { kUp = 0, kDown = 1 };

constexpr int kSlimTokens = 4;

// Whether the one-wave kernel runs a projection (`rows` output rows an expert,
// reductions of `kdim`) of a batch of T tokens.  Up to 4 tokens the union is
// small (at most T K experts) and the four-wave items of the other kernel leave
// CUs idle or unevenly loaded; measured up + down, with every shape tried ahead:
// T = 1 +12 to +44%, T = 4 +2 to +28%.  From 8 tokens its waves each staging the
// activations for themselves costs more than it gains where buckets fill (T = 8
// in 4 experts, MXFP4: -16%; bf16 T = 8: -3%).  The other kernel keeps
// * an up projection with so many one-wave items that an XCD's 32 CUs run them in
//   several rounds: bf16, 768 an XCD (64 experts, H = 2048, I = 3072) -4%, 896 (8
//   experts, H = 4096, I = 14336) -6 to -11%, while 360 and 384 (gpt-oss shape; 32
//   experts, H = 4096, I = 3072) give -10 to +1% where T K experts are active and
//   +9 to +13% where the tokens share theirs, and 192 +2 to +44%; MXFP4 gains up
//   to 768 (+2 to +23%) and at 896 with 1 and 2 tokens (+11 to +23%), with 3 and
//   4 it loses 4 to 8% of the layer;
// * from 3 tokens, a down projection over so many values that every wave stages
//   the activations again and again (14336: the layer -4 to -8%);
// * a bf16 down projection with several four-wave items for each of the 256 CUs,
//   or with one where the reduction is too short to make up for a start of its
//   own in every wave (768 values, T = 2 and 4: -7% and -9%; 1024, T = 2 to 4:
//   -3%; 1408, T = 4 in 16 experts: -13%; 3072, T = 4 in 27 experts: -10%).
inline bool ffn_slim_pays(FfnMode mode, WeightFmt fmt, int T, int K, int E, int rows, int kdim) {
  if (T > kSlimTokens) return false;
  const int experts = std::min(E, T * K);
  if (mode == kUp) {
    const int xcd_items = rows / 16 * ((experts + kNumXcd - 1) / kNumXcd);
    return fmt == kBf16 ? xcd_items <= 512 : T <= 2 || xcd_items <= 800;
  }
  if (T > 2 && kdim > 8192) return false;
  return fmt == kMxfp4 || (rows + 127) / 128 * experts < (kdim < 1536 ? 256 : 512);
}

constexpr int kWideTokens = 128;  // tokens of one item of the wide kernel

// Items an expert's rows make for one token group: 128 rows of W1 and of W3
// (up) or 256 rows of W2 (down) each.
inline int wide_tiles(FfnMode mode, int rows) { return mode == kUp ? (rows + 127) / 128 : (rows + 255) / 256; }

// Whether the wide kernel runs a projection of a batch of T > 64 tokens.  Its
// items are twice as long as the small-batch kernel's, so there must be enough
// of them to give every CU one: with E experts and T K / 128 further token
// groups about 310 (measured: 312 items +4%, 330 items +15%, but 300 items of
// a ragged shape -4 to -13%, 280 items -6% and 171 items -14%).
//
// With bf16 weights the buckets must also be large enough for the MFMAs to
// show: 20 tokens on average for the up projection (25 tokens +6%; 16 tokens
// even; 18.5 tokens -1%; 12.5 tokens of one domain -2%) and 12 for the down
// projection, which gains from staging h in whole lines (12.5 tokens +1%, of
// one domain +6%; 8 tokens -2%); 32 where the reduction is short and an item's
// start weighs more (256 values: 9 and 16 tokens -6% and -7%, 62 tokens +14%).
//
// MXFP4 streams a quarter of the bytes and gains earlier.  Over six shapes
// and six kinds of routing (uniform over all, 64, 32, 16 and top-k experts, and
// skewed): up from 4 tokens (4 to 12 tokens +4% in the mean, 12 to 32 +9%, more
// +20%); down from 8, below which it is even, and with fewer than 600 items
// from 32 (60 experts of I = 1408, 496 to 576 items: -1 to -30%).
inline bool ffn_wide_pays(FfnMode mode, WeightFmt fmt, int T, int K, int E, int rows, int kdim) {
  const long long items = (long long)wide_tiles(mode, rows) * (E + T * K / kWideTokens);
  if (T <= 64 || items < 310) return false;
  if (fmt == kMxfp4) return T * K >= (mode == kUp ? 4 : items < 600 ? 32 : 8) * E;
  return T * K >= (kdim < 512 ? 32 : mode == kUp ? 20 : 12) * E;
}

// The tokens of an item: 128, 64 or 32.  The host sees the batch, not the union,
// so the device decides, from the union's buckets cut to `cap` tokens: `groups`
// in all, t16 the buckets' 16-token tiles, cmax the largest bucket; an expert has
// `tiles` row bands.  The largest cap is taken for which wide_cap_fits.
//
// bf16: an item is bound by its weights, which every group reads again, so
// groups are cut only while there would not be an item for each CU: below 256
// (400 tokens in 8 Qwen3 experts, up: 192 items of 128 tokens 64 us, 336 of 64
// tokens 56), and to 32 only below 160 (60 experts of I = 1408, 256 tokens in 16,
// down: 28 us with 64-token groups, 38 with 32).
//
// MXFP4: an item is bound by its products, so the longest one counts.  An item
// costs about 3 tiles for its start and weights and 1 for each token tile.
// Groups are cut while there are fewer items than CUs, or so few more (up to 352)
// that a CU with two works while most have ended (gpt-oss shape, 256 tokens in 16
// experts, down: 288 items 66 us, 480 items 49); and, where buckets are uneven,
// while the longest item takes longer than a 512th of all the work, which the 512
// resident workgroups would otherwise wait for (64 experts of H = 4096, I = 1024,
// 80 tokens with skewed picks, up: 108 -> 74 us).  Even buckets gain nothing from
// more, shorter items (256 tokens in 64 Qwen3 experts, up: 42 us, 53 cut to 32).
constexpr int kWideStart = 3;
constexpr int wide_longest(int cap, int cmax) {
  const int groups = cmax > cap ? (cmax + cap - 1) / cap : 1;
  return kWideStart + ((cmax + 15) / 16 + groups - 1) / groups;
}
// The longest item within a quarter of the mean one.
constexpr bool wide_even(int cap, int groups, int t16, int cmax) {
  return 4 * wide_longest(cap, cmax) * groups <= 5 * (kWideStart * groups + t16);
}
constexpr bool wide_cap_fits(WeightFmt fmt, int cap, int tiles, int groups, int t16, int cmax) {
  const int items = tiles * groups;
  if (cap <= 32) return true;
  if (fmt == kBf16) return items >= (cap > 64 ? 256 : 160);
  if (items < 256 || (items > 256 && items < 352)) return false;
  return wide_even(cap, groups, t16, cmax) ||
         tiles * (kWideStart * groups + t16) >= 512 * wide_longest(cap, cmax);
}

// Whether whole experts go round-robin over the XCDs, so that an expert's
// activations are fetched into one XCD's L2, instead of the union's (expert, row
// band) units, which balance the XCDs: while every bucket is one item's, and for
// MXFP4 only if the buckets are even and the U experts divide evenly (within a
// quarter) among the XCDs (8 experts of I = 14336, 66 tokens with skewed picks,
// up: 182 us whole, 123 by bands).
constexpr bool wide_whole(WeightFmt fmt, int cap, int groups, int t16, int cmax, int U) {
  if (cmax > cap) return false;
  return fmt == kBf16 || (wide_even(cap, groups, t16, cmax) && (U + kNumXcd - 1) / kNumXcd * kNumXcd * 4 <= 5 * U);
}

// Workgroups of the wide kernel an XCD: an expert's bands for its share of E
// experts and of the further groups of 128 tokens, but at least the two a CU
// that are resident.  The device cuts groups smaller where few experts are
// active, and with no more workgroups than 128-token groups would need, the
// last few items made a second round (37 experts, H = 1056, I = 544, T = 1000:
// 46 items an XCD on 40 workgroups, up 50.2 -> 38.2 us with 64).
constexpr int kWideResident = 64;
inline int wide_slots(int tiles, int T, int K, int E) {
  const int per_xcd = (E + kNumXcd - 1) / kNumXcd;
  const int extra = (T * K / kWideTokens + kNumXcd - 1) / kNumXcd;
  return std::max(tiles * (per_xcd + extra), kWideResident);
}

}  // namespace eldr
