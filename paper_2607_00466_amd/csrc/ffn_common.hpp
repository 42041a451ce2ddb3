// Shared by the expert FFN's kernels: weight formats, launch arguments, the
// bf16 pair split, the FP4 expansion and the dealing of a large batch's items.
#pragma once

#include "common.hpp"

namespace eldr {

constexpr int kKStep = 32;        // k per MFMA
constexpr int kFragElems = 512;   // bf16 values in one packed 16 x 32 weight fragment (1 KB)

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

template <int FMT>
__host__ __device__ constexpr int slot_steps() {
  return FMT == kBf16 ? 1 : 2;
}

enum FfnMode { kUp = 0, kDown = 1 };

struct FfnArgs {
  const uint4* src;            // up: x [T, H] fp32; down: h [T*K, I] as bf16 pairs
  const uint16_t* wa;          // bf16, packed by band: up W1 and W3; down W2
  const int32_t* offsets;      // [E+1]
  const int32_t* perm_token;   // [T*K]
  const int32_t* union_ids;    // [E]: the union in dispatch order (moe_bucket's second half)
  const int32_t* union_size;   // [1]
  void* dst;                   // up: h [T*K, I] as bf16 pairs; down: y_perm [T*K, H] fp32
  int rows;                    // output rows per expert: up I, down H
  int kdim;                    // reduction length: up H, down I
  int tiles;                   // row bands per expert
  int experts;                 // E
  const u32x4* qcodes;         // MXFP4: packed FP4 codes (up: W1 and W3; down: W2)
  const uint32_t* qscales;     // MXFP4: packed E8M0 scales
  // Routed up launches (the buckets built in the kernel from the routing):
  const int32_t* ids;          // [T, K] each token's experts
  int T, K;
  int32_t* b_counts;           // moe_bucket's outputs, written by workgroup 0
  int32_t* b_offsets;
  int32_t* b_perm_token;
  int32_t* b_pair_pos;
  int32_t* b_union_ids;
  int32_t* b_union_size;
};

template <int N>
struct Int {
  static constexpr int value = N;
};

// Calls f(Int<0>{}), ..., f(Int<N-1>{}) -- a loop whose index is a constant.
template <int N, typename F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(Int<I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Split two fp32 values into bf16 high parts and rounded remainders with the
// packed round-to-nearest-even convert: hi = rne(v), lo = rne(v - hi).
__device__ __forceinline__ void split2(uint32_t a, uint32_t b, uint32_t& hi, uint32_t& lo) {
#pragma clang fp contract(off)  // v may be a product: the remainder is that of the rounded value
  const f32x2 v = {__uint_as_float(a), __uint_as_float(b)};
  const bf16x2 h = __builtin_convertvector(v, bf16x2);
  const f32x2 r = v - __builtin_convertvector(h, f32x2);
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
}

// 8 fp32 values (as raw bits) -> 8 bf16 high parts and 8 bf16 low parts.
__device__ __forceinline__ void split8_pk(const u32x4& a, const u32x4& b, u32x4& hi, u32x4& lo) {
  uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
  split2(a.x, a.y, h0, l0);
  split2(a.z, a.w, h1, l1);
  split2(b.x, b.y, h2, l2);
  split2(b.z, b.w, h3, l3);
  hi = u32x4{h0, h1, h2, h3};
  lo = u32x4{l0, l1, l2, l3};
}

// 8 FP4 E2M1 codes (a dword, the first in the low nibble) times the E8M0
// scale in the low byte of sc, as the 8 bf16 values of an MFMA operand.  The
// scaled convert multiplies exactly (an E2M1 value has two significant bits)
// for scale codes 1 .. 252.
__device__ __forceinline__ u32x4 expand_fp4(uint32_t w, uint32_t sc) {
  const float x = __uint_as_float((sc & 0xffu) << 23);
  return u32x4{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, x, 0)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, x, 1)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, x, 2)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, x, 3))};
}

// Inclusive prefix sum over the 64 lanes of a wave: shifts within rows of 16
// lanes (lanes shifted in from outside the row read 0), then the totals of
// rows 0 and 2 broadcast into rows 1 and 3, then that of rows 0-1 into 2-3.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}


// Work items of a batch whose buckets may exceed one token group of GROUP
// tokens: calls item(e, band, first slot of the bucket, first token of the
// group, tokens, whole, shared) for each; whole: whole experts are dealt (one
// item a workgroup), shared: the band is read by other groups too.
//
// The union lists its experts in dispatch order (moe_bucket: more
// 16-token tiles first).  A projection's units are (expert, row band)
// pairs in that order, band by band: unit tiles * u + t is band t of the
// expert at union position u, and unit k goes to XCD k % 8.  So every XCD gets an
// equal share of every expert's bands (exactly equal when the band count
// is a multiple of 8, within one band otherwise) and the XCDs' loads match
// however skewed the buckets are; an XCD's items follow the union order,
// so the largest buckets start first; and an expert's items there are its
// bands in order with each band's token groups adjacent, reading the same
// weights side by side through the XCD's L2.
//
// Every wave holds the whole union, four positions a lane (4 * lane + j;
// union_ids is -1 past the union and is read together with union_size):
// id, bucket start and size, and the first item and number of items of
// the expert on this XCD.  Loads are issued unconditionally (from clamped
// indices), so the wave waits for two round trips rather than one a slot.
template <int GROUP, bool EVEN, class Item>
__device__ __forceinline__ void deal_large_batch(const FfnArgs& a, const int xcd, const int slot, const int slots,
                                                 Item&& item) {
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  static_assert(MOE_MAX_E <= 4 * kWave, "four union positions a lane");
  int e_j[4], sb_j[4], hi_j[4], c_j[4], n_j[4], first_j[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) e_j[j] = a.union_ids[min(4 * lane + j, a.experts - 1)];
  const int U = *a.union_size;  // U <= 0 (empty or invalid routing): no items
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ec = e_j[j] >= 0 && e_j[j] < a.experts ? e_j[j] : 0;
    sb_j[j] = a.offsets[ec];
    hi_j[j] = a.offsets[ec + 1];
  }
  // (keeps the compiler from sinking a load into the branch that uses it)
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(sb_j[j]), "+v"(hi_j[j]));
  int lane_n = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int u = 4 * lane + j;
    const bool member = u < min(U, a.experts) && e_j[j] >= 0 && e_j[j] < a.experts;
    c_j[j] = member ? max(hi_j[j] - sb_j[j], 0) : 0;
    const int g = (c_j[j] + GROUP - 1) / GROUP;
    const int band0 = (xcd - a.tiles * u) & (kNumXcd - 1);  // first band on this XCD
    const int nb = band0 < a.tiles ? (a.tiles - 1 - band0) / kNumXcd + 1 : 0;
    n_j[j] = nb * g;
    first_j[j] = lane_n;
    lane_n += n_j[j];
  }
  // When every bucket fits one token group, the batch is not skewed enough
  // to need the band dealing: whole experts go round-robin over the XCDs as
  // for small batches, so that an expert's activations (x rows for up, h
  // for down) are fetched into one XCD's L2 rather than into all eight.
  int cmax = max(max(c_j[0], c_j[1]), max(c_j[2], c_j[3]));
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) cmax = max(cmax, __shfl_xor(cmax, off));
  const bool whole = __builtin_amdgcn_readfirstlane(cmax) <= GROUP;
  int total = slot + 1, w_e = 0, w_sb = 0, w_c = 0;
  // The table moves to LDS for the item loop: held in registers it would
  // stay live across every item and crowd the 128-token passes.
  __shared__ int4 lk_first[kWave], lk_n[kWave], lk_c[kWave], lk_e[kWave], lk_sb[kWave];
  if (whole) {
    const int u = (slot / a.tiles) * kNumXcd + xcd;
    if (u >= U || u >= a.experts) return;  // also covers U < 0 (invalid routing)
    // union position u: its entries, from the lane that holds them
    const int ls = u / 4, js = u % 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j == js) {
        w_e = __builtin_amdgcn_readlane(e_j[j], ls);
        w_sb = __builtin_amdgcn_readlane(sb_j[j], ls);
        w_c = __builtin_amdgcn_readlane(c_j[j], ls);
      }
    }
  } else {
    const int incl = wave_inclusive_sum(lane_n);
    total = __builtin_amdgcn_readlane(incl, kWave - 1);
    if (slot >= total) return;
    if (wave == 0) {
      const int f0 = incl - lane_n;
      lk_first[lane] = make_int4(first_j[0] + f0, first_j[1] + f0, first_j[2] + f0, first_j[3] + f0);
      lk_n[lane] = make_int4(n_j[0], n_j[1], n_j[2], n_j[3]);
      lk_c[lane] = make_int4(c_j[0], c_j[1], c_j[2], c_j[3]);
      lk_e[lane] = make_int4(e_j[0], e_j[1], e_j[2], e_j[3]);
      lk_sb[lane] = make_int4(sb_j[0], sb_j[1], sb_j[2], sb_j[3]);
    }
    __syncthreads();
  }
  for (int it = slot; it < total; it += slots) {
    if (whole) {
      if (w_c > 0) item(w_e, slot % a.tiles, w_sb, 0, w_c, true, false);
      break;
    }
    // the union position whose items cover this one
    const int4 f4 = lk_first[lane];
    const int4 n4 = lk_n[lane];
    const int fj[4] = {f4.x, f4.y, f4.z, f4.w};
    const int nj[4] = {n4.x, n4.y, n4.z, n4.w};
    int js = -1, ls = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned long long hit = __ballot(nj[j] > 0 && fj[j] <= it && it < fj[j] + nj[j]);
      if (hit != 0) {
        js = j;
        ls = __ffsll(hit) - 1;
      }
    }
    if (js < 0) break;  // not reached: the ranges cover [0, total)
    js = __builtin_amdgcn_readfirstlane(js);
    ls = __builtin_amdgcn_readfirstlane(ls);
    // union position 4 * ls + js: its entries, read at a uniform address
    auto pick = [&](const int4* v) { return reinterpret_cast<const int*>(v)[4 * ls + js]; };
    const int cu = pick(lk_c);
    const int g = (cu + GROUP - 1) / GROUP;
    const int r = it - pick(lk_first);
    const int band = r / g;
    const int group = r - band * g;
    const int tile = ((xcd - a.tiles * (4 * ls + js)) & (kNumXcd - 1)) + kNumXcd * band;
    // An expert's groups: GROUP tokens each and the rest in the last, or (EVEN)
    // as many whole tiles in each as make them equal within one tile.
    const int per = EVEN ? ((cu + 15) / 16 + g - 1) / g * 16 : GROUP;
    const int p0 = group * per;
    const int c = min(per, cu - p0);
    if (c > 0) item(pick(lk_e), tile, pick(lk_sb), p0, c, false, g > 1);
  }
}

}  // namespace eldr
