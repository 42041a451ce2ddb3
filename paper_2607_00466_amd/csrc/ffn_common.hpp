// Shared by the expert FFN's kernels: launch arguments, the
// bf16 pair split, the FP4 expansion and the dealing of a large batch's items.
#pragma once

#include "common.hpp"

namespace eldr {

constexpr int kKStep = 32;        // k per MFMA
constexpr int kFragElems = 512;   // bf16 values in one packed 16 x 32 weight fragment (1 KB)

template <int FMT>
__host__ __device__ constexpr int slot_steps() {
  return FMT == kBf16 ? 1 : 2;
}

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


// The union of a large batch, held by every wave: positions 4 lane + j in
// dispatch order (union_ids is -1 past the union and is read together with
// union_size): id, bucket start and size (0 past the union, or for an invalid
// routing).  Loads are issued unconditionally (from clamped indices), so the
// wave waits for two round trips rather than one a position.
struct UnionLanes {
  int e[4], sb[4], c[4];
  int U;
};

__device__ __forceinline__ UnionLanes load_union(const FfnArgs& a) {
  static_assert(MOE_MAX_E <= 4 * kWave, "four union positions a lane");
  const int lane = threadIdx.x % kWave;
  UnionLanes L;
  int hi[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) L.e[j] = a.union_ids[min(4 * lane + j, a.experts - 1)];
  L.U = *a.union_size;  // U <= 0 (empty or invalid routing): no items
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ec = L.e[j] >= 0 && L.e[j] < a.experts ? L.e[j] : 0;
    L.sb[j] = a.offsets[ec];
    hi[j] = a.offsets[ec + 1];
  }
  // (keeps the compiler from sinking a load into the branch that uses it)
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(L.sb[j]), "+v"(hi[j]));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool member = 4 * lane + j < min(L.U, a.experts) && L.e[j] >= 0 && L.e[j] < a.experts;
    L.c[j] = member ? max(hi[j] - L.sb[j], 0) : 0;
  }
  return L;
}

// The largest bucket (uniform).
__device__ __forceinline__ int union_max(const UnionLanes& L) {
  int m = max(max(L.c[0], L.c[1]), max(L.c[2], L.c[3]));
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
  return __builtin_amdgcn_readfirstlane(m);
}

// Union position u's entries, from the lane that holds them (u uniform).
struct UnionEntry {
  int e, sb, c;
};
__device__ __forceinline__ UnionEntry union_entry(const UnionLanes& L, const int u) {
  UnionEntry r{0, 0, 0};
  const int ls = u / 4, js = u % 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (j == js) {
      r.e = __builtin_amdgcn_readlane(L.e[j], ls);
      r.sb = __builtin_amdgcn_readlane(L.sb[j], ls);
      r.c = __builtin_amdgcn_readlane(L.c[j], ls);
    }
  }
  return r;
}

// The items of one XCD when (expert, row band) units are dealt round-robin.
// The union lists its experts in dispatch order (moe_bucket: more 16-token
// tiles first); unit tiles * u + t is band t of the expert at union position
// u, and unit k goes to XCD k % 8.  So every XCD gets an equal share of every
// expert's bands (exactly equal when the band count is a multiple of 8, within
// one band otherwise) and the XCDs' loads match however skewed the buckets
// are; an XCD's items follow the union order, so the largest buckets start
// first; and an expert's items there are its bands in order with each band's
// token groups adjacent, reading the same weights side by side through the
// XCD's L2.  The table lies in LDS for the item loop: held in registers it
// would stay live across every item and crowd the 128-token passes.
struct ItemTable {
  int4 first[kWave], n[kWave], c[kWave], e[kWave], sb[kWave];
};
struct Item {
  int e, tile, sb, c, group, groups;  // c: tokens of the whole bucket
};

// Fills the table (uniform; ends with a barrier) and returns the item count.
template <class Groups>
__device__ __forceinline__ int deal_bands(const FfnArgs& a, const UnionLanes& L, ItemTable& tab, const int xcd,
                                          Groups&& groups) {
  const int lane = threadIdx.x % kWave;
  int n[4], first[4], lane_n = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int band0 = (xcd - a.tiles * (4 * lane + j)) & (kNumXcd - 1);  // first band on this XCD
    const int nb = band0 < a.tiles ? (a.tiles - 1 - band0) / kNumXcd + 1 : 0;
    n[j] = nb * groups(L.c[j]);
    first[j] = lane_n;
    lane_n += n[j];
  }
  const int incl = wave_inclusive_sum(lane_n);
  const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
  if (threadIdx.x < kWave) {
    const int f0 = incl - lane_n;
    tab.first[lane] = make_int4(first[0] + f0, first[1] + f0, first[2] + f0, first[3] + f0);
    tab.n[lane] = make_int4(n[0], n[1], n[2], n[3]);
    tab.c[lane] = make_int4(L.c[0], L.c[1], L.c[2], L.c[3]);
    tab.e[lane] = make_int4(L.e[0], L.e[1], L.e[2], L.e[3]);
    tab.sb[lane] = make_int4(L.sb[0], L.sb[1], L.sb[2], L.sb[3]);
  }
  __syncthreads();
  return total;
}

// Item `it` of the XCD (it < deal_bands' count): the union position whose
// items cover it, its band and its token group.
template <class Groups>
__device__ __forceinline__ Item find_item(const FfnArgs& a, const ItemTable& tab, const int xcd, const int it,
                                          Groups&& groups) {
  const int lane = threadIdx.x % kWave;
  const int4 f4 = tab.first[lane];
  const int4 n4 = tab.n[lane];
  const int fj[4] = {f4.x, f4.y, f4.z, f4.w};
  const int nj[4] = {n4.x, n4.y, n4.z, n4.w};
  int js = 0, ls = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const unsigned long long hit = __ballot(nj[j] > 0 && fj[j] <= it && it < fj[j] + nj[j]);
    if (hit != 0) {
      js = j;
      ls = __ffsll(hit) - 1;
    }
  }
  js = __builtin_amdgcn_readfirstlane(js);
  ls = __builtin_amdgcn_readfirstlane(ls);
  // union position 4 * ls + js: its entries, read at a uniform address
  auto pick = [&](const int4* v) { return reinterpret_cast<const int*>(v)[4 * ls + js]; };
  Item r;
  r.c = pick(tab.c);
  r.groups = groups(r.c);
  const int k = it - pick(tab.first);
  const int band = k / r.groups;
  r.group = k - band * r.groups;
  r.tile = ((xcd - a.tiles * (4 * ls + js)) & (kNumXcd - 1)) + kNumXcd * band;
  r.e = pick(tab.e);
  r.sb = pick(tab.sb);
  return r;
}

}  // namespace eldr
