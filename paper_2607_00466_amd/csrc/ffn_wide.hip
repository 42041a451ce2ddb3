// moe_expert_ffn for batches whose buckets are large: prefill chunks and the
// larger decode batches.
//
// What bounds it: from about 100 tokens an expert the MFMAs (two products a
// weight, one with each part of the bf16 pair), below that the weight stream.
// The small-batch kernel gives a wave 32 weight rows: every activation
// fragment it reads from LDS feeds two row tiles, and at 128 tokens the LDS
// reads alone (16 KB a wave and k-step) take as long as the products.
//
// * An item is 256 weight rows (up: 128 of W1 and the same of W3; down: of W2)
//   by up to 128 tokens of one expert; each of its 4 waves owns four 16-row
//   tiles, so a fragment read feeds four row tiles (the LDS is busy a fifth of the
//   time).
//   Two workgroups share a CU: 128 accumulator registers of the 256 a lane
//   has, and 70 KB of LDS each.
// * Weights go from memory to registers, as fragments, a ring of k-steps
//   ahead; the two packed bands of an item keep their layout.
// * Activations are staged in LDS in whole lines (8 lanes read a token's 128
//   bytes of a k-step).  With a lane to a token, as the small-batch kernel
//   stages, each 16-byte lane read was a cache access of its own, and the L1's
//   tag rate bounded the kernel (busy 68% of the time; 36 accesses a load
//   instruction against 18 now: 461 -> 432 us).
// * A chunk's next one is requested when the chunk starts and published when
//   it ends.  Vector loads return in order, so that wait covers the weights
//   requested before it too: chunks are as long as the ring.
// * A bucket over 128 tokens is cut into groups of equal size within a tile.
// * A slot's products are added in the same order as in every other kernel of
//   the expert FFN, so its result is the same bits.
//
// Measured (up + down by the rules that choose the kernels, before it -> with it;
// picks uniform over the experts named): Qwen3-30B-A3B shape, bf16, T = 4096 884
// -> 691 us (the up products 709 -> 949 TFLOP/s), T = 1000 303 -> 260, T = 512
// 245 -> 226, T = 256 in 64 experts (down alone takes it) 131 -> 126; gpt-oss
// shape, MXFP4: T = 2048 1070 -> 857 us, T = 1000 660 -> 541, T = 256 341 -> 335.
#include "ffn_wide.hpp"

namespace eldr {

constexpr int kWideThreads = 256;  // 4 waves
constexpr int kWideBuf = 32768;    // bytes of one staging buffer: 16 fragment pairs of 2 KB

// One item: expert e's wave slots from 8 tile on by the c tokens (1 .. 16 NTB)
// from bucket slot `first`.  SHARED: other items read the same rows for other
// tokens side by side, so the weight loads are ordinary (cacheable) ones.
template <int MODE, int FMT, int NTB, bool SHARED>
__device__ __forceinline__ void wide_pass(const FfnArgs& a, unsigned char (&lds)[2][kWideBuf], const int e,
                                          const int tile, const int first, const int c) {
  // k-steps of a chunk (what one buffer holds, at most 8), and of weights in
  // flight (what the accumulators leave room for).
  constexpr int C = NTB == 1 ? 8 : 16 / NTB;
  constexpr int G = C * NTB / 4;  // units of 16 tokens by one k-step a wave stages of a chunk
  constexpr int kSlot = slot_steps<FMT>();
  static_assert(C % kSlot == 0, "whole ring slots");
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int K = a.kdim;
  const int nk = K / kKStep;
  const int nslot = nk / kSlot;
  const int arow = lane & 15;
  const int kgrp = lane >> 4;
  const int nt = (c + 15) / 16;

  // ---- weights: wave slots (16 rows of W1 and of W3, or 32 rows of W2) 2p and
  // 2p + 1 of the expert, p = 4 tile + wave, lie side by side in a packed band.
  constexpr int kSlotRows = MODE == kUp ? 16 : 32;
  const int ns = a.rows / kSlotRows;
  const int s0 = 2 * (4 * tile + wave);
  const int s0c = min(s0, (ns - 1) & ~1);
  const int band = s0c / 4;
  const int wb = min(4, ns - 4 * band);
  const int in_band = s0c - 4 * band;
  const int second = s0c + 1 < ns ? 1 : 0;
  const uint16_t* pa = a.wa;
  size_t step_elems = 0;
  const u32x4* pq = a.qcodes;
  const uint32_t* ps = a.qscales;
  if constexpr (FMT == kBf16) {
    constexpr int kMats = MODE == kUp ? 2 : 1;
    step_elems = (size_t)wb * 2 * kFragElems;
    pa += ((size_t)e * a.rows + (size_t)band * 4 * kSlotRows) * (size_t)K * kMats +
          (size_t)(2 * in_band) * kFragElems;
  } else {
    const size_t q0 = ((size_t)e * ns + 4 * band) * nslot + in_band;
    pq += q0 * 64;
    ps += q0 * 16;
  }
  u32x4 ring[C / kSlot][FMT == kBf16 ? 4 : 2];
  uint32_t rsc[C / kSlot][2];
  auto ring_load = [&](const int i, const int si) {
    if constexpr (FMT == kBf16) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const u32x4* q = reinterpret_cast<const u32x4*>(pa + (size_t)si * step_elems +
                                                        (f < 2 ? f : f - 2 + 2 * second) * kFragElems) + lane;
        ring[i][f] = SHARED ? *q : __builtin_nontemporal_load(q);
      }
    } else {
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const size_t o = (size_t)si * wb + f * second;
        const u32x4* q = pq + o * 64 + lane;
        const uint32_t* r = ps + o * 16 + arow;
        ring[i][f] = SHARED ? *q : __builtin_nontemporal_load(q);
        rsc[i][f] = SHARED ? *r : __builtin_nontemporal_load(r);
      }
    }
  };

  // ---- activations.  A unit is 16 tokens of one k-step: 16 rows of 128 bytes
  // in memory, a 2 KB piece of a staging buffer.  A wave stages units wave,
  // wave + 4, ... of a chunk (k-step u / NTB, token tile u % NTB) with two
  // loads each; eight lanes read a row's 128 bytes, so a load touches whole
  // lines, and eight rows, in an order that puts neighbouring octets'
  // LDS writes on different banks.
  //
  // In LDS a unit is 128 places of 16 bytes: 8 values of the high (q = 0 .. 3,
  // the k-group) or low part (q = 4 .. 7) of token n are at place
  // 16 q + (n ^ q ^ 4 (n / 8)).  For one q the 16 tokens, and for one token
  // the 8 q, fall on places that differ mod 8, so neither the products'
  // reads (one q, 8 tokens a cycle) nor the staging writes conflict.
  const int oct = lane / 8, piece = lane % 8;
  auto place = [](const int q, const int n) { return (16 * q + (n ^ q ^ ((n >> 3) << 2))) * 16; };
  const unsigned char* src = reinterpret_cast<const unsigned char*>(a.src);
  if constexpr (MODE == kDown) src += (size_t)first * K * 4;
  uint32_t roff[NTB == 8 ? 2 : 1][2];  // byte offsets of the staged rows (x: below 2^28; h: 128 rows)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n16 = (oct >> 1) + 4 * (oct & 1) + 8 * h;
#pragma unroll
    for (int j = 0; j < (NTB == 8 ? 2 : 1); ++j) {
      const int n = min(((wave + 4 * j) % NTB) * 16 + n16, c - 1);
      const uint32_t r = MODE == kUp ? (uint32_t)a.perm_token[first + n] : (uint32_t)n;
      roff[j][h] = r * (uint32_t)K * 4 + piece * 16;
    }
  }
  // place(q + 4, n) is place(q, n) ^ 64 and 1024 bytes on, place(q, n + 8)
  // place(q, n) ^ 64 and 128 bytes on (q < 4, n < 8), so two registers hold
  // all the places of a thread's pieces.
  const int n0 = (oct >> 1) + 4 * (oct & 1);
  const int put0 = MODE == kUp ? place(piece / 2, n0) + (piece % 2) * 8 : place((piece % 2) * 4 + piece / 2, n0);
  const int put1 = put0 ^ 64;
  const int get_hi = place(kgrp, arow), get_lo = (get_hi ^ 64) + 1024;
  u32x4 stg[G][2];
  auto fetch = [&](const int ks0) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int ks = min(ks0 + (wave + 4 * j) / NTB, nk - 1);
      const unsigned char* s = src + (size_t)ks * 128;
#pragma unroll
      for (int h = 0; h < 2; ++h) stg[j][h] = *reinterpret_cast<const u32x4*>(s + roff[NTB == 8 ? j % 2 : 0][h]);
    }
  };
  auto publish = [&](const int buf) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      unsigned char* d = &lds[buf][(wave + 4 * j) * 2048];
      if constexpr (MODE == kUp) {
        // 4 values of two rows: half a place of each part
        uint2 hi, lo;
        split2(stg[j][0].x, stg[j][0].y, hi.x, lo.x);
        split2(stg[j][0].z, stg[j][0].w, hi.y, lo.y);
        *reinterpret_cast<uint2*>(d + put0) = hi;
        *reinterpret_cast<uint2*>(d + put1 + 1024) = lo;
        split2(stg[j][1].x, stg[j][1].y, hi.x, lo.x);
        split2(stg[j][1].z, stg[j][1].w, hi.y, lo.y);
        *reinterpret_cast<uint2*>(d + put1 + 128) = hi;
        *reinterpret_cast<uint2*>(d + put0 + 1152) = lo;
      } else {
        // a whole place of one part of two rows
        *reinterpret_cast<u32x4*>(d + put0) = stg[j][0];
        *reinterpret_cast<u32x4*>(d + put1 + 128) = stg[j][1];
      }
    }
  };

  f32x4 acc[NTB][4];
#pragma unroll
  for (int t = 0; t < NTB; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[t][r] = f32x4{0.f, 0.f, 0.f, 0.f};

  // k-step s, the I-th of its chunk: the products, then the refill of the ring
  // slot they have read (the scheduling barrier keeps it there).
  auto kstep = [&](const int buf, auto I, const int s) {
    constexpr int slot = decltype(I)::value / kSlot, sub = decltype(I)::value % kSlot;
    u32x4 w[4];
    if constexpr (FMT == kBf16) {
#pragma unroll
      for (int f = 0; f < 4; ++f) w[f] = ring[slot][f];
    } else {
#pragma unroll
      for (int f = 0; f < 4; ++f)
        w[f] = expand_fp4(ring[slot][f / 2][2 * (f % 2) + sub], rsc[slot][f / 2] >> (8 * (2 * (f % 2) + sub)));
    }
    const unsigned char* bb = &lds[buf][decltype(I)::value * NTB * 2048];
    // Tile t's products, with tile t + 1's operands already requested; tiles
    // past the bucket are left out (lanes past it hold its last token, and
    // their columns are not stored).
    u32x4 bh[2], bl[2];
    bh[0] = *reinterpret_cast<const u32x4*>(bb + get_hi);
    bl[0] = *reinterpret_cast<const u32x4*>(bb + get_lo);
    static_for<NTB>([&](auto T_) {
      constexpr int t = decltype(T_)::value;
      if (t <= NTB / 2 || t < nt) {  // (a pass of NTB tiles has more than NTB / 2)
        if constexpr (t + 1 < NTB) {
          bh[(t + 1) % 2] = *reinterpret_cast<const u32x4*>(bb + (t + 1) * 2048 + get_hi);
          bl[(t + 1) % 2] = *reinterpret_cast<const u32x4*>(bb + (t + 1) * 2048 + get_lo);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = mfma16x16x32(w[r], bh[t % 2], acc[t][r]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = mfma16x16x32(w[r], bl[t % 2], acc[t][r]);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    if constexpr (sub == kSlot - 1) ring_load(slot, min((s + C) / kSlot, nslot - 1));
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- the k loop.  Chunk ch is in buffer ch % 2; the next one is requested
  // when it starts and published when it ends.
  __syncthreads();  // the previous item has finished with LDS
#pragma unroll
  for (int i = 0; i < C / kSlot; ++i) ring_load(i, min(i, nslot - 1));
  fetch(0);
  publish(0);
  __syncthreads();
  int buf = 0;
  auto chunk = [&](const int ks, auto TAIL) __attribute__((always_inline)) {
    fetch(ks + C);
    static_for<C>([&](auto I) {
      if (!decltype(TAIL)::value || ks + decltype(I)::value < nk) kstep(buf, I, ks + decltype(I)::value);
    });
    buf ^= 1;
    publish(buf);
    __syncthreads();
  };
  const int full = nk - nk % C;
  for (int ks = 0; ks < full; ks += C) chunk(ks, Int<0>{});
  if (full < nk) chunk(full, Int<1>{});

  // ---- epilogue: lane holds rows .. + 4 kgrp + i of token arow of a tile
  const int rsub = 4 * kgrp;
  const bool ok0 = s0 < ns, ok1 = s0 + 1 < ns;
#pragma unroll
  for (int t = 0; t < NTB; ++t) {
    const int n = t * 16 + arow;
    if (n < c) {
      const size_t sl = (size_t)(first + n);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 0 ? !ok0 : !ok1) continue;
        if constexpr (MODE == kUp) {
          uint32_t v[4], hi[2], lo[2];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(silu(acc[t][2 * h][i]) * acc[t][2 * h + 1][i]);
          split2(v[0], v[1], hi[0], lo[0]);
          split2(v[2], v[3], hi[1], lo[1]);
          const int col = (s0 + h) * 16 + rsub;
          unsigned char* g = static_cast<unsigned char*>(a.dst) + sl * (size_t)a.rows * 4 + (col / 8) * 32 + (col % 8) * 2;
          *reinterpret_cast<uint2*>(g) = make_uint2(hi[0], hi[1]);
          *reinterpret_cast<uint2*>(g + 16) = make_uint2(lo[0], lo[1]);
        } else {
          float* y = static_cast<float*>(a.dst) + sl * a.rows + (s0 + h) * 32 + rsub;
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            const f32x4 v = acc[t][2 * h + f];
            *reinterpret_cast<float4*>(y + 16 * f) = make_float4(v[0], v[1], v[2], v[3]);
          }
        }
      }
    }
  }
}

template <int MODE, int FMT>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ffn_wide_kernel(FfnArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][kWideBuf];
  __shared__ ItemTable tab;
  const int xcd = blockIdx.x % kNumXcd;
  const int slot = blockIdx.x / kNumXcd;
  const int slots = gridDim.x / kNumXcd;
  UnionLanes L = load_union(a);
  // Tokens an item takes at most, and how the items are dealt.
  constexpr WeightFmt fmt = WeightFmt(FMT);
  const int cmax = union_max(L);
  int cap = 2 * kWideTokens, n, t16;
  do {  // the union's groups and, above them, its 16-token tiles (both below 2^13), in one sum
    cap /= 2;
    int part = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) part += (L.c[j] + cap - 1) / cap + ((L.c[j] + 15) / 16 << 16);
    const int sum = __builtin_amdgcn_readlane(wave_inclusive_sum(part), kWave - 1);
    n = sum & 0xffff;
    t16 = sum >> 16;
  } while (!wide_cap_fits(fmt, cap, a.tiles, n, t16, cmax));
  const bool whole = wide_whole(fmt, cap, n, t16, cmax, L.U);
  auto groups = [cap](const int c) { return (c + cap - 1) / cap; };
  UnionEntry x{0, 0, 0};
  int total = slot + 1;
  if (whole) {
    const int u = (slot / a.tiles) * kNumXcd + xcd;
    if (u >= L.U || u >= a.experts) return;  // also covers U < 0 (invalid routing)
    x = union_entry(L, u);
    if (x.c <= 0) return;
  } else {
    total = deal_bands(a, L, tab, xcd, groups);
  }
  for (int it = slot; it < total; it += slots) {
    int e = x.e, tile = slot % a.tiles, first = x.sb, c = x.c;
    bool shared = false;
    if (!whole) {
      const Item m = find_item(a, tab, xcd, it, groups);
      // groups of as many whole tiles as make them equal within one
      const int per = ((m.c + 15) / 16 + m.groups - 1) / m.groups * 16;
      e = m.e;
      tile = m.tile;
      first = m.sb + m.group * per;
      c = min(per, m.c - m.group * per);
      shared = m.groups > 1;
    }
    e = __builtin_amdgcn_readfirstlane(e);
    tile = __builtin_amdgcn_readfirstlane(tile);
    first = __builtin_amdgcn_readfirstlane(first);
    c = __builtin_amdgcn_readfirstlane(c);
    auto pass = [&](auto NTB) __attribute__((always_inline)) {
      constexpr int n = decltype(NTB)::value;
      if (shared)
        wide_pass<MODE, FMT, n, true>(a, lds, e, tile, first, c);
      else
        wide_pass<MODE, FMT, n, false>(a, lds, e, tile, first, c);
    };
    if (c > 64)
      pass(Int<8>{});
    else if (c > 32)
      pass(Int<4>{});
    else if (c > 16)
      pass(Int<2>{});
    else
      pass(Int<1>{});
    if (whole) break;
  }
}

template <int MODE, int FMT>
void launch_ffn_wide(FfnArgs a, int T, int K, int E, hipStream_t s) {
  a.tiles = wide_tiles(FfnMode(MODE), a.rows);
  hipLaunchKernelGGL((ffn_wide_kernel<MODE, FMT>), dim3(kNumXcd * wide_slots(a.tiles, T, K, E)), dim3(kWideThreads), 0,
                     s, a);
}

template void launch_ffn_wide<kUp, kBf16>(FfnArgs, int, int, int, hipStream_t);
template void launch_ffn_wide<kDown, kBf16>(FfnArgs, int, int, int, hipStream_t);
template void launch_ffn_wide<kUp, kMxfp4>(FfnArgs, int, int, int, hipStream_t);
template void launch_ffn_wide<kDown, kMxfp4>(FfnArgs, int, int, int, hipStream_t);

}  // namespace eldr
