// moe_expert_ffn for batches of at most 4 tokens.
//
// What bounds it: latency and the number of CUs that stream.  A token's top-8
// experts make 96 up items of four waves in the Qwen3-30B-A3B shape, and a CU
// draws at most about 40 GB/s from one workgroup.  Here an item is one wave
// and its 16 rows of W1 and W3 (32 of W2), a workgroup of its own: 384 and 512
// of them, spread evenly over the CUs, with no barrier in the loop.
//
// * Each wave stages its item's activations for itself, in whole lines, in 8 KB
//   of LDS: 64, 32 or 16 k-steps of the 1, 2 or 4 tokens its bucket can hold.
//   They are requested before the weights, so that only they are waited for,
//   and a one-token bucket of up to 2048 values is staged once.
// * 8 k-steps of weights are in flight a wave.  16 measured 2 to 5% slower (the
//   first products wait behind the longer burst), and two or four waves a
//   workgroup up to 12% slower.
// * Routed up launches build the buckets in one wave: every bucket is one
//   16-token tile, so the dispatch order is the ascending one, and the first
//   workgroup, which has no item, writes moe_bucket's outputs.
// * The products are added in the other kernels' order: the same bits.
//
// Measured (up + down by the rules that choose the kernels, four-wave items ->
// with it; random experts): Qwen3-30B-A3B shape T = 1 28.6 -> 18.8 us, T = 3 (up
// alone takes it) 48.7 -> 42.4; gpt-oss shape MXFP4 T = 1 35.7 -> 29.1, T = 4 50.6
// -> 44.5, bf16 T = 1 71.4 -> 59.4.
#include "ffn_slim.hpp"

namespace eldr {

constexpr int kSlimRows = 64;  // staged rows (a token's k-step, 128 bytes each)
constexpr int kSlimRing = 8;   // k-steps of weights in flight

// One item: the c tokens (1 .. 4) of expert e by wave band `wb` (16 rows of W1
// and of W3, or 32 rows of W2).  row_of(n): the row of a.src that token n
// reads; first: its bucket's first slot.
template <int MODE, int FMT, class RowOf>
__device__ __forceinline__ void slim_item(const FfnArgs& a, unsigned char* lds, const int e, const int wb,
                                          const int first, const int c, RowOf&& row_of) {
  constexpr int kSlot = slot_steps<FMT>();
  constexpr int R = kSlimRing;
  const int lane = threadIdx.x;
  const int K = a.kdim;
  const int nk = K / kKStep;
  const int nslot = nk / kSlot;
  const int arow = lane & 15;
  const int kgrp = lane >> 4;

  // ---- weights: the wave's fragments of each k-step, in their packed band
  constexpr int kBandRows = MODE == kUp ? 16 : 32;
  const int ns = a.rows / kBandRows;
  const int band = wb / 4;
  const int waves_b = min(4, ns - 4 * band);
  const int in_band = wb - 4 * band;
  const uint16_t* pa = a.wa;
  size_t step_elems = 0;
  const u32x4* pq = a.qcodes;
  const uint32_t* ps = a.qscales;
  if constexpr (FMT == kBf16) {
    constexpr int kMats = MODE == kUp ? 2 : 1;
    step_elems = (size_t)waves_b * 2 * kFragElems;
    pa += ((size_t)e * a.rows + (size_t)band * 4 * kBandRows) * (size_t)K * kMats + (size_t)(2 * in_band) * kFragElems;
  } else {
    const size_t q0 = ((size_t)e * ns + 4 * band) * nslot + in_band;
    pq += q0 * 64;
    ps += q0 * 16;
  }
  u32x4 ring[R / kSlot][FMT == kBf16 ? 2 : 1];
  uint32_t rsc[R / kSlot];
  auto ring_load = [&](const int i, const int si) __attribute__((always_inline)) {
    if constexpr (FMT == kBf16) {
#pragma unroll
      for (int f = 0; f < 2; ++f)
        ring[i][f] = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4*>(pa + (size_t)si * step_elems + f * kFragElems) + lane);
    } else {
      const size_t o = (size_t)si * waves_b;
      ring[i][0] = __builtin_nontemporal_load(pq + o * 64 + lane);
      rsc[i] = __builtin_nontemporal_load(ps + o * 16 + arow);
    }
  };

  // ---- activations: row r of a chunk is token r % cp of k-step r / cp, cp the
  // power of two that holds c.  Eight lanes move a row, 16 bytes each.
  const int lc = c <= 1 ? 0 : c <= 2 ? 1 : 2;
  const int cp = 1 << lc;
  const int CK = kSlimRows >> lc;  // k-steps of a chunk: a multiple of the ring
  static_assert(kSlimRows / kSlimTokens % kSlimRing == 0, "chunks start with the ring");
  const int oct = lane / 8, piece = lane % 8;
  // place of 16 bytes q of row r (q = 0 .. 3: high parts of k-group q, 4 .. 7:
  // low parts); neighbouring tokens' places differ, so that reading one q of
  // all tokens does not meet on a bank
  auto place = [&](const int r, const int q) { return r * 128 + ((q ^ (r & (cp - 1))) * 16); };
  const unsigned char* rowp = reinterpret_cast<const unsigned char*>(a.src) +
                              (size_t)row_of(min(oct & (cp - 1), c - 1)) * K * 4 + piece * 16;
  // rows past the last k-step are neither requested nor published (uniform)
  auto past = [&](const int i, const int ks0) { return i > 0 && (ks0 << lc) + 8 * i >= nk << lc; };
  u32x4 stg[kSlimRows / 8];
  auto fetch = [&](const int ks0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kSlimRows / 8; ++i) {
      if (past(i, ks0)) break;
      stg[i] = *reinterpret_cast<const u32x4*>(rowp + (size_t)min(ks0 + ((8 * i + oct) >> lc), nk - 1) * 128);
    }
  };
  // One wave: its LDS operations complete in order, only the compiler is held.
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto publish = [&](const int ks0) __attribute__((always_inline)) {
    wave_sync();
#pragma unroll
    for (int i = 0; i < kSlimRows / 8; ++i) {
      if (past(i, ks0)) break;
      const int r = 8 * i + oct;
      if constexpr (MODE == kUp) {
        uint2 hi, lo;
        split2(stg[i].x, stg[i].y, hi.x, lo.x);
        split2(stg[i].z, stg[i].w, hi.y, lo.y);
        *reinterpret_cast<uint2*>(lds + place(r, piece / 2) + (piece % 2) * 8) = hi;
        *reinterpret_cast<uint2*>(lds + place(r, 4 + piece / 2) + (piece % 2) * 8) = lo;
      } else {
        *reinterpret_cast<u32x4*>(lds + place(r, (piece % 2) * 4 + piece / 2)) = stg[i];
      }
    }
    wave_sync();
  };
  // (lanes past the bucket read its last token; their columns are not stored)
  const int mine = min(arow, c - 1);
  const int get_hi = place(mine, kgrp), get_lo = place(mine, 4 + kgrp);

  fetch(0);
#pragma unroll
  for (int i = 0; i < R / kSlot; ++i) ring_load(i, min(i, nslot - 1));
  publish(0);
  if (CK < nk) fetch(CK);

  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  auto block = [&](const int s0, auto TAIL) __attribute__((always_inline)) {
    if ((s0 & (CK - 1)) == 0 && s0 > 0) {  // the next chunk
      publish(s0);
      if (s0 + CK < nk) fetch(s0 + CK);
    }
    const unsigned char* bb = lds + ((s0 & (CK - 1)) << lc) * 128;
    static_for<R>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if (!decltype(TAIL)::value || s0 + i < nk) {
        const u32x4 bh = *reinterpret_cast<const u32x4*>(bb + (i << lc) * 128 + get_hi);
        const u32x4 bl = *reinterpret_cast<const u32x4*>(bb + (i << lc) * 128 + get_lo);
        constexpr int slot = i / kSlot, sub = i % kSlot;
        u32x4 w0, w1;
        if constexpr (FMT == kBf16) {
          w0 = ring[slot][0];
          w1 = ring[slot][1];
        } else {
          w0 = expand_fp4(ring[slot][0][sub], rsc[slot] >> (8 * sub));
          w1 = expand_fp4(ring[slot][0][2 + sub], rsc[slot] >> (8 * (2 + sub)));
        }
        acc0 = mfma16x16x32(w0, bh, acc0);
        acc1 = mfma16x16x32(w1, bh, acc1);
        acc0 = mfma16x16x32(w0, bl, acc0);
        acc1 = mfma16x16x32(w1, bl, acc1);
        if constexpr (sub == kSlot - 1) ring_load(slot, min((s0 + i + R) / kSlot, nslot - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };
  const int full = nk - nk % R;
  for (int s = 0; s < full; s += R) block(s, Int<0>{});
  if (full < nk) block(full, Int<1>{});

  // ---- epilogue: lane holds rows 4 kgrp .. + 3 of token arow
  if (arow < c) {
    const size_t sl = (size_t)(first + arow);
    if constexpr (MODE == kUp) {
      uint32_t v[4], hi[2], lo[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(silu(acc0[i]) * acc1[i]);
      split2(v[0], v[1], hi[0], lo[0]);
      split2(v[2], v[3], hi[1], lo[1]);
      const int col = wb * 16 + 4 * kgrp;
      unsigned char* g = static_cast<unsigned char*>(a.dst) + sl * (size_t)a.rows * 4 + (col / 8) * 32 + (col % 8) * 2;
      *reinterpret_cast<uint2*>(g) = make_uint2(hi[0], hi[1]);
      *reinterpret_cast<uint2*>(g + 16) = make_uint2(lo[0], lo[1]);
    } else {
      float* y = static_cast<float*>(a.dst) + sl * a.rows + wb * 32 + 4 * kgrp;
      *reinterpret_cast<float4*>(y) = make_float4(acc0[0], acc0[1], acc0[2], acc0[3]);
      *reinterpret_cast<float4*>(y + 16) = make_float4(acc1[0], acc1[1], acc1[2], acc1[3]);
    }
  }
}

// a.tiles: wave bands an expert.  An XCD's items are those of the union
// positions xcd, xcd + 8, ..., expert by expert; ROUTED grids start with 8
// workgroups more, the first of which writes the buckets out.
template <int MODE, int FMT, bool ROUTED>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void ffn_slim_kernel(FfnArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kSlimRows * 128];
  const int lane = threadIdx.x;
  const int xcd = blockIdx.x % kNumXcd;
  const int slot = (int)(blockIdx.x / kNumXcd) - (ROUTED ? 1 : 0);
  const int u = slot / a.tiles * kNumXcd + xcd;
  const int wb = slot % a.tiles;
  if constexpr (ROUTED) {
    if (slot < 0 && blockIdx.x != 0) return;
    // The buckets: bit t of an expert's mask when token t picked it; one pair
    // a lane, then four experts a lane.
    __shared__ uint32_t mask_s[MOE_MAX_E];
    static_assert(kSlimTokens * MOE_MAX_K <= kWave && MOE_MAX_E == 4 * kWave, "one pair, four experts a lane");
    const int E = a.experts, P = a.T * a.K;
    const int id = a.ids[min(lane, P - 1)];
    const int t = lane / a.K;
    const bool in = id >= 0 && id < E;
#pragma unroll
    for (int j = 0; j < 4; ++j) mask_s[4 * lane + j] = 0u;
    __syncthreads();
    if (lane < P && in) atomicOr(&mask_s[id], 1u << t);
    __syncthreads();
    uint32_t m[4];
    int n[4], f[4], sn = 0, sf = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      m[j] = mask_s[4 * lane + j];
      n[j] = __popc(m[j]);
      f[j] = n[j] > 0 ? 1 : 0;
      sn += n[j];
      sf += f[j];
    }
    const int in_n = wave_inclusive_sum(sn);
    const int in_f = wave_inclusive_sum(sf);
    const int pairs = __builtin_amdgcn_readlane(in_n, kWave - 1);
    const int U = __builtin_amdgcn_readlane(in_f, kWave - 1);
    const bool ok = pairs == P;  // a bad or repeated pick leaves fewer bits than pairs
    int off[4], pos[4], bn = in_n - sn, bf = in_f - sf;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      off[j] = bn;
      pos[j] = bf;
      bn += n[j];
      bf += f[j];
    }
    if (slot < 0) {
      __shared__ int off_s[MOE_MAX_E];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int e = 4 * lane + j;
        off_s[e] = off[j];
        if (e < E) {
          a.b_counts[e] = n[j];
          a.b_offsets[e] = off[j];
          if (f[j]) {
            a.b_union_ids[pos[j]] = e;
            a.b_union_ids[E + pos[j]] = e;
          }
          if (e >= U) {
            a.b_union_ids[e] = -1;
            a.b_union_ids[E + e] = -1;
          }
        }
      }
      if (lane == 0) {
        a.b_offsets[E] = pairs;
        *a.b_union_size = ok ? U : -1;
      }
      __syncthreads();
      if (ok && lane < P) {
        const int sl = off_s[id] + __popc(mask_s[id] & ((1u << t) - 1u));
        a.b_perm_token[sl] = t;
        a.b_pair_pos[lane] = sl;
      }
      return;
    }
    if (!ok || u >= U) return;
    // the expert at union position u
    int e = 0, first = 0;
    uint32_t mask = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned long long hit = __ballot(f[j] && pos[j] == u);
      if (hit != 0) {
        const int ls = __ffsll(hit) - 1;
        e = 4 * ls + j;
        first = __builtin_amdgcn_readlane(off[j], ls);
        mask = (uint32_t)__builtin_amdgcn_readlane((int)m[j], ls);
      }
    }
    // token n of the bucket: the n-th set bit
    slim_item<MODE, FMT>(a, lds, e, wb, first, __popc(mask), [&](const int nth) {
      uint32_t v = mask;
#pragma unroll
      for (int i = 0; i < kSlimTokens - 1; ++i) v = i < nth ? v & (v - 1) : v;
      return __builtin_ctz(v);
    });
  } else {
    const int U = *a.union_size;
    if (u >= U) return;  // also covers U < 0 (invalid routing)
    const int e = a.union_ids[u];
    if (e < 0 || e >= a.experts) return;  // not reached for a union member
    const int first = a.offsets[e];
    const int c = min(a.offsets[e + 1] - first, kSlimTokens);
    if (c > 0)
      slim_item<MODE, FMT>(a, lds, e, wb, first, c,
                           [&](const int n) { return MODE == kUp ? a.perm_token[first + n] : first + n; });
  }
}

template <int MODE, int FMT, bool ROUTED>
void launch_ffn_slim(const FfnArgs& args, int T, int K, int E, hipStream_t s) {
  FfnArgs a = args;
  a.tiles = a.rows / (MODE == kUp ? 16 : 32);
  const int per_xcd = (std::min(E, T * K) + kNumXcd - 1) / kNumXcd;
  hipLaunchKernelGGL((ffn_slim_kernel<MODE, FMT, ROUTED>), dim3(kNumXcd * (a.tiles * per_xcd + (ROUTED ? 1 : 0))),
                     dim3(kWave), 0, s, a);
}

template void launch_ffn_slim<kUp, kBf16, true>(const FfnArgs&, int, int, int, hipStream_t);
template void launch_ffn_slim<kUp, kBf16, false>(const FfnArgs&, int, int, int, hipStream_t);
template void launch_ffn_slim<kDown, kBf16, false>(const FfnArgs&, int, int, int, hipStream_t);
template void launch_ffn_slim<kUp, kMxfp4, true>(const FfnArgs&, int, int, int, hipStream_t);
template void launch_ffn_slim<kUp, kMxfp4, false>(const FfnArgs&, int, int, int, hipStream_t);
template void launch_ffn_slim<kDown, kMxfp4, false>(const FfnArgs&, int, int, int, hipStream_t);

}  // namespace eldr
