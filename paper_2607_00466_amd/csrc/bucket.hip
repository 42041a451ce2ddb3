// moe_bucket: per-expert buckets of (token, expert) pairs and the union of
// distinct experts, in one launch.
//
// Latency bounds it: a few dependent passes over ids that fit the L2.  Every
// workgroup builds all the bitmaps and counts for itself (integer work on the
// same ids, so they agree without any exchange) and writes its own stretch of
// the pairs; workgroup 0 also writes the per-expert outputs.  One workgroup
// alone spent a prefill chunk on the scattered stores of perm_token (a cache
// line a lane), on ids loaded one at a time, and on bitmaps whose rows, a
// multiple of the LDS banks apart, put a wave's atomics on one bank.  Measured
// before and after (top-8 of 128): T = 4096 52.5 -> 12.7 us, T = 1000 14.3 ->
// 6.4, T = 512 7.2 -> 6.0; T <= 256 within 0.1.
//
// Each expert gets a bitmap over tokens in LDS (bit t set when token t picked
// it).  A slot's rank inside its bucket is the number of set bits below t,
// so buckets list their tokens in ascending order without any sort, and the
// result does not depend on the order in which threads ran.  The union is
// listed twice: in ascending id, then in dispatch order -- experts with more
// 16-token tiles (the expert FFN's unit of work per item) first, equal ones
// by ascending id -- so the FFN starts its longest items first while batches
// of small buckets stream the experts in address order.  An expert's
// dispatch position is the number of experts with a larger (tiles, -id) key.
#include "common.hpp"

namespace eldr {

constexpr int kBucketThreads = 1024;
constexpr int kOrderTokens = 16;        // union order: buckets compared in tiles of 16 tokens

// LARGE: several threads an expert (see bucket_launch).  IN_PLACE: pair_pos holds
// the ids and is overwritten.
template <bool LARGE, bool IN_PLACE>
__global__ __launch_bounds__(kBucketThreads) void bucket_kernel(
    const int32_t* __restrict__ topk_ids, int T, int E, int K, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm_token, int32_t* __restrict__ pair_pos,
    int32_t* __restrict__ union_ids, int32_t* __restrict__ union_size) {
  const int32_t* ids = IN_PLACE ? pair_pos : topk_ids;
  extern __shared__ uint32_t smem[];
  // union order keys, larger first: 16-token tiles (<= 256) above 255 - e
  // (e < 256); 0 past E, below every expert with tokens
  __shared__ __attribute__((aligned(16))) int key_s[MOE_MAX_E];
  __shared__ int bad;
  __shared__ int total_pairs, total_union;
  const int W = (T + 31) / 32;
  const int S = bucket_stride(T);
  const int EW = E * S;
  uint32_t* mask = smem;                                          // [E][S] token bitmaps
  uint16_t* pre = reinterpret_cast<uint16_t*>(mask + EW);         // [E][S] bits before word w
  int32_t* cnt = reinterpret_cast<int32_t*>(pre + ((EW + 1) & ~1));  // [E]
  int32_t* off = cnt + E;                                         // [E]
  int32_t* usc = off + E;                                         // [E] position, ascending union
  int32_t* rnk = usc + E;                                         // [E] position, dispatch order
  const int tid = threadIdx.x;
  const int P = T * K;
  // the pair's token: p + 1/2 is exact, and 1 / K is off by less than the
  // quotient's distance to a whole number (at least 1 / (2 K))
  const float inv_k = 1.0f / (float)K;
  auto token_of = [&](const int p) { return (int)(((float)p + 0.5f) * inv_k); };

  for (int i = tid; i < EW; i += kBucketThreads) mask[i] = 0u;
  if (tid == 0) bad = 0;
  __syncthreads();

  // A batch of ids in flight a thread.  A repeated pick leaves fewer bits than
  // pairs, which the total shows.
  constexpr int kBatch = LARGE ? 8 : 2;
  for (int p0 = tid; p0 < P; p0 += kBucketThreads * kBatch) {
    int ev[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) ev[i] = ids[min(p0 + i * kBucketThreads, P - 1)];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int p = p0 + i * kBucketThreads;
      const int t = token_of(p);
      const bool in = ev[i] >= 0 && ev[i] < E;
      if (p < P && in) atomicOr(&mask[ev[i] * S + (t >> 5)], 1u << (t & 31));
      if (p < P && !in) bad = 1;
    }
  }
  __syncthreads();

  // Bits before each word, and each expert's count.  Large: 16 threads an
  // expert (8 or 4 where E is above 64 or 128) sum a stretch of its words
  // each, scan the sums, and write.
  if constexpr (LARGE) {
    const int log_per = E <= 64 ? 4 : E <= 128 ? 3 : 2;
    const int per = 1 << log_per;
    const int e = tid >> log_per;
    const int sub = tid & (per - 1);
    const int words = (W + per - 1) >> log_per;
    const int w0 = min(sub * words, W), w1 = min(w0 + words, W);
    int sum = 0;
    if (e < E)
      for (int w = w0; w < w1; ++w) sum += __popc(mask[e * S + w]);
    int incl = sum;
    for (int o = 1; o < per; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (sub >= o) incl += v;
    }
    if (e < E) {
      int run = incl - sum;
      for (int w = w0; w < w1; ++w) {
        pre[e * S + w] = (uint16_t)run;
        run += __popc(mask[e * S + w]);
      }
      if (sub == per - 1) {
        cnt[e] = run;
        key_s[e] = (((run + kOrderTokens - 1) / kOrderTokens) << 8) | (MOE_MAX_E - 1 - e);
      }
    }
  } else {
    for (int e = tid; e < E; e += kBucketThreads) {
      int run = 0;
      for (int w = 0; w < W; ++w) {
        pre[e * S + w] = (uint16_t)run;
        run += __popc(mask[e * S + w]);
      }
      cnt[e] = run;
      key_s[e] = (((run + kOrderTokens - 1) / kOrderTokens) << 8) | (MOE_MAX_E - 1 - e);
    }
  }
  for (int e = E + tid; e < MOE_MAX_E; e += kBucketThreads) key_s[e] = 0;
  __syncthreads();

  // Exclusive scans of counts and of (counts > 0) over E <= 256 experts by
  // wave 0: 4 consecutive experts per lane, then a shuffle scan over lanes.
  // Meanwhile the other waves rank each expert: R adjacent threads split the
  // keys (in runs of 4, read 16 bytes at a time) and sum their counts.
  static_assert(kBucketThreads >= kWave + 2 * MOE_MAX_E, "two ranking threads an expert");
  if (tid >= kWave) {
    const int R = E <= (kBucketThreads - kWave) / 4 ? 4 : 2;
    const int q = tid - kWave;
    const int e = q / R;
    const int quads = (E + 3) / 4;
    const int per = (quads + R - 1) / R;
    const int q0 = (q % R) * per;
    const int q1 = min(quads, q0 + per);
    int above = 0;
    if (e < E) {
      const int key = key_s[e];
      const int4* k4 = reinterpret_cast<const int4*>(key_s);
      for (int i = q0; i < q1; ++i) {
        const int4 k = k4[i];
        above += (k.x > key) + (k.y > key) + (k.z > key) + (k.w > key);
      }
    }
    above += __shfl_xor(above, 1);
    if (R == 4) above += __shfl_xor(above, 2);
    if (e < E && q % R == 0) rnk[e] = above;
  } else {
    const int lane = tid;
    int c[4], f[4], sc = 0, sf = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane * 4 + i;
      c[i] = e < E ? cnt[e] : 0;
      f[i] = c[i] > 0 ? 1 : 0;
      sc += c[i];
      sf += f[i];
    }
    int ic = sc, jf = sf;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int nc = __shfl_up(ic, o);
      const int nf = __shfl_up(jf, o);
      if (lane >= o) {
        ic += nc;
        jf += nf;
      }
    }
    int bc = ic - sc, bf = jf - sf;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane * 4 + i;
      if (e < E) {
        off[e] = bc;
        usc[e] = bf;
      }
      bc += c[i];
      bf += f[i];
    }
    if (lane == kWave - 1) {
      total_pairs = ic;
      total_union = jf;
    }
  }
  __syncthreads();

  const bool ok = (bad == 0) && (total_pairs == P);
  if (ok) {
    // this workgroup's stretch of the pairs
    const int per_wg = (P + gridDim.x - 1) / gridDim.x;
    const int p1 = min(P, (int)(blockIdx.x + 1) * per_wg);
    for (int p = blockIdx.x * per_wg + tid; p < p1; p += kBucketThreads) {
      const int t = token_of(p);
      const int e = ids[p];
      const int w = t >> 5;
      const uint32_t below = mask[e * S + w] & ((1u << (t & 31)) - 1u);
      const int slot = off[e] + pre[e * S + w] + __popc(below);
      perm_token[slot] = t;
      pair_pos[p] = slot;
    }
  }
  if (blockIdx.x != 0) return;
  const int U = total_union;
  for (int e = tid; e < E; e += kBucketThreads) {
    counts[e] = cnt[e];
    offsets[e] = off[e];
    if (cnt[e] > 0) {
      union_ids[usc[e]] = e;
      union_ids[E + rnk[e]] = e;
    }
  }
  for (int u = tid; u < E; u += kBucketThreads)
    if (u >= U) {
      union_ids[u] = -1;
      union_ids[E + u] = -1;
    }
  if (tid == 0) {
    offsets[E] = total_pairs;
    *union_size = ok ? U : -1;
  }
}

}  // namespace eldr

extern "C" int moe_bucket(const int32_t* topk_ids, moe_dims d, int32_t* counts, int32_t* offsets,
                          int32_t* perm_token, int32_t* pair_pos, int32_t* union_ids,
                          int32_t* union_size, void* stream) {
  using namespace eldr_host;
  int st = check_dims(d);
  if (st != MOE_OK) return st;
  if (!counts || !offsets || !union_ids || !union_size) return MOE_ERR_INVALID;
  if (d.T > 0 && (!topk_ids || !perm_token || !pair_pos)) return MOE_ERR_INVALID;
  if (!aligned4(topk_ids) || !aligned4(counts) || !aligned4(offsets) || !aligned4(perm_token) ||
      !aligned4(pair_pos) || !aligned4(union_ids) || !aligned4(union_size))
    return MOE_ERR_UNSUPPORTED;
  if ((long long)d.E * ((d.T + 31) / 32) > eldr::kBucketMaxWords) return MOE_ERR_UNSUPPORTED;
  const bool in_place = topk_ids == pair_pos;
  const eldr::BucketLaunch l = eldr::bucket_launch(d.T, d.E, d.K, in_place);
  const auto kernel = l.large ? (in_place ? eldr::bucket_kernel<true, true> : eldr::bucket_kernel<true, false>)
                              : (in_place ? eldr::bucket_kernel<false, true> : eldr::bucket_kernel<false, false>);
  // Above 64 KiB (bitmaps, prefixes and tables: from about 10,200 bitmap words)
  // the kernel's dynamic LDS limit has to be raised, on the current device,
  // before the launch; the call is cheap and shapes that need it are
  // prefill-sized, so it is made on every such call rather than cached.
  if (l.lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.lds) != hipSuccess)
    return MOE_ERR_HIP;
  hipLaunchKernelGGL(kernel, dim3(l.wgs), dim3(eldr::kBucketThreads), l.lds, reinterpret_cast<hipStream_t>(stream),
                     topk_ids, d.T, d.E, d.K, counts, offsets, perm_token, pair_pos, union_ids, union_size);
  return launch_status();
}
