// HIP kernels of the combinatorial candidate search: binning of the hit pool
// by (layer, phi, z), either by way of buckets of consecutive bins or hit by
// hit, then the search itself in one launch (one thread per
// candidate slot, one wave per block; per layer of the plan the selection,
// the extend with its window scan, and at the end the final pass that writes
// the kept candidates).
#include "kf_kernels.hpp"
#include "kf_search.hpp"
#include "kf_search_launch.hpp"

namespace kf {

// ---- binning -------------------------------------------------------------------

__global__ void __launch_bounds__(256) fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    p[i] = v;
}

__device__ __forceinline__ int layer_of_hit(const BinTable& t, int32_t h) {
  int lo = 0, hi = t.n_layers;   // off[lo] <= h < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (t.off[mid] <= h) lo = mid;
    else hi = mid;
  }
  return lo;
}

// a layer's bins
struct LayerBins {
  int32_t base, nphi, nz;
  float lo, hi;
};

__device__ __forceinline__ LayerBins bins_of_layer(const BinTable& t, int L) {
  return {t.base[L], t.nphi[L], t.nz[L], t.lo[L], t.hi[L]};
}

// -1: a layer that is never searched
__device__ __forceinline__ int32_t bin_of_hit(const LayerBins& l, float x, float y, float z) {
  if (l.nphi == 0) return -1;
  const float phi = atan2f(y, x);
  return l.base + phi_bin(phi, l.nphi) * l.nz + z_bin(z, l.lo, l.hi, l.nz);
}

// ---- binning by buckets ----
//
// About one hit falls into a bin, and hits arrive in no order, so moving them
// one by one costs an atomic per hit in memory (counters) and three partial
// cache lines per hit (48 bytes, whose neighbours other dies' caches hold).
// Here the bins are taken in buckets of consecutive ones.  A block takes
// kSplitHits consecutive hits, orders them by bucket in LDS and appends each
// run to its bucket, one atomic per run, in mostly whole lines.  Then one
// block per bucket orders its hits by bin with LDS counters, within a region
// that its own cache holds, and writes the bins' offsets.  Bound by the four
// passes over the payload: 2.78M hits, 23 us to count, 60 to split (152 with
// each thread storing its own hits), 50 to order (67 without LDS).  Smaller
// buckets make the split's runs shorter (2^9 bins), larger ones the ordering
// slower than that gains (2^11 bins: 86 us).
constexpr int kCountBlock = 512, kCountPer = 8;   // bucket counters: threads, hits per thread
constexpr int kCountHits = kCountBlock * kCountPer;
constexpr int kSplitBlock = 512, kSplitPer = 2;   // splitting
constexpr int kSplitHits = kSplitBlock * kSplitPer;
constexpr int kMaxBuckets = 4096;      // LDS counters of a splitting block
constexpr int kMinBucketShift = 10, kMaxBucketShift = 13;   // log2 of the bins per bucket
constexpr int kMaxBucketBins = 1 << kMaxBucketShift;   // LDS counters of an ordering block
constexpr int kOrderBlock = 1024, kOrderPer = 2;   // ordering: threads, hits per thread in one go
constexpr int kOrderHits = 1536;   // hits ordered in one go (72 KB of LDS, two blocks on a CU)
static_assert(kOrderHits <= kOrderBlock * kOrderPer && kOrderBlock <= 1 << kMinBucketShift, "ordering block");

// log2 of the bins per bucket
static int bucket_shift(int64_t n_bins) {
  int shift = kMinBucketShift;
  while ((int64_t(kMaxBuckets) << shift) < n_bins) ++shift;
  return shift;
}

int64_t pool_buckets(int64_t n_bins) {
  const int shift = bucket_shift(n_bins);
  return (n_bins + (int64_t(1) << shift) - 1) >> shift;
}

// The layers of a block's hits [h0, h1), and the buckets [b0, b1] they can
// fall into (none where b1 < b0).
struct SplitRange {
  int l0, l1;
  int32_t b0, b1;
};

__device__ __forceinline__ SplitRange split_range(const BinTable& t, int64_t h0, int64_t h1, int shift) {
  SplitRange r;
  r.l0 = layer_of_hit(t, int32_t(h0));
  r.l1 = layer_of_hit(t, int32_t(h1 - 1));
  r.b0 = t.base[r.l0] >> shift;
  r.b1 = (t.base[r.l1] + t.nphi[r.l1] * t.nz[r.l1] - 1) >> shift;
  return r;
}

// hits per bucket; every hit's bin is kept for the next pass
__global__ void __launch_bounds__(kCountBlock) bucket_count_kernel(BinTable t, const float* pos, int64_t n, int shift,
                                                                   int32_t* count, int32_t* bin_of) {
  extern __shared__ int32_t in_bucket[];
  const int64_t h0 = int64_t(blockIdx.x) * kCountHits, h1 = h0 + kCountHits < n ? h0 + kCountHits : n;
  const SplitRange r = split_range(t, h0, h1, shift);
  const int nb = r.b1 - r.b0 + 1;
  for (int b = threadIdx.x; b < nb; b += kCountBlock) in_bucket[b] = 0;
  __syncthreads();
  // (most blocks lie within one layer)
  float x[kCountPer], y[kCountPer], z[kCountPer];
#pragma unroll
  for (int k = 0; k < kCountPer; ++k) {
    const int64_t h = h0 + k * kCountBlock + threadIdx.x, hh = h < h1 ? h : h0;
    x[k] = pos[hh];
    y[k] = pos[n + hh];
    z[k] = pos[2 * n + hh];
  }
  const LayerBins first = bins_of_layer(t, r.l0);
#pragma unroll
  for (int k = 0; k < kCountPer; ++k) {
    const int64_t h = h0 + k * kCountBlock + threadIdx.x;
    if (h < h1) {
      LayerBins l = first;
      if (r.l0 != r.l1) l = bins_of_layer(t, layer_of_hit(t, int32_t(h)));
      const int32_t b = bin_of_hit(l, x[k], y[k], z[k]);
      bin_of[h] = b;
      if (b >= 0) atomicAdd(&in_bucket[(b >> shift) - r.b0], 1);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += kCountBlock)
    if (in_bucket[b]) atomicAdd(&count[r.b0 + b], in_bucket[b]);
}

// Exclusive scan of the buckets' counts into base[0 .. nb] and cursor (one
// block; nb <= kMaxBuckets).
__global__ void __launch_bounds__(1024) bucket_scan_kernel(const int32_t* count, int nb, int32_t* base,
                                                           int32_t* cursor) {
  constexpr int kItems = kMaxBuckets / 1024;
  __shared__ int32_t s[1024];
  const int i0 = int(threadIdx.x) * kItems;
  int32_t v[kItems], tot = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    v[k] = i0 + k < nb ? count[i0 + k] : 0;
    tot += v[k];
  }
  s[threadIdx.x] = tot;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int32_t add = int(threadIdx.x) >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  int32_t run = s[threadIdx.x] - tot;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (i0 + k < nb) base[i0 + k] = cursor[i0 + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 1023) base[nb] = run;
}

// copy every hit to its bucket's part of `split` (bin in the place of phi)
__global__ void __launch_bounds__(kSplitBlock) bucket_split_kernel(BinTable t, const float* pos, const float* cov,
                                                                   const int32_t* id, const int32_t* module, int64_t n,
                                                                   int shift, const int32_t* bin_of, int32_t* cursor,
                                                                   PoolHit* split) {
  __shared__ float4 hit[kSplitHits * 3];   // the block's hits, ordered by bucket
  __shared__ int32_t dst[kSplitHits];      // their places in `split`
  __shared__ int32_t wave_sum[kSplitBlock / 64];
  extern __shared__ int32_t in_bucket[];   // [nb] counts, then first places in `hit`; [nb] first places in `split`
  const int tid = int(threadIdx.x);
  const int64_t h0 = int64_t(blockIdx.x) * kSplitHits, h1 = h0 + kSplitHits < n ? h0 + kSplitHits : n;
  const SplitRange r = split_range(t, h0, h1, shift);
  const int nb = r.b1 - r.b0 + 1;
  int32_t* const run = in_bucket + (nb > 0 ? nb : 0);
  for (int b = tid; b < nb; b += kSplitBlock) in_bucket[b] = 0;
  __syncthreads();
  int32_t bin[kSplitPer], rank[kSplitPer];
  float4 v[kSplitPer][3];
#pragma unroll
  for (int k = 0; k < kSplitPer; ++k) {
    const int64_t h = h0 + k * kSplitBlock + tid;
    const int64_t hh = h < h1 ? h : h0;
    bin[k] = h < h1 ? bin_of[h] : -1;
    v[k][0] = make_float4(pos[hh], pos[n + hh], pos[2 * n + hh], __int_as_float(bin[k]));
    v[k][1] = make_float4(cov[hh], cov[n + hh], cov[2 * n + hh], cov[3 * n + hh]);
    v[k][2] = make_float4(cov[4 * n + hh], cov[5 * n + hh], __int_as_float(id[hh]),
                          __int_as_float(module ? module[hh] : -1));
  }
#pragma unroll
  for (int k = 0; k < kSplitPer; ++k) rank[k] = bin[k] >= 0 ? atomicAdd(&in_bucket[(bin[k] >> shift) - r.b0], 1) : 0;
  __syncthreads();
  // exclusive scan of the counts, kSplitBlock buckets at a time
  int32_t placed = 0;
  for (int c0 = 0; c0 < nb; c0 += kSplitBlock) {
    const int b = c0 + tid;
    const int32_t c = b < nb ? in_bucket[b] : 0;
    int32_t sum = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t up = __shfl_up(sum, o);
      if ((tid & 63) >= o) sum += up;
    }
    if ((tid & 63) == 63) wave_sum[tid >> 6] = sum;
    __syncthreads();
    int32_t before = placed, all = 0;
#pragma unroll
    for (int w = 0; w < kSplitBlock / 64; ++w) {
      if (w < (tid >> 6)) before += wave_sum[w];
      all += wave_sum[w];
    }
    if (b < nb) {
      in_bucket[b] = before + sum - c;
      if (c) run[b] = atomicAdd(&cursor[r.b0 + b], c);
    }
    placed += all;
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < kSplitPer; ++k) {
    if (bin[k] < 0) continue;
    const int b = (bin[k] >> shift) - r.b0;
    const int32_t i = in_bucket[b] + rank[k];
    dst[i] = run[b] + rank[k];
#pragma unroll
    for (int x = 0; x < 3; ++x) hit[i * 3 + x] = v[k][x];
  }
  __syncthreads();
  float4* const out = reinterpret_cast<float4*>(split);
  for (int j = tid; j < placed * 3; j += kSplitBlock) out[int64_t(dst[j / 3]) * 3 + j % 3] = hit[j];
}

// One block per bucket: its hits in bin order into the pool, and its bins'
// offsets (the last bucket's block also writes bin_off[n_bins]).  A bucket of
// up to kOrderHits hits is read once and written from LDS in whole lines;
// larger ones are counted and moved in two passes.
__global__ void __launch_bounds__(kOrderBlock) bucket_order_kernel(const PoolHit* split, const int32_t* base, int shift,
                                                                   int64_t n_bins, PoolBins o) {
  __shared__ float4 hit[kOrderHits * 3];
  __shared__ int32_t wave_sum[kOrderBlock / 64];
  extern __shared__ int32_t at[];   // [bins per bucket] counts, then places
  const int tid = int(threadIdx.x);
  const int per = (1 << shift) / kOrderBlock;   // bins per thread
  const int64_t bin0 = int64_t(blockIdx.x) << shift;
  const int32_t h0 = base[blockIdx.x], n_hits = base[blockIdx.x + 1] - h0;
  const bool once = n_hits <= kOrderHits;
  const float4* const in = reinterpret_cast<const float4*>(split + h0);
  float4* const out = reinterpret_cast<float4*>(o.hits + h0);
  for (int b = tid; b < (1 << shift); b += kOrderBlock) at[b] = 0;
  __syncthreads();
  float4 v[kOrderPer][3];
  int32_t rank[kOrderPer];
  if (once) {
#pragma unroll
    for (int k = 0; k < kOrderPer; ++k) {
      const int h = k * kOrderBlock + tid;
      if (h < n_hits) {
#pragma unroll
        for (int x = 0; x < 3; ++x) v[k][x] = in[h * 3 + x];
      }
    }
#pragma unroll
    for (int k = 0; k < kOrderPer; ++k)
      if (k * kOrderBlock + tid < n_hits) rank[k] = atomicAdd(&at[__float_as_int(v[k][0].w) - int32_t(bin0)], 1);
  } else {
    for (int64_t h = tid; h < n_hits; h += kOrderBlock)
      atomicAdd(&at[__float_as_int(in[h * 3].w) - int32_t(bin0)], 1);
  }
  __syncthreads();
  int32_t tot = 0;
  for (int k = 0; k < per; ++k) tot += at[tid * per + k];
  int32_t sum = tot;
#pragma unroll
  for (int w = 1; w < 64; w <<= 1) {
    const int32_t up = __shfl_up(sum, w);
    if ((tid & 63) >= w) sum += up;
  }
  if ((tid & 63) == 63) wave_sum[tid >> 6] = sum;
  __syncthreads();
  int32_t run = sum - tot;
#pragma unroll
  for (int w = 0; w < kOrderBlock / 64; ++w)
    if (w < (tid >> 6)) run += wave_sum[w];
  for (int k = 0; k < per; ++k) {
    const int32_t c = at[tid * per + k];
    at[tid * per + k] = run;
    run += c;
  }
  __syncthreads();
  for (int b = tid; b < (1 << shift); b += kOrderBlock)
    if (bin0 + b < n_bins) o.bin_off[bin0 + b] = h0 + at[b];
  if (tid == 0 && blockIdx.x == gridDim.x - 1) o.bin_off[n_bins] = h0 + n_hits;
  if (once) {
#pragma unroll
    for (int k = 0; k < kOrderPer; ++k) {
      if (k * kOrderBlock + tid < n_hits) {
        const int32_t i = at[__float_as_int(v[k][0].w) - int32_t(bin0)] + rank[k];
        v[k][0].w = atan2f(v[k][0].y, v[k][0].x);
#pragma unroll
        for (int x = 0; x < 3; ++x) hit[i * 3 + x] = v[k][x];
      }
    }
    __syncthreads();
    for (int j = tid; j < n_hits * 3; j += kOrderBlock) out[j] = hit[j];
  } else {
    __syncthreads();   // the bins' places are read above and moved below
    for (int64_t h = tid; h < n_hits; h += kOrderBlock) {
      float4 a = in[h * 3];
      const float4 b = in[h * 3 + 1], c = in[h * 3 + 2];
      const int64_t i = atomicAdd(&at[__float_as_int(a.w) - int32_t(bin0)], 1);
      a.w = atan2f(a.y, a.x);
      out[i * 3] = a;
      out[i * 3 + 1] = b;
      out[i * 3 + 2] = c;
    }
  }
}

// ---- binning hit by hit ----

// count hits per bin; each hit keeps its rank inside its bin
__global__ void __launch_bounds__(256) bin_count_kernel(BinTable t, const float* pos, int64_t n, int32_t* count,
                                                        int32_t* bin_of, int32_t* rank) {
  const int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (h >= n) return;
  const int L = layer_of_hit(t, int32_t(h));
  const int32_t b = bin_of_hit(bins_of_layer(t, L), pos[h], pos[n + h], pos[2 * n + h]);
  bin_of[h] = b;
  if (b >= 0) rank[h] = atomicAdd(&count[b], 1);
}

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;   // per thread

// exclusive scan of counts[0..n) into off, block by block; block totals out
__global__ void __launch_bounds__(kScanBlock) scan_blocks_kernel(const int32_t* in, int64_t n, int32_t* out,
                                                                 int32_t* block_sum) {
  __shared__ int32_t s[kScanBlock];
  const int64_t base = int64_t(blockIdx.x) * kScanBlock * kScanItems + int64_t(threadIdx.x) * kScanItems;
  int32_t v[kScanItems];
  int32_t tot = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0;
    tot += v[k];
  }
  s[threadIdx.x] = tot;
  __syncthreads();
  for (int o = 1; o < kScanBlock; o <<= 1) {
    const int32_t add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  int32_t run = s[threadIdx.x] - tot;   // exclusive prefix of this thread
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == kScanBlock - 1) block_sum[blockIdx.x] = s[threadIdx.x];
}

// exclusive scan of the block totals (one block, chunks with a carry);
// total[0] = grand total
__global__ void __launch_bounds__(1024) scan_sums_kernel(int32_t* sums, int64_t nb, int32_t* total) {
  __shared__ int32_t s[1024];
  __shared__ int32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
    const int64_t i = c0 + threadIdx.x;
    const int32_t v = i < nb ? sums[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int32_t add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (i < nb) sums[i] = carry + s[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry += s[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) total[0] = carry;
}

__global__ void __launch_bounds__(256) scan_add_kernel(int32_t* out, int64_t n, const int32_t* sums,
                                                       const int32_t* total) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] += sums[i / (kScanBlock * kScanItems)];
  if (i == n) out[n] = total[0];
}

// copy every hit to its binned position (x, y, z, phi, covariance, id,
// module: three 16-byte stores)
__global__ void __launch_bounds__(256) bin_scatter_kernel(BinTable t, const float* pos, const float* cov,
                                                          const int32_t* id, const int32_t* module, int64_t n,
                                                          const int32_t* bin_off, const int32_t* bin_of,
                                                          const int32_t* rank, PoolBins o) {
  const int64_t h = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (h >= n || bin_of[h] < 0) return;
  const int64_t d = int64_t(bin_off[bin_of[h]]) + rank[h];
  const float x = pos[h], y = pos[n + h];
  float4* dst = reinterpret_cast<float4*>(o.hits + d);
  dst[0] = make_float4(x, y, pos[2 * n + h], atan2f(y, x));
  dst[1] = make_float4(cov[h], cov[n + h], cov[2 * n + h], cov[3 * n + h]);
  dst[2] = make_float4(cov[4 * n + h], cov[5 * n + h], __int_as_float(id[h]), __int_as_float(module ? module[h] : -1));
}

// ---- search ------------------------------------------------------------------

// The whole search in one launch.  Block b owns the seeds [b * spb,
// (b + 1) * spb), spb = blockDim.x / beam, and their slots: thread i <
// spb * beam is slot b * spb * beam + i.  At every layer the slot first
// runs the previous layer's selection for itself (its candidate and that
// candidate's state, read from its seed's slots in LDS), then, after a
// block barrier, its extend, which leaves its child list and the state it
// goes on with in LDS for the next selection; a second barrier closes the
// layer.  After the last layer come the last selection and the final pass.
// A seed's slots exchange data only with each other, so blocks never wait
// for one another: each runs its seeds through the layers at its own pace.
// B: a compile-time bound on beam (2, 4, 6 or 8), the size of the child
// lists held in registers and LDS.
template <int B>
__global__ void __launch_bounds__(kSearchBlock, kSearchWaves) search_kernel(SearchArgs a,
                                                                          const SearchLayer* __restrict__ layers) {
  __shared__ SlotExchange<B> X;
  const int spb = kSearchBlock / a.beam;
  const int i = int(threadIdx.x);
  const int64_t seed0 = int64_t(blockIdx.x) * spb;
  const int64_t s = seed0 * a.beam + i;
  const int64_t t = seed0 + i;
  const bool slot = i < spb * a.beam && s < a.n * a.beam;
  // the seeds' status words collect the bits of their slots' steps
  if (i < spb && t < a.n) a.status[t] = 0u;
  __syncthreads();
  Cand k;
  k.live = false;
  for (int step = 0; step < a.plan_len; ++step) {
    if (slot) {
      if (step == 0)
        seed_candidate(a, s, k);
      else
        select_slot<B>(a, X, step - 1, s, i, k);
    }
    __syncthreads();
    const SearchLayer& L = layers[step];
    uint32_t st = 0;
    float score = 0.f;
    ScanWindow w;
    w.scan = false;
    const bool open = slot && extend_open<B>(a, X, L, layers[step > 0 ? step - 1 : 0], step, s, i, k, score, w, st);
    Kids<B> K;
    kids_init(K);
    scan_window<B>(a, X, L, w, i, k.p, k.c, score, K, st);
    if (open) extend_close<B>(a, X, i, k, score, K);
    if (st) atomicOr(&a.status[s / a.beam], st);
    __syncthreads();
  }
  if (slot) select_slot<B>(a, X, a.plan_len - 1, s, i, k);
  __syncthreads();
  if (slot) {
    const uint32_t st = finish_candidate(a, layers[a.plan_len - 1], s, k);
    if (st) atomicOr(&a.status[s / a.beam], st);
  }
}

static unsigned blocks(int64_t n, int b) { return unsigned((n + b - 1) / b); }

// By buckets while the second copy of the pool they need stays small (1.6 GB)
// and a bucket's counters fit into LDS; larger pools and finer binnings are
// binned hit by hit.  (2.78M hits in 2.46M bins: 140 us by buckets, 317 us hit
// by hit.)
bool pool_by_buckets(int64_t n, int64_t n_bins) {
  return n <= kMaxSplitHits && n_bins <= int64_t(kMaxBuckets) * kMaxBucketBins;
}

hipError_t launch_bin_pool(const BinTable& t, const float* pos, const float* cov, const int32_t* id,
                           const int32_t* module, int64_t n, int64_t n_bins, const SearchWork& w, hipStream_t s) {
  if (pool_by_buckets(n, n_bins)) {
    const int shift = bucket_shift(n_bins);
    const int nb = int(pool_buckets(n_bins));
    const unsigned lds = unsigned(nb * sizeof(int32_t));   // at most 16 KB
    hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks(nb, 256)), dim3(256), 0, s, w.count, int64_t(nb), 0);
    if (n > 0)
      hipLaunchKernelGGL(bucket_count_kernel, dim3(blocks(n, kCountHits)), dim3(kCountBlock), lds, s, t, pos, n, shift,
                         w.count, w.bin_of);
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(1024), 0, s, w.count, nb, w.bucket_base, w.cursor);
    if (n > 0)
      hipLaunchKernelGGL(bucket_split_kernel, dim3(blocks(n, kSplitHits)), dim3(kSplitBlock), 2 * lds, s, t, pos, cov, id,
                         module, n, shift, w.bin_of, w.cursor, w.split);
    hipLaunchKernelGGL(bucket_order_kernel, dim3(unsigned(nb)), dim3(kOrderBlock), unsigned(sizeof(int32_t) << shift), s, w.split, w.bucket_base, shift,
                       n_bins, w.pool);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(fill_i32_kernel, dim3(1024), dim3(256), 0, s, w.count, n_bins, 0);
  if (n > 0)
    hipLaunchKernelGGL(bin_count_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, t, pos, n, w.count, w.bin_of,
                       w.rank);
  const int64_t nb = (n_bins + kScanBlock * kScanItems - 1) / (kScanBlock * kScanItems);
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(unsigned(nb)), dim3(kScanBlock), 0, s, w.count, n_bins,
                     w.pool.bin_off, w.block_sum);
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, s, w.block_sum, nb, w.total);
  hipLaunchKernelGGL(scan_add_kernel, dim3(blocks(n_bins + 1, 256)), dim3(256), 0, s, w.pool.bin_off, n_bins,
                     w.block_sum, w.total);
  if (n > 0)
    hipLaunchKernelGGL(bin_scatter_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, t, pos, cov, id, module, n,
                       w.pool.bin_off, w.bin_of, w.rank, w.pool);
  return hipGetLastError();
}

hipError_t launch_search(SearchArgs a, const SearchLayer* layers, SearchLayer* d_layers, hipStream_t s) {
  hipError_t e = hipMemcpyAsync(d_layers, layers, size_t(a.plan_len) * sizeof(SearchLayer), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  const int spb = kSearchBlock / a.beam;
  const dim3 grid(blocks(a.n, spb)), block(kSearchBlock);
  const SearchLayer* L = d_layers;
  if (a.beam <= 2)
    hipLaunchKernelGGL(search_kernel<2>, grid, block, 0, s, a, L);
  else if (a.beam <= 4)
    hipLaunchKernelGGL(search_kernel<4>, grid, block, 0, s, a, L);
  else if (a.beam <= 6)
    hipLaunchKernelGGL(search_kernel<6>, grid, block, 0, s, a, L);
  else
    hipLaunchKernelGGL(search_kernel<kMaxBeam>, grid, block, 0, s, a, L);
  return hipGetLastError();
}

}  // namespace kf
