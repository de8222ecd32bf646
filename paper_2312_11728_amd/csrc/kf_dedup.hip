// Duplicate removal among found tracks (one track per seed, one hit id per
// layer of the plan).  Tracks t and u are duplicates when they carry the same
// hit id at >= 1 layer and at >= frac * min(n_t, n_u) layers (n: hit count);
// u outranks t on (score, then lower index); t is removed when an outranking
// track is its duplicate, and dup_of[t] names the highest-ranked one.
//
// The candidate partners of a track are the tracks that share one of its hit
// ids: the (hit id, track) entries of all tracks go into a hash table of
// linked lists, an entry 16 bytes with all that ranks it, so that a step
// along a list is one load.  A group of lanes per track, one lane per layer,
// then walks the lists of its hit ids and compares its track's hit list with
// each outranking partner's, layer by layer; the highest-ranked duplicate is
// the minimum of a 64-bit rank key over what the lanes met, whatever the
// order of the lists.  Bound by launches and the latency of the walk: three
// kernels, 34 us for 20k tracks of 17 layers (sorting the entries by hit id
// took 12 to 20 launches and 150 us).
#include <algorithm>

#include "kf_dedup.hpp"

namespace kf {

namespace {

// An entry of a list: the next entry's index (-1: the last), the hit id, the
// track and its score.
struct alignas(16) DedupNode {
  int32_t next, hit, track;
  float score;
};

__device__ inline bool has_candidate(float s) { return s > -__builtin_huge_valf(); }

// heads of the hash table: 2^bits, at least the number of entries
int table_bits(int64_t m) {
  int bits = 8;
  while ((int64_t(1) << bits) < m) ++bits;
  return bits;
}

__device__ inline uint32_t slot_of(int32_t h, int bits) {
  return (uint32_t(h) * 2654435769u) >> (32 - bits);   // 2^32 / golden ratio: neighbouring ids spread
}

__global__ void __launch_bounds__(256) dedup_clear_kernel(int4* head, int64_t n4) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n4) head[i] = make_int4(-1, -1, -1, -1);
}

// Entry i = t * n_layers + l into its list, unless it is a miss or its track
// has no candidate.
__global__ void __launch_bounds__(256) dedup_insert_kernel(DedupArgs a, DedupNode* node, int32_t* head, int bits) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t m = a.n * a.n_layers;
  if (i >= m) return;
  const int64_t t = i / a.n_layers;
  const int l = int(i - t * a.n_layers);
  const int32_t h = a.hits[t * a.hit_stride + l];
  const float s = a.score[t * a.score_stride];
  if (h < 0 || !has_candidate(s)) return;
  const int32_t next = atomicExch(&head[slot_of(h, bits)], int32_t(i));
  node[i] = DedupNode{next, h, int32_t(t), s};
}

// The rank of track u as an unsigned key: smaller is higher ranked (score
// descending, then index ascending); -0 and +0 rank alike.
__device__ inline unsigned long long rank_key(float s, int64_t u) {
  if (s == 0.0f) s = 0.0f;
  const uint32_t b = __float_as_uint(s);
  const uint32_t ord = (b & 0x80000000u) ? ~b : (b | 0x80000000u);   // increasing with s
  return (static_cast<unsigned long long>(~ord) << 32) | static_cast<uint32_t>(u);
}

// G lanes per track (a power of two >= n_layers), lane l of the group walking
// the list of t's hit id at layer l: of the tracks there that outrank t and
// are its duplicates, the highest-ranked.
template <int G>
__global__ void __launch_bounds__(256) dedup_scan_kernel(DedupArgs a, const DedupNode* node, const int32_t* head,
                                                         int bits) {
  const int l = int(threadIdx.x) % G;
  const int L = a.n_layers;
  const int64_t stride = int64_t(gridDim.x) * (256 / G);
  for (int64_t t = (int64_t(blockIdx.x) * 256 + threadIdx.x) / G; t < a.n; t += stride) {   // whole groups
    const int32_t* ht = a.hits + t * a.hit_stride;
    const float st = a.score[t * a.score_stride];
    const bool has = has_candidate(st);
    const int32_t h = l < L ? ht[l] : -1;
    unsigned long long mine = ~0ull;
    if (has && h >= 0) {
      for (int32_t i = head[slot_of(h, bits)]; i >= 0;) {
        const DedupNode e = node[i];
        i = e.next;
        const int64_t u = e.track;
        const float su = e.score;
        if (e.hit != h || u == t) continue;
        if (!(su > st || (su == st && u < t))) continue;   // u does not outrank t
        const unsigned long long ku = rank_key(su, u);
        if (ku >= mine) continue;   // ranks below a duplicate found already
        const int32_t* hu = a.hits + u * a.hit_stride;
        // both rows, eight layers' loads at a time (a layer past the last one
        // repeats it and does not count)
        int nt = 0, nu = 0, shared = 0;
        for (int k0 = 0; k0 < L; k0 += 8) {
          int32_t x[8], y[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int kk = k0 + k < L ? k0 + k : L - 1;
            x[k] = ht[kk];
            y[k] = hu[kk];
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const bool in = k0 + k < L;
            nt += (in && x[k] >= 0) ? 1 : 0;
            nu += (in && y[k] >= 0) ? 1 : 0;
            shared += (in && y[k] >= 0 && x[k] == y[k]) ? 1 : 0;
          }
        }
        const int nmin = nt < nu ? nt : nu;
        // exact: a float times an integer <= 64 is exact in double
        if (shared >= 1 && double(shared) >= double(a.frac) * double(nmin)) mine = ku;
      }
    }
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
      const unsigned long long other = __shfl_xor(mine, o);
      mine = other < mine ? other : mine;
    }
    if (l == 0) {
      a.keep[t] = (has && mine == ~0ull) ? 1 : 0;
      if (a.dup_of) a.dup_of[t] = (has && mine != ~0ull) ? int32_t(uint32_t(mine)) : -1;
    }
  }
}

size_t up256(size_t b) { return (b + 255) / 256 * 256; }

template <int G>
void launch_scan(const DedupArgs& a, const DedupNode* node, const int32_t* head, int bits, hipStream_t s) {
  const unsigned grid = unsigned(std::min<int64_t>((a.n * G + 255) / 256, 1 << 20));
  hipLaunchKernelGGL(dedup_scan_kernel<G>, dim3(grid), dim3(256), 0, s, a, node, head, bits);
}

}  // namespace

size_t dedup_workspace_bytes(int64_t n, int32_t n_layers) {
  const int64_t m = n * n_layers;
  return up256(size_t(m) * sizeof(DedupNode)) + (size_t(4) << table_bits(m));
}

hipError_t launch_dedup(const DedupArgs& a, void* work, size_t work_bytes, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const int64_t m = a.n * a.n_layers;
  if (work_bytes < dedup_workspace_bytes(a.n, a.n_layers)) return hipErrorInvalidValue;
  DedupNode* node = static_cast<DedupNode*>(work);
  int32_t* head = reinterpret_cast<int32_t*>(static_cast<char*>(work) + up256(size_t(m) * sizeof(DedupNode)));
  const int bits = table_bits(m);
  const int64_t n4 = (int64_t(1) << bits) / 4;
  hipLaunchKernelGGL(dedup_clear_kernel, dim3(unsigned((n4 + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<int4*>(head), n4);
  hipLaunchKernelGGL(dedup_insert_kernel, dim3(unsigned((m + 255) / 256)), dim3(256), 0, s, a, node, head, bits);
  if (a.n_layers <= 16)
    launch_scan<16>(a, node, head, bits, s);
  else if (a.n_layers <= 32)
    launch_scan<32>(a, node, head, bits, s);
  else
    launch_scan<64>(a, node, head, bits, s);
  return hipGetLastError();
}

}  // namespace kf
