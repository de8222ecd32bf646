// Kernels of the final fit with outlier rejection: the set-up of the per-entry
// masks, and per round the decisions (the worst used hit by unbiased chi2
// rejected, or the track closed with the round's backward-fit result) together
// with the sub-batch of the tracks left open.  The unbiased chi2 itself is
// computed entry-parallel beside the backward pass whose combination it
// reuses.
#include <cmath>

#include "kf_backward.hpp"

namespace kf {

namespace {

constexpr int kFinalBlock = 256;

// Set-up, one thread per track (its open flag) and per entry: the tracks'
// entries are the one range [hit_offsets[0], hit_offsets[n]), written
// thread by thread.
template <typename T>
__global__ void __launch_bounds__(kFinalBlock) final_init_kernel(FinalRoundArgs<T> a) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < a.n) a.open_orig[i] = kFinalOpen;
  if (i < 2 && a.counts) a.counts[i] = 0;
  const int64_t e = int64_t(a.hit_offsets[0]) + i;
  if (e >= a.hit_offsets[a.n] || e >= a.n_hits) return;
  a.outlier[e] = 0;
  a.used[e] = a.hit_valid[e] ? 1 : 0;
  if (a.hit_chi2) a.hit_chi2[e] = T(NAN);
}

// One track per thread: its decision; true if it stays open.
template <typename T>
__device__ __forceinline__ bool decide(const FinalRoundArgs<T>& a, int64_t t, int64_t to, int64_t e0o, int len) {
  const uint8_t op = a.open_orig[to];
  const uint32_t bst = a.b_status[t];
  const bool refitted = !(bst & TRK_BAD_INPUT);
  const int n_e = len < a.max_len ? len : a.max_len;
  double worst = -INFINITY;
  int worst_r = -1, n_used = 0;
  // kAhead entries' loads at a time (past the end the last entry again)
  constexpr int kAhead = 10;
  for (int r0 = 0; r0 < n_e; r0 += kAhead) {
    bool used[kAhead];
    T c2[kAhead];   // NaN unless refitted (launch_final_chi2), undefined on an unused entry
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int r = r0 + k < n_e ? r0 + k : n_e - 1;
      used[k] = a.used_orig[e0o + r] != 0;
      c2[k] = a.pred_state[int64_t(r) * a.n + t];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (r0 + k >= n_e || !used[k]) continue;
      ++n_used;
      if (a.hit_chi2) a.hit_chi2[e0o + r0 + k] = c2[k];
      if (double(c2[k]) > worst) {   // NaN never counts; the first entry among equals
        worst = double(c2[k]);
        worst_r = r0 + k;
      }
    }
  }
  const bool reject = a.round < a.max_reject && refitted && worst_r >= 0 && worst > a.chi2_cut &&
                      n_used - 1 >= a.min_keep;
  if (reject) {
    a.outlier[e0o + worst_r] = 1;
    a.used_orig[e0o + worst_r] = 0;
    a.open_orig[to] = kFinalOpen | kFinalRejected;
    return true;
  }
  // closed: this round's backward-fit result
#pragma unroll
  for (int i = 0; i < 6; ++i) a.state_out[i * a.ld + to] = a.b_state[i * a.n + t];
#pragma unroll
  for (int i = 0; i < 21; ++i) a.cov_out[i * a.ld + to] = a.b_cov[i * a.n + t];
  a.charge_out[to] = a.b_charge[t];
  a.chi2_out[to] = a.b_chi2[t];
  a.ndf_out[to] = a.b_ndf[t];
  a.status_out[to] = bst | ((op & kFinalRejected) ? TRK_OUTLIER : 0u);
  a.open_orig[to] = 0;
  return false;
}

// A round's decisions, and the tracks left open with their entries into the
// next round's sub-batch: the first kRoundTracks threads of a block decide,
// count the block's open tracks and their entries and reserve their places
// with one 64-bit atomic (tracks in the high half, entries in the low half, so
// that both go up together and the offsets stay those of consecutive tracks);
// then all its threads copy the entries, 16 lanes a track.  The order of the
// blocks in the sub-batch is of no consequence: every track is fitted by
// itself.  Bound by latency, hence the many threads per track; one launch in
// place of eight (100k tracks, first round: 46 us, from 26 for the decisions,
// 63 for a copy by one lane a track and 25 for two scans and the flags).
constexpr int kRoundTracks = 128, kRoundBlock = 512;

template <typename T>
__global__ void __launch_bounds__(kRoundBlock) final_round_kernel(FinalRoundArgs<T> a) {
  __shared__ int32_t src[kRoundTracks], dst[kRoundTracks], num[kRoundTracks];   // the block's open tracks
  __shared__ unsigned long long wave_sum[kRoundTracks / 64], base;
  const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  const int64_t t = int64_t(blockIdx.x) * kRoundTracks + tid;
  int64_t to = 0, e0o = 0;
  int len = 0;
  bool open = false;
  if (tid < kRoundTracks && t < a.n) {
    to = a.map ? int64_t(a.map[t]) : t;   // the caller's track and entries
    e0o = a.orig_offsets[to];
    len = int(a.orig_offsets[to + 1] - e0o);
    open = decide(a, t, to, e0o, len);
  }
  if (!a.sub_map) return;
  if (blockIdx.x == 0 && tid < 2) a.next_counts[tid] = 0;
  const unsigned long long mine = open ? (1ull << 32) + uint32_t(len) : 0ull;
  unsigned long long sum = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long up = __shfl_up(sum, o);
    if (lane >= o) sum += up;
  }
  if (lane == 63 && tid < kRoundTracks) wave_sum[wave] = sum;
  __syncthreads();
  unsigned long long before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kRoundTracks / 64; ++w) {
    if (w < wave) before += wave_sum[w];
    all += wave_sum[w];
  }
  if (all == 0) return;   // the whole block
  // counts[0] (tracks) is the low word in memory: the halves are swapped
  if (tid == 0) {
    const unsigned long long swapped = (all >> 32) | (all << 32);
    const unsigned long long old = atomicAdd(reinterpret_cast<unsigned long long*>(a.counts), swapped);
    base = (old >> 32) | (old << 32);
  }
  __syncthreads();
  if (open) {
    const unsigned long long place = base + before + (sum - mine);
    const int32_t i = int32_t(place >> 32), d0 = int32_t(uint32_t(place));
    a.sub_map[i] = int32_t(to);
    a.sub_offsets[i] = d0;
    a.sub_offsets[i + 1] = d0 + len;   // what the next track writes too, if there is one
    const int k = int((before + (sum - mine)) >> 32);
    src[k] = int32_t(e0o);
    dst[k] = d0;
    num[k] = len;
  }
  __syncthreads();
  const int n_open = int(all >> 32);
  const int64_t nh = a.n_hits;
  for (int k = tid >> 4; k < n_open; k += kRoundBlock / 16) {
    const int64_t s0 = src[k], d0 = dst[k];
    const int m = num[k];
    for (int r0 = tid & 15; r0 < m; r0 += 32) {
      // entries r0 and r0 + 16 (or r0 again): all loads, then the stores
      const int64_t e[2] = {s0 + r0, s0 + (r0 + 16 < m ? r0 + 16 : r0)};
      int16_t lay[2];
      uint8_t used[2];
      T v[2][9];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        lay[h] = a.orig_layer[e[h]];
        used[h] = a.used_orig[e[h]];
#pragma unroll
        for (int x = 0; x < 3; ++x) v[h][x] = a.orig_pos[x * nh + e[h]];
#pragma unroll
        for (int x = 0; x < 6; ++x) v[h][3 + x] = a.orig_cov[x * nh + e[h]];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t d = d0 + (e[h] - s0);
        a.sub_layer[d] = lay[h];
        a.sub_used[d] = used[h];
#pragma unroll
        for (int x = 0; x < 3; ++x) a.sub_pos[x * nh + d] = v[h][x];
#pragma unroll
        for (int x = 0; x < 6; ++x) a.sub_cov[x * nh + d] = v[h][3 + x];
      }
    }
  }
}

}  // namespace

template <typename T>
hipError_t launch_final_init(const FinalRoundArgs<T>& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const int64_t m = a.n > a.n_hits ? a.n : a.n_hits;
  hipLaunchKernelGGL(final_init_kernel<T>, dim3(unsigned((m + kFinalBlock - 1) / kFinalBlock)), dim3(kFinalBlock), 0,
                     s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_final_round(const FinalRoundArgs<T>& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(final_round_kernel<T>, dim3(unsigned((a.n + kRoundTracks - 1) / kRoundTracks)),
                     dim3(kRoundBlock), 0, s, a);
  return hipGetLastError();
}

template hipError_t launch_final_init<float>(const FinalRoundArgs<float>&, hipStream_t);
template hipError_t launch_final_init<double>(const FinalRoundArgs<double>&, hipStream_t);
template hipError_t launch_final_round<float>(const FinalRoundArgs<float>&, hipStream_t);
template hipError_t launch_final_round<double>(const FinalRoundArgs<double>&, hipStream_t);

}  // namespace kf
