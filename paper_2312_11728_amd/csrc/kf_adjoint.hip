// HIP kernels of the reverse pass: one track per lane for the adjoint sweep,
// then a deterministic two-stage reduction of the hit-position gradients into
// the per-layer alignment gradient (fixed summation order: the result does
// not depend on scheduling).
#include "kf_adjoint.hpp"
#include "kf_stage.hpp"

namespace kf {

// Entries of track t that a reverse sweep over the stored states takes: the
// range of the fit, cut by adjoint_stop_kernel's count if the fit was stopped.
template <typename T, typename Acc>
__device__ __forceinline__ void completed_range(const AdjArgs<T>& a, int64_t t, const Acc& acc, int len, int& k0,
                                                int& n) {
  fitted_range(acc, len, a.f.max_len, k0, n);
  if (n > 0 && was_stopped(a, t)) n = int(a.grad_seed[t]);
}

// Reverse sweep without stored states (seg > 1 and no workspace), one track
// per lane: each state is recomputed from its segment's checkpoint.
template <typename T>
__global__ void __launch_bounds__(256) adjoint_recompute_kernel(AdjArgs<T> a, GeomArgs g) {
  __shared__ GeomLds<T> sg;
  __shared__ T sal[2 * kMaxLayers];
  stage_align(sal, a.f, g);
  stage_geometry(sg, g);
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= a.f.n) return;
  const int64_t e0 = a.f.hit_offsets[t];
  const int len = int(a.f.hit_offsets[t + 1] - e0);
  CsrTrack<T> acc{a.f, e0};
  int k0, n;
  completed_range(a, t, acc, len, k0, n);
  adjoint_sweep<false>(a, TrackGeom<T>{sg.kind, sg.pos, sg.x0, g.n_layers, T(g.bz), T(g.mass)},
                       a.f.align ? sal : nullptr, t, acc, len, e0, k0, n);
}

// Reverse sweep of tracks [w0, w0 + 64) (one wave; every lane must call it)
// over the stored states, the steps of adjoint_sweep<true>.  The hits come
// through LDS, the entries of a chunk counted down from each track's last; a
// processed entry's gradient takes the place of its hit there, and the chunk's
// gradients are written in the order of its loads.
template <typename T, int J>
__device__ void adjoint_wave_staged(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t w0,
                                    StageBuf<T, J>& sb) {
  const FitArgs<T>& f = a.f;
  const int lane = int(threadIdx.x) & 63;
  const int64_t t = w0 + lane, nh = f.n_hits;
  const bool in_range = t < f.n;
  int64_t e_last = 0;
  int n_done = 0;
  double wchi = 1.0;
  if (in_range) {
    const int64_t e0 = f.hit_offsets[t];
    const int len = int(f.hit_offsets[t + 1] - e0);
    int k0;
    completed_range(a, t, CsrTrack<T>{f, e0}, len, k0, n_done);
    e_last = e0 + k0 + n_done - 1;
    // entries outside the fit: before the first valid one, past max_len or
    // the track's stop
    for (int k = 0; k < len; ++k) {
      if (k == k0) k += n_done;
      if (k >= len) break;
      a.grad_hit[e0 + k] = a.grad_hit[nh + e0 + k] = a.grad_hit[2 * nh + e0 + k] = T(0);
    }
    if (a.w) wchi = double(a.w[t]);
  }
  sb.e0[lane] = int32_t(n_done > 0 ? e_last : 0);
  sb.len[lane] = n_done;
  const int kmax = wave_max(n_done);
  double pb[6], cb[21];
#pragma unroll
  for (int i = 0; i < 6; ++i) pb[i] = 0.0;
#pragma unroll
  for (int i = 0; i < 21; ++i) cb[i] = 0.0;
  int q_after = 0;
  const StoredStates<T> stored(a, t);
  wave_sync();
  StageRows<J> rows;
  stage_rows(sb, rows);
  for (int j0 = 0; j0 < kmax; j0 += J) {
    stage_chunk<-1>(f, rows, j0, sb);
    wave_sync();
    const int jn = min(J, kmax - j0);
    for (int jj = 0; jj < jn; ++jj) {
      const int j = n_done - 1 - (j0 + jj);
      if (j < 0) continue;
      const int32_t lv = sb.lv[jj][lane];
      const bool valid = (lv >> 16) != 0;
      const int lay = int16_t(lv & 0xffff);
      T p[6], c[21], m[3], V[6];
      int q, prev = lay;
      if (j >= 1) {
        stored.before(j, p, c, q);
        prev = jj + 1 < J ? int16_t(sb.lv[jj + 1][lane] & 0xffff) : f.hit_layer[e_last - (j0 + jj) - 1];
      } else {
        stored.seed(p, c, q);
      }
#pragma unroll
      for (int x = 0; x < 3; ++x) m[x] = sb.v[x][jj][lane];
#pragma unroll
      for (int x = 0; x < 6; ++x) V[x] = sb.v[3 + x][jj][lane];
      double hb[3];
      step_vjp(p, c, q, j0 + jj == 0 ? q : q_after, j, lay, prev, valid, m, V, g, sal, wchi, pb, cb, hb);
#pragma unroll
      for (int x = 0; x < 3; ++x) sb.v[x][jj][lane] = T(hb[x]);
      q_after = q;
    }
    wave_sync();   // every lane's gradients are there
#pragma unroll
    for (int r = 0; r < J; ++r) {
      const int l = r * (64 / J) + lane / J, jj = lane % J;
      if (j0 + jj <= rows.last[r]) {
        const int64_t e = int64_t(rows.e0[r]) - (j0 + jj);
#pragma unroll
        for (int x = 0; x < 3; ++x) a.grad_hit[x * nh + e] = sb.v[x][jj][l];
      }
    }
    wave_sync();   // and are read before the next chunk is staged
  }
  if (in_range) {
#pragma unroll
    for (int i = 0; i < 6; ++i) a.grad_seed[i * f.ld + t] = T(pb[i]);
  }
}

// The reverse sweep over stored states.  It runs at one wave per SIMD (the
// adjoints, the state and the Jacobian fill the registers) and so holds the
// sweep alone: the forward steps that find where a stopped track ended are
// taken by adjoint_stop_kernel, which leaves the number of completed entries
// in grad_seed, and the states come from the checkpoints or the refill pass.
// Hits and their gradients go through LDS: lanes are tracks, whose entries lie
// a track's length apart, and read directly every 8-byte value moved a cache
// line of its own.  100k tracks of 20 entries, FP64: 365 us (786 us with dense
// 6x6 products, the forward steps and direct reads in this kernel; 543 us with
// direct reads and the Jacobian's intermediates in memory); one wave's chain
// of 20 entries takes 125 us.
constexpr int kAdjointBlock = 256;

template <typename T>
__global__ void __launch_bounds__(kAdjointBlock) adjoint_kernel(AdjArgs<T> a, GeomArgs g) {
  constexpr int J = stage_entries<T, 1>();
  __shared__ GeomLds<T> sg;
  __shared__ T sal[2 * kMaxLayers];
  __shared__ StageBuf<T, J> sb[kAdjointBlock / 64];
  stage_align(sal, a.f, g);
  stage_geometry(sg, g);
  const int64_t w0 = int64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63u);
  adjoint_wave_staged<T, J>(a, TrackGeom<T>{sg.kind, sg.pos, sg.x0, g.n_layers, T(g.bz), T(g.mass)},
                            a.f.align ? sal : nullptr, w0, sb[threadIdx.x >> 6]);
}

// Per stopped track, the entries that the forward fit completed, into
// grad_seed[0][t] (at most 64; the sweep overwrites it with the gradient).
template <typename T>
__global__ void __launch_bounds__(256) adjoint_stop_kernel(AdjArgs<T> a, GeomArgs g) {
  __shared__ GeomLds<T> sg;
  __shared__ T sal[2 * kMaxLayers];
  stage_align(sal, a.f, g);
  stage_geometry(sg, g);
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= a.f.n || !was_stopped(a, t)) return;
  const int64_t e0 = a.f.hit_offsets[t];
  CsrTrack<T> acc{a.f, e0};
  int k0, n;
  fitted_range(acc, int(a.f.hit_offsets[t + 1] - e0), a.f.max_len, k0, n);
  if (n > 0)
    n = steps_done(a, TrackGeom<T>{sg.kind, sg.pos, sg.x0, g.n_layers, T(g.bz), T(g.mass)}, a.f.align ? sal : nullptr,
                   t, acc, k0, n);
  a.grad_seed[t] = T(n);
}

// The states the reverse sweep reads (seg > 1 with a state buffer), one
// thread per track, at the forward fit's occupancy rather than under the
// reverse pass's registers: for every entry j >= 1 (relative to the track's
// first valid entry), the state before it -- the checkpoint at the start of
// each segment, then the segment's forward steps -- stored in slot j - 1.
// These are the steps fill_segment takes, in the same order on the same
// values.  The wave's hits come through LDS a few entries per track at a
// time, as in the forward fit: all rows of a chunk are loaded before any is
// written, consecutive lanes reading consecutive entries of one track (a
// slot past a track's end loads its last entry and is never read).
constexpr int kRefillBlock = 256;

template <typename T, int J>
__device__ void refill_wave_staged(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t w0,
                                   StageBuf<T, J>& sb) {
  const FitArgs<T>& f = a.f;
  const int lane = int(threadIdx.x) & 63;
  const int64_t t = w0 + lane;
  const bool in_range = t < f.n;
  int64_t e0 = 0;
  int len = 0;
  if (in_range) {
    e0 = f.hit_offsets[t];
    len = int(f.hit_offsets[t + 1] - e0);
    if (len > f.max_len) len = f.max_len;
  }
  sb.e0[lane] = int32_t(e0);
  sb.len[lane] = len;
  const int kmax = wave_max(len);
  const int64_t n = f.n, cst = f.ld * int64_t(f.n_seg);
  T p[6], c[21];
  int q = 0, prev = 0, prev_lay = 0, k0 = -1;
  wave_sync();
  StageRows<J> rows;
  stage_rows(sb, rows);
  for (int j0 = 0; j0 < kmax; j0 += J) {
    stage_chunk<1>(f, rows, j0, sb);
    wave_sync();
    const int jn = min(J, kmax - j0);
    for (int jj = 0; jj < jn; ++jj) {
      const int k = j0 + jj;
      if (!in_range || k >= len) continue;
      const int32_t lv = sb.lv[jj][lane];
      const bool valid = (lv >> 16) != 0;
      const int lay = int16_t(lv & 0xffff);
      if (k0 < 0) {
        if (valid) k0 = k;   // entry j = 0: its state is the seed
        prev_lay = lay;
        continue;
      }
      const int j = k - k0;
      if ((j - 1) % f.seg == 0) {
        // a segment starts: its checkpoint, after entry j - 1 of layer prev_lay
        const T* base = f.ckpt + int64_t((j - 1) / f.seg) * f.ld + t;
#pragma unroll
        for (int i = 0; i < 6; ++i) p[i] = base[i * cst];
#pragma unroll
        for (int i = 0; i < 21; ++i) c[i] = base[(6 + i) * cst];
        q = int(base[27 * cst]);
        prev = prev_lay;
      }
      T* slot = a.seg_buf + int64_t(j - 1) * kSegVals * n + t;
#pragma unroll
      for (int i = 0; i < 6; ++i) slot[i * n] = p[i];
#pragma unroll
      for (int i = 0; i < 21; ++i) slot[(6 + i) * n] = c[i];
      slot[27 * n] = T(q);
      if (j % f.seg != 0 && j + 1 < len - k0 && known_layer(g, lay)) {
        T m[3], V[6];
#pragma unroll
        for (int x = 0; x < 3; ++x) m[x] = sb.v[x][jj][lane];
#pragma unroll
        for (int x = 0; x < 6; ++x) V[x] = sb.v[3 + x][jj][lane];
        T c2;
        uint32_t sst = 0;
        step_forward(p, c, q, j, lay, prev, valid, m, V, g, sal, c2, sst);
        prev = lay;
      }
      prev_lay = lay;
    }
    wave_sync();   // every lane has read the chunk before the next one is staged
  }
}

template <typename T>
__global__ void __launch_bounds__(kRefillBlock, sizeof(T) == 4 ? 2 : 1) refill_kernel(AdjArgs<T> a, GeomArgs g) {
  constexpr int J = stage_entries<T, sizeof(T) == 4 ? 2 : 1>();
  __shared__ GeomLds<T> sg;
  __shared__ T sal[2 * kMaxLayers];
  __shared__ StageBuf<T, J> sb[kRefillBlock / 64];
  stage_align(sal, a.f, g);
  stage_geometry(sg, g);
  const int64_t w0 = int64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63u);
  refill_wave_staged<T, J>(a, TrackGeom<T>{sg.kind, sg.pos, sg.x0, g.n_layers, T(g.bz), T(g.mass)},
                           a.f.align ? sal : nullptr, w0, sb[threadIdx.x >> 6]);
}

// Stage 1: one wave per kAlignPerBlock consecutive entries of the batch
// (entries hit_offsets[0] .. hit_offsets[n]), lane l taking entries l,
// l + 64, ... of the block's range, so that every load of the wave is
// coalesced.  A barrel hit h with gradient hb contributes
// (h_x hb_y - h_y hb_x)/R to the r-phi offset of its layer (the rotation
// m = R(a/R) h keeps the cross product; the sum is divided by R once) and hb_z
// to the z offset; disk hits and holes contribute 0.  Each lane adds into its
// own LDS column; then lane l adds the 64 columns of layer l, starting with
// column l (equal columns would meet in one LDS bank).  Fixed order
// throughout: the result does not depend on scheduling.  The columns are those
// of the layers there are (dynamic LDS, 1 KB a layer in FP64), so that a CU
// holds all its blocks at once.  Bound by memory latency, then bandwidth (90
// MB for 2M FP64 entries): 31 us, from 82 us with 64 columns of every possible
// layer, a division per entry and all lanes of the last sum in one bank.
template <typename T>
__global__ void __launch_bounds__(64) align_partial_kernel(AdjArgs<T> a, GeomArgs g) {
  extern __shared__ double align_columns[];
  T* part = reinterpret_cast<T*>(align_columns);   // [2][n_layers][64]
  const int lane = threadIdx.x, nl = g.n_layers;
  for (int l = 0; l < 2 * nl; ++l) part[l * 64 + lane] = T(0);
  const bool barrel_lane = lane < nl && g.kind[lane] == 0;
  const uint64_t barrel = __ballot(barrel_lane);   // bit l: layer l is a barrel
  const int64_t nh = a.f.n_hits;
  const int64_t first = a.f.hit_offsets[0], last = a.f.hit_offsets[a.f.n];
  const int64_t b0 = first + int64_t(blockIdx.x) * kAlignPerBlock;
  // kAhead iterations' loads, from clamped indices, then their sums without a
  // branch: entries that do not contribute add zero to layer 0
  constexpr int kAhead = 8;
  for (int k = 0; k < kAlignPerBlock / 64; k += kAhead) {
    T hx[kAhead], hy[kAhead], gx[kAhead], gy[kAhead], gz[kAhead];
    int lay[kAhead];
    bool use[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t e = b0 + int64_t(k + u) * 64 + lane;
      use[u] = e < last;
      const int64_t ee = align_load_entry(e, last);
      use[u] = use[u] && a.f.hit_valid[ee] != 0;
      lay[u] = a.f.hit_layer[ee];
      hx[u] = a.f.hit_pos[ee];
      hy[u] = a.f.hit_pos[nh + ee];
      gx[u] = a.grad_hit[ee];
      gy[u] = a.grad_hit[nh + ee];
      gz[u] = a.grad_hit[2 * nh + ee];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const bool in = use[u] && lay[u] >= 0 && lay[u] < nl && (barrel >> (lay[u] & 63) & 1);
      T* col = part + (in ? lay[u] : 0) * 64 + lane;
      const T dphi = hx[u] * gy[u] - hy[u] * gx[u];
      col[0] += in ? dphi : T(0);
      col[nl * 64] += in ? gz[u] : T(0);
    }
  }
  __syncthreads();
  if (lane >= nl) return;
  T dphi = T(0), dz = T(0);
#pragma unroll 8
  for (int k = 0; k < 64; ++k) {
    const int col = (k + lane) & 63;
    dphi += part[lane * 64 + col];
    dz += part[(nl + lane) * 64 + col];
  }
  // [component][layer][block], which stage 2 reads along the blocks
  T* out = a.partial + int64_t(lane) * gridDim.x + blockIdx.x;
  out[0] = barrel_lane ? dphi / T(g.pos[lane]) : T(0);
  out[int64_t(kMaxLayers) * gridDim.x] = dz;
}

// Stage 2: one block per (component, layer): thread k adds the partials of
// blocks k, k + 256, ... in order, then a fixed tree over the threads.
template <typename T>
__global__ void __launch_bounds__(256) align_final_kernel(AdjArgs<T> a, int32_t n_layers, int64_t n_blocks) {
  __shared__ T red[256];
  const int c = blockIdx.x / n_layers, l = blockIdx.x % n_layers;
  const T* part = a.partial + (int64_t(c) * kMaxLayers + l) * n_blocks;
  T acc = T(0);
  for (int64_t b = threadIdx.x; b < n_blocks; b += 256) acc += part[b];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (int(threadIdx.x) < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.grad_align[c * n_layers + l] = red[0];
}

template <typename T>
hipError_t launch_adjoint(const AdjArgs<T>& a, const GeomArgs& g, hipStream_t s) {
  if (a.f.n > 0) {
    const int64_t grid = (a.f.n + 255) / 256;
    if (a.seg_buf)
      hipLaunchKernelGGL(refill_kernel<T>, dim3(unsigned((a.f.n + kRefillBlock - 1) / kRefillBlock)), dim3(kRefillBlock), 0,
                         s, a, g);
    if (a.fwd_status) hipLaunchKernelGGL(adjoint_stop_kernel<T>, dim3(unsigned(grid)), dim3(256), 0, s, a, g);
    if (a.seg_buf || a.f.seg == 1)
      hipLaunchKernelGGL(adjoint_kernel<T>, dim3(unsigned((a.f.n + kAdjointBlock - 1) / kAdjointBlock)),
                         dim3(kAdjointBlock), 0, s, a, g);
    else
      hipLaunchKernelGGL(adjoint_recompute_kernel<T>, dim3(unsigned(grid)), dim3(256), 0, s, a, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.grad_align) {
    // no tracks: nothing contributes (and the offsets may be absent)
    const int64_t nb = a.f.n > 0 ? adjoint_partial_blocks(a.f.n_hits) : 0;
    const unsigned lds = unsigned(2 * g.n_layers * 64 * sizeof(T));   // at most 64 KB
    if (nb > 0) hipLaunchKernelGGL(align_partial_kernel<T>, dim3(unsigned(nb)), dim3(64), lds, s, a, g);
    hipLaunchKernelGGL(align_final_kernel<T>, dim3(unsigned(2 * g.n_layers)), dim3(256), 0, s, a, g.n_layers, nb);
  }
  return hipGetLastError();
}

template hipError_t launch_adjoint<float>(const AdjArgs<float>&, const GeomArgs&, hipStream_t);
template hipError_t launch_adjoint<double>(const AdjArgs<double>&, const GeomArgs&, hipStream_t);

}  // namespace kf
