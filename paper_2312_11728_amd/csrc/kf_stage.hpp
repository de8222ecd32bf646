// Per-block staging of the detector description (and the alignment) in LDS,
// shared by the fit and adjoint kernels, and the per-wave staging buffer of
// the hit entries used by the staged fit kernels (forward and backward).
#pragma once

#include "kf_kernels.hpp"

namespace kf {

// ---- geometry staged in LDS --------------------------------------------------
template <typename T>
struct GeomLds {
  T pos[kMaxLayers];
  T x0[kMaxLayers];
  int kind[kMaxLayers];
};

template <typename T>
__device__ __forceinline__ void stage_geometry(GeomLds<T>& sg, const GeomArgs& g) {
  for (int i = threadIdx.x; i < g.n_layers; i += blockDim.x) {
    sg.pos[i] = T(g.pos[i]);
    sg.x0[i] = T(g.x0[i]);
    sg.kind[i] = g.kind[i];
  }
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ void stage_align(T* sal, const FitArgs<T>& a, const GeomArgs& g) {
  if (a.align) {
    for (int i = threadIdx.x; i < g.n_layers; i += blockDim.x) {
      sal[i] = a.align[i];
      sal[kMaxLayers + i] = a.align[g.n_layers + i];
    }
  }
}

// ---- hits of a wave staged in LDS, a few entries per track at a time ----------

// entries per track and chunk: the LDS of a 256-thread block (4 waves) plus
// the state backup must allow the WAVES blocks per CU the register budget
// allows
template <typename T, int WAVES>
constexpr int stage_entries() {
  return sizeof(T) == 4 ? (WAVES == 1 ? 8 : 4) : (WAVES == 1 ? 4 : 1);
}

template <typename T, int J>
struct StageBuf {
  T v[9][J][64];        // hit x, y, z, then the 6 covariance terms
  int32_t lv[J][64];    // layer (low 16 bits) | valid << 16
  int32_t e0[64];       // first entry of each lane's track
  int32_t len[64];      // entries of each lane's track (0: no track)
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

// The rows of a chunk that a lane copies: row r of every chunk is entry
// j0 + jj of the track in slot r * (64 / J) + lane / J, jj = lane % J, so that
// consecutive lanes read consecutive entries of one track (64 / J runs of J
// contiguous values a load).  The slot of a row is the same in every chunk:
// its track's first entry and last index stay in registers.
template <int J>
struct StageRows {
  int32_t e0[J], last[J];   // last < 0: no entries
};

template <typename T, int J>
__device__ __forceinline__ void stage_rows(const StageBuf<T, J>& sb, StageRows<J>& rows) {
  const int lane = int(threadIdx.x) & 63;
#pragma unroll
  for (int r = 0; r < J; ++r) {
    const int l = r * (64 / J) + lane / J;
    rows.e0[r] = sb.e0[l];
    rows.last[r] = sb.len[l] - 1;
  }
}

// Off: the type of a byte offset from the arrays' starts, which do not depend
// on the lane.  32 bits, where every array is below 4 GB, leave an address
// one shift per row and element size instead of a 64-bit addition per load.
template <typename Off, typename T, int J>
__device__ __forceinline__ void load_rows(const FitArgs<T>& a, const uint32_t (&e)[J], int32_t (&lv)[J],
                                          T (&v)[J][9]) {
  const int64_t nh = a.n_hits;
#pragma unroll
  for (int r = 0; r < J; ++r) {
    const Off o = Off(e[r]);
    const uint16_t lay = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(a.hit_layer) + o * 2);
    lv[r] = int32_t(lay) | (a.hit_valid[o] ? (1 << 16) : 0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      v[r][k] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.hit_pos + k * nh) + o * Off(sizeof(T)));
#pragma unroll
    for (int k = 0; k < 6; ++k)
      v[r][3 + k] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.hit_cov + k * nh) + o * Off(sizeof(T)));
  }
}

// Copies entries [j0, j0 + J) of the wave's 64 tracks into LDS (DIR 1: counted
// up from each track's e0; -1: down).  All rows are loaded before any is
// written, so a chunk costs one memory round trip.  A slot past the end of
// its track loads the track's last entry, one without entries entry 0 (the
// caller stages only while some track has an entry, so n_hits > 0); those
// slots are never read.
template <int DIR, typename T, int J>
__device__ __forceinline__ void stage_chunk(const FitArgs<T>& a, const StageRows<J>& rows, int j0, StageBuf<T, J>& sb) {
  const int lane = int(threadIdx.x) & 63;
  const int jj = lane % J;
  uint32_t e[J];
#pragma unroll
  for (int r = 0; r < J; ++r) {
    const int k = min(j0 + jj, rows.last[r]);
    e[r] = uint32_t(rows.last[r] < 0 ? 0 : rows.e0[r] + DIR * k);
  }
  int32_t lv[J];
  T v[J][9];
  if (a.n_hits <= int64_t(0xffffffffu / sizeof(T)))
    load_rows<uint32_t>(a, e, lv, v);
  else
    load_rows<uint64_t>(a, e, lv, v);
#pragma unroll
  for (int r = 0; r < J; ++r) {
    const int l = r * (64 / J) + lane / J;
    sb.lv[jj][l] = lv[r];
#pragma unroll
    for (int k = 0; k < 9; ++k) sb.v[k][jj][l] = v[r][k];
  }
}

}  // namespace kf
