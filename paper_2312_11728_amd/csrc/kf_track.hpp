// The per-track layer loop of the forward fit, callable from device and host
// code: the kernels run it with one track per lane.
#pragma once

#include "kf_kernels.hpp"
#include "kf_math.hpp"
#include "kf_surface.hpp"

namespace kf {

// Spacing of the hits of a spaced seed (mode 1), cm in the transverse plane:
// wide enough to give closely spaced disk hits a usable lever arm, and below
// the 3 cm between the two innermost barrel layers of the toy detectors, so
// that whether a barrel hit pair qualifies is never decided by rounding.
constexpr double kSeedSpacing = 2.5;

// Seed of track t from three of its valid hits (mode 0: the first three;
// mode 1: the first, then each next one >= kSeedSpacing away in the
// transverse plane from the previously chosen one), with the charge and the
// status (KF_TRK_BAD_INPUT without three such hits; the state is then zero).
template <typename T>
struct SeedOut {
  T p[6];
  int q;
  uint32_t st;
};

// Not inlined: the seeding kernel and the fits that seed their own tracks
// call one compiled copy, so both give the same bits.
template <typename T>
KF_HD __attribute__((noinline)) SeedOut<T> seed_of_track(const int32_t* __restrict__ off,
                                                        const uint8_t* __restrict__ valid,
                                                        const T* __restrict__ pos, int64_t nh, int64_t t, int mode,
                                                        T bz) {
  const int64_t e0 = off[t], e1 = off[t + 1];
  int64_t pick[3] = {-1, -1, -1};
  int cnt = 0;
  T lx = T(0), ly = T(0);
  for (int64_t e = e0; e < e1 && cnt < 3; ++e) {
    if (!valid[e]) continue;
    const T hx = pos[e], hy = pos[nh + e];
    bool take = (cnt == 0);
    if (!take) {
      if (mode == 0) {
        take = true;
      } else {
        const T dx = hx - lx, dy = hy - ly;
        take = k_sqrt(dx * dx + dy * dy) >= T(kSeedSpacing);
      }
    }
    if (take) {
      pick[cnt++] = e;
      lx = hx;
      ly = hy;
    }
  }
  SeedOut<T> o;
#pragma unroll
  for (int i = 0; i < 6; ++i) o.p[i] = T(0);
  o.q = 1;
  o.st = 0;
  if (cnt == 3) {
    T h[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) h[k][c] = pos[c * nh + pick[k]];
    seed_from_hits(h[0], h[1], h[2], bz, o.p, o.q);
  } else {
    o.st |= TRK_BAD_INPUT;
  }
  return o;
}

// the seed covariance: wide and diagonal, so that the first hits decide
template <typename T>
KF_HD inline void seed_covariance(T c[21]) {
  const T diag[6] = {T(1), T(1), T(1), T(1), T(0.01), T(0.01)};
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j) c[sym(i, j)] = (i == j) ? diag[i] : T(0);
}

template <typename T>
KF_HD inline void seed_track(const SeedArgs<T>& a, int64_t t) {
  const SeedOut<T> o = seed_of_track(a.hit_offsets, a.hit_valid, a.hit_pos, a.n_hits, t, int(a.mode), T(a.bz));
  T c[21];
  seed_covariance(c);
#pragma unroll
  for (int i = 0; i < 6; ++i) a.seed_state[i * a.ld + t] = o.p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) a.seed_cov[i * a.ld + t] = c[i];
  a.seed_charge[t] = int8_t(o.q);
  a.trk_status[t] = o.st;
}

template <typename T>
struct TrackGeom {
  const int* kind;
  const T* pos;
  const T* x0;
  int n_layers;
  T bz;
  T mass;
};

template <typename T>
KF_HD inline void write_checkpoint(const FitArgs<T>& a, int64_t t, int slot, const T p[6], const T c[21], int q) {
  const int64_t stride = a.ld * int64_t(a.n_seg);
  T* base = a.ckpt + int64_t(slot) * a.ld + t;
#pragma unroll
  for (int i = 0; i < 6; ++i) base[i * stride] = p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) base[(6 + i) * stride] = c[i];
  base[27 * stride] = T(q);
}

// Entry access for the per-track loop: the caller's CSR arrays ...
template <typename T>
struct CsrTrack {
  const FitArgs<T>& a;
  int64_t e0;
  KF_HD inline bool valid(int k) const { return a.hit_valid[e0 + k] != 0; }
  KF_HD inline int layer(int k) const { return a.hit_layer[e0 + k]; }
  KF_HD inline void load(int k, int& lay, bool& val, T m[3], T V[6]) const {
    const int64_t e = e0 + k, nh = a.n_hits;
    lay = a.hit_layer[e];
    val = a.hit_valid[e] != 0;
    m[0] = a.hit_pos[e];
    m[1] = a.hit_pos[nh + e];
    m[2] = a.hit_pos[2 * nh + e];
#pragma unroll
    for (int i = 0; i < 6; ++i) V[i] = a.hit_cov[i * nh + e];
  }
};

// ... or the packed tile-transposed copy (slot s of its tile).
template <typename T>
struct PackedTrack {
  const PackedHits<T>& pk;
  int64_t base;  // tile_base + s % kTile
  KF_HD inline bool valid(int k) const { return (pk.lv[base + int64_t(k) * kTile] >> 16) != 0; }
  KF_HD inline void load(int k, int& lay, bool& val, T m[3], T V[6]) const {
    const int64_t i = base + int64_t(k) * kTile, st = pk.stride;
    const int32_t lv = pk.lv[i];
    lay = int16_t(lv & 0xffff);
    val = (lv >> 16) != 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) m[c] = pk.hit[c * st + i];
#pragma unroll
    for (int c = 0; c < 6; ++c) V[c] = pk.hit[(3 + c) * st + i];
  }
};

// alignment correction of a barrel hit (a rotation by a_rphi / R about the
// beam axis and a shift a_z along it)
template <typename T>
KF_HD inline void align_hit(T m[3], const T* __restrict__ sal, int lay, T pos) {
  T sa, ca;
  k_sincos(sal[lay] * k_rcp(pos), &sa, &ca);
  const T hx = m[0], hy = m[1];
  m[0] = ca * hx - sa * hy;
  m[1] = sa * hx + ca * hy;
  m[2] += sal[kMaxLayers + lay];
}

// One entry of the forward fit: transport to layer `lay` (entry j > 0; the
// first entry only adds its own layer's material), then, for a valid hit, the
// alignment correction of the hit (barrel layers: rotation by a_rphi / R about
// the beam axis and a shift a_z along it) and the update.  m is overwritten
// with the aligned hit.  Returns false when the crossing fails; c2 is the
// entry's chi2 contribution (0 for a hole).
template <int R2 = kFuseAny, typename T, typename PreMaterial = NoPreMaterial>
KF_HD inline bool step_forward(T p[6], T c[21], int& q, int j, int lay, int prev, bool valid, T m[3], const T V[6],
                               const TrackGeom<T>& g, const T* __restrict__ sal, T& c2, uint32_t& sst,
                               const PreMaterial& pre = PreMaterial()) {
  const int kind = g.kind[lay];
  if (j > 0) {
    if (!propagate<R2>(p, c, q, kind, g.pos[lay], g.x0[lay], lay == prev, true, g.bz, g.mass, sst,
                       static_cast<T*>(nullptr), static_cast<NoTape*>(nullptr), pre))
      return false;
  } else {
    add_material_here<R2>(p, c, kind, g.x0[lay], g.mass, sst);
  }
  c2 = T(0);
  if (valid) {
    if (sal && kind == 0) align_hit(m, sal, lay, g.pos[lay]);
    update(p, c, q, m, V, c2, sst);
  }
  return true;
}

// The covariance a fit carries from entry to entry: the 6x6 one in FP32, the
// 5x5 one of the surface frame in FP64.  In FP64 the surface frame saves a
// third of the step.  In FP32 the 6x6 step keeps its rounding: while 1/pT is
// compatible with zero its rounding decides the charge that a filtered state
// is kept with, which the smoother and the final fit's decisions depend on,
// so that another rounding (the 5x5 form's errors are no larger) changes one
// smoothed entry in a million visibly.
template <typename T>
constexpr bool kOnSurface = sizeof(T) == 8;

// A track on its way through the forward or backward fit.  bk: room for 28
// values at bk[k * bk_stride], kept out of registers (in LDS on the device).
// FP32: s.p, s.q and c6 hold the state, bk the backup of a step.  FP64:
// done = 0: no entry completed, bk holds the starting state and its 6x6
// covariance.  done = 1: the first entry completed, bk holds its result (a
// 6x6 covariance of full rank, which a checkpoint or the output may need) and
// s the covariance confined to the track's plane.  done = 2: s is
// on the last completed entry's surface; bk is the backup of a step.
template <typename T>
struct FitState {
  SurfState<T> s;
  T c6[kOnSurface<T> ? 1 : 21];
  int done, prev, nval;
  int ck_next, ck_slot;   // the next entry with a checkpoint before it, its slot
  uint32_t st;
  T chi2;
};

template <typename T>
KF_HD inline void save_full(T* bk, int bk_stride, const T p[6], const T c[21]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) bk[i * bk_stride] = p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) bk[(6 + i) * bk_stride] = c[i];
}

template <typename T>
KF_HD inline void load_full(const T* bk, int bk_stride, T p[6], T c[21]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) p[i] = bk[i * bk_stride];
#pragma unroll
  for (int i = 0; i < 21; ++i) c[i] = bk[(6 + i) * bk_stride];
}

// the track's state and 6x6 covariance after its last completed entry
template <typename T>
KF_HD inline void current_state(const FitState<T>& f, const T* bk, int bk_stride, T p[6], T c[21]) {
  if (kOnSurface<T> && f.done < 2) {
    load_full(bk, bk_stride, p, c);
    return;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) p[i] = f.s.p[i];
  if constexpr (kOnSurface<T>) {
    expand_cov(f.s, c);
  } else {
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = f.c6[i];
  }
}

// the starting state of a fit
template <typename T>
KF_HD inline void start_state(FitState<T>& f, T* bk, int bk_stride, const T p[6], const T c[21], int q) {
  f.s.q = q;
  f.done = 0;
  f.prev = 0;
  f.nval = 0;
  f.ck_next = 1;
  f.ck_slot = 0;
  f.chi2 = T(0);
  if constexpr (kOnSurface<T>) {
    save_full(bk, bk_stride, p, c);
  } else {
#pragma unroll
    for (int i = 0; i < 6; ++i) f.s.p[i] = p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) f.c6[i] = c[i];
  }
}

// One entry of the forward (BACK false) or backward fit: layer check,
// checkpoint (forward), the step to the entry's layer with its material and,
// for a valid hit, the update; rolled back when it turns non-finite.  j:
// index relative to the track's first entry (forward: its first valid one),
// which takes its layer's material where the track is.  pre is called with
// the state on a later entry's surface before the layer's material.  Returns
// false when the track stops here (the reason is in f.st).
//
// Surface frame: the first entry works on the starting state's 6x6 covariance
// and leaves it confined to the track's plane.  The 6x6 update has one place,
// for the first entry and for the lanes that update5 turns away: most waves
// pass it by.
template <bool BACK, int R2, typename T, typename PreMaterial = NoPreMaterial>
KF_HD inline bool fit_entry(const FitArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t, int j,
                            int lay, bool valid, T m[3], const T V[6], FitState<T>& f, T* bk, int bk_stride,
                            const PreMaterial& pre = PreMaterial()) {
  if (lay < 0 || lay >= g.n_layers) {
    f.st |= TRK_BAD_INPUT;
    return false;
  }
  if constexpr (!kOnSurface<T>) {
    T* p = f.s.p;
    T* c = f.c6;
    if (!BACK && a.ckpt && j == f.ck_next) {
      write_checkpoint(a, t, f.ck_slot, p, c, f.s.q);
      f.ck_next += a.seg < kMaxLen ? a.seg : kMaxLen;
      ++f.ck_slot;
    }
    save_full(bk, bk_stride, p, c);
    const int q = f.s.q;
    uint32_t sst = 0;
    T c2;
    if (!step_forward<R2>(p, c, f.s.q, j, lay, f.prev, valid, m, V, g, sal, c2, sst, pre)) {
      f.st |= sst;
      return false;
    }
    f.st |= sst;
    if (!all_finite(p, c, c2)) {
      f.st |= TRK_NONFINITE;
      load_full(bk, bk_stride, p, c);
      f.s.q = q;
      return false;
    }
    f.chi2 += c2;
    f.nval += valid ? 1 : 0;
    f.prev = lay;
    return true;
  }
  SurfState<T>& s = f.s;
  const int q = s.q, kind = g.kind[lay];
  const T x0 = g.x0[lay];
  uint32_t sst = 0;
  T c2 = T(0), C[21];
  bool six = j == 0;   // C holds the covariance
  if (six) {
    load_full(bk, bk_stride, s.p, C);
    add_material_here(s.p, C, kind, x0, g.mass, sst);
  } else {
    if (!BACK && a.ckpt && j == f.ck_next) {
      T p[6];
      current_state(f, bk, bk_stride, p, C);
      write_checkpoint(a, t, f.ck_slot, p, C, q);
      f.ck_next += a.seg < kMaxLen ? a.seg : kMaxLen;
      ++f.ck_slot;
    }
    if (f.done == 2) {
#pragma unroll
      for (int i = 0; i < 6; ++i) bk[i * bk_stride] = s.p[i];
#pragma unroll
      for (int i = 0; i < 15; ++i) bk[(6 + i) * bk_stride] = s.c[i];
      bk[21 * bk_stride] = s.tx;
      bk[22 * bk_stride] = s.ty;
    }
    if (!propagate5(s, kind, g.pos[lay], x0, lay == f.prev, g.bz, g.mass, sst, pre)) {
      f.st |= sst;
      return false;
    }
  }
  if (valid) {
    if (sal && kind == 0) align_hit(m, sal, lay, g.pos[lay]);
    if (j > 0 && !update5(s, m, V, c2, sst)) {
      six = true;
      expand_cov(s, C);
    }
  }
  bool ok;
  if (six) {
    if (valid) update(s.p, C, s.q, m, V, c2, sst);
    ok = all_finite(s.p, C, c2);
    if (ok && j == 0) {
      save_full(bk, bk_stride, s.p, C);
      confine_to_track_plane(C, g.bz, s);
    } else {
      compress_cov(C, s);
    }
  } else {
    ok = all_finite5(s, c2);
  }
  f.st |= sst;
  if (!ok) {
    f.st |= TRK_NONFINITE;
    s.q = q;
    if (f.done == 2) {
#pragma unroll
      for (int i = 0; i < 6; ++i) s.p[i] = bk[i * bk_stride];
#pragma unroll
      for (int i = 0; i < 15; ++i) s.c[i] = bk[(6 + i) * bk_stride];
      s.tx = bk[21 * bk_stride];
      s.ty = bk[22 * bk_stride];
      s.kind = g.kind[f.prev];
    }
    return false;
  }
  f.done = j == 0 ? 1 : 2;
  f.chi2 += c2;
  f.nval += valid ? 1 : 0;
  f.prev = lay;
  return true;
}

// The starting state of track t: the given seed, or (make_seeds) the seed
// made from its hits, whose status bits go to st.
template <typename T>
KF_HD inline void load_seed(const FitArgs<T>& a, int64_t t, T bz, T p[6], T c[21], int& q, uint32_t& st) {
  if (a.make_seeds == 0) {
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = a.seed_state[i * a.ld + t];
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = a.seed_cov[i * a.ld + t];
    q = a.seed_charge[t];
    return;
  }
  const SeedOut<T> o = seed_of_track(a.hit_offsets, a.hit_valid, a.hit_pos, a.n_hits, t, a.make_seeds - 1, bz);
#pragma unroll
  for (int i = 0; i < 6; ++i) p[i] = o.p[i];
  q = o.q;
  st |= o.st;
  seed_covariance(c);
  if (a.seed_state_out) {
#pragma unroll
    for (int i = 0; i < 6; ++i) a.seed_state_out[i * a.ld + t] = p[i];
  }
  if (a.seed_cov_out) {
#pragma unroll
    for (int i = 0; i < 21; ++i) a.seed_cov_out[i * a.ld + t] = c[i];
  }
  if (a.seed_charge_out) a.seed_charge_out[t] = int8_t(q);
}

template <typename T>
KF_HD inline void begin_fit(const FitArgs<T>& a, int64_t t, T bz, FitState<T>& f, T* bk, int bk_stride) {
  T p[6], c[21];
  f.st = 0;
  int q;
  load_seed(a, t, bz, p, c, q, f.st);
  start_state(f, bk, bk_stride, p, c, q);
}

template <typename T>
KF_HD inline void store_fit(const FitArgs<T>& a, int64_t t, const T p[6], const T c[21], int q, T chi2, int nval,
                            uint32_t st) {
#pragma unroll
  for (int i = 0; i < 6; ++i) a.state_out[i * a.ld + t] = p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) a.cov_out[i * a.ld + t] = c[i];
  a.charge_out[t] = int8_t(q);
  a.chi2[t] = chi2;
  a.ndf[t] = 2 * nval - 5;
  a.trk_status[t] = st;
}

// Forward fit of track t whose entries are read through `acc` (len entries).
// sal: alignment staged as [rphi x kMaxLayers][z x kMaxLayers] or null.
// Leading holes are skipped: the fit starts at the first valid entry.
template <typename T, typename Acc>
KF_HD inline void fit_track(const FitArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                            const Acc& acc, int len, T* bk, int bk_stride) {
  FitState<T> f;
  begin_fit(a, t, g.bz, f, bk, bk_stride);
  if (len > a.max_len) {
    f.st |= TRK_BAD_INPUT;
    len = a.max_len;
  }
  int k0 = 0;
  while (k0 < len && !acc.valid(k0)) ++k0;
  if (k0 >= len) {
    f.st |= TRK_BAD_INPUT;
  } else {
    // entry data are loaded one entry ahead so that the loads of entry k+1
    // overlap the arithmetic of entry k
    int lay_n;
    bool valid_n;
    T m_n[3], V_n[6];
    acc.load(k0, lay_n, valid_n, m_n, V_n);
    for (int k = k0; k < len; ++k) {
      const int lay = lay_n;
      const bool valid = valid_n;
      T m[3], V[6];
#pragma unroll
      for (int i = 0; i < 3; ++i) m[i] = m_n[i];
#pragma unroll
      for (int i = 0; i < 6; ++i) V[i] = V_n[i];
      if (k + 1 < len) acc.load(k + 1, lay_n, valid_n, m_n, V_n);
      if (!fit_entry<false, kFuseY>(a, g, sal, t, k - k0, lay, valid, m, V, f, bk, bk_stride)) break;
    }
  }
  T p[6], c[21];
  current_state(f, bk, bk_stride, p, c);
  store_fit(a, t, p, c, f.s.q, f.chi2, f.nval, f.st);
}

// Fit of the track in slot / index `i`: LAYOUT 2 reads the packed layout,
// LAYOUT 1 the CSR arrays in length-sorted slot order, LAYOUT 0 the CSR arrays
// with slot = track.
template <typename T, int LAYOUT>
KF_HD inline void fit_slot(const FitArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t i, T* bk,
                           int bk_stride) {
  if constexpr (LAYOUT == 1) {
    const int64_t t = a.pk.order[i];
    const int64_t e0 = a.hit_offsets[t];
    const int len = int(a.hit_offsets[t + 1] - e0);
    CsrTrack<T> acc{a, e0};
    fit_track(a, g, sal, t, acc, len, bk, bk_stride);
  } else if constexpr (LAYOUT == 2) {
    const int64_t t = a.pk.order[i];
    const int len = int(a.hit_offsets[t + 1] - a.hit_offsets[t]);
    PackedTrack<T> acc{a.pk, a.pk.tile_base[i / kTile] + (i % kTile)};
    fit_track(a, g, sal, t, acc, len, bk, bk_stride);
  } else {
    const int64_t e0 = a.hit_offsets[i];
    const int len = int(a.hit_offsets[i + 1] - e0);
    CsrTrack<T> acc{a, e0};
    fit_track(a, g, sal, i, acc, len, bk, bk_stride);
  }
}

}  // namespace kf
