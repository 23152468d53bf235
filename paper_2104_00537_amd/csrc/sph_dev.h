// Per-particle device routines shared by the single-case and the batched
// kernels: the cell key, the sorted-order gather with its interaction view,
// and the symplectic update (Sections 2.5.2 and 5.1 of the DualSPHysics v5.0
// paper).
#pragma once

#include "sph_internal.h"

namespace sph {

// Along a periodic component k (period L > 0, Section 2.7) a coordinate that
// left [o, o + L) re-enters at the other end: x - L, or x + L (o if that
// rounds to o + L).
__device__ inline double wrap_coord(const KParams& kp, int k, double x) {
  const double L = k == 0 ? kp.px : (k == 1 ? kp.py : kp.pz);
  if (!(L > 0.0)) return x;
  const double o = k == 0 ? kp.ox : (k == 1 ? kp.oy : kp.oz);
  if (x >= o + L) return __dsub_rn(x, L);
  if (x < o) {
    x = __dadd_rn(x, L);
    if (x >= o + L) x = o;
  }
  return x;
}

// Cell index per axis = floor((x - origin) * inv): one FP64 subtraction and
// one FP64 multiplication (no contraction is possible), x fastest; inv is the
// inverse cell size, times x_sub along x.  Outside
// the grid, and for particles excluded earlier, the key is ncell_total, so
// they sort last and lie in no cell range.  Periodic components take the
// wrapped coordinate (and its last cell if the product rounds up to the
// end).
template <typename X>  // x(k): the coordinate along component k
__device__ inline uint32_t cell_key_at(const KParams& kp, int dim, X&& x) {
  const double org[3] = {kp.ox, kp.oy, kp.oz};
  const int nc[3] = {kp.ncx, kp.ncy, kp.ncz};
  int c[3] = {0, 0, 0};
  for (int k = 0; k < dim; ++k) {
    const double d = __dsub_rn(wrap_coord(kp, k, x(k)), org[k]);
    const double s = __dmul_rn(d, k == 0 ? kp.inv_csx : kp.inv_cs);
    double f = floor(s);
    if (((kp.periodic >> k) & 1) && f == (double)nc[k]) f -= 1.0;
    if (!(f >= 0.0) || !(f < (double)nc[k])) return kp.ncell_total;
    c[k] = (int)f;
  }
  return (uint32_t)(c[0] + nc[0] * (c[1] + nc[1] * c[2]));
}
__device__ inline uint32_t cell_key_local(const KParams& kp, const double* __restrict__ pos,
                                          const uint8_t* __restrict__ type, int64_t n,
                                          int64_t i) {
  if (is_excluded(type[i])) return kp.ncell_total;
  return cell_key_at(kp, kp.dim, [&](int k) { return pos[k * n + i]; });
}

// Counts the calling lane's particle in its cell k (lanes that take part, in
// any combination) and returns a rank of its own there.  Neighbouring lanes
// of one cell make one atomic: an input that a step before left sorted has
// its cells' members in runs.
__device__ inline uint32_t count_in_cell(bool take, uint32_t k, uint32_t* __restrict__ count) {
  const int lane = threadIdx.x & 63;
  const uint32_t prev = (uint32_t)__shfl_up((int)k, 1, 64);
  const uint64_t taking = __ballot(take);
  const bool before = lane > 0 && ((taking >> (lane - 1)) & 1ull);
  const bool head = take && !(before && prev == k);
  const uint64_t heads = __ballot(head);
  // the run's first lane, and one past its last: the next head or idle lane
  const uint64_t upto = (2ull << lane) - 1ull;  // (lanes 0..lane)
  const int first = 63 - (int)__builtin_clzll((heads & upto) | 1ull);
  const uint64_t stop = (heads | ~taking) & ~((2ull << first) - 1ull);
  const int end = stop ? (int)__builtin_ctzll(stop) : 64;
  uint32_t base = 0;
  if (head) base = atomicAdd(&count[k], (uint32_t)(end - lane));
  base = (uint32_t)__shfl((int)base, first, 64);
  return base + (uint32_t)(lane - first);
}

// The sorted index of particle src among the members of its cell k: the
// cell's first index plus the members with a lower input index (ties of the
// stable sort keep input order).
__device__ inline int64_t stable_slot(const uint2* __restrict__ member,
                                      const uint32_t* __restrict__ cell_start, uint32_t k,
                                      uint32_t src) {
  const uint32_t c0 = cell_start[k], c1 = cell_start[k + 1];
  uint32_t below = 0, m = c0;
  for (; m + 4u <= c1; m += 4u) {  // (coarse cells: loads in flight together)
    const uint32_t a = member[m].x, b = member[m + 1u].x, c = member[m + 2u].x,
                   d = member[m + 3u].x;
    below += (a < src ? 1u : 0u) + (b < src ? 1u : 0u) + (c < src ? 1u : 0u) + (d < src ? 1u : 0u);
  }
  for (; m < c1; ++m) below += member[m].x < src ? 1u : 0u;
  return (int64_t)c0 + below;
}

// (rho/rho0)^gamma - 1 of the Tait equation (Eq. 28: P = B_t times this), in
// FP64; for gamma = 7 as the expansion of (1+u)^7 - 1 in u = rho/rho0 - 1,
// which keeps the small pressures of a nearly incompressible fluid free of
// cancellation.
__device__ inline double tait_ratio(const KParams& kp, double r) {
  const double u = r / kp.rho0 - 1.0;
  if (kp.gamma == 7.0)
    return u * (7.0 + u * (21.0 + u * (35.0 + u * (35.0 + u * (21.0 + u * (7.0 + u))))));
  return pow(r / kp.rho0, kp.gamma) - 1.0;
}

__device__ inline void write_view(const KParams& kp, int64_t i, const double* x, const float* v,
                                  float rho, uint8_t t, uint32_t lkey, float4* __restrict__ pr,
                                  float4* __restrict__ vp);

// Gathers particle src into sorted slot i and writes the two float4 the
// interaction reads (the "view"):
//   pr = {local position (dim components), 0, +rho fluid / -rho wall}
//   vp = {velocity (dim components), 0, P}
// lkey is the particle's key relative to its case.  Local positions follow
// the precision scheme of Section 5.1 (FP64 positions, short FP32 distances,
// so the error does not grow with the domain): along y and z the FP32 offset
// x - (origin + c cs) from the particle's cell, evaluated in FP64; along x a
// 32-bit fixed-point position modulo kFrameCells cells (the bits are stored
// in the float slot), whose differences are exact modulo that period.  P is the
// Tait pressure of Eq. 28, per particle in FP64 (tait_ratio).  Returns true if
// the particle was excluded by this call (it left the grid).
__device__ inline bool reorder_one(const KParams& kp, int64_t n, int64_t i, int64_t src,
                                   uint32_t lkey, const sph_state& in, const sph_state& out,
                                   const sph_state& cin, const sph_state& cout, int carry,
                                   float4* __restrict__ pr, float4* __restrict__ vp) {
  // (all loads first: the compiler cannot move them across the stores)
  double x[3] = {0.0, 0.0, 0.0};
  float v[3] = {0.f, 0.f, 0.f};
  for (int d = 0; d < kp.dim; ++d) {
    x[d] = in.pos[d * n + src];
    v[d] = in.vel[d * n + src];
  }
  const float rho = in.rho[src];
  uint8_t t = in.type[src];
  const bool ids = in.id && out.id;
  const uint32_t id = ids ? in.id[src] : 0u;
  const bool live = !(t & SPH_EXCLUDED);
  for (int d = 0; d < kp.dim; ++d) {
    if (live) x[d] = wrap_coord(kp, d, x[d]);
    out.pos[d * n + i] = x[d];
    out.vel[d * n + i] = v[d];
  }
  out.rho[i] = rho;
  bool newly = false;
  if (lkey == kp.ncell_total && !(t & SPH_EXCLUDED)) {
    t |= SPH_EXCLUDED;
    newly = true;
  }
  out.type[i] = t;
  if (ids) out.id[i] = id;
  if (in.normal && out.normal)
    for (int d = 0; d < kp.dim; ++d) out.normal[d * n + i] = in.normal[d * n + src];
  if (in.vel64 && out.vel64) {  // an all-FP64 state's velocities and densities
    for (int d = 0; d < kp.dim; ++d) out.vel64[d * n + i] = in.vel64[d * n + src];
    out.rho64[i] = in.rho64[src];
  }
  if (carry) {
    for (int d = 0; d < kp.dim; ++d) {
      cout.pos[d * n + i] = cin.pos[d * n + src];
      cout.vel[d * n + i] = cin.vel[d * n + src];
    }
    cout.rho[i] = cin.rho[src];
    if (cin.vel64 && cout.vel64) {
      for (int d = 0; d < kp.dim; ++d) cout.vel64[d * n + i] = cin.vel64[d * n + src];
      cout.rho64[i] = cin.rho64[src];
    }
  }
  if (t & SPH_EXCLUDED) {
    pr[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    vp[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    return newly;
  }
  write_view(kp, i, x, v, rho, t, lkey, pr, vp);
  return newly;
}

// The view entry of sorted slot i (a live particle) from its position x
// (FP64), velocity v, density rho and type t, relative to the cell of key
// lkey (see reorder_one).  The position may lie slightly outside that cell
// (a view refreshed after the particle moved): the offsets then fall
// outside [0, cs), which the interaction handles like any other.
__device__ inline void write_view(const KParams& kp, int64_t i, const double* x, const float* v,
                                  float rho, uint8_t t, uint32_t lkey, float4* __restrict__ pr,
                                  float4* __restrict__ vp) {
  const int c0 = (int)(lkey % (uint32_t)kp.ncx);
  const uint32_t rest = lkey / (uint32_t)kp.ncx;
  const int c[3] = {c0, (int)(rest % (uint32_t)kp.ncy), (int)(rest / (uint32_t)kp.ncy)};
  const double org[3] = {kp.ox, kp.oy, kp.oz};
  float o[3] = {0.f, 0.f, 0.f};
  for (int d = 1; d < kp.dim; ++d) o[d] = (float)(x[d] - (org[d] + (double)c[d] * kp.cs));
  // x: fixed-point position modulo kFrameCells cells, 2^32 units per period
  const double fr = (x[0] - org[0]) * kp.inv_frame;
  const double f = fr - floor(fr);
  o[0] = __uint_as_float((uint32_t)(uint64_t)(f * 4294967296.0));
  const double pw = tait_ratio(kp, (double)rho);
  pr[i] = make_float4(o[0], o[1], o[2], is_fluid(t) ? rho : -rho);
  vp[i] = make_float4(v[0], v[1], v[2], (float)(kp.b_tait * pw));
}

// Imposed wall motion along x: D(t) = (A/w^2)(1 - cos wt), v(t) = (A/w) sin wt.
__device__ inline double motion_disp(const KParams& kp, double t) {
  if (kp.motion_omega == 0.0) return 0.0;
  const double w = kp.motion_omega;
  return kp.motion_amp / (w * w) * (1.0 - cos(w * t));
}
__device__ inline double motion_vel(const KParams& kp, double t) {
  if (kp.motion_omega == 0.0) return 0.0;
  return kp.motion_amp / kp.motion_omega * sin(kp.motion_omega * t);
}

// One particle of the symplectic update: PHASE 0 is the predictor (Eq. 33
// lines 1-2, Eq. 34 line 1) and saves state n; PHASE 1 the corrector (Eq. 33
// lines 3-4, Eq. 34 line 2) from the saved state.  dmove / vmove are the
// imposed wall displacement since t and velocity at the phase's end time.
// Returns true if the new state is not finite or the density not positive.
// disp2 (PHASE 0) receives the squared distance the particle moved.
template <int PHASE>
__device__ inline bool symplectic_one(const KParams& kp, int64_t n, int64_t i, double dt,
                                      double dmove, double vmove, const sph_state& saved,
                                      const sph_state& s, const float* __restrict__ ace,
                                      const float* __restrict__ arho, double& disp2) {
  const uint8_t t = s.type[i];
  if (PHASE == 0) {
    for (int d = 0; d < kp.dim; ++d) {
      saved.pos[d * n + i] = s.pos[d * n + i];
      saved.vel[d * n + i] = s.vel[d * n + i];
    }
    saved.rho[i] = s.rho[i];
  }
  if (is_excluded(t)) return false;
  bool bad = false;
  if (is_fluid(t)) {
    for (int d = 0; d < kp.dim; ++d) {
      const double a = (double)ace[d * n + i];
      if (PHASE == 0) {
        const double v = (double)s.vel[d * n + i];
        const double x0 = s.pos[d * n + i], x1 = x0 + 0.5 * dt * v;
        s.pos[d * n + i] = x1;
        disp2 += (x1 - x0) * (x1 - x0);
        const float v1 = (float)(v + 0.5 * dt * a);
        s.vel[d * n + i] = v1;
        bad |= !isfinite(v1);
      } else {
        const double vn = (double)saved.vel[d * n + i];
        const double v1 = vn + dt * a;
        s.pos[d * n + i] = saved.pos[d * n + i] + dt * 0.5 * (v1 + vn);
        const float v1f = (float)v1;
        s.vel[d * n + i] = v1f;
        bad |= !isfinite(v1f);
      }
    }
  } else if ((t & 0x7f) == SPH_BOUND_MOVING) {
    s.pos[i] = saved.pos[i] + dmove;
    s.vel[i] = (float)vmove;
    if (PHASE == 0) disp2 += dmove * dmove;
  }
  double r;
  if (PHASE == 0) {
    r = (double)s.rho[i] + 0.5 * dt * (double)arho[i];
  } else {
    const double eps = -((double)arho[i] / (double)s.rho[i]) * dt;
    r = (double)saved.rho[i] * (2.0 - eps) / (2.0 + eps);
  }
  const float rf = (float)r;
  s.rho[i] = rf;
  return bad || !(rf > 0.f) || !isfinite(rf);
}

// The predictor (symplectic_one<0>) and the view refresh of its result in one
// pass: the particle's new position, velocity and density go to the state and,
// from registers, to its view entry, relative to the cell of its key from the
// last binning.  All loads come before the first store: the state's arrays may
// alias as far as the compiler knows, so it moves none across.  A particle that
// leaves the grid along an open component is excluded, as a binning would; its
// view entry gets NaN offsets and zero density, so it meets no target in the
// cell range it still sits in (newly is set).
template <int DIM>
__device__ inline bool predict_view_one(const KParams& kp, int64_t n, int64_t i, double dt,
                                        double dmove, double vmove, const sph_state& saved,
                                        const sph_state& s, const float* __restrict__ ace,
                                        const float* __restrict__ arho,
                                        const uint32_t* __restrict__ key,
                                        float4* __restrict__ pr, float4* __restrict__ vp,
                                        double& disp2, bool& newly) {
  double x[3] = {0.0, 0.0, 0.0};
  float v[3] = {0.f, 0.f, 0.f}, a[3] = {0.f, 0.f, 0.f};
  const uint8_t t = s.type[i];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    x[d] = s.pos[d * n + i];
    v[d] = s.vel[d * n + i];
    a[d] = ace[d * n + i];
  }
  const float rho = s.rho[i], ar = arho[i];
  const uint32_t lkey = key[i];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    saved.pos[d * n + i] = x[d];
    saved.vel[d * n + i] = v[d];
  }
  saved.rho[i] = rho;
  if (is_excluded(t)) return false;  // (its view entry was written by the binning)
  bool bad = false;
  if (is_fluid(t)) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const double v0 = (double)v[d];
      const double x0 = x[d], x1 = x0 + 0.5 * dt * v0;
      s.pos[d * n + i] = x[d] = x1;
      disp2 += (x1 - x0) * (x1 - x0);
      s.vel[d * n + i] = v[d] = (float)(v0 + 0.5 * dt * (double)a[d]);
      bad |= !isfinite(v[d]);
    }
  } else if ((t & 0x7f) == SPH_BOUND_MOVING) {
    s.pos[i] = x[0] = x[0] + dmove;
    s.vel[i] = v[0] = (float)vmove;
    disp2 += dmove * dmove;
  }
  const float rf = (float)((double)rho + 0.5 * dt * (double)ar);
  s.rho[i] = rf;
  if (cell_key_at(kp, DIM, [&](int k) { return x[k]; }) == kp.ncell_total) {
    s.type[i] = t | SPH_EXCLUDED;
    newly = true;
    const float nan = __builtin_nanf("");
    pr[i] = make_float4(0.f, nan, nan, 0.f);
    vp[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  } else {
    write_view(kp, i, x, v, rf, t, lkey, pr, vp);
  }
  return bad || !(rf > 0.f) || !isfinite(rf);
}

// As symplectic_one for an all-FP64 state (vel64 and rho64 set in s and
// saved): the same update in FP64 from FP64 rates, with the FP32 copies of
// velocity and density rewritten as their roundings.
template <int PHASE>
__device__ inline bool symplectic_one_f64(const KParams& kp, int64_t n, int64_t i, double dt,
                                          double dmove, double vmove, const sph_state& saved,
                                          const sph_state& s, const double* __restrict__ ace,
                                          const double* __restrict__ arho, double& disp2) {
  const uint8_t t = s.type[i];
  if (PHASE == 0) {
    for (int d = 0; d < kp.dim; ++d) {
      saved.pos[d * n + i] = s.pos[d * n + i];
      saved.vel[d * n + i] = s.vel[d * n + i];
      saved.vel64[d * n + i] = s.vel64[d * n + i];
    }
    saved.rho[i] = s.rho[i];
    saved.rho64[i] = s.rho64[i];
  }
  if (is_excluded(t)) return false;
  bool bad = false;
  if (is_fluid(t)) {
    for (int d = 0; d < kp.dim; ++d) {
      const double a = ace[d * n + i];
      double v1;
      if (PHASE == 0) {
        const double v = s.vel64[d * n + i];
        const double x0 = s.pos[d * n + i], x1 = x0 + 0.5 * dt * v;
        s.pos[d * n + i] = x1;
        disp2 += (x1 - x0) * (x1 - x0);
        v1 = v + 0.5 * dt * a;
      } else {
        const double vn = saved.vel64[d * n + i];
        v1 = vn + dt * a;
        s.pos[d * n + i] = saved.pos[d * n + i] + dt * 0.5 * (v1 + vn);
      }
      s.vel64[d * n + i] = v1;
      s.vel[d * n + i] = (float)v1;
      bad |= !isfinite(v1);
    }
  } else if ((t & 0x7f) == SPH_BOUND_MOVING) {
    s.pos[i] = saved.pos[i] + dmove;
    s.vel64[i] = vmove;
    s.vel[i] = (float)vmove;
    if (PHASE == 0) disp2 += dmove * dmove;
  }
  double r;
  if (PHASE == 0) {
    r = s.rho64[i] + 0.5 * dt * arho[i];
  } else {
    const double eps = -(arho[i] / s.rho64[i]) * dt;
    r = saved.rho64[i] * (2.0 - eps) / (2.0 + eps);
  }
  s.rho64[i] = r;
  s.rho[i] = (float)r;
  return bad || !(r > 0.0) || !isfinite(r);
}

// One particle of the Verlet update (Section 2.5.1): MODE 0 is Eq. 30
// (v^{n+1} = v^{n-1} + 2 dt F, rho^{n+1} = rho^{n-1} + 2 dt R), MODE 1 is
// Eq. 31 (v^{n+1} = v^n + dt F, rho^{n+1} = rho^n + dt R, the intermediate
// step); both move fluid particles by r += dt v^n + dt^2/2 F.  `prev` holds
// the velocity and density of step n-1 and receives those of step n.  Moving
// walls take their imposed position and velocity (dmove since t, vmove at
// t + dt).  Returns true if the new state is not finite or the density not
// positive.
template <int MODE>
__device__ inline bool verlet_one(const KParams& kp, int64_t n, int64_t i, double dt,
                                  double dmove, double vmove, const sph_state& prev,
                                  const sph_state& s, const float* __restrict__ ace,
                                  const float* __restrict__ arho) {
  const uint8_t t = s.type[i];
  if (is_excluded(t)) return false;
  bool bad = false;
  const bool fluid = is_fluid(t);
  for (int d = 0; d < kp.dim; ++d) {
    const float vn = s.vel[d * n + i];
    if (fluid) {
      const double a = (double)ace[d * n + i];
      s.pos[d * n + i] = s.pos[d * n + i] + dt * (double)vn + 0.5 * dt * dt * a;
      const double v1 = MODE == 0 ? (double)prev.vel[d * n + i] + 2.0 * dt * a
                                  : (double)vn + dt * a;
      const float v1f = (float)v1;
      s.vel[d * n + i] = v1f;
      bad |= !isfinite(v1f);
    }
    prev.vel[d * n + i] = vn;
  }
  if ((t & 0x7f) == SPH_BOUND_MOVING) {
    s.pos[i] = s.pos[i] + dmove;
    s.vel[i] = (float)vmove;
  }
  const float rn = s.rho[i];
  const double r = MODE == 0 ? (double)prev.rho[i] + 2.0 * dt * (double)arho[i]
                             : (double)rn + dt * (double)arho[i];
  prev.rho[i] = rn;
  const float rf = (float)r;
  s.rho[i] = rf;
  return bad || !(rf > 0.f) || !isfinite(rf);
}

}  // namespace sph
