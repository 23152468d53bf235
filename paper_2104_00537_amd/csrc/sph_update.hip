// System update (Section 5.1): the variable time step of Eq. 35, the
// symplectic position-Verlet update of Eq. 33-34 and the Verlet update of
// Eq. 30-31, with the imposed motion of moving walls (Eq. 37).
#include "sph_dev.h"
#include "sph_kernels.h"

namespace sph {

// The per-block partials of the last interaction pass summed over a block of
// THREADS threads; the result is complete in thread 0.  (Maxima and whole
// numbers: the same in any order.)
struct RedSums {
  float fmax, vmax;
  unsigned long long count, count_wall, nfluid;
};
template <int THREADS>
__device__ inline RedSums reduce_partials(const BlockRed* __restrict__ red, int64_t nblk) {
  __shared__ RedSums part[THREADS / 64];
  RedSums r{0.f, 0.f, 0ull, 0ull, 0ull};
  for (int64_t b = threadIdx.x; b < nblk; b += 4 * THREADS) {
    BlockRed q[4];  // (loads in flight together)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      q[u] = b + u * THREADS < nblk ? red[b + u * THREADS] : BlockRed{0.f, 0.f, 0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      r.fmax = fmaxf(r.fmax, q[u].fmax);
      r.vmax = fmaxf(r.vmax, q[u].vmax);
      r.count += q[u].count;
      r.count_wall += q[u].count_wall;
      r.nfluid += q[u].nfluid;
    }
  }
  r.fmax = wave_max(r.fmax);
  r.vmax = wave_max(r.vmax);
  for (int off = 32; off > 0; off >>= 1) {
    r.count += __shfl_xor(r.count, off, 64);
    r.count_wall += __shfl_xor(r.count_wall, off, 64);
    r.nfluid += __shfl_xor(r.nfluid, off, 64);
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < THREADS / 64; ++w) {
      r.fmax = fmaxf(r.fmax, part[w].fmax);
      r.vmax = fmaxf(r.vmax, part[w].vmax);
      r.count += part[w].count;
      r.count_wall += part[w].count_wall;
      r.nfluid += part[w].nfluid;
    }
  }
  return r;
}

// Eq. 35 from the sums.
__device__ inline double time_step(const KParams& kp, const RedSums& r) {
  if (r.nfluid == 0) return INFINITY;
  const double f = (double)r.fmax, v = (double)r.vmax;
  const double dtf = f > 0.0 ? sqrt(kp.h / f) : INFINITY;
  const double dtcv = kp.h / (kp.c0 + v);
  return kp.cfl * (dtf < dtcv ? dtf : dtcv);
}

__device__ inline void write_time_step(const KParams& kp, const RedSums& r, double d, double* dt,
                                       uint64_t* inter, float* maxima, uint32_t* err) {
  *dt = d;
  if (!(d >= kp.dt_floor) || !isfinite(d)) set_error(err, SPH_ERR_DT_FLOOR);
  if (inter) {
    inter[0] += (uint64_t)r.count;
    inter[1] += (uint64_t)r.count_wall;
  }
  if (maxima) {
    maxima[0] = r.fmax;
    maxima[1] = r.vmax;
  }
}

constexpr int kRedThreads = 1024;

__global__ __launch_bounds__(kRedThreads) void k_reduce_dt(KParams kp,
                                                           const BlockRed* __restrict__ red,
                                                           WsHeader* __restrict__ hdr,
                                                           double* __restrict__ dt,
                                                           uint64_t* __restrict__ inter,
                                                           float* __restrict__ maxima) {
  const RedSums r = reduce_partials<kRedThreads>(red, hdr->nred);
  if (threadIdx.x == 0) write_time_step(kp, r, time_step(kp, r), dt, inter, maxima, &hdr->err);
}

// The time and the imposed motion of a phase, in shm: dt (given in thread 0),
// the walls' move since t and their velocity at the phase's end.  tadv, when
// given, is the time to advance by dt: without imposed motion no block needs
// t, so block 0 advances it and the update needs no second kernel (4.5 us in
// eager launches, 1.3 us in a graph).
__device__ inline void phase_times(const KParams& kp, double dt, const double* __restrict__ tp,
                                   double* __restrict__ tadv, double share, double (&shm)[3]) {
  if (threadIdx.x == 0) {
    shm[0] = dt;
    shm[1] = shm[2] = 0.0;
    if (kp.motion_omega != 0.0) {
      const double t = *tp, t1 = t + share * dt;
      shm[1] = motion_disp(kp, t1) - motion_disp(kp, t);
      shm[2] = motion_vel(kp, t1);
    } else if (tadv && blockIdx.x == 0) {
      *tadv += dt;
    }
  }
  __syncthreads();
}

// phase 0: predictor, saving state n; phase 1: corrector from the saved state.
// The predictor also records the largest distance a particle moved (for an
// interaction that reuses the cells of the last binning).  F64S: an all-FP64
// state, whose rates ace and arho are FP64 arrays.  RED (the corrector): one
// more block, the first, does the work of k_reduce_dt for the pass that made
// the rates, whose time step (*rdt) the corrector does not use: beside the
// update instead of before it, in a launch less.
struct RedArgs {
  const BlockRed* red;
  WsHeader* hdr;
  double* dt;
  uint64_t* inter;
};
template <int PHASE, bool F64S, bool RED>
__global__ __launch_bounds__(kBlock) void k_symplectic(KParams kp, int64_t n,
                                                       const double* __restrict__ dtp,
                                                       const double* __restrict__ tp,
                                                       double* __restrict__ tadv,
                                                       sph_state saved, sph_state s,
                                                       const void* __restrict__ ace,
                                                       const void* __restrict__ arho,
                                                       uint32_t* __restrict__ err,
                                                       uint32_t* __restrict__ disp, RedArgs ra) {
  if (RED && blockIdx.x == 0) {
    const RedSums r = reduce_partials<kBlock>(ra.red, ra.hdr->nred);
    if (threadIdx.x == 0) {
      write_time_step(kp, r, time_step(kp, r), ra.dt, ra.inter, nullptr, err);
      if (tadv) *tadv += *dtp;
    }
    return;
  }
  __shared__ double shm[3];
  phase_times(kp, threadIdx.x == 0 ? *dtp : 0.0, tp, RED ? nullptr : tadv,
              PHASE == 0 ? 0.5 : 1.0, shm);
  const int64_t i = (int64_t)(blockIdx.x - (RED ? 1 : 0)) * blockDim.x + threadIdx.x;
  double disp2 = 0.0;
  bool bad = false;
  if (i < n) {
    if constexpr (F64S)
      bad = symplectic_one_f64<PHASE>(kp, n, i, shm[0], shm[1], shm[2], saved, s,
                                      static_cast<const double*>(ace),
                                      static_cast<const double*>(arho), disp2);
    else
      bad = symplectic_one<PHASE>(kp, n, i, shm[0], shm[1], shm[2], saved, s,
                                  static_cast<const float*>(ace),
                                  static_cast<const float*>(arho), disp2);
  }
  if (bad) set_error(err, SPH_ERR_NONFINITE);
  if (PHASE == 0) record_displacement(disp2, disp);
}

// The predictor with the view refresh of its result (predict_view_one): one
// pass that reads 61 and writes 112 bytes per 3-D particle in place of two of
// together 218, bound by that traffic for large cases (1.32M particles: 34.4 +
// 20.0 -> 37.4 us; 8.8M: 217 + 154 -> 270 us) and by launches for small ones.
// RED: with the reduction of the pass's partials, done by every block for
// itself (block 0 writes the results).
//
// Up to kFuseReduceMaxN particles the blocks' own reductions cost less than
// the launch they replace (a step of 4k particles in 2-D: 54.1 -> 51.2 us, of
// 168k in 3-D 274.8 -> 272.3 us); at 1.32M particles, 5170 blocks that read
// 5170 partials each, they cost more (1297 -> 1310 us).
constexpr int64_t kFuseReduceMaxN = 262144;
template <int DIM, bool RED>
__global__ __launch_bounds__(kBlock) void k_predict_view(
    KParams kp, int64_t n, double* __restrict__ dtp, const double* __restrict__ tp,
    sph_state saved, sph_state s, const float* __restrict__ ace, const float* __restrict__ arho,
    const uint32_t* __restrict__ key, float4* __restrict__ pr, float4* __restrict__ vp,
    uint32_t* __restrict__ err, uint32_t* __restrict__ disp, RedArgs ra) {
  __shared__ double shm[3];
  double dt = 0.0;
  if (RED) {
    const RedSums r = reduce_partials<kBlock>(ra.red, ra.hdr->nred);
    if (threadIdx.x == 0) {
      dt = time_step(kp, r);
      if (blockIdx.x == 0) write_time_step(kp, r, dt, ra.dt, ra.inter, nullptr, err);
    }
  } else if (threadIdx.x == 0) {
    dt = *dtp;
  }
  phase_times(kp, dt, tp, nullptr, 0.5, shm);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double disp2 = 0.0;
  if (i < n) {
    bool newly = false;
    if (predict_view_one<DIM>(kp, n, i, shm[0], shm[1], shm[2], saved, s, ace, arho, key, pr, vp,
                              disp2, newly))
      set_error(err, SPH_ERR_NONFINITE);
    if (newly) set_error(err, SPH_ERR_EXCLUDED);
  }
  record_displacement(disp2, disp);
}

// Verlet update (Eq. 30 for MODE 0, Eq. 31 for MODE 1) of the sorted state.
template <int MODE>
__global__ void k_verlet(KParams kp, int64_t n, const double* __restrict__ dtp,
                         const double* __restrict__ tp, double* __restrict__ tadv,
                         sph_state prev, sph_state s,
                         const float* __restrict__ ace, const float* __restrict__ arho,
                         uint32_t* __restrict__ err) {
  __shared__ double shm[3];
  phase_times(kp, threadIdx.x == 0 ? *dtp : 0.0, tp, tadv, 1.0, shm);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (verlet_one<MODE>(kp, n, i, shm[0], shm[1], shm[2], prev, s, ace, arho))
    set_error(err, SPH_ERR_NONFINITE);
}

__global__ void k_advance_time(const double* __restrict__ dt, double* __restrict__ t) {
  if (threadIdx.x == 0) *t = *t + *dt;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int64_t len, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < len) p[i] = v;
}

hipError_t launch_reduce_dt(const KParams& kp, int64_t n, double* dt, uint64_t* interactions,
                            float* maxima, void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  hipLaunchKernelGGL(k_reduce_dt, dim3(1), dim3(kRedThreads), 0, st, kp, ws_ptr<BlockRed>(ws, L.red),
                     ws_ptr<WsHeader>(ws, L.err), dt, interactions, maxima);
  return hipGetLastError();
}

hipError_t launch_symplectic(const KParams& kp, int64_t n, int phase, const double* dt, double* t,
                             sph_state& saved, sph_state& s, const float* ace, const float* arho,
                             void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  WsHeader* hdr = ws_ptr<WsHeader>(ws, L.err);
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  double* tadv = phase == 1 && n > 0 && kp.motion_omega == 0.0 ? t : nullptr;
  if (n > 0) {
    uint32_t* disp = ws_ptr<uint32_t>(ws, L.disp);
    const bool f64s = s.vel64 != nullptr;
#define SPH_SYMP(PH, F)                                                                      \
  hipLaunchKernelGGL((k_symplectic<PH, F, false>), dim3(grid), dim3(kBlock), 0, st, kp, n, dt, t, \
                     tadv, saved, s, (const void*)ace, (const void*)arho, &hdr->err, disp, RedArgs{})
    if (phase == 0) {
      if (f64s) SPH_SYMP(0, true); else SPH_SYMP(0, false);
    } else {
      if (f64s) SPH_SYMP(1, true); else SPH_SYMP(1, false);
    }
#undef SPH_SYMP
  }
  if (phase == 1 && !tadv)
    hipLaunchKernelGGL(k_advance_time, dim3(1), dim3(64), 0, st, dt, t);
  return hipGetLastError();
}

hipError_t launch_update(const KParams& kp, int64_t n, int phase, double* dt, double* dt_half,
                         uint64_t* interactions, double* t, sph_state& saved, sph_state& s,
                         const float* ace, const float* arho, const uint32_t* key, void* ws,
                         hipStream_t st) {
  const WsLayout L = ws_layout(n);
  WsHeader* hdr = ws_ptr<WsHeader>(ws, L.err);
  uint32_t* disp = ws_ptr<uint32_t>(ws, L.disp);
  const BlockRed* red = ws_ptr<BlockRed>(ws, L.red);
  // (one buffer for both time steps: the corrector's blocks would read it while
  // its first block writes it)
  if (n == 0 || (phase == 1 && dt_half == dt)) {
    hipError_t e = launch_reduce_dt(kp, n, phase == 0 ? dt : dt_half, interactions, nullptr, ws, st);
    return e != hipSuccess ? e : launch_symplectic(kp, n, phase, dt, t, saved, s, ace, arho, ws, st);
  }
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  if (phase == 1) {
    const bool moving = kp.motion_omega != 0.0;
    hipLaunchKernelGGL((k_symplectic<1, false, true>), dim3(grid + 1), dim3(kBlock), 0, st, kp, n,
                       dt, t, moving ? nullptr : t, saved, s, (const void*)ace, (const void*)arho,
                       &hdr->err, disp, RedArgs{red, hdr, dt_half, interactions});
    if (moving) hipLaunchKernelGGL(k_advance_time, dim3(1), dim3(64), 0, st, dt, t);
    return hipGetLastError();
  }
  const RedArgs ra{red, hdr, dt, interactions};
  const bool fuse = n <= kFuseReduceMaxN;
  if (!fuse) {
    const hipError_t e = launch_reduce_dt(kp, n, dt, interactions, nullptr, ws, st);
    if (e != hipSuccess) return e;
  }
#define SPH_PV(D, F)                                                                         \
  hipLaunchKernelGGL((k_predict_view<D, F>), dim3(grid), dim3(kBlock), 0, st, kp, n, dt, t,  \
                     saved, s, ace, arho, key, ws_ptr<float4>(ws, L.view_pr),                \
                     ws_ptr<float4>(ws, L.view_vp), &hdr->err, disp, ra)
  if (kp.dim == 2) {
    if (fuse) SPH_PV(2, true); else SPH_PV(2, false);
  } else {
    if (fuse) SPH_PV(3, true); else SPH_PV(3, false);
  }
#undef SPH_PV
  return hipGetLastError();
}

hipError_t launch_verlet(const KParams& kp, int64_t n, int mode, const double* dt, double* t,
                          sph_state& prev, sph_state& s, const float* ace, const float* arho,
                          void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  uint32_t* err = ws_ptr<uint32_t>(ws, L.err);
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  double* tadv = n > 0 && kp.motion_omega == 0.0 ? t : nullptr;
  if (n > 0) {
    if (mode == 0)
      hipLaunchKernelGGL(k_verlet<0>, dim3(grid), dim3(kBlock), 0, st, kp, n, dt, t, tadv, prev, s,
                         ace, arho, err);
    else
      hipLaunchKernelGGL(k_verlet<1>, dim3(grid), dim3(kBlock), 0, st, kp, n, dt, t, tadv, prev, s,
                         ace, arho, err);
  }
  if (!tadv) hipLaunchKernelGGL(k_advance_time, dim3(1), dim3(64), 0, st, dt, t);
  return hipGetLastError();
}

hipError_t launch_clear_error(void* ws, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, ws_ptr<uint32_t>(ws, 0), (int64_t)1, 0u);
  return hipGetLastError();
}

}  // namespace sph
