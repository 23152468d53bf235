// Modified dynamic boundary condition (Section 2.6.2 of the DualSPHysics
// v5.0 paper, Eq. 38-39): wall densities and velocities from ghost nodes.
//
// A first kernel lists the wall particles; then kMdbcLanes lanes per listed
// wall.  Its ghost node G = r_B + normal_B is binned like a particle; the rows
// of G's neighbour cells are dealt to the wall's lanes and walked as in the
// interaction (one range per row, cut to the support sphere of G), candidates
// are screened in FP32 on the view's offsets with a margin, and the pairs
// that pass are tested and summed in FP64 on the FP64 positions.  The lanes'
// sums are added by shuffles, and the (d+1) x (d+1) corrected system is
// solved by Gaussian elimination with partial pivoting in registers.  Only
// wall entries of the state density and of the interaction view are written;
// the fluid entries that the walk reads are never changed, and the sign of a
// wall's view density (the only thing read of a wall candidate) stays
// negative.
#include "sph_dev.h"
#include "sph_kernels.h"

namespace sph {

// Lanes per wall.  Walls are a part of the particles (145k of 442k in a 3-D
// dam break: 2270 wavefronts with one lane each, two per SIMD), so their
// pass is bound by the latency of its loads and not by FP64 arithmetic
// (vector units 0.3 busy).  At that size k_mdbc takes 292, 203, 194 and
// 204 us with 1, 2, 4 and 8 lanes, and 184 us with 4 and registers held to
// 128 for a fourth wavefront per SIMD (280 us with one lane and full-range
// FP64 division and square root).
constexpr int kMdbcLanes = 4;

// 1/a (a > 0, infinity included; no denormals) and sqrt(a) (a >= 0, finite;
// below 1e-290 taken as 0) to about one ulp by Newton steps from the
// hardware's approximations: without the scaling and the special cases of the
// full versions, which take most of their instructions.
__device__ inline double rcp64(double a) {
  const double y = __builtin_amdgcn_rcp(a);
  const double x = fma(y, fma(-a, y, 1.0), y);
  return y > 0.0 ? fma(x, fma(-a, x, 1.0), x) : 0.0;
}
__device__ inline double sqrt64(double a) {
  if (!(a > 1e-290)) return 0.0;
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, a), h, g);
  return fma(fma(-g, g, a), h, g);
}

// Kernel value and gradient factor (grad W = F r) in FP64: Wendland C2
// (Eq. 11), W = alpha_D (1 - q/2)^4 (2q + 1), F = kfab (1 - q/2)^3, or cubic
// spline (Eq. 10), with alpha_D and kfab of the case.
__device__ inline void kernel_wf64(const KParams& kp, double r, double& w, double& f) {
  const double q = r * kp.inv_h;
  if (kp.kernel == 0) {
    const double u = 1.0 - 0.5 * q;
    const double u3 = u * u * u;
    w = kp.w_alpha * u3 * u * (2.0 * q + 1.0);
    f = kp.f_coef * u3;
  } else if (q <= 1.0) {
    w = kp.w_alpha * (1.0 - 1.5 * q * q + 0.75 * q * q * q);
    f = kp.f_coef * (-3.0 + 2.25 * q);
  } else {
    const double u = 2.0 - q;
    w = kp.w_alpha * 0.25 * u * u * u;
    f = -0.75 * kp.f_coef * u * u / q;
  }
}

// Solves the M x M system A x = b in place (x returned in b) by Gaussian
// elimination with partial pivoting; the row exchanges are compare-and-swap
// steps with fixed indices, so the arrays stay in registers.  Returns the
// determinant (0 if a pivot vanished).
template <int M>
__device__ inline double solve_small(double (&A)[M][M], double (&b)[M]) {
  double det = 1.0;
#pragma unroll
  for (int c = 0; c < M; ++c) {
#pragma unroll
    for (int r = c + 1; r < M; ++r) {
      if (fabs(A[r][c]) > fabs(A[c][c])) {
#pragma unroll
        for (int k = 0; k < M; ++k) {
          const double t = A[c][k];
          A[c][k] = A[r][k];
          A[r][k] = t;
        }
        const double t = b[c];
        b[c] = b[r];
        b[r] = t;
        det = -det;
      }
    }
    if (A[c][c] == 0.0) return 0.0;
    det *= A[c][c];
    const double inv = 1.0 / A[c][c];
#pragma unroll
    for (int r = c + 1; r < M; ++r) {
      const double f = A[r][c] * inv;
#pragma unroll
      for (int k = c; k < M; ++k) A[r][k] -= f * A[c][k];
      b[r] -= f * b[c];
    }
  }
#pragma unroll
  for (int c = M - 1; c >= 0; --c) {
    double s = b[c];
#pragma unroll
    for (int k = c + 1; k < M; ++k) s -= A[c][k] * b[k];
    b[c] = s / A[c][c];
  }
  return det;
}

__global__ void k_zero_wall_count(WsHeader* __restrict__ hdr) {
  if (threadIdx.x == 0) hdr->nwall = 0u;
}

// The wall particles (not excluded) of the sorted state, appended to a work
// list in any order; each wall's result depends only on its own inputs, so the
// order does not matter.  A block takes kListRounds rounds of its threads and
// makes one atomic for all of them (6.9 us for 441k particles): with one per
// wavefront the atomics on the one counter, about 5 ns each, took 41 us.
constexpr int kListRounds = 8;
__global__ __launch_bounds__(kBlock) void k_wall_list(int64_t n, const uint8_t* __restrict__ type,
                                                      uint32_t* __restrict__ list,
                                                      WsHeader* __restrict__ hdr) {
  constexpr int kWaves = kBlock / 64;
  __shared__ uint32_t first[kListRounds * kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * (kBlock * kListRounds) + threadIdx.x;
  uint64_t mask[kListRounds];
#pragma unroll
  for (int r = 0; r < kListRounds; ++r) {
    const int64_t i = i0 + r * kBlock;
    mask[r] = __ballot(i < n && !is_excluded(type[i]) && !is_fluid(type[i]));
    if (lane == 0) first[r * kWaves + wave] = (uint32_t)__popcll(mask[r]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (int k = 0; k < kListRounds * kWaves; ++k) {
      const uint32_t c = first[k];
      first[k] = total;
      total += c;
    }
    const uint32_t base = total ? atomicAdd(&hdr->nwall, total) : 0u;
    for (int k = 0; k < kListRounds * kWaves; ++k) first[k] += base;
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kListRounds; ++r)
    if ((mask[r] >> lane) & 1ull)
      list[first[r * kWaves + wave] + (uint32_t)__popcll(mask[r] & below)] =
          (uint32_t)(i0 + r * kBlock);
}

// The sum of v over the kMdbcLanes adjacent lanes of a wall, in every lane.
__device__ inline double lanes_sum(double v) {
  for (int off = 1; off < kMdbcLanes; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <int DIM, int R>
__global__ __launch_bounds__(kBlock, 4) void k_mdbc(KParams kp, int64_t n, sph_state s,
                                                 const uint32_t* __restrict__ cstart,
                                                 float4* __restrict__ pr,
                                                 float4* __restrict__ vp,
                                                 const uint32_t* __restrict__ list,
                                                 const WsHeader* __restrict__ hdr, int64_t w0) {
  constexpr int M = DIM + 1;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int sub = (int)(t % kMdbcLanes);
  const int64_t wall = w0 + t / kMdbcLanes;
  if (wall >= (int64_t)hdr->nwall) return;  // (all lanes of a wall together)
  const int64_t i = list[wall];
  double g[3] = {0.0, 0.0, 0.0}, rb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    rb[d] = s.pos[d * n + i];
    g[d] = rb[d] + (double)s.normal[d * n + i];
  }
  // key cell of the ghost node; a ghost node outside the grid has no fluid
  // around it (the wall is treated as dry)
  const double org[3] = {kp.ox, kp.oy, kp.oz};
  const int nc[3] = {kp.ncx, kp.ncy, kp.ncz};
  int c[3] = {0, 0, 0};
  bool inside = true;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const double f = floor((g[d] - org[d]) * (d == 0 ? kp.inv_csx : kp.inv_cs));
    inside = inside && f >= 0.0 && f < (double)nc[d];
    c[d] = inside ? (int)f : 0;
  }
  // sums of the corrected system: sw = sum V w, swr = sum V w r,
  // sfr = sum V F r, sfrr = sum V F r r^T (symmetric, upper part), b0 =
  // sum m w, bf = sum m F r (m is applied after the sums); and the Shepard
  // velocity sum
  double sw = 0.0, swr[3] = {0.0, 0.0, 0.0}, sfr[3] = {0.0, 0.0, 0.0};
  double sfrr[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const double mb = kp.mass_f;
  double b0 = 0.0, bf[3] = {0.0, 0.0, 0.0}, sv[3] = {0.0, 0.0, 0.0};
  // the ghost node in the view's frame: fixed-point x (as the reorder writes
  // it), y and z relative to the ghost's cell
  const double fr = (g[0] - kp.ox) * kp.inv_frame;
  const uint32_t xg = (uint32_t)(uint64_t)((fr - floor(fr)) * 4294967296.0);
  const float yg = DIM >= 2 ? (float)(g[1] - (kp.oy + (double)c[1] * kp.cs)) : 0.f;
  const float zg = DIM == 3 ? (float)(g[2] - (kp.oz + (double)c[2] * kp.cs)) : 0.f;
  const int fcells = kFrameCells << kp.lg_xsub;
  const float fx =
      (float)(int32_t)(xg - ((uint32_t)(c[0] % fcells) << (29 - kp.lg_xsub))) * kp.unit_x_f;
  const float cs = kp.cs_f;
  // FP32 pre-test with a margin far above its rounding; the FP64 test on the
  // FP64 positions decides
  const float pre2 = kp.support2_f * 1.0002f;
  const int reach = R * kp.x_sub;
  const int xlo = c[0] - reach < 0 ? 0 : c[0] - reach;
  const int xhi = c[0] + reach >= kp.ncx ? kp.ncx - 1 : c[0] + reach;
  constexpr int kRowsY = 2 * R + 1;
  constexpr int kRows = kRowsY * (DIM == 3 ? 2 * R + 1 : 1);
  for (int q = sub; q < (inside ? kRows : 0); q += kMdbcLanes) {
    const int dz = (DIM == 3 ? -R : 0) + q / kRowsY, dy = q % kRowsY - R;
    const int z = c[2] + dz;
    if (z < 0 || z >= kp.ncz) continue;
    const float ez0 = (float)dz * cs - zg;
    const float ez = DIM == 3 ? (dz > 0 ? ez0 : (dz < 0 ? -(ez0 + cs) : 0.f)) : 0.f;
    {
      const int y = c[1] + dy;
      if (y < 0 || y >= kp.ncy) continue;
      const float ey0 = (float)dy * cs - yg;
      const float ey = dy > 0 ? ey0 : (dy < 0 ? -(ey0 + cs) : 0.f);
      const float w2 = pre2 - ey * ey - ez * ez;
      if (!(w2 > 0.f)) continue;
      const float wx = sqrtf(w2);
      int x0 = c[0] + (int)floorf((fx - wx) * kp.inv_csx_f);
      int x1 = c[0] + (int)floorf((fx + wx) * kp.inv_csx_f);
      x0 = x0 < xlo ? xlo : x0;
      x1 = x1 > xhi ? xhi : x1;
      const uint32_t row = (uint32_t)kp.ncx * ((uint32_t)y + (uint32_t)kp.ncy * (uint32_t)z);
      const uint32_t j1 = cstart[row + x1 + 1];
      const float ys = yg - (float)dy * cs, zs = zg - (float)dz * cs;
      // groups of 4 candidates: their views are loaded together (padded), the
      // screened ones then load their FP64 positions and velocities together
      for (uint32_t j = cstart[row + x0]; j < j1; j += 4) {
        const float4* q = pr + j;
        float4 pb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pb[u] = q[u];
        bool hit[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float ex = (float)(int32_t)(xg - __float_as_uint(pb[u].x)) * kp.unit_x_f;
          const float ey1 = ys - pb[u].y, ez1 = DIM == 3 ? zs - pb[u].z : 0.f;
          hit[u] = j + u < j1 && pb[u].w > 0.f && ex * ex + ey1 * ey1 + ez1 * ez1 < pre2;
        }
        double pbx[4][3];
        float4 vb4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (hit[u]) {
#pragma unroll
            for (int d = 0; d < DIM; ++d) pbx[u][d] = s.pos[d * n + j + u];
            vb4[u] = vp[j + u];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (!hit[u]) continue;
          double r[3] = {0.0, 0.0, 0.0}, r2 = 0.0;
#pragma unroll
          for (int d = 0; d < DIM; ++d) {
            r[d] = pbx[u][d] - g[d];
            r2 += r[d] * r[d];
          }
          if (!(r2 < kp.support2)) continue;
          double w, f;
          kernel_wf64(kp, sqrt64(r2), w, f);
          const double vb = mb * rcp64((double)pb[u].w);
          const double vw = vb * w, vf = vb * f;
          sw += vw;
          b0 += w;
#pragma unroll
          for (int a = 0; a < DIM; ++a) {
            swr[a] += vw * r[a];
            sfr[a] += vf * r[a];
            bf[a] += f * r[a];
          }
          sfrr[0] += vf * r[0] * r[0];
          sfrr[1] += vf * r[0] * r[1];
          sfrr[3] += vf * r[1] * r[1];
          if (DIM == 3) {
            sfrr[2] += vf * r[0] * r[2];
            sfrr[4] += vf * r[1] * r[2];
            sfrr[5] += vf * r[2] * r[2];
          }
          sv[0] += vw * (double)vb4[u].x;
          sv[1] += vw * (double)vb4[u].y;
          if (DIM == 3) sv[2] += vw * (double)vb4[u].z;
        }
      }
    }
  }
  sw = lanes_sum(sw);
  b0 = mb * lanes_sum(b0);
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    swr[a] = lanes_sum(swr[a]);
    sfr[a] = lanes_sum(sfr[a]);
    bf[a] = mb * lanes_sum(bf[a]);
    sv[a] = lanes_sum(sv[a]);
  }
#pragma unroll
  for (int a = 0; a < 6; ++a)
    if (DIM == 3 || a == 0 || a == 1 || a == 3) sfrr[a] = lanes_sum(sfrr[a]);
  if (sub != 0) return;
  double rho_b = kp.rho0;
  double vout[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int d = 0; d < DIM; ++d) vout[d] = (double)s.vel[d * n + i];
  if (sw > 0.0) {
    double A[M][M], x[M];
    A[0][0] = sw;
    x[0] = b0;
    const int sym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      A[0][1 + a] = swr[a];
      A[1 + a][0] = sfr[a];
      x[1 + a] = bf[a];
#pragma unroll
      for (int k = 0; k < DIM; ++k) A[1 + a][1 + k] = sfrr[sym[a][k]];
    }
    const double det = solve_small<M>(A, x);
    if (fabs(det) >= 1e-3) {
      rho_b = x[0];
#pragma unroll
      for (int d = 0; d < DIM; ++d) rho_b += (rb[d] - g[d]) * x[1 + d];
    } else {
      rho_b = b0 / sw;
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) vout[d] = 2.0 * vout[d] - sv[d] / sw;
  }
  const float rf = (float)rho_b;
  s.rho[i] = rf;
  pr[i].w = -rf;
  const double pw = tait_ratio(kp, (double)rf);
  vp[i] = make_float4((float)vout[0], (float)vout[1], DIM == 3 ? (float)vout[2] : 0.f,
                      (float)(kp.b_tait * pw));
}

hipError_t launch_mdbc(const KParams& kp, int64_t n, const sph_state& s, const uint32_t* key,
                       const uint32_t* cell_start, void* ws, hipStream_t st) {
  (void)key;
  const WsLayout L = ws_layout(n);
  float4* pr = ws_ptr<float4>(ws, L.view_pr);
  float4* vp = ws_ptr<float4>(ws, L.view_vp);
  WsHeader* hdr = ws_ptr<WsHeader>(ws, L.err);
  // the work list lives in the sort's key buffer, free once the cells are
  // binned (sph_bin_cells must not run between this and the next launch)
  uint32_t* list = ws_ptr<uint32_t>(ws, L.keyA);
  const int64_t chunk = kBlock * kListRounds;
  hipLaunchKernelGGL(k_zero_wall_count, dim3(1), dim3(64), 0, st, hdr);
  hipLaunchKernelGGL(k_wall_list, dim3((unsigned)((n + chunk - 1) / chunk)), dim3(kBlock), 0, st,
                     n, s.type, list, hdr);
  // room for every particle being a wall (blocks past the list leave at once),
  // kLaunchWalls walls a launch: a launch has fewer than 2^32 threads
  constexpr int64_t kLaunchWalls = (int64_t)1 << 29;
  static_assert(kLaunchWalls * kMdbcLanes < ((int64_t)1 << 32), "threads of a launch");
#define SPH_MDBC(D, RR)                                                                    \
  hipLaunchKernelGGL((k_mdbc<D, RR>), dim3(grid), dim3(kBlock), 0, st, kp, n, s, cell_start, \
                     pr, vp, list, hdr, w0)
  for (int64_t w0 = 0; w0 < n; w0 += kLaunchWalls) {
    const int64_t walls = n - w0 < kLaunchWalls ? n - w0 : kLaunchWalls;
    const unsigned grid = (unsigned)((walls * kMdbcLanes + kBlock - 1) / kBlock);
    if (kp.dim == 2) {
      if (kp.cell_div == 1) SPH_MDBC(2, 1); else SPH_MDBC(2, 2);
    } else {
      if (kp.cell_div == 1) SPH_MDBC(3, 1); else SPH_MDBC(3, 2);
    }
  }
#undef SPH_MDBC
  return hipGetLastError();
}

}  // namespace sph
