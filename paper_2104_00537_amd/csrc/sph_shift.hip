// Particle shifting (Section 2.8 of the DualSPHysics v5.0 paper: Eq. 40-41
// with the concentration and its gradient of Eq. 53) on gfx950.
//
// Two gathers over the interaction view of the state n+1/2: the
// concentration C of every particle, then, for fluid particles, its
// gradient and the shift, added to the corrected FP64 positions.  One lane
// per particle in sorted order (a few where the case is too small to fill the
// GPU), blocks placed per XCD as in the interaction; sums per lane, no
// atomics.  Bound by the candidates' 16 bytes through the L1 data path (0.86
// busy at 958k particles) and, for small cases, by the latency of the loads.
#include "sph_kernels.h"
#include "sph_pair.h"
#include "sph_slots.h"

namespace sph {

// W / w_alpha of the cubic spline (Eq. 10).
__device__ inline float spline_w_f(float q) {
  if (q <= 1.f) return fmaf(q * q, fmaf(0.75f, q, -1.5f), 1.f);
  const float u = 2.f - q;
  return 0.25f * u * u * u;
}

// c + vb W(r) / w_alpha for the case's kernel: Wendland C2 (Eq. 11), with the
// operations of the interaction's own sum (pair_terms), or cubic spline (Eq. 10).
__device__ inline float add_conc(const KParams& kp, float r2, float vb, float c) {
  const float s = __builtin_amdgcn_sqrtf(r2);
  if (kp.kernel == 0) {
    const float w = fmaf(s, kp.mhalf_inv_h_f, 1.f);
    return conc_wendland(w * w * w * vb, w, c);
  }
  return fmaf(vb, spline_w_f(s * kp.inv_h_f), c);
}

// F_ab / kfab with grad_a W_ab = F_ab r_ab (as in the interaction's pair terms).
__device__ inline float kernel_f_f(const KParams& kp, float r2) {
  const float s = __builtin_amdgcn_sqrtf(r2);
  if (kp.kernel == 0) {
    const float w = fmaf(s, kp.mhalf_inv_h_f, 1.f);
    return w * w * w;
  }
  const float q = s * kp.inv_h_f, u = 2.f - q;
  return q <= 1.f ? fmaf(2.25f, q, -3.f) : -0.75f * u * u * __builtin_amdgcn_rcpf(q);
}

// The sums of a target over its neighbours: C_a / (m_f w_alpha) (GRAD false), or
// grad C_a / (m_f kfab).
template <int DIM, bool GRAD>
struct ShiftAcc {
  float s[GRAD ? DIM : 1];
};

// One group of 4 consecutive candidates from byte offset o of the view (see
// gather_group): positions loaded together and tested, then for the gradient
// the concentrations of the hits, then their terms.  Only the candidates before
// byte offset o1 count (the view is padded by kViewPad entries): whole groups in a
// loop of their own and a masked one behind it made a wavefront take a round more
// per row than its longest lane needs (1.37M particles of a batch, both kernels:
// 803 us, masked throughout 741).
template <int DIM, bool GRAD, typename O>
__device__ __forceinline__ void shift_group(const KParams& kp, uint32_t xa, float ys, float zs,
                                            O o, O o1, const float4* __restrict__ pr,
                                            const float* __restrict__ conc, float ca,
                                            ShiftAcc<DIM, GRAD>& acc) {
  constexpr int NU = 4;
  float4 pb[NU];
  load_group<NU>(pr, o, pb);
  bool hit[NU];
  float dxs[NU], dys[NU], dzs[NU], r2s[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    r2s[u] = pair_geom<DIM>(kp, xa, ys, zs, pb[u], dxs[u], dys[u], dzs[u]);
    hit[u] = r2s[u] < kp.support2_f && o + 16u * u < o1;
    // (the density is loaded with the position: left alone, the compiler loads
    // it by itself once the test has passed)
    asm volatile("" ::"v"(pb[u].w));
  }
  float cb[NU];
  if (GRAD) {
    const O oc = o >> 2;
    if (hit[0]) cb[0] = at_byte<0>(conc, oc);
    if (hit[1]) cb[1] = at_byte<1>(conc, oc);
    if (hit[2]) cb[2] = at_byte<2>(conc, oc);
    if (hit[3]) cb[3] = at_byte<3>(conc, oc);
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (!hit[u]) continue;
    const float vb =  // V_b / m_f
        (pb[u].w > 0.f ? 1.f : kp.mass_ratio_f) * __builtin_amdgcn_rcpf(fabsf(pb[u].w));
    if (GRAD) {
      const float w = vb * (cb[u] - ca) * kernel_f_f(kp, r2s[u]);
      acc.s[0] = fmaf(w, dxs[u], acc.s[0]);
      acc.s[1 % (GRAD ? DIM : 1)] = fmaf(w, dys[u], acc.s[1 % (GRAD ? DIM : 1)]);
      if (DIM == 3) acc.s[2 % (GRAD ? DIM : 1)] = fmaf(w, dzs[u], acc.s[2 % (GRAD ? DIM : 1)]);
    } else {
      acc.s[0] = add_conc(kp, r2s[u], vb, acc.s[0]);
    }
  }
}

// The sums of one target (view position pa, key cell (cx, cy, cz), cell keys
// offset by cbase) over the rows of lane `sub` of its LPT (walk_rows), in masked
// groups of 4.
template <int DIM, int R, bool PER, bool GRAD, int LPT, bool WIDE>
__device__ __forceinline__ ShiftAcc<DIM, GRAD> shift_walk(const KParams& kp, uint32_t cbase,
                                               const float4& pa, int cx, int cy, int cz,
                                               const float4* __restrict__ pr,
                                               const uint32_t* __restrict__ cstart, float cull2,
                                               const float* __restrict__ conc, float ca,
                                               int sub, int stride) {
  ShiftAcc<DIM, GRAD> acc{};
  auto walk = [&](auto o, auto o1, uint32_t xv, float ys, float zs) {
    for (; o < o1; o += 64u)
      shift_group<DIM, GRAD>(kp, xv, ys, zs, o, o1, pr, conc, ca, acc);
  };
  walk_rows<DIM, R, PER, LPT, WIDE>(kp, cbase, pa, cx, cy, cz, cstart, cull2, sub, stride, walk);
  return acc;
}

// The sum of v over the `lanes` adjacent lanes of a target (uniform), in every lane.
__device__ inline float lanes_sum(float v, int lanes) {
  for (int off = 1; off < lanes; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// The target, the lane's place among the target's lanes and their number, LPT or
// one: after an interaction with one lane per target, shifting takes one too
// (thread t target t, the sums in the order of the one-lane kernel).
template <int LPT>
__device__ inline int64_t shift_lane(const WsHeader* __restrict__ hdr, int& sub, int& lanes) {
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  lanes = LPT > 1 && hdr->one_lane == 0u ? LPT : 1;
  sub = lanes == 1 ? 0 : (int)(t % LPT);
  return lanes == 1 ? t : t / LPT;
}

// The culling radius squared of a walk: the support (with a margin above the
// FP32 error of the offsets) when the cells are those of the view's own
// binning; widened by the largest recorded displacement when they are reused
// (R above the cells' stencil), with SPH_ERR_MARGIN past half a cell, or
// when particles moved since the binning but the cells' own reach is used.
template <int R>
__device__ inline float shift_cull2(const KParams& kp, const uint32_t* __restrict__ disp,
                                    uint32_t* __restrict__ err) {
  if (R <= kp.cell_div) {
    // the cells' own reach after particles moved since the binning: pairs
    // may be missed
    if (blockIdx.x == 0 && threadIdx.x == 0 && read_displacement(disp) > 0.f)
      set_error(err, SPH_ERR_MARGIN);
    return kp.support2_f * 1.0002f;
  }
  const float delta = read_displacement(disp);
  const float rc = __builtin_amdgcn_sqrtf(kp.support2_f) * 1.0001f + delta;
  if (!(2.f * delta < kp.cs_f) && blockIdx.x == 0 && threadIdx.x == 0)
    set_error(err, SPH_ERR_MARGIN);
  return rc * rc;
}

// C_a = sum_b V_b W_ab (Eq. 53), every non-excluded particle, a included, of one
// target (cell keys offset by cbase) in every lane of
// its LPT; lanes without a target (`live` false) take part in the sums over lanes.
template <int DIM, int R, bool PER, int LPT, bool WIDE>
__device__ inline float conc_one(const KParams& kp, bool live, uint32_t cbase, int64_t i,
                                 const float4* __restrict__ pr,
                                 const uint32_t* __restrict__ key,
                                 const uint32_t* __restrict__ cstart, float cull2, int sub,
                                 int lanes) {
  ShiftAcc<DIM, false> acc{};
  if (live) {
    const float4 pa = pr[i];
    int cx, cy, cz;
    key_cell(kp, key[i] - cbase, cx, cy, cz);
    acc = shift_walk<DIM, R, PER, false, LPT, WIDE>(kp, cbase, pa, cx, cy, cz, pr, cstart, cull2,
                                                    nullptr, 0.f, sub, lanes);
  }
  return conc_scale(kp) * lanes_sum(acc.s[0], lanes);
}

// grad C_a = sum_b V_b (C_b - C_a) F_ab r_ab and dr_a = -A_s h |v_a| dt grad C_a
// (Eq. 40-41, 53) for one fluid target i, with the tangential projection
// below the surface threshold (Eq. 54, a_n = 0); dr_a is added to the
// positions (and written to `shift` when given) by lane 0 of the target's LPT.
template <int DIM, int R, bool PER, int LPT, bool WIDE>
__device__ inline void shift_one(const KParams& kp, bool live, uint32_t cbase, int64_t n,
                                 int64_t i, const float4* __restrict__ pr,
                                 const float4* __restrict__ vp,
                                 const uint32_t* __restrict__ key,
                                 const uint32_t* __restrict__ cstart,
                                 const float* __restrict__ conc, const double* __restrict__ dtp,
                                 float cull2, double* __restrict__ pos, float* __restrict__ shift,
                                 int sub, int lanes) {
  ShiftAcc<DIM, true> acc{};
  float ca = 0.f;
  if (live) {
    ca = conc[i];
    const float4 pa = pr[i];
    int cx, cy, cz;
    key_cell(kp, key[i] - cbase, cx, cy, cz);
    acc = shift_walk<DIM, R, PER, true, LPT, WIDE>(kp, cbase, pa, cx, cy, cz, pr, cstart, cull2,
                                                   conc, ca, sub, lanes);
  }
  const float kfab = kp.kfab_mf_f;
  const float g0 = kfab * lanes_sum(acc.s[0], lanes), g1 = kfab * lanes_sum(acc.s[1], lanes),
              g2 = DIM == 3 ? kfab * lanes_sum(acc.s[DIM - 1], lanes) : 0.f;
  if (!live || sub != 0) return;
  // sums over components as explicit fma chains: a zero component (2-D cases,
  // and 2-D slots of a batch in the packed (x, 0, z) layout) adds exactly
  // nothing, so both layouts round alike
  const float4 va = vp[i];
  const float speed =
      __builtin_amdgcn_sqrtf(fmaf(va.z, va.z, fmaf(va.y, va.y, va.x * va.x)));
  const float ds = kp.shift_k_f * speed * (float)*dtp;
  float d[3] = {-ds * g0, -ds * g1, DIM == 3 ? -ds * g2 : 0.f};
  if (kp.shift_fs_f > 0.f && ca < kp.shift_fs_f) {
    const float gg = fmaf(g2, g2, fmaf(g1, g1, g0 * g0));
    if (gg > 0.f) {
      const float k = fmaf(d[2], g2, fmaf(d[1], g1, d[0] * g0)) / gg;
      d[0] = fmaf(-k, g0, d[0]);
      d[1] = fmaf(-k, g1, d[1]);
      d[2] = fmaf(-k, g2, d[2]);
    }
  }
  for (int c = 0; c < DIM; ++c) {
    pos[c * n + i] += (double)d[c];
    if (shift) shift[c * n + i] = d[c];
  }
}

template <int DIM, int R, bool PER, int LPT, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_shift_conc(KParams kp, int64_t n,
                                                       const float4* __restrict__ pr,
                                                       const uint32_t* __restrict__ key,
                                                       const uint32_t* __restrict__ cstart,
                                                       const uint8_t* __restrict__ type,
                                                       float* __restrict__ conc,
                                                       const uint32_t* __restrict__ disp,
                                                       WsHeader* __restrict__ hdr) {
  int sub, lanes;
  const int64_t i = shift_lane<LPT>(hdr, sub, lanes);
  const float cull2 = shift_cull2<R>(kp, disp, &hdr->err);
  const bool live = i < n && !is_excluded(type[i]);
  const float c =
      conc_one<DIM, R, PER, LPT, WIDE>(kp, live, 0u, i, pr, key, cstart, cull2, sub, lanes);
  if (i < n && sub == 0) conc[i] = live ? c : 0.f;
}

template <int DIM, int R, bool PER, int LPT, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_shift_apply(
    KParams kp, int64_t n, const float4* __restrict__ pr, const float4* __restrict__ vp,
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ cstart,
    const uint8_t* __restrict__ type, const float* __restrict__ conc,
    const double* __restrict__ dtp, double* __restrict__ pos, float* __restrict__ shift,
    const uint32_t* __restrict__ disp, WsHeader* __restrict__ hdr) {
  int sub, lanes;
  const int64_t i = shift_lane<LPT>(hdr, sub, lanes);
  const float cull2 = shift_cull2<R>(kp, disp, &hdr->err);
  const uint8_t ty = i < n ? type[i] : (uint8_t)0;
  const bool live = i < n && is_fluid(ty) && !is_excluded(ty);
  if (i < n && !live && shift && sub == 0)
    for (int d = 0; d < DIM; ++d) shift[d * n + i] = 0.f;
  shift_one<DIM, R, PER, LPT, WIDE>(kp, live, 0u, n, i, pr, vp, key, cstart, conc, dtp, cull2,
                                    pos, shift, sub, lanes);
}

// ------------------------------------------------------------- batches --
// Shifting over the slots of a batch (packed 3-component arrays, cell keys
// offset per slot): each slot with its own constants, dt and displacement
// record; slots whose A_s is zero are left as they are (C = 0, no shift).
// The lanes of a wave are taken slot by slot (one pass when the wave lies in
// one slot), so every pass has its slot's constants uniform.

// The culling radius squared of a slot's walk, as shift_cull2 with the
// slot's own displacement record and error word (reported by lane `leader`).
template <int R>
__device__ inline float batch_shift_cull2(const KParams& kp, const uint32_t* __restrict__ disp,
                                          uint32_t* __restrict__ err,
                                          uint32_t* __restrict__ slot_err, int leader) {
  const float delta = read_displacement(disp);
  if (R <= kp.cell_div) {
    // the cells' own reach after particles moved since the binning
    if (delta > 0.f && (threadIdx.x & 63) == leader) {
      set_error(err, SPH_ERR_MARGIN);
      set_error(slot_err, SPH_ERR_MARGIN);
    }
    return kp.support2_f * 1.0002f;
  }
  const float rc = __builtin_amdgcn_sqrtf(kp.support2_f) * 1.0001f + delta;
  if (!(2.f * delta < kp.cs_f) && (threadIdx.x & 63) == leader) {
    set_error(err, SPH_ERR_MARGIN);
    set_error(slot_err, SPH_ERR_MARGIN);
  }
  return rc * rc;
}

template <int R, bool APPLY, bool PER, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_batch_shift(
    const SlotEntry* __restrict__ tab, int ns, int64_t n, const float4* __restrict__ pr,
    const float4* __restrict__ vp, const uint32_t* __restrict__ key,
    const uint32_t* __restrict__ cstart, const uint8_t* __restrict__ type,
    float* __restrict__ conc, const double* __restrict__ dt, double* __restrict__ pos,
    float* __restrict__ shift, const uint32_t* __restrict__ disp, uint32_t* __restrict__ err,
    uint32_t* __restrict__ slot_err) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  const int sa = i < n ? find_slot(tab, ns, i) : -1;
  bool todo = i < n;
  while (__ballot(todo) != 0ull) {
    const int leader = (int)__builtin_ctzll(__ballot(todo));
    const int rs = __builtin_amdgcn_readlane(sa, leader);
    const bool mine = todo && sa == rs;
    todo = todo && !mine;
    // (a copy: the walk's asm statement would have the table read again after it,
    // which cost a batch of 68k particles 186 us in place of 160)
    const KParams kp = tab[rs].kp;
    if (!(kp.shift_k_f > 0.f)) {  // no shifting in this slot
      if (mine && !APPLY) conc[i] = 0.f;
      if (mine && APPLY && shift)
        for (int d = 0; d < 3; ++d) shift[d * n + i] = 0.f;
      continue;
    }
    const uint32_t cbase = tab[rs].cbase;
    const float cull2 =
        batch_shift_cull2<R>(kp, disp + (size_t)rs * kDispSlots, err, &slot_err[rs], leader);
    if (!mine) continue;
    const uint8_t t = type[i];
    if (!APPLY) {
      const bool live = !is_excluded(t);
      const float c = conc_one<3, R, PER, 1, WIDE>(kp, live, cbase, i, pr, key, cstart, cull2, 0, 1);
      conc[i] = live ? c : 0.f;
    } else {
      const bool live = is_fluid(t) && !is_excluded(t);
      if (!live && shift)
        for (int d = 0; d < 3; ++d) shift[d * n + i] = 0.f;
      shift_one<3, R, PER, 1, WIDE>(kp, live, cbase, n, i, pr, vp, key, cstart, conc, &dt[rs],
                                    cull2, pos, shift, 0, 1);
    }
  }
}

// Lanes per target for a case of n particles, as for the interaction
// (lanes_per_target), of fewer kinds.  Measured, both kernels together, us with
// 1 / 4 / 16 lanes (dam breaks on reused cells):
//   3-D    7k: 166 / 69 / 32    21k: 167 / 67 / 41    33k: 163 / 69 / 54
//         58k: 169 / 79 / 88   127k: 175 / 136 / 166  168k: 182 / 179 / 225
//         filled box          140k: 186 / 183 / 236  175k: 210 / 230 / 289
//   2-D    4k: 26 / 16          54k: 27 / 22           84k: 29 / 29
static int shift_lanes(int dim, int64_t n) {
  if (dim == 2) return n <= 65536 ? 4 : 1;
  return n <= 49152 ? 16 : n <= 147456 ? 4 : 1;
}

hipError_t launch_shifting(const KParams& kp, int64_t n, const sph_state& s, const uint32_t* key,
                           const uint32_t* cell_start, const double* dt, float* conc,
                           float* shift, bool reuse, bool given, void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  const float4* pr = ws_ptr<float4>(ws, L.view_pr);
  const float4* vp = ws_ptr<float4>(ws, L.view_vp);
  float* c = conc ? conc : ws_ptr<float>(ws, L.keyA);
  const uint32_t* disp = ws_ptr<uint32_t>(ws, L.disp);
  WsHeader* hdr = ws_ptr<WsHeader>(ws, L.err);
  const bool per = kp.periodic != 0;
  // a large case or grid takes the walk with 64-bit offsets, one lane per target
  // (a large grid may hold few particles: they need no speed)
  const bool wide = !walk_fits_32(n, kp.ncell_total);
  const int lanes = wide ? 1 : shift_lanes(kp.dim, n);
  // reused cells: one more cell of reach, cut widened by the displacement
  const int reach = kp.cell_div + (reuse ? 1 : 0);
#define SPH_SHIFT(D, RR, PE, LP, WI)                                                          \
  do {                                                                                        \
    const dim3 grid(n > 0 ? (unsigned)((n * LP + kBlock - 1) / kBlock) : 1u);                 \
    if (!given)                                                                               \
      hipLaunchKernelGGL((k_shift_conc<D, RR, PE, LP, WI>), grid, dim3(kBlock), 0, st, kp, n, \
                         pr, key, cell_start, s.type, c, disp, hdr);                          \
    hipLaunchKernelGGL((k_shift_apply<D, RR, PE, LP, WI>), grid, dim3(kBlock), 0, st, kp, n,  \
                       pr, vp, key, cell_start, s.type, c, dt, s.pos, shift, disp, hdr);      \
  } while (0)
#define SPH_SHIFT_L2(RR, PE)                      \
  if (lanes == 4) SPH_SHIFT(2, RR, PE, 4, false); \
  else if (wide) SPH_SHIFT(2, RR, PE, 1, true);   \
  else SPH_SHIFT(2, RR, PE, 1, false)
#define SPH_SHIFT_L3(RR, PE)                           \
  if (lanes == 16) SPH_SHIFT(3, RR, PE, 16, false);    \
  else if (lanes == 4) SPH_SHIFT(3, RR, PE, 4, false); \
  else if (wide) SPH_SHIFT(3, RR, PE, 1, true);        \
  else SPH_SHIFT(3, RR, PE, 1, false)
#define SPH_SHIFT_R(D)                                                                  \
  if (reach == 1) { if (per) { SPH_SHIFT_L##D(1, true); } else { SPH_SHIFT_L##D(1, false); } }      \
  else if (reach == 2) { if (per) { SPH_SHIFT_L##D(2, true); } else { SPH_SHIFT_L##D(2, false); } } \
  else { if (per) { SPH_SHIFT_L##D(3, true); } else { SPH_SHIFT_L##D(3, false); } }
  if (kp.dim == 2) {
    SPH_SHIFT_R(2);
  } else {
    SPH_SHIFT_R(3);
  }
#undef SPH_SHIFT_R
#undef SPH_SHIFT_L3
#undef SPH_SHIFT_L2
#undef SPH_SHIFT
  return hipGetLastError();
}

hipError_t launch_batch_shifting(const BatchDesc& B, const sph_state& s, const uint32_t* key,
                                 const uint32_t* cell_start, const double* dt, float* conc,
                                 float* shift, bool reuse, void* ws, hipStream_t st) {
  const int64_t n = B.n_total;
  const BatchWsLayout W = batch_ws_layout(B.n_slots, n);
  const SlotEntry* tab = (const SlotEntry*)B.table;
  const float4* pr = ws_ptr<float4>(ws, W.base.view_pr);
  const float4* vp = ws_ptr<float4>(ws, W.base.view_vp);
  float* c = conc ? conc : ws_ptr<float>(ws, W.base.keyA);
  const uint32_t* disp = ws_ptr<uint32_t>(ws, W.disp);
  uint32_t* err = ws_ptr<uint32_t>(ws, W.base.err);
  uint32_t* serr = ws_ptr<uint32_t>(ws, W.slot_err);
  const int64_t g = (n + kBlock - 1) / kBlock;
  const unsigned grid = (unsigned)(g > 0 ? g : 1);
  // reused cells: one more cell of reach, cut widened by each slot's record
  const int reach = B.cell_div + (reuse ? 1 : 0);
  const bool per = (B.flags & SPH_BATCH_PERIODIC) != 0;
  const bool wide = !walk_fits_32(n, (uint64_t)B.key_cells);
#define SPH_BSHIFT_P(RR, PE, WI)                                                                \
  do {                                                                                          \
    hipLaunchKernelGGL((k_batch_shift<RR, false, PE, WI>), dim3(grid), dim3(kBlock), 0, st, tab, \
                       B.n_slots, n, pr, vp, key, cell_start, s.type, c, dt, s.pos, shift, disp, \
                       err, serr);                                                              \
    hipLaunchKernelGGL((k_batch_shift<RR, true, PE, WI>), dim3(grid), dim3(kBlock), 0, st, tab, \
                       B.n_slots, n, pr, vp, key, cell_start, s.type, c, dt, s.pos, shift, disp, \
                       err, serr);                                                              \
  } while (0)
#define SPH_BSHIFT(RR)                                                          \
  do {                                                                          \
    if (wide) { if (per) SPH_BSHIFT_P(RR, true, true); else SPH_BSHIFT_P(RR, false, true); } \
    else { if (per) SPH_BSHIFT_P(RR, true, false); else SPH_BSHIFT_P(RR, false, false); }    \
  } while (0)
  if (reach == 1) {
    SPH_BSHIFT(1);
  } else if (reach == 2) {
    SPH_BSHIFT(2);
  } else {
    SPH_BSHIFT(3);
  }
#undef SPH_BSHIFT
#undef SPH_BSHIFT_P
  return hipGetLastError();
}

}  // namespace sph
