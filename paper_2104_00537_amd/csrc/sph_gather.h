// The interaction over the rows of neighbour cells (gather_walk): its kernel
// and the launch over its variants for one dimension.  The 2-D and the 3-D
// variants are instantiated in a source each, which compile side by side.
#pragma once

#include "sph_dev.h"
#include "sph_kernels.h"
#include "sph_pair.h"

namespace sph {

// ------------------------------------------------- interaction: gather --
// The target's own terms from its view entry (sorted slot i).
template <bool GEN>
__device__ __forceinline__ void target_data(const KParams& kp, int64_t i,
                                            const float4* __restrict__ pr,
                                            const float4* __restrict__ vp,
                                            const uint8_t* __restrict__ type, TargetData& T) {
  const float4 pa = pr[i], va = vp[i];
  T.fluid = pa.w > 0.f;
  T.rho = fabsf(pa.w);
  T.irho = __builtin_amdgcn_rcpf(T.rho);
  T.ik = kp.kvc_f * T.irho;
  T.p = va.w;
  T.vx = va.x;
  T.vy = va.y;
  T.vz = va.z;
  T.flt = GEN && kp.floating && is_floating(type[i]);
}

// Wavefronts per SIMD that the registers are held to (1: not held).  The walk
// fills its waits with other wavefronts, and a case of few rounds of wavefronts
// ends on a partly filled one, so that one more or less per SIMD shows (us per
// pass; R = 2 / 3):
//   2-D, 503k: 7 (by its scalar registers) 66.6 / 66.1, 8: 56.0 / 55.3; larger
//     and smaller cases within 2 % either way
//   3-D, 1.32M: 7 573 / 576, 8 (it spills) 591 / 593; 1.58M: 699 / 703, 723 / 723
//   3-D periodic, 958k: 6 604 / 610, 7 574 / 579, 8 621 / 630
//   3-D with options, 441k: 5 304 / 307, 6 266 / 268, 7 271 / 272
// At other sizes from 230k to 2M particles these numbers are within 2 % of the
// compiler's own or faster.
// With several lanes per target the registers are left to the compiler, which
// gives the 2 lanes of the default formulation in 3-D 6 wavefronts.  A case of more
// wavefronts than that ends on a second round of few of them and, from kHoldMinN
// particles on (HOLD), is faster held to 7 (us per pass, 6 / 7: open block 207k
// 167 / 143, 229k 178 / 153; filled box 221k 165 / 142; dam break, half of it walls
// whose targets end early, 216k 120 / 123, 234k 129 / 135, 253k 144 / 139).
constexpr int64_t kHoldMinN = 221184;
constexpr int gather_waves(int dim, bool plain, bool gen, int lpt, bool hold) {
  if (hold) return 7;
  if (!plain || (dim == 2 && gen) || (dim == 3 && lpt > 1)) return 1;
  return dim == 2 ? 8 : gen ? 6 : 7;
}

// LPT lanes per target particle (sorted order): 1 is the production kernel of
// large cases; more deal each target's rows to that many lanes, for cases too
// small to fill the GPU (see lanes_per_target).
template <int DIM, int R, bool DIAG, bool EQM, bool GEN, bool PER, int LPT, bool CONC = false,
          bool HOLD = false>
__global__ __launch_bounds__(kBlock, gather_waves(DIM, EQM && !DIAG, GEN, LPT, HOLD)) void
k_interact_gather(
    KParams kp, int64_t n, const float4* __restrict__ pr, const float4* __restrict__ vp,
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ cstart,
    const uint8_t* __restrict__ type, const double* __restrict__ pos64, float* __restrict__ ace,
    float* __restrict__ arho, float* __restrict__ visc, uint32_t* __restrict__ nbr,
    BlockRed* __restrict__ red, WsHeader* __restrict__ hdr, const uint32_t* __restrict__ disp,
    float* __restrict__ conc) {
  static_assert(LPT >= 1 && LPT <= kMaxLanes && (LPT & (LPT - 1)) == 0, "a power of two");
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  const int64_t i = t / LPT;
  const int sub = (int)(t % LPT);
  float fmag = 0.f, vmax_out = 0.f;
  uint32_t cnt_out = 0, cnt_wall = 0, nfl = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) hdr->one_lane = LPT == 1 ? 1u : 0u;
  // cells reused after a view refresh (R above the cells' own stencil): cull
  // with the support widened by the largest displacement since the binning
  float cull2 = kp.support2_f * 1.0002f;
  if (R > kp.cell_div) {
    const float delta = read_displacement(disp);
    const float rc = __builtin_amdgcn_sqrtf(kp.support2_f) * 1.0001f + delta;
    cull2 = rc * rc;
    if (!(2.f * delta < kp.cs_f) && blockIdx.x == 0 && threadIdx.x == 0)
      set_error(&hdr->err, SPH_ERR_MARGIN);
  } else if (blockIdx.x == 0 && threadIdx.x == 0 && read_displacement(disp) > 0.f) {
    // particles moved since the binning (a predictor ran) but the walk keeps
    // the cells' own reach: pairs may be missed
    set_error(&hdr->err, SPH_ERR_MARGIN);
  }
  if constexpr (LPT == 1) {
    if (i < n) {
      PairAcc acc{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0u};
      TargetData T{false, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, false, 0.f};
      uint32_t c64 = 0;
      // with modified DBC the wall densities come from Eq. 38 (sph_mdbc): wall
      // targets take no sums
      if (!is_excluded(type[i]) && (kp.boundary == 0 || is_fluid(type[i]))) {
        target_data<GEN>(kp, i, pr, vp, type, T);
        const float4 pa = pr[i];
        int cx, cy, cz;
        key_cell(kp, key[i], cx, cy, cz);
        gather_walk<DIM, R, DIAG, EQM, GEN, PER, 1, CONC>(kp, 0u, n, i, pa, T, cx, cy, cz, pr, vp,
                                                          cstart, pos64, acc, c64, cull2);
        if (T.fluid) acc.cnt -= 1u;  // the self pair: counted, added nothing
        const uint32_t c = DIAG ? c64 : acc.cnt;
        write_target<DIM>(kp, n, i, T, acc, c, ace, arho, visc, nbr, fmag, vmax_out, nfl);
        if (CONC) conc[i] = conc_scale(kp) * acc.conc;
        cnt_out = acc.cnt;
        cnt_wall = T.fluid ? 0u : acc.cnt;
      } else {
        write_zero<DIM>(n, i, ace, arho, visc, nbr);
        if (CONC) conc[i] = 0.f;
      }
    }
  } else {
    PairAcc acc{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0u};
    TargetData T{false, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, false, 0.f};
    uint32_t c64 = 0;
    const bool active =
        i < n && !is_excluded(type[i]) && (kp.boundary == 0 || is_fluid(type[i]));
    if (active) {
      target_data<GEN>(kp, i, pr, vp, type, T);
      const float4 pa = pr[i];
      int cx, cy, cz;
      key_cell(kp, key[i], cx, cy, cz);
      gather_walk<DIM, R, DIAG, EQM, GEN, PER, LPT, CONC>(kp, 0u, n, i, pa, T, cx, cy, cz, pr,
                                                          vp, cstart, pos64, acc, c64, cull2,
                                                          sub);
    }
    combine_lanes<LPT, CONC>(acc, c64);  // every lane: the sums of its target's lanes
    if (i < n && sub == 0) {
      if (active) {
        if (T.fluid) acc.cnt -= 1u;  // the self pair: counted, added nothing
        const uint32_t c = DIAG ? c64 : acc.cnt;
        write_target<DIM>(kp, n, i, T, acc, c, ace, arho, visc, nbr, fmag, vmax_out, nfl);
        if (CONC) conc[i] = conc_scale(kp) * acc.conc;
        cnt_out = acc.cnt;
        cnt_wall = T.fluid ? 0u : acc.cnt;
      } else {
        write_zero<DIM>(n, i, ace, arho, visc, nbr);
        if (CONC) conc[i] = 0.f;
      }
    }
  }
  write_block_red<kBlock / 64>(fmag, vmax_out, cnt_out, cnt_wall, nfl, red, hdr);
}

// Lanes per target for a case of n particles.  One wavefront that walks its
// targets' rows alone takes about 100 us in 3-D and 17 us in 2-D, whatever
// the case's size: a chain of dependent loads (ranges, candidates,
// velocities, row after row).  While wavefronts are too few to hide it,
// dealing the rows to more lanes shortens the chain; once the GPU is full the
// extra instructions cost (rows of different lengths in step, the sums over
// lanes).  The lines lie where measured times cross (us per pass, 1 / 2 / 4 /
// 8 / 16 lanes; 3-D dam breaks and 2-D dam breaks, one MI355X):
//   3-D   13k: 104 / 60 / 36 / 23 / 19      25k: 102 / 59 / 36 / 28 / 28
//         66k: 105 / 64 / 50 / 50 / 55     127k: 121 / 81 / 84 / 89 / 106
//        223k: 164 / 124 / 144 / 158 / 189  441k: 220 / 234 / 292 / 321 / 387
//   2-D   14k: 17 / 12 / 9.7 / 9.6 / 10     54k: 18 / 14 / 15 / 16 / 24
//        185k: 25 / 27 / 33 / 41 / 69
// The last lines of 3-D differ with the kind of case, the more so as a step's second
// pass, on reused cells, is slower with two lanes (us, both passes, 1 / 2 lanes, held
// as above):
//   sloshing tank   242k: 328 / 280   266k: 350 / 306
//   dam break       253k: 314 / 286   273k: 321 / 300   315k: 363 / 377
//   filled box      221k: 356 / 296   244k: 366 / 359   260k: 374 / 387
//   open block      229k: 344 / 317   252k: 375 / 385   286k: 407 / 440
// With options (gen) two lanes have 5 wavefronts per SIMD and lose sooner (cubic
// spline, periodic with all options):
//   dam break       234k: 397 / 347   253k: 393 / 390
//   sloshing tank   219k: 382 / 364   242k: 391 / 403
//   filled box      184k: 394 / 373   192k: 402 / 399   229k: 427 / 441
//   channel         202k: 548 / 533   209k: 548 / 546   223k: 490 / 532
// The lines lie where no kind loses more than about 5 %.
inline int lanes_per_target(int dim, int64_t n, bool gen, bool per) {
  if (dim == 2) return n <= 32768 ? 4 : n <= 122880 ? 2 : 1;
  if (n <= 98304) return n <= 24576 ? 16 : n <= 65536 ? 8 : 4;
  return n <= (!gen ? kLanesMaxN : per ? 212992 : 235520) ? 2 : 1;
}

template <int DIM>
hipError_t launch_gather(const KParams& kp, int64_t n, const sph_state& s, const uint32_t* key,
                         const uint32_t* cell_start, float* ace, float* arho, float* visc,
                         uint32_t* nbr, uint32_t flags, const InteractScratch& w,
                         hipStream_t st) {
  const bool diag = (flags & SPH_DIAG_COUNT_F64) != 0;
  // reused cells: one more cell of reach (the kernels read the displacement)
  const int reach = kp.cell_div + ((flags & SPH_INTERACT_REUSE_CELLS) ? 1 : 0);
  const bool eqm = kp.mass_f == kp.mass_b;
  const bool gen = kp.kernel != 0 || kp.viscosity != 0 || kp.ddt == 2 || kp.floating != 0;
  const bool per = kp.periodic != 0;
  int lanes = (flags & SPH_INTERACT_ONE_LANE) ? 1 : lanes_per_target(kp.dim, n, gen, per);
  const bool hold = n > kHoldMinN;
  // the diagnostic count and unequal masses come with one lane or four, and lose
  // with four sooner (us per pass, 1 / 4 lanes):
  //   3-D, unequal masses   100k: 117 / 91    140k: 127 / 124, reused cells 129 / 142
  //        count            100k: 236 / 224   140k: 277 / 299   304k: 417 / 598
  //   2-D, unequal masses    54k: 17 / 15     105k: 21 / 23
  //        count             54k: 25 / 22     105k: 30 / 36
  if ((diag || !eqm) && lanes > 1) lanes = n <= (DIM == 2 ? 65536 : 131072) ? 4 : 1;
#define SPH_LAUNCH(D, RR, G, PP, GG, PE, LP, HO)                                              \
  hipLaunchKernelGGL((k_interact_gather<D, RR, G, PP, GG, PE, LP, false, HO>),                \
                     dim3(n > 0 ? (unsigned)((n * LP + kBlock - 1) / kBlock) : 1u),           \
                     dim3(kBlock), 0, st, kp, n, w.pr, w.vp, key, cell_start, s.type, s.pos, ace, \
                     arho, visc, nbr, w.red, w.hdr, w.disp, nullptr)
// The formulation and the periodic components are chosen apart: the general pair
// terms test the case's options for every pair, which a periodic case in the
// default formulation need not pay (958k particles in a periodic channel:
// 715 -> 608 us a pass; the same operations, the same results).
#define SPH_LAUNCH_F(D, RR, G, PP, LP)                  \
  if (per && gen) SPH_LAUNCH(D, RR, G, PP, true, true, LP, false); \
  else if (per) SPH_LAUNCH(D, RR, G, PP, false, true, LP, false); \
  else if (gen) SPH_LAUNCH(D, RR, G, PP, true, false, LP, false); \
  else SPH_LAUNCH(D, RR, G, PP, false, false, LP, false)
#define SPH_LAUNCH_1(D, RR, G, PP)                      \
  if (lanes == 1) { SPH_LAUNCH_F(D, RR, G, PP, 1); }    \
  else { SPH_LAUNCH_F(D, RR, G, PP, 4); }
#define SPH_LAUNCH_2(RR)                                         \
  if (lanes == 1) { SPH_LAUNCH_F(2, RR, false, true, 1); }       \
  else if (lanes == 2) { SPH_LAUNCH_F(2, RR, false, true, 2); }  \
  else { SPH_LAUNCH_F(2, RR, false, true, 4); }
#define SPH_LAUNCH_3(RR)                                         \
  if (lanes == 1) { SPH_LAUNCH_F(3, RR, false, true, 1); }       \
  else if (lanes == 2 && hold && !gen) {                         \
    if (per) SPH_LAUNCH(3, RR, false, true, false, true, 2, true); \
    else SPH_LAUNCH(3, RR, false, true, false, false, 2, true);  \
  } else if (lanes == 2) { SPH_LAUNCH_F(3, RR, false, true, 2); } \
  else if (lanes == 4) { SPH_LAUNCH_F(3, RR, false, true, 4); }  \
  else if (lanes == 8) { SPH_LAUNCH_F(3, RR, false, true, 8); }  \
  else { SPH_LAUNCH_F(3, RR, false, true, 16); }
#define SPH_LAUNCH_R(D, RR)                                      \
  if (diag && eqm) { SPH_LAUNCH_1(D, RR, true, true); }          \
  else if (diag) { SPH_LAUNCH_1(D, RR, true, false); }           \
  else if (!eqm) { SPH_LAUNCH_1(D, RR, false, false); }          \
  else { SPH_LAUNCH_##D(RR); }
  if constexpr (DIM == 2) {
    if (reach == 1) { SPH_LAUNCH_R(2, 1); }
    else if (reach == 2) { SPH_LAUNCH_R(2, 2); }
    else { SPH_LAUNCH_R(2, 3); }
  } else {
    if (reach == 1) { SPH_LAUNCH_R(3, 1); }
    else if (reach == 2) { SPH_LAUNCH_R(3, 2); }
    else { SPH_LAUNCH_R(3, 3); }
  }
#undef SPH_LAUNCH_R
#undef SPH_LAUNCH_3
#undef SPH_LAUNCH_2
#undef SPH_LAUNCH_1
#undef SPH_LAUNCH_F
#undef SPH_LAUNCH
  return hipGetLastError();
}

extern template hipError_t launch_gather<2>(const KParams&, int64_t, const sph_state&,
                                            const uint32_t*, const uint32_t*, float*, float*,
                                            float*, uint32_t*, uint32_t, const InteractScratch&,
                                            hipStream_t);
extern template hipError_t launch_gather<3>(const KParams&, int64_t, const sph_state&,
                                            const uint32_t*, const uint32_t*, float*, float*,
                                            float*, uint32_t*, uint32_t, const InteractScratch&,
                                            hipStream_t);

}  // namespace sph
