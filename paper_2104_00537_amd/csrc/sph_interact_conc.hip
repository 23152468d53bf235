// The interaction with the concentration of Eq. 53 (pair_terms' CONC), for the
// pass before a particle shifting: on reused cells, in the default formulation
// with equal masses.  A walk of its own for the concentration costs 350 us at
// 958k particles of a periodic channel, of which the tests of the candidates and
// their 16 bytes through the L1 data path are nearly all; three operations more
// per pair in the interaction's walk cost about 10 us (616 -> 626).
#include "sph_gather.h"

namespace sph {

hipError_t launch_interact_conc(const KParams& kp, int64_t n, const sph_state& s,
                                const uint32_t* key, const uint32_t* cell_start, float* ace,
                                float* arho, float* conc, uint32_t flags, void* ws,
                                hipStream_t st) {
  const WsLayout L = ws_layout(n);
  float* c = conc ? conc : ws_ptr<float>(ws, L.keyA);
  const bool per = kp.periodic != 0;
  int lanes = (flags & SPH_INTERACT_ONE_LANE) ? 1 : lanes_per_target(kp.dim, n, false, per);
  // C takes registers: in a periodic channel two lanes per target have 5 wavefronts
  // per SIMD and are held to 7 sooner than without it, and one lane is faster sooner
  // (us per pass, two lanes / held / one: channel 168k 179 / 195 / 228, 194k 252 / 223
  // / 243; filled box 192k 149 / 151 / 170, 238k 200 / 195 / 182; dam break 234k 149
  // / - / 171, 253k 164 / - / 169)
  const bool hold = n > (per ? 184320 : kHoldMinN);
  if (lanes == 2 && kp.dim == 3 && n > (per ? 229376 : 235520)) lanes = 1;
#define SPH_CONC(D, RR, PE, LP, HO)                                                            \
  hipLaunchKernelGGL((k_interact_gather<D, RR, false, true, false, PE, LP, true, HO>),         \
                     dim3((unsigned)((n * LP + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,    \
                     kp, n, ws_ptr<float4>(ws, L.view_pr), ws_ptr<float4>(ws, L.view_vp), key, \
                     cell_start, s.type, s.pos, ace, arho, nullptr, nullptr,                   \
                     ws_ptr<BlockRed>(ws, L.red), ws_ptr<WsHeader>(ws, L.err),                 \
                     ws_ptr<uint32_t>(ws, L.disp), c)
#define SPH_CONC_L2(RR, PE)                  \
  if (lanes == 1) SPH_CONC(2, RR, PE, 1, false);    \
  else if (lanes == 2) SPH_CONC(2, RR, PE, 2, false); \
  else SPH_CONC(2, RR, PE, 4, false)
#define SPH_CONC_L3(RR, PE)                           \
  if (lanes == 1) SPH_CONC(3, RR, PE, 1, false);      \
  else if (lanes == 2 && hold) SPH_CONC(3, RR, PE, 2, true); \
  else if (lanes == 2) SPH_CONC(3, RR, PE, 2, false); \
  else if (lanes == 4) SPH_CONC(3, RR, PE, 4, false); \
  else if (lanes == 8) SPH_CONC(3, RR, PE, 8, false); \
  else SPH_CONC(3, RR, PE, 16, false)
#define SPH_CONC_P(D, RR)                      \
  if (per) { SPH_CONC_L##D(RR, true); }        \
  else { SPH_CONC_L##D(RR, false); }
  if (kp.dim == 2) {
    if (kp.cell_div == 1) { SPH_CONC_P(2, 2); }
    else { SPH_CONC_P(2, 3); }
  } else {
    if (kp.cell_div == 1) { SPH_CONC_P(3, 2); }
    else { SPH_CONC_P(3, 3); }
  }
#undef SPH_CONC_P
#undef SPH_CONC_L3
#undef SPH_CONC_L2
#undef SPH_CONC
  return hipGetLastError();
}

}  // namespace sph
