// Neighbour list (Section 5.1 of the DualSPHysics v5.0 paper): cell keys, a
// stable counting sort of the particles by key, cell ranges and the reorder
// of the particle state into sorted structure-of-arrays.
//
// The cell ranges are an output anyway, so the sort is built on them: one
// pass counts the particles of every cell, a scan of the counts gives the
// ranges, and each particle is placed in its cell's range in whatever order
// the counting atomics met them.  That order differs from run to run; the
// reorder restores the stable one by ranking each particle among the members
// of its cell by input index (a cell of h/x_sub holds about one particle, so
// there is little to rank).  Particles outside the grid are kept apart: they
// may be many, and their order follows from a scan of their numbers per
// wavefront.  Six kernels in all.
#include "sph_dev.h"
#include "sph_kernels.h"

namespace sph {

// ------------------------------------------------------ keys and counting --
// The number of excluded particles of the calling wavefront (to xcount) and
// the calling lane's rank among them.
__device__ inline uint32_t rank_excluded(bool excluded, int64_t i, int64_t n,
                                         uint32_t* __restrict__ xcount) {
  const uint64_t mask = __ballot(excluded);
  const int lane = threadIdx.x & 63;
  if (lane == 0 && i < n) xcount[i >> 6] = (uint32_t)__popcll(mask);
  return (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
}

// (a new binning also restarts the record of the largest displacement)
__global__ __launch_bounds__(kBlock) void k_count_cells(
    KParams kp, int64_t n, const double* __restrict__ pos, const uint8_t* __restrict__ type,
    uint32_t* __restrict__ key, uint32_t* __restrict__ rank, uint32_t* __restrict__ count,
    uint32_t* __restrict__ xcount, uint32_t* __restrict__ disp, WsHeader* __restrict__ hdr) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i == 0) {
    for (int k = 0; k < kDispSlots; ++k) disp[k] = 0u;
    hdr->bin_gen = hdr->bin_gen + 1u;
    hdr->one_lane = 0u;
  }
  const uint32_t k = i < n ? cell_key_local(kp, pos, type, n, i) : 0u;
  const bool excluded = i < n && k == kp.ncell_total;
  uint32_t r = rank_excluded(excluded, i, n, xcount);
  const uint32_t rc = count_in_cell(i < n && !excluded, k, count);
  if (i >= n) return;
  if (!excluded) r = rc;
  key[i] = k;
  rank[i] = r;
}

// ------------------------------------------------------- exclusive scans --
// Exclusive prefix sum of one value per thread over a 256-thread block.
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t base = 0, all = 0;
  for (int w = 0; w < kBlock / 64; ++w) {
    if (w < wave) base += wsum[w];
    all += wsum[w];
  }
  __syncthreads();
  if (total) *total = all;
  return base + x - v;
}

// The scanned sequence: the counts of the `cells` cells, then the numbers of
// excluded particles per wavefront.  Its exclusive prefix sums are the cells'
// first sorted indices, start[cells] (the number of particles in cells) and
// the first sorted index of each wavefront's excluded particles.  Each of at
// most kScanBlocks blocks takes one chunk of whole scan tiles, so the sums of
// the chunks fit the workspace whatever the number of cells.
typedef uint32_t uint4a4 __attribute__((ext_vector_type(4), aligned(4)));
struct ScanSeq {
  uint32_t* start;
  uint32_t* xcount;
  int64_t cells;
  int64_t len;
  __device__ uint32_t get(int64_t e) const { return e < cells ? start[e] : xcount[e - cells]; }
  __device__ void put(int64_t e, uint32_t v) const {
    if (e <= cells) start[e] = v;
    if (e >= cells) xcount[e - cells] = v;
  }
};

__global__ __launch_bounds__(kBlock) void k_scan_sums(ScanSeq q, int64_t chunk,
                                                      uint32_t* __restrict__ sums) {
  const int64_t e0 = (int64_t)blockIdx.x * chunk;
  const int64_t e1 = e0 + chunk < q.len ? e0 + chunk : q.len;
  uint32_t s = 0;
  const int64_t ev = e1 < q.cells ? e1 : q.cells;  // (chunks start at whole vectors)
  for (int64_t e = e0 + 4 * (int64_t)threadIdx.x; e < e1; e += 4 * kBlock) {
    if (e + 4 <= ev) {
      const uint4a4 v = *reinterpret_cast<const uint4a4*>(q.start + e);
      s += v.x + v.y + v.z + v.w;
    } else {
      for (int k = 0; k < 4; ++k)
        if (e + k < e1) s += q.get(e + k);
    }
  }
  uint32_t total;
  block_exclusive_scan(s, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void k_scan_apply(ScanSeq q, int64_t chunk,
                                                       const uint32_t* __restrict__ sums) {
  // the sum of the chunks before this one
  uint32_t before = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += kBlock) before += sums[b];
  uint32_t run;
  block_exclusive_scan(before, &run);
  const int64_t e0 = (int64_t)blockIdx.x * chunk;
  const int64_t e1 = e0 + chunk < q.len ? e0 + chunk : q.len;
  for (int64_t t = e0; t < e1; t += kScanTile) {
    const int64_t base = t + threadIdx.x * kScanItems;
    const bool whole = base + kScanItems <= e1 && base + kScanItems <= q.cells;
    uint32_t v[kScanItems], s = 0;
    if (whole) {
      const uint4a4* p = reinterpret_cast<const uint4a4*>(q.start + base);
#pragma unroll
      for (int k = 0; k < kScanItems; k += 4) {
        const uint4a4 a = p[k / 4];
        v[k] = a.x;
        v[k + 1] = a.y;
        v[k + 2] = a.z;
        v[k + 3] = a.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) v[k] = base + k < e1 ? q.get(base + k) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    uint32_t total;
    uint32_t x = run + block_exclusive_scan(s, &total);
    if (whole) {
      uint4a4* p = reinterpret_cast<uint4a4*>(q.start + base);
#pragma unroll
      for (int k = 0; k < kScanItems; k += 4) {
        uint4a4 a;
        a.x = x;
        a.y = a.x + v[k];
        a.z = a.y + v[k + 1];
        a.w = a.z + v[k + 2];
        p[k / 4] = a;
        x = a.w + v[k + 3];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) {
        if (base + k < e1) q.put(base + k, x);
        x += v[k];
      }
    }
    run += total;
  }
}

__global__ __launch_bounds__(kBlock) void k_zero_cells(uint32_t* __restrict__ p, int64_t len) {
  const int64_t e = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
  if (e + 4 <= len) {
    *reinterpret_cast<uint4a4*>(p + e) = uint4a4{0u, 0u, 0u, 0u};
  } else {
    for (int64_t k = e; k < len; ++k) p[k] = 0u;
  }
}

void launch_zero_cells(uint32_t* cell_start, int64_t cells, hipStream_t st) {
  const int64_t g = (cells + 4 * kBlock - 1) / (4 * kBlock);
  if (g > 0)
    hipLaunchKernelGGL(k_zero_cells, dim3((unsigned)g), dim3(kBlock), 0, st, cell_start, cells);
}

void launch_scan_cells(uint32_t* cell_start, int64_t cells, uint32_t* xcount, int64_t n,
                       uint32_t* sums, hipStream_t st) {
  const int64_t waves = (n + 63) / 64;
  // (at least one entry after the cells': their total goes to it)
  const int64_t len = cells + (waves > 0 ? waves : 1);
  int64_t chunk = (len + kScanBlocks - 1) / kScanBlocks;
  chunk = (chunk + kScanTile - 1) / kScanTile * kScanTile;
  const unsigned blocks = (unsigned)((len + chunk - 1) / chunk);
  const ScanSeq q{cell_start, xcount, cells, len};
  hipLaunchKernelGGL(k_scan_sums, dim3(blocks), dim3(kBlock), 0, st, q, chunk, sums);
  hipLaunchKernelGGL(k_scan_apply, dim3(blocks), dim3(kBlock), 0, st, q, chunk, sums);
}

// ------------------------------------------------------------- placement --
// The members of each cell, {input index, key}, in its range (in any order),
// excluded particles in theirs (in input order).
__global__ __launch_bounds__(kBlock) void k_place(int64_t n, uint32_t ncell_total,
                                                  const uint32_t* __restrict__ key,
                                                  const uint32_t* __restrict__ rank,
                                                  const uint32_t* __restrict__ cell_start,
                                                  const uint32_t* __restrict__ xstart,
                                                  uint2* __restrict__ member) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t k = key[i];
  member[(k < ncell_total ? cell_start[k] : xstart[i >> 6]) + rank[i]] =
      make_uint2((uint32_t)i, k);
}

// --------------------------------------------------------------- reorder --
__global__ __launch_bounds__(kBlock) void k_reorder(
    KParams kp, int64_t n, const uint2* __restrict__ member,
    const uint32_t* __restrict__ cell_start, uint32_t* __restrict__ perm,
    uint32_t* __restrict__ key, sph_state in, sph_state out, sph_state cin, sph_state cout,
    int carry, float4* __restrict__ pr, float4* __restrict__ vp, uint32_t* __restrict__ err) {
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (t >= n) return;
  const uint32_t src = member[t].x, k = member[t].y;
  const int64_t i = k < kp.ncell_total ? stable_slot(member, cell_start, k, src) : t;
  perm[i] = src;
  key[i] = k;
  if (reorder_one(kp, n, i, src, k, in, out, cin, cout, carry, pr, vp))
    set_error(err, SPH_ERR_EXCLUDED);
}

// ------------------------------------------------------------ view refresh --
// Rewrites the view of sorted slot i from the state's current position,
// velocity and density, relative to the cell its key (from the last
// binning) names; positions are not wrapped (they stay relative to that
// cell).  A particle that is now outside the grid along an open component
// is excluded, as a binning would; its view entry gets NaN offsets and zero
// density, so it meets no target in the cell range it still sits in.
__global__ void k_refresh_view(KParams kp, int64_t n, const uint32_t* __restrict__ key,
                               sph_state s, float4* __restrict__ pr, float4* __restrict__ vp,
                               uint32_t* __restrict__ err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint8_t t = s.type[i];
  if (t & SPH_EXCLUDED) return;  // its entry was written by the binning
  if (cell_key_local(kp, s.pos, s.type, n, i) == kp.ncell_total) {
    s.type[i] = t | SPH_EXCLUDED;
    set_error(err, SPH_ERR_EXCLUDED);
    const float nan = __builtin_nanf("");
    pr[i] = make_float4(0.f, nan, nan, 0.f);
    vp[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  double x[3] = {0.0, 0.0, 0.0};
  float v[3] = {0.f, 0.f, 0.f};
  for (int d = 0; d < kp.dim; ++d) {
    x[d] = s.pos[d * n + i];
    v[d] = s.vel[d * n + i];
  }
  write_view(kp, i, x, v, s.rho[i], t, key[i], pr, vp);
}

hipError_t launch_refresh_view(const KParams& kp, int64_t n, const sph_state& s,
                               const uint32_t* key, void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  if (n > 0)
    hipLaunchKernelGGL(k_refresh_view, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock),
                       0, st, kp, n, key, s, ws_ptr<float4>(ws, L.view_pr),
                       ws_ptr<float4>(ws, L.view_vp), ws_ptr<uint32_t>(ws, L.err));
  return hipGetLastError();
}

// ------------------------------------------------------------------ host --
hipError_t launch_bin_cells(const KParams& kp, int64_t n, const sph_state& in, sph_state& out,
                            const sph_state* cin, sph_state* cout, uint32_t* key,
                            uint32_t* perm, uint32_t* cell_start, void* ws, hipStream_t st) {
  const WsLayout L = ws_layout(n);
  uint32_t* ikey = ws_ptr<uint32_t>(ws, L.keyA);
  uint32_t* rank = ws_ptr<uint32_t>(ws, L.rank);
  uint2* member = ws_ptr<uint2>(ws, L.member);
  uint32_t* xcount = ws_ptr<uint32_t>(ws, L.xcount);
  const unsigned gridn = (unsigned)((n + kBlock - 1) / kBlock);
  launch_zero_cells(cell_start, kp.ncell_total, st);
  if (n > 0)
    hipLaunchKernelGGL(k_count_cells, dim3(gridn), dim3(kBlock), 0, st, kp, n, in.pos, in.type,
                       ikey, rank, cell_start, xcount, ws_ptr<uint32_t>(ws, L.disp),
                       ws_ptr<WsHeader>(ws, L.err));
  launch_scan_cells(cell_start, kp.ncell_total, xcount, n, ws_ptr<uint32_t>(ws, L.scan_part), st);
  if (n > 0) {
    hipLaunchKernelGGL(k_place, dim3(gridn), dim3(kBlock), 0, st, n, kp.ncell_total, ikey, rank,
                       cell_start, xcount, member);
    sph_state ci{}, co{};
    const int carry = (cin && cout) ? 1 : 0;
    if (carry) {
      ci = *cin;
      co = *cout;
    }
    hipLaunchKernelGGL(k_reorder, dim3(gridn), dim3(kBlock), 0, st, kp, n, member,
                       cell_start, perm, key, in, out, ci, co, carry,
                       ws_ptr<float4>(ws, L.view_pr), ws_ptr<float4>(ws, L.view_vp),
                       ws_ptr<uint32_t>(ws, L.err));
  }
  return hipGetLastError();
}

}  // namespace sph
