// The binning of coarse grids: cell keys, a stable LSD radix sort in LDS, cell
// ranges and the reorder.
//
// The counting sort (sph_bin.hip) ranks each particle among the members of its
// cell, at the cell's population squared, and counts cells with atomics, which
// collide where the cells are few.  With the usual cells, of about one particle
// to a few tens, both are small; a coarse grid (coarse_cells) takes the radix
// sort, whose cost does not depend on the population.  Same keys, permutation and
// ranges.
#include "sph_dev.h"
#include "sph_kernels.h"
#include "sph_slots.h"

namespace sph {

constexpr int kSortItems = 8;  // keys per thread of a tile
constexpr int kSortTile = kBlock * kSortItems;

// The keys by input index.  (A kernel of its own: with the first digit's counts,
// eight keys a thread, too few wavefronts wait for the positions.  A new binning
// also restarts the record of the largest displacement.)
__global__ __launch_bounds__(kBlock) void k_cell_keys(
    KParams kp, int64_t n, const double* __restrict__ pos, const uint8_t* __restrict__ type,
    uint32_t* __restrict__ key, uint32_t* __restrict__ disp, WsHeader* __restrict__ hdr) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  if (i == 0) {
    for (int k = 0; k < kDispSlots; ++k) disp[k] = 0u;
    hdr->bin_gen = hdr->bin_gen + 1u;
    hdr->one_lane = 0u;
  }
  key[i] = cell_key_local(kp, pos, type, n, i);
}

__global__ __launch_bounds__(kBlock) void k_batch_cell_keys(
    const SlotEntry* __restrict__ tab, int ns, int64_t n, const double* __restrict__ pos,
    const uint8_t* __restrict__ type, uint32_t* __restrict__ key, SlotAccum* __restrict__ acc,
    uint32_t* __restrict__ disp) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < (int64_t)ns * kAccCopies) acc[i] = SlotAccum{0u, 0u, 0u, 0u, 0ull, 0ull};
  if (i < (int64_t)ns * kDispSlots) disp[i] = 0u;
  if (i >= n) return;
  const int s = find_slot(tab, ns, i);
  key[i] = tab[s].cbase + cell_key_local(tab[s].kp, pos, type, n, i);
}

// The counts of digit (key >> shift) & (2^bits - 1) of the block's tile, to column
// blockIdx.x of hist (one row of nblk entries per digit).
__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint32_t* __restrict__ keys,
                                                       int64_t n, int64_t nblk, int shift,
                                                       int bits, uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  const int bins = 1 << bits;
  for (int b = threadIdx.x; b < bins; b += kBlock) h[b] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  const uint32_t mask = (uint32_t)bins - 1u;
  for (int r = 0; r < kSortItems; ++r) {
    const int64_t i = base + r * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & mask], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += kBlock) hist[(int64_t)b * nblk + blockIdx.x] = h[b];
}

// Exclusive prefix sum of one value per thread over the block (and their total).
__device__ inline uint32_t block_prefix(uint32_t v, uint32_t* total) {
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

// Scan of kScanTile counts per block; the tiles' totals go to part.
__global__ __launch_bounds__(kBlock) void k_tile_scan(uint32_t* __restrict__ data, int64_t len,
                                                      uint32_t* __restrict__ part) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  uint32_t v[kScanItems], s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < len ? data[base + k] : 0u;
    s += v[k];
  }
  uint32_t total;
  uint32_t run = block_prefix(s, &total);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < len) data[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Scatter of one pass over digit (key >> shift) & (2^bits - 1), bits <= 8; offs
// holds the first position of each digit of each tile, or, with part, that
// position within its scan tile, whose totals part holds (at most kFusedParts: each
// block adds them up itself, a launch less than a whole scan).  Wave w of a block owns
// keys [w*512, (w+1)*512) of the block's tile (8 rounds of 64); a wave ranks the
// keys of a round among themselves with ballots (lanes holding the same digit, in
// lane order) and keeps a running count per digit in its own LDS row, so each key
// gets its position within the wave's digit run without block barriers.  The
// tile is then sorted by digit in LDS (digit-major, then wave, then position) and
// written out from there, so that consecutive threads store consecutive addresses
// of a digit's run.  Tile order is wave-major, round, lane -- the input order -- so
// the pass is stable.  vin null: the values are the entries' own indices.
constexpr int kFusedParts = 2 * kBlock;

__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n, int shift, int bits,
    const uint32_t* __restrict__ offs, int64_t nblk, const uint32_t* __restrict__ part,
    int64_t parts) {
  __shared__ uint32_t pp[kFusedParts];
  if (part) {
    const int64_t p0 = 2 * (int64_t)threadIdx.x;
    const uint32_t v0 = p0 < parts ? part[p0] : 0u;
    const uint32_t v1 = p0 + 1 < parts ? part[p0 + 1] : 0u;
    const uint32_t ex = block_prefix(v0 + v1, nullptr);
    pp[p0] = ex;
    pp[p0 + 1] = ex + v0;
  }
  __shared__ uint32_t wrun[kBlock / 64][256];  // per-wave digit counts, then local bases
  __shared__ uint32_t dstart[256];             // first local position of each digit
  __shared__ uint32_t gbase[256];              // global position of each digit's run
  __shared__ uint32_t sk[kSortTile], sv[kSortTile];
  const int bins = 1 << bits;
  const uint32_t mask = (uint32_t)bins - 1u;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  for (int b = lane; b < 256; b += 64) wrun[wave][b] = 0;
  const int64_t tile0 = (int64_t)blockIdx.x * kSortTile;
  const int64_t base = tile0 + (int64_t)wave * (64 * kSortItems);
  uint32_t kk[kSortItems], vv[kSortItems], pos[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const int64_t i = base + r * 64 + lane;
    const bool valid = i < n;
    const uint32_t key = valid ? kin[i] : 0u;
    const uint32_t d = (key >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __ballot(valid && bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(peers & lt);
    const uint32_t prior = wrun[wave][d];
    pos[r] = prior + rank;
    // the first lane of each digit group advances the wave's running count
    // (this wave's reads of the round came first, in program order)
    if (valid && rank == 0) wrun[wave][d] = prior + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();  // (the next round's reads come after)
    kk[r] = key;
    vv[r] = valid ? (vin ? vin[i] : (uint32_t)i) : 0u;
  }
  __syncthreads();
  // digit totals of the tile, their exclusive scan, and the per-wave bases
  const int b = threadIdx.x;  // one digit per thread (bins <= kBlock)
  uint32_t tot = 0;
  if (b < bins)
    for (int w = 0; w < kBlock / 64; ++w) tot += wrun[w][b];
  const uint32_t ds = block_prefix(b < bins ? tot : 0u, nullptr);
  if (b < bins) {
    dstart[b] = ds;
    const int64_t o = (int64_t)b * nblk + blockIdx.x;
    gbase[b] = offs[o] + (part ? pp[o / kScanTile] : 0u);
    uint32_t s = ds;
    for (int w = 0; w < kBlock / 64; ++w) {
      const uint32_t c = wrun[w][b];
      wrun[w][b] = s;
      s += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    if (base + r * 64 + lane < n) {
      const uint32_t lp = wrun[wave][(kk[r] >> shift) & mask] + pos[r];
      sk[lp] = kk[r];
      sv[lp] = vv[r];
    }
  }
  __syncthreads();
  const int64_t cnt = n - tile0 < kSortTile ? n - tile0 : kSortTile;
  for (int p = threadIdx.x; p < cnt; p += kBlock) {
    const uint32_t key = sk[p];
    const uint32_t d = (key >> shift) & mask;
    const uint32_t dst = gbase[d] + ((uint32_t)p - dstart[d]);
    kout[dst] = key;
    vout[dst] = sv[p];
  }
}

// cell_start[c] = first sorted index whose key is >= c (lower bound), for
// c = 0..last.  A block takes kCsCells consecutive cells: two of its waves find
// the lower bounds of its first cell and of the next block's first cell in the
// whole key array by a 64-ary search (each round probes 64 evenly spaced keys of
// the current range; the probes below the target, a prefix, narrow it to one gap
// between probes), and each cell's lower bound is then found within that range.
constexpr int kCsCells = 2048;

__global__ __launch_bounds__(kBlock) void k_cell_start(const uint32_t* __restrict__ key,
                                                       int64_t n, uint32_t last,
                                                       uint32_t* __restrict__ start) {
  __shared__ int64_t bound[2];
  const int64_t c0 = (int64_t)blockIdx.x * kCsCells;
  const int64_t c1 = c0 + kCsCells < (int64_t)last + 1 ? c0 + kCsCells : (int64_t)last + 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (wave < 2) {
    const int64_t c = wave == 0 ? c0 : c1;
    int64_t lo = 0, hi = n;
    while (hi > lo) {
      const int64_t step = (hi - lo + 63) / 64;
      const int64_t p = lo + (int64_t)lane * step;
      const bool below = p < hi && (int64_t)key[p] < c;
      const int64_t cnt = __popcll(__ballot(below));
      const int64_t pc = lo + cnt * step;
      const int64_t nlo = cnt == 0 ? lo : lo + (cnt - 1) * step + 1;
      hi = pc < hi ? pc : hi;
      lo = nlo;
    }
    if (lane == 0) bound[wave] = lo;
  }
  __syncthreads();
  for (int64_t c = c0 + threadIdx.x; c < c1; c += kBlock) {
    int64_t lo = bound[0], hi = bound[1];
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((int64_t)key[mid] < c) lo = mid + 1;
      else hi = mid;
    }
    start[c] = (uint32_t)lo;
  }
}

__global__ __launch_bounds__(kBlock) void k_reorder_sorted(
    KParams kp, int64_t n, const uint32_t* __restrict__ perm, const uint32_t* __restrict__ key,
    sph_state in, sph_state out, sph_state cin, sph_state cout, int carry,
    float4* __restrict__ pr, float4* __restrict__ vp, uint32_t* __restrict__ err) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  if (reorder_one(kp, n, i, perm[i], key[i], in, out, cin, cout, carry, pr, vp))
    set_error(err, SPH_ERR_EXCLUDED);
}

__global__ __launch_bounds__(kBlock) void k_batch_reorder_sorted(
    const SlotEntry* __restrict__ tab, int ns, int64_t n, const uint32_t* __restrict__ perm,
    const uint32_t* __restrict__ key, sph_state in, sph_state out, sph_state cin, sph_state cout,
    int carry, float4* __restrict__ pr, float4* __restrict__ vp, uint32_t* __restrict__ err,
    uint32_t* __restrict__ slot_err) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int s = find_slot(tab, ns, i);  // (every slot keeps its particle range)
  if (reorder_one(tab[s].kp, n, i, perm[i], key[i] - tab[s].cbase, in, out, cin, cout, carry, pr,
                  vp)) {
    set_error(err, SPH_ERR_EXCLUDED);
    set_error(&slot_err[s], SPH_ERR_EXCLUDED);
  }
}

// ------------------------------------------------------------------ host --
// The stable sort of the n keys 0..last in the workspace's keyA region: sorted keys
// to `key`, the permutation to `perm`, the ranges to cell_start (last + 1 entries).
// The workspace's sort regions hold two sets of keys and values; the counts are kept
// where the views will be written (256 words per 2048 particles and one, less than
// the views of any case of at least kCoarseMinN).
static void radix_sort_cells(int64_t n, uint32_t last, uint32_t* key, uint32_t* perm,
                             uint32_t* cell_start, const WsLayout& L, void* ws,
                             hipStream_t st) {
  uint32_t* kA = ws_ptr<uint32_t>(ws, L.keyA);
  uint32_t* vA = ws_ptr<uint32_t>(ws, L.rank);
  uint32_t* kB = ws_ptr<uint32_t>(ws, L.member);
  uint32_t* vB = kB + n;
  uint32_t* hist = ws_ptr<uint32_t>(ws, L.view_pr);
  uint32_t* part = ws_ptr<uint32_t>(ws, L.scan_part);
  const int64_t nblk = (n + kSortTile - 1) / kSortTile;
  int total_bits = 1;  // enough for keys 0..last
  while (total_bits < 32 && ((uint64_t)1 << total_bits) <= (uint64_t)last) ++total_bits;
  const int passes = (total_bits + 7) / 8;
  const int per = (total_bits + passes - 1) / passes;
  const uint32_t* ksrc = kA;
  const uint32_t* vsrc = nullptr;  // the input order on the first pass
  for (int p = 0; p < passes; ++p) {
    const int shift = p * per;
    const int bits = shift + per <= total_bits ? per : total_bits - shift;
    uint32_t* kdst = p == passes - 1 ? key : (p & 1) ? kA : kB;
    uint32_t* vdst = p == passes - 1 ? perm : (p & 1) ? vA : vB;
    hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nblk), dim3(kBlock), 0, st, ksrc, n, nblk,
                       shift, bits, hist);
    const int64_t parts = ((nblk << bits) + kScanTile - 1) / kScanTile;
    const bool fused = parts <= kFusedParts;
    if (fused)
      hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)parts), dim3(kBlock), 0, st, hist,
                         nblk << bits, part);
    else
      launch_scan_cells(hist, nblk << bits, ws_ptr<uint32_t>(ws, L.xcount), 0, part, st);
    hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)nblk), dim3(kBlock), 0, st, ksrc, vsrc,
                       kdst, vdst, n, shift, bits, hist, nblk, fused ? part : nullptr, parts);
    ksrc = kdst;
    vsrc = vdst;
  }
  hipLaunchKernelGGL(k_cell_start, dim3((unsigned)(((int64_t)last + kCsCells) / kCsCells)),
                     dim3(kBlock), 0, st, key, n, last, cell_start);
}

hipError_t launch_bin_cells_radix(const KParams& kp, int64_t n, const sph_state& in,
                                  sph_state& out, const sph_state* cin, sph_state* cout,
                                  uint32_t* key, uint32_t* perm, uint32_t* cell_start, void* ws,
                                  hipStream_t st) {
  const WsLayout L = ws_layout(n);
  const unsigned grid = (unsigned)((n + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_cell_keys, dim3(grid), dim3(kBlock), 0, st, kp, n, in.pos, in.type,
                     ws_ptr<uint32_t>(ws, L.keyA), ws_ptr<uint32_t>(ws, L.disp),
                     ws_ptr<WsHeader>(ws, L.err));
  radix_sort_cells(n, kp.ncell_total, key, perm, cell_start, L, ws, st);
  const int carry = cin && cout ? 1 : 0;
  hipLaunchKernelGGL(k_reorder_sorted, dim3(grid), dim3(kBlock), 0, st, kp, n, perm, key, in, out,
                     carry ? *cin : sph_state{}, carry ? *cout : sph_state{}, carry,
                     ws_ptr<float4>(ws, L.view_pr), ws_ptr<float4>(ws, L.view_vp),
                     ws_ptr<uint32_t>(ws, L.err));
  return hipGetLastError();
}

hipError_t launch_batch_bin_cells_radix(const BatchDesc& B, const sph_state& in, sph_state& out,
                                        const sph_state* cin, sph_state* cout, uint32_t* key,
                                        uint32_t* perm, uint32_t* cell_start, void* ws,
                                        hipStream_t st) {
  const int64_t n = B.n_total;
  const BatchWsLayout W = batch_ws_layout(B.n_slots, n);
  const SlotEntry* tab = (const SlotEntry*)B.table;
  const int64_t nd = (int64_t)B.n_slots * (kDispSlots > kAccCopies ? kDispSlots : kAccCopies);
  const int64_t nk = n > nd ? n : nd;
  hipLaunchKernelGGL(k_batch_cell_keys, dim3((unsigned)((nk + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, st, tab, B.n_slots, n, in.pos, in.type,
                     ws_ptr<uint32_t>(ws, W.base.keyA), ws_ptr<SlotAccum>(ws, W.accum),
                     ws_ptr<uint32_t>(ws, W.disp));
  radix_sort_cells(n, (uint32_t)B.key_cells, key, perm, cell_start, W.base, ws, st);
  const int carry = cin && cout ? 1 : 0;
  hipLaunchKernelGGL(k_batch_reorder_sorted, dim3((unsigned)((n + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, st, tab, B.n_slots, n, perm, key, in, out,
                     carry ? *cin : sph_state{}, carry ? *cout : sph_state{}, carry,
                     ws_ptr<float4>(ws, W.base.view_pr), ws_ptr<float4>(ws, W.base.view_vp),
                     ws_ptr<uint32_t>(ws, W.base.err), ws_ptr<uint32_t>(ws, W.slot_err));
  return hipGetLastError();
}

}  // namespace sph
