// Binning of the omnidirectional rasterizer, gfx950: depth sort of the (Gaussian, view) items view
// by view, pair emission, stable LSD radix sort of the pairs by global tile, per-tile ranges.
//
// The pairs must end up ordered by the 64-bit key (global tile << 32 | depth bits), ties by
// Gaussian index.  Instead of sorting 64-bit keys over all pairs, each view's items (far fewer than
// its pairs) are first sorted by their 32-bit depth; pairs are then emitted in (view, depth) order
// and sorted stably by tile id alone.  The result is the same permutation as a stable sort of the
// 64-bit keys of index-ordered pairs, since a tile belongs to one view.
//
// Culled items leave the sort in its first pass (or the ranks' placement), so everything after it
// handles the kept items only: a view that sees a part of the scene costs that part.
//
// Radix sort: reduce-then-scan (no inter-workgroup spinning, so no forward-progress assumption):
// per-block digit histograms, exclusive scans per digit across blocks, then a stable scatter in which
// each wavefront ranks its keys by ballots over the digit's bits (multi-split).
// Every count the kernels need (kept items, pairs) is read from device memory, so the whole
// chain runs without a host round trip and can be captured in a graph.
#include "common.h"

namespace odgs {
namespace {

__device__ inline uint32_t wave_incl_scan(uint32_t x) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  return x;
}

// Inclusive scan across a block of NT threads.  `lds` holds NT / 64 words; contains two barriers.
template <int NT>
__device__ inline uint32_t block_incl_scan(uint32_t x, uint32_t* lds, uint32_t& total) {
  const uint32_t incl = wave_incl_scan(x);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  if (lane == kWave - 1) lds[w] = incl;
  __syncthreads();
  uint32_t pre = 0;
  total = 0;
#pragma unroll
  for (int k = 0; k < NT / kWave; ++k) {
    pre += (k < w) ? lds[k] : 0u;
    total += lds[k];
  }
  __syncthreads();
  return incl + pre;
}
__device__ inline uint32_t block_incl_scan256(uint32_t x, uint32_t* lds, uint32_t& total) {
  return block_incl_scan<256>(x, lds, total);
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t value, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

// A key no kept item has (a kept depth is a finite float): culled items.
constexpr uint32_t kCulledKey = 0xffffffffu;

// Keys of segment `seg` (a view's items, or the whole pair list): all n_host, or the first n_dev[seg].
__device__ inline uint32_t active_count(const uint32_t* n_dev, int seg, uint32_t n_host) {
  return n_dev ? min(n_dev[seg], n_host) : n_host;
}

// Lanes of the wavefront with the same digit of `dbits` (<= MAX) bits as this one, among those with
// `valid` set.
template <int MAX>
__device__ inline uint64_t digit_peers(uint32_t d, int dbits, bool valid) {
  uint64_t peers = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
  for (int b = 0; b < MAX; ++b) {
    if (b >= dbits) break;  // uniform
    const bool bit = (d >> b) & 1u;
    const uint64_t bb = __builtin_amdgcn_ballot_w64(bit);
    peers &= bit ? bb : ~bb;
  }
  return peers;
}

// Per-block histogram of the digit of `dbits` (<= 8) bits at `shift`: hist[block][digit], `nblocks`
// blocks per segment of `stride` keys.  Each wavefront counts into its own LDS histogram (a quarter
// of the same-address atomics).  DROP: culled keys are not counted.  AGG (for a pass over a key's
// top digit, which takes few distinct values): the lanes of a round holding the same digit are found
// by ballots over its bits and only the lowest of them adds their number, instead of one contended
// atomic per key.
template <bool DROP, bool AGG>
__global__ __launch_bounds__(kSortThreads) void radix_hist_kernel(const uint32_t* __restrict__ keys, uint32_t stride,
                                                                 const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                                 int nblocks, int shift, int dbits,
                                                                 uint32_t* __restrict__ hist) {
  const uint32_t dmask = (1u << dbits) - 1u;
  constexpr int NW = kSortThreads / kWave;
  __shared__ uint32_t h[NW][256];
  const int t = threadIdx.x, wave = t >> 6, lane = t & (kWave - 1);
  const int seg = (int)blockIdx.x / nblocks, c = (int)blockIdx.x - seg * nblocks;
  const uint32_t n = active_count(n_dev, seg, n_host);
  const uint32_t start = (uint32_t)c * (uint32_t)kSortBlockItems;
  if (start >= n) return;  // uniform: blocks past the keys are neither scanned nor scattered
  keys += (size_t)seg * stride;
#pragma unroll
  for (int w = 0; w < NW; ++w) h[w][t] = 0;
  __syncthreads();
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  uint32_t k[kSortIpt];
#pragma unroll
  for (int r = 0; r < kSortIpt; ++r)  // unconditional loads stay in flight together
    k[r] = keys[min(start + (uint32_t)(r * kSortThreads + t), n - 1)];
#pragma unroll
  for (int r = 0; r < kSortIpt; ++r) {
    const bool valid = start + (uint32_t)(r * kSortThreads + t) < n && !(DROP && k[r] == kCulledKey);
    const uint32_t d = (k[r] >> shift) & dmask;
    if constexpr (AGG) {
      const uint64_t peers = digit_peers<8>(d, dbits, valid);
      if (valid && (peers & below) == 0ull) atomicAdd(&h[wave][d], (uint32_t)__popcll(peers));
    } else {
      if (valid) atomicAdd(&h[wave][d], 1u);
    }
  }
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) sum += h[w][t];
  hist[(size_t)blockIdx.x * 256 + t] = sum;
}

// Exclusive scan of hist[block][digit] over the blocks of each segment that hold keys, in place, and
// the digit totals tot[segment][digit]: a workgroup per COLS digits (pieces of the rows) and segment,
// COLS threads along the digits and 1024 / COLS groups of consecutive blocks.
template <int COLS>
__global__ __launch_bounds__(1024) void radix_scan_kernel(uint32_t* __restrict__ hist,
                                                          const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                          int nblocks, int bins, uint32_t* __restrict__ tot) {
  constexpr int G = 1024 / COLS;
  __shared__ uint32_t s[G][COLS + 1];
  __shared__ uint32_t wtot[1024 / kWave];
  const int t = threadIdx.x, col = t % COLS, g = t / COLS, seg = (int)blockIdx.y;
  const int d = (int)blockIdx.x * COLS + col;
  const uint32_t n = active_count(n_dev, seg, n_host);
  const int rows = min(nblocks, (int)((n + (uint32_t)kSortBlockItems - 1) / (uint32_t)kSortBlockItems));
  uint32_t* h = hist + (size_t)seg * nblocks * bins + d;
  const int chunk = (rows + G - 1) / G, r0 = min(rows, g * chunk), r1 = min(rows, r0 + chunk);
  uint32_t sum = 0;
#pragma unroll 8
  for (int r = r0; r < r1; ++r) sum += h[(size_t)r * bins];
  s[g][col] = sum;
  __syncthreads();
  // exclusive prefix over the groups of each digit: G consecutive threads per digit
  {
    const int c2 = t / G, g2 = t % G, lane = t & (kWave - 1), w = t >> 6;
    const uint32_t x = s[g2][c2];
    constexpr int SPAN = G < kWave ? G : kWave;
    uint32_t incl = x;
#pragma unroll
    for (int off = 1; off < SPAN; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off);
      if ((lane % SPAN) >= off) incl += y;
    }
    if (lane == kWave - 1) wtot[w] = incl;
    __syncthreads();
    if constexpr (G > kWave) {
      for (int k = c2 * (G / kWave); k < w; ++k) incl += wtot[k];
    }
    if (g2 == G - 1) tot[(size_t)seg * bins + (int)blockIdx.x * COLS + c2] = incl;
    s[g2][c2] = incl - x;
  }
  __syncthreads();
  uint32_t run = s[g][col];
#pragma unroll 8
  for (int r = r0; r < r1; ++r) {
    const uint32_t x = h[(size_t)r * bins];
    h[(size_t)r * bins] = run;
    run += x;
  }
}

struct ScatterArgs {
  const uint32_t* kin;
  const uint32_t* vin;  // nullptr: the values are the input positions
  uint32_t* kout;
  uint32_t* vout;
  const uint32_t* n_dev;  // live keys per segment (nullptr: n_host)
  uint32_t n_host;
  uint32_t stride;  // keys from one segment to the next, in input and output
  int nblocks;      // blocks per segment
  int shift, dbits;
  const uint32_t* hist;  // [block][digit]: scanned over the blocks, or (FOLD) the counts themselves
  const uint32_t* tot;   // [segment][digit] (not with FOLD)
  uint32_t* live_out;    // first pass over items: kept keys per segment
  uint32_t* packed_out;  // last pass over items: the segments are written without gaps, their sum here
  uint2* ranges;         // single pass over tile ids: every tile's [start, end)
  int tiles;
};

// Stable scatter of one digit pass.  DROP: culled keys are left out (and the kept ones counted).
// Phase 1: each wavefront ranks its own contiguous part of the block's keys (rounds of 64 in
// input order; per round a multi-split by dbits ballots gives the rank among same-digit peers, added
// to the wavefront's running per-digit count in LDS) with no block barriers; one exclusive prefix
// over the wavefronts per digit then makes the ranks block-wide and stable.  Phase 2 places the
// keys digit-sorted in LDS; phase 3 writes them out in that order, so consecutive threads store
// consecutive addresses of each digit's output run.
// FOLD: the block sums the earlier blocks' counts of each digit itself (few blocks per segment), which
// saves the scan's launch.
//
// At small sizes the kernel is one chain of rounds per wavefront (11 us at 6,000 keys with 256 threads
// and 16 rounds; 8 us with 512 threads and eight), at large ones bound by its scattered stores: at 4M
// items of eight views a pass takes 34 us (39 us over all views at once: a view's segment is small enough
// for the stores of neighbouring blocks to meet in the caches).
template <int NT, int BINS, bool DROP, bool FOLD>
__global__ __launch_bounds__(NT) void radix_scatter_kernel(ScatterArgs a) {
  const uint32_t dmask = (1u << a.dbits) - 1u;
  constexpr int NW = NT / kWave;
  constexpr int PER_WAVE = kSortBlockItems / NW;
  constexpr int ROUNDS = PER_WAVE / kWave;
  constexpr int DPT = BINS >= NT ? BINS / NT : 1;  // consecutive digits per thread
  __shared__ uint32_t s_key[kSortBlockItems];
  __shared__ uint32_t s_val[kSortBlockItems];
  __shared__ uint16_t wh[NW][BINS];  // per-wavefront running digit counts, then local placement starts
  __shared__ uint32_t gshift[BINS];  // global start minus local start of each digit for this block
  __shared__ uint32_t lds[NW];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t >> 6;
  const int seg = (int)blockIdx.x / a.nblocks, c = (int)blockIdx.x - seg * a.nblocks;
  const uint32_t n = active_count(a.n_dev, seg, a.n_host);
  const uint32_t start = (uint32_t)c * (uint32_t)kSortBlockItems;
  uint32_t base = (uint32_t)seg * a.stride;  // first output position of the segment
  if (a.packed_out) {
    base = 0;
    for (int u = 0; u < seg; ++u) base += a.n_dev[u];  // uniform
    if (blockIdx.x == 0 && t == 0) {
      uint32_t kept = 0;
      const int segs = (int)gridDim.x / a.nblocks;
      for (int u = 0; u < segs; ++u) kept += a.n_dev[u];
      *a.packed_out = kept;
    }
  }
  if (start >= n && !(a.ranges && blockIdx.x == 0)) return;  // uniform across the block
  const uint32_t nb = start < n ? min((uint32_t)kSortBlockItems, n - start) : 0u;
  // the keys first: their latency overlaps the digit offsets below
  const size_t in0 = (size_t)seg * a.stride + start;
  uint32_t key[ROUNDS], val[ROUNDS], rank[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t li = (uint32_t)(wave * PER_WAVE + r * kWave + lane);
    const bool in = li < nb;
    key[r] = in ? a.kin[in0 + li] : 0u;
    val[r] = in ? (a.vin ? a.vin[in0 + li] : (uint32_t)(in0 + li)) : 0u;
  }
  for (int k = t; k < NW * BINS / 2; k += NT) reinterpret_cast<uint32_t*>(wh)[k] = 0;
  // global start of each digit: the digits below it in the whole segment, and its keys in earlier blocks
  uint32_t gstart[DPT], total;
  {
    uint32_t dt[DPT], sum = 0;
    if constexpr (FOLD) {
      static_assert(DPT == 1, "one digit per thread");
      const int rows = min(a.nblocks, (int)((n + (uint32_t)kSortBlockItems - 1) / (uint32_t)kSortBlockItems));
      const uint32_t* h = a.hist + (size_t)seg * a.nblocks * BINS;
      // NT / BINS groups of threads take every other (...) row each
      constexpr int G = NT / BINS;
      const int d = t % BINS, g = t / BINS;
      uint32_t pre = 0, all = 0;
#pragma unroll 8
      for (int r = g; r < rows; r += G) {
        const uint32_t x = h[(size_t)r * BINS + d];
        all += x;
        pre += r < c ? x : 0u;
      }
      if constexpr (G > 1) {  // combined in the key buffer, unused so far
        s_key[t] = pre;
        s_val[t] = all;
        __syncthreads();
        if (g == 0) {
#pragma unroll
          for (int k = 1; k < G; ++k) {
            pre += s_key[t + k * BINS];
            all += s_val[t + k * BINS];
          }
        } else {
          pre = all = 0;
        }
      }
      dt[0] = sum = all;
      gstart[0] = base + pre;
    } else {
#pragma unroll
      for (int j = 0; j < DPT; ++j) {
        const int d = t * DPT + j;
        dt[j] = d < BINS ? a.tot[(size_t)seg * BINS + d] : 0u;
        gstart[j] = base + (d < BINS && nb > 0 ? a.hist[(size_t)blockIdx.x * BINS + d] : 0u);
        sum += dt[j];
      }
    }
    uint32_t run = block_incl_scan<NT>(sum, lds, total) - sum;
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      const int d = t * DPT + j;
      if (a.ranges && blockIdx.x == 0 && d < a.tiles) a.ranges[d] = make_uint2(run, run + dt[j]);
      gstart[j] += run;
      run += dt[j];
    }
  }
  const uint32_t out_end = base + total;
  if (DROP && c == 0 && t == 0) a.live_out[seg] = total;
  if (nb == 0) return;  // uniform
  const uint64_t lanes_below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t li = (uint32_t)(wave * PER_WAVE + r * kWave + lane);
    const bool valid = li < nb && !(DROP && key[r] == kCulledKey);
    const uint32_t d = (key[r] >> a.shift) & dmask;
    const uint64_t peers = digit_peers<BINS == 256 ? 8 : 11>(d, a.dbits, valid);
    const uint32_t wr = __popcll(peers & lanes_below);
    // every lane of a peer group reads the group's running count, then its first lane advances it
    // (one wavefront's LDS operations execute in order)
    const uint32_t cnt = wh[wave][d];
    __builtin_amdgcn_wave_barrier();
    rank[r] = cnt + wr;
    if (valid && wr == 0) wh[wave][d] = (uint16_t)(cnt + (uint32_t)__popcll(peers));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // per digit: block-local start (exclusive prefix over digits of the block totals) plus the
  // wavefront's exclusive prefix, folded into one placement start per (wavefront, digit); and
  // the digit's global-minus-local shift for the write-out (one LDS read per key in each phase)
  uint32_t placed;
  {
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      const int d = t * DPT + j;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += d < BINS ? wh[w][d] : 0u;
    }
    uint32_t run = block_incl_scan<NT>(sum, lds, placed) - sum;
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      const int d = t * DPT + j;
      if (d < BINS) {
        gshift[d] = gstart[j] - run;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const uint32_t x = wh[w][d];
          wh[w][d] = (uint16_t)run;
          run += x;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t li = (uint32_t)(wave * PER_WAVE + r * kWave + lane);
    if (li < nb && !(DROP && key[r] == kCulledKey)) {
      const uint32_t d = (key[r] >> a.shift) & dmask;
      const uint32_t p = wh[wave][d] + rank[r];
      s_key[p] = key[r];
      s_val[p] = val[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortBlockItems / NT; ++r) {
    const uint32_t i = r * NT + t;
    if (i < placed) {
      const uint32_t k = s_key[i];
      const uint32_t d = (k >> a.shift) & dmask;
      const uint32_t pos = gshift[d] + i;  // unsigned wrap-around: global start + (i - local start)
      if (pos < out_end) {  // always true for a consistent histogram; keeps a corrupted one in bounds
        a.kout[pos] = k;
        a.vout[pos] = s_val[i];
      }
    }
  }
}

// Sum of the tile counts of each block of depth-sorted items.
constexpr int kScanIpt = 4;
constexpr int kScanBlockItems = 256 * kScanIpt;

// Coarse binning (16x16 tiles, every W and H a multiple of 32): an item's pairs are the 32x32
// tiles its 16x16-tile rectangle r touches, columns c0 .. c0 + nc - 1 (an unwrapped range, taken
// modulo W / 32 like r's own columns) and rows r0 .. r0 + nr - 1, each pair carrying the mask of
// the four 16x16 tiles b = 2 by + bx of its 32x32 tile that r covers.
struct CoarseRect {
  int c0, nc, r0, nr;
};

__device__ inline CoarseRect coarse_rect(const Rect& r, int ntx16) {
  CoarseRect c{0, 0, 0, 0};
  if (r.ncols == 0 || r.nrows == 0) return c;
  if (r.ncols >= ntx16) {  // every column (col0 = 0)
    c.nc = ntx16 >> 1;
  } else {
    c.c0 = r.col0 >> 1;
    c.nc = ((r.col0 + r.ncols - 1) >> 1) - c.c0 + 1;
  }
  c.r0 = r.row0 >> 1;
  c.nr = ((r.row0 + r.nrows - 1) >> 1) - c.r0 + 1;
  return c;
}

// Mask of the 16x16 tiles of 32x32 tile (column cu, unwrapped; row ru) that r covers.
__device__ inline uint32_t coarse_mask(const Rect& r, int ntx16, int cu, int ru) {
  uint32_t m = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int x = 2 * cu + (b & 1), y = 2 * ru + (b >> 1);
    const bool col = r.ncols >= ntx16 || (x >= r.col0 && x < r.col0 + r.ncols);
    const bool row = y >= r.row0 && y < r.row0 + r.nrows;
    m |= (col && row) ? (1u << b) : 0u;
  }
  return m;
}

// Key bits above the coarse tile id: the 16x16-tile mask (coarse tile ids stay below 2^27).
constexpr int kMaskShift = 28;
constexpr uint32_t kTileIdMask = (1u << kMaskShift) - 1u;

// Pairs of an item: its 16x16 (or the plan's) tiles, or the 32x32 tiles with coarse binning.
__device__ inline uint32_t item_pairs(const Rect& r, int coarse, int ntx16) {
  if (!coarse) return (uint32_t)r.ncols * (uint32_t)r.nrows;
  const CoarseRect cr = coarse_rect(r, ntx16);
  return (uint32_t)(cr.nc * cr.nr);
}

// Gathers the items' tile rectangles into (view, depth) order (the one random access of binning; the
// offset and emission passes then read them sequentially), writes each item's pair count in that
// order (scnt; 32x32 tiles with coarse binning) and reduces the counts per block.  Workgroups go to
// the eight XCDs in turn, so those of one XCD take one consecutive eighth of the items: the
// rectangles an XCD gathers are those of few views, which its own L2 holds (4M items of eight views:
// 77 -> 38 us against a gather in depth order over all views).
__global__ __launch_bounds__(256) void count_reduce_kernel(const uint32_t* __restrict__ sorted_ids,
                                                           const uint32_t* __restrict__ kept,
                                                           const Rect* __restrict__ rect, int64_t n, ViewTable vt,
                                                           int coarse, Rect* __restrict__ srect,
                                                           uint32_t* __restrict__ scnt,
                                                           uint32_t* __restrict__ block_sum) {
  __shared__ uint32_t lds[4];
  __shared__ int s_w16[ODGS_MAX_VIEWS];  // 16x16 tiles per row of each view (coarse binning)
  const uint32_t items = *kept;
  const uint32_t blocks = (items + (uint32_t)kScanBlockItems - 1) / (uint32_t)kScanBlockItems;
  const uint32_t per = (blocks + 7) / 8, b = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= per || b >= blocks) return;  // uniform
  if (threadIdx.x < vt.n_views) s_w16[threadIdx.x] = vt.W[threadIdx.x] / 16;
  __syncthreads();
  const uint32_t start = b * (uint32_t)kScanBlockItems;
  // all loads first (indices clamped into the list), so the four gathers are in flight together
  uint32_t id[kScanIpt];
  Rect r[kScanIpt];
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) id[k] = sorted_ids[min(start + k * 256 + threadIdx.x, items - 1)];  // coalesced
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) r[k] = rect[id[k]];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) {
    const uint32_t j = start + k * 256 + threadIdx.x;
    if (j < items) {
      srect[j] = r[k];
      const uint32_t c = item_pairs(r[k], coarse, coarse ? s_w16[id[k] / (uint32_t)n] : 0);  // ids are below 2^31
      scnt[j] = c;
      s += c;
    }
  }
  uint32_t total;
  block_incl_scan256(s, lds, total);
  if (threadIdx.x == 0) block_sum[b] = total;
}

// The pair total into the status record of a new pair list (no forward has composited it yet).
__device__ inline void set_pair_total(uint64_t total, int64_t capacity, odgs_status* __restrict__ status) {
  const uint32_t gen = status->bin_gen + 1u;
  status->bin_gen = gen;
  status->fwd_gen = ~gen;
  status->n_pairs = (int64_t)total;
  status->n_pairs_stored = (int32_t)((int64_t)total < capacity ? (int64_t)total : capacity);
  if ((int64_t)total > capacity) status->flags |= ODGS_STATUS_OVERFLOW;
}

// Exclusive scan of the block sums (in place, as 64-bit offsets) and the pair total.
__global__ __launch_bounds__(256) void count_top_kernel(const uint32_t* __restrict__ block_sum,
                                                        uint64_t* __restrict__ block_off,
                                                        const uint32_t* __restrict__ kept, int64_t capacity,
                                                        odgs_status* __restrict__ status) {
  constexpr int IPT = 16;  // consecutive block sums per thread and round
  const int nblocks = (int)((*kept + (uint32_t)kScanBlockItems - 1) / (uint32_t)kScanBlockItems);
  __shared__ uint64_t wtot[4];
  uint64_t carry = 0;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  for (int base = 0; base < nblocks; base += 256 * IPT) {
    const int k0 = base + (int)threadIdx.x * IPT;
    uint32_t x[IPT];
    uint64_t sum = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      x[j] = k0 + j < nblocks ? block_sum[k0 + j] : 0u;
      sum += x[j];
    }
    uint64_t incl = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint64_t y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) wtot[w] = incl;
    __syncthreads();
    uint64_t pre = 0;
    for (int q = 0; q < w; ++q) pre += wtot[q];
    const uint64_t total = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    __syncthreads();
    uint64_t run = carry + pre + incl - sum;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (k0 + j < nblocks) block_off[k0 + j] = run;
      run += x[j];
    }
    carry += total;
  }
  if (threadIdx.x == 0) set_pair_total(carry, capacity, status);
}

// First pair position of every depth-sorted item (clamped to the capacity: items starting past
// it emit nothing).  Pairs of one item are contiguous and items follow depth order, so a later
// stable sort by tile keeps (depth, index) order inside every tile.
__global__ __launch_bounds__(256) void item_offsets_kernel(const uint32_t* __restrict__ scnt,
                                                           const uint64_t* __restrict__ block_off,
                                                           const uint32_t* __restrict__ kept, int64_t capacity,
                                                           uint32_t* __restrict__ ioff) {
  __shared__ uint32_t lds[4];
  const int64_t items = *kept;
  if ((int64_t)blockIdx.x * kScanBlockItems >= items) return;  // uniform
  const int64_t start = (int64_t)blockIdx.x * kScanBlockItems;
  uint32_t cnt[kScanIpt];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) {
    const int64_t j = start + threadIdx.x * kScanIpt + k;
    cnt[k] = j < items ? scnt[j] : 0u;
    s += cnt[k];
  }
  uint32_t total;
  const uint32_t incl = block_incl_scan256(s, lds, total);
  uint64_t off = block_off[blockIdx.x] + (incl - s);
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) {
    const int64_t j = start + threadIdx.x * kScanIpt + k;
    if (j < items) ioff[j] = (uint32_t)(off < (uint64_t)capacity ? off : (uint64_t)capacity);
    off += cnt[k];
  }
}

// Small launches (sort_by_rank) take two kernels instead of the radix sort, the counts and their scans:
// fifteen launches whose length at such sizes is their start-up and their chains of dependent steps.
// The first counts, for every item, the items of its view that come before it in (depth, index) order,
// by comparing it with all of them; the second places the items by that rank.  Measured, all of the
// binning as a graph: 51 against 86 us at 1,500 Gaussians and a 256x128 view (115 before the scans were
// folded), 73 against 102 us at 8,000 and 512x256, but 113 against 103 us at 12,000: the line lies at
// 8,192.  With many views the two meet (40 views of 2,000: 204 and 202 us), at 2^28 comparisons.
constexpr int kRankThreads = 256;
constexpr int kRankKeys = 256;  // keys a workgroup compares its items with: a thread's chain of adds sets the length
constexpr int kPlaceThreads = 1024;
constexpr int kRankItems = 8192;            // Gaussians, eight per thread of the placing workgroup
constexpr int64_t kRankPairs = 1ll << 28;  // comparisons over all views

__global__ __launch_bounds__(kRankThreads) void depth_rank_kernel(const uint32_t* __restrict__ dkey, int n,
                                                                  uint32_t* __restrict__ rank) {
  __shared__ uint4 s_key[kRankKeys / 4];
  const int t = threadIdx.x, i0 = (int)blockIdx.x * kRankThreads, j0 = (int)blockIdx.y * kRankKeys, i = i0 + t;
  const uint32_t* keys = dkey + (int64_t)blockIdx.z * n;
#pragma unroll
  for (int k = 0; k < kRankKeys / kRankThreads; ++k) {
    const int j = j0 + k * kRankThreads + t;
    reinterpret_cast<uint32_t*>(s_key)[k * kRankThreads + t] = j < n ? keys[j] : kCulledKey;  // (below no limit)
  }
  const uint32_t key = i < n ? keys[i] : kCulledKey;
  __syncthreads();
  // an equal key comes before if its index does: the limit is one higher for the keys before item i
  uint32_t c[4] = {0u, 0u, 0u, 0u};
  if (j0 + kRankKeys <= i0 || j0 >= i0 + kRankThreads) {
    const uint32_t lim = j0 < i0 ? key + 1u : key;
#pragma unroll 8
    for (int k = 0; k < kRankKeys / 4; ++k) {
      const uint4 x = s_key[k];
      c[0] += x.x < lim ? 1u : 0u;
      c[1] += x.y < lim ? 1u : 0u;
      c[2] += x.z < lim ? 1u : 0u;
      c[3] += x.w < lim ? 1u : 0u;
    }
  } else {
    const int before = i - j0;
#pragma unroll 8
    for (int k = 0; k < kRankKeys / 4; ++k) {
      const uint4 x = s_key[k];
      c[0] += x.x < key + (4 * k < before ? 1u : 0u) ? 1u : 0u;
      c[1] += x.y < key + (4 * k + 1 < before ? 1u : 0u) ? 1u : 0u;
      c[2] += x.z < key + (4 * k + 2 < before ? 1u : 0u) ? 1u : 0u;
      c[3] += x.w < key + (4 * k + 3 < before ? 1u : 0u) ? 1u : 0u;
    }
  }
  const uint32_t all = (c[0] + c[1]) + (c[2] + c[3]);
  if (key != kCulledKey && all != 0) atomicAdd(&rank[(int64_t)blockIdx.z * n + i], all);
}

// One workgroup per view: its kept items in rank order behind those of the views before it (which it
// counts by reading their rectangles), with their rectangles and first pair positions.  IPT: items
// per thread (the smallest of 2, 4, 8 that holds n).  Leaves the ranks cleared.
template <int IPT>
__global__ __launch_bounds__(kPlaceThreads) void rank_place_kernel(
    const uint32_t* __restrict__ dkey, const Rect* __restrict__ rect, int n, ViewTable vt, int coarse, int64_t capacity,
    uint32_t* __restrict__ rank, uint32_t* __restrict__ sorted_ids, Rect* __restrict__ srect,
    uint32_t* __restrict__ ioff, uint32_t* __restrict__ kept_out, odgs_status* __restrict__ status) {
  constexpr int NW = kPlaceThreads / kWave;
  __shared__ uint32_t s_cnt[IPT * kPlaceThreads];  // pair counts by rank
  __shared__ uint16_t s_id[IPT * kPlaceThreads];
  __shared__ uint64_t lds64[NW][3];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t >> 6, view = (int)blockIdx.x;
  const int64_t item0 = (int64_t)view * n;
  const int w16 = vt.W[view] / 16;
  uint32_t key[IPT], rk[IPT];
  Rect rc[IPT];
#pragma unroll
  for (int r = 0; r < IPT; ++r) {
    const int64_t i = item0 + min(r * kPlaceThreads + t, n - 1);
    key[r] = dkey[i];
    rk[r] = rank[i];
    rc[r] = rect[i];
    s_cnt[r * kPlaceThreads + t] = 0;
    s_id[r * kPlaceThreads + t] = 0;
  }
  // kept items and pairs of the views before this one
  uint64_t v3[3] = {0, 0, 0};  // kept here; kept and pairs before
  for (int u = 0; u < view; ++u) {
    const int wu = vt.W[u] / 16;
#pragma unroll 4
    for (int k = t; k < n; k += kPlaceThreads) {
      const uint32_t c = item_pairs(rect[(int64_t)u * n + k], coarse, wu);
      v3[1] += c != 0 ? 1u : 0u;
      v3[2] += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < IPT; ++r) {
    const int i = r * kPlaceThreads + t;
    if (i < n && key[r] != kCulledKey) {
      ++v3[0];
      rank[item0 + i] = 0;
      if (rk[r] < (uint32_t)n) {  // always true for ranks of these keys; keeps others in bounds
        s_cnt[rk[r]] = item_pairs(rc[r], coarse, w16);
        s_id[rk[r]] = (uint16_t)i;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v3[k] += __shfl_xor(v3[k], off);
    if (lane == 0) lds64[wave][k] = v3[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    v3[k] = 0;
    for (int w = 0; w < NW; ++w) v3[k] += lds64[w][k];
  }
  const int live = (int)v3[0];
  const int64_t out0 = (int64_t)v3[1];
  // consecutive positions per thread, and a 64-bit scan of their counts
  const int ipt = (live + kPlaceThreads - 1) / kPlaceThreads, p0 = t * ipt;
  uint32_t id[IPT], cnt[IPT];
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const bool in = k < ipt && p0 + k < live;
    id[k] = in ? s_id[p0 + k] : 0u;
    cnt[k] = in ? s_cnt[p0 + k] : 0u;
    rc[k] = rect[item0 + id[k]];
    mine += cnt[k];
  }
  uint64_t incl = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint64_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  __syncthreads();
  if (lane == kWave - 1) lds64[wave][0] = incl;
  __syncthreads();
  uint64_t off = v3[2], all = v3[2];
  for (int w = 0; w < NW; ++w) {
    off += w < wave ? lds64[w][0] : 0ull;
    all += lds64[w][0];
  }
  off += incl - mine;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (k < ipt && p0 + k < live) {
      const int64_t j = out0 + p0 + k;
      sorted_ids[j] = (uint32_t)(item0 + id[k]);
      srect[j] = rc[k];
      ioff[j] = (uint32_t)(off < (uint64_t)capacity ? off : (uint64_t)capacity);
    }
    off += cnt[k];
  }
  if (view == (int)gridDim.x - 1 && t == 0) {
    *kept_out = (uint32_t)(out0 + live);
    set_pair_total(all, capacity, status);
  }
}

// Pair-parallel emission: block b writes the pairs of sort block b, [b * kSortBlockItems,
// (b + 1) * kSortBlockItems), in rounds of kEmitPairs, four consecutive pairs per thread, so
// stores are coalesced whatever the items' sizes.  Per round the block locates its items with one
// search over the item offsets, stages them in LDS, and each thread finds the item of its first
// pair by a binary search in LDS.  The block also counts the low tile digit of its pairs: the
// histogram the tile sort's first pass needs (hist[b][digit]), so that pass does not
// read the keys once more to count them.
constexpr int kEmitRun = 4;  // consecutive pairs per thread
constexpr int kEmitPairs = 256 * kEmitRun;
constexpr int kEmitRounds = kSortBlockItems / kEmitPairs;
static_assert(kEmitRounds * kEmitPairs == kSortBlockItems, "whole rounds per sort block");

// Last index in [0, n) with a[idx] <= x, for nondecreasing a with a[0] <= x, searched by one
// whole wavefront: each round probes 64 evenly spaced entries of the interval at once and keeps
// the stretch between the last probe <= x and the next one, so about four rounds of dependent
// loads cover millions of entries (a binary search takes twenty-odd).  Uniform result.
__device__ inline int64_t wave_last_le(const uint32_t* __restrict__ a, int64_t n, uint32_t x) {
  const int lane = threadIdx.x & (kWave - 1);
  int64_t lo = 0, hi = n;  // a[lo] <= x; hi == n or a[hi] > x
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t idx = lo + (int64_t)lane * step;
    const bool le = idx < hi && a[idx] <= x;  // true on a prefix of the lanes, lane 0 included
    const int k = __popcll(__builtin_amdgcn_ballot_w64(le)) - 1;
    lo += (int64_t)k * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// One round of emit_pairs_kernel: pairs [p0, p1), also counted into the wavefront's histogram.
template <bool COARSE>
__device__ inline void emit_round(const uint32_t* __restrict__ sorted_ids, const uint32_t* __restrict__ ioff,
                                  const Rect* __restrict__ srect, int64_t items, int64_t n, const ViewTable& vt,
                                  int tile, uint32_t* __restrict__ pkey, uint32_t* __restrict__ pval, uint32_t p0,
                                  uint32_t p1, uint32_t* s_off, uint32_t* s_item, Rect* s_rect, uint32_t* s_tb,
                                  uint16_t* s_ntx, const int64_t* s_range, uint32_t* hw, uint32_t dmask,
                                  const uint32_t* s_vtb, const uint16_t* s_vntx) {
  // s_range: the items holding pairs p0 and p1 - 1
  const int64_t i0 = s_range[0];
  const int m = (int)(s_range[1] - i0 + 1);  // <= kEmitPairs: every listed item owns >= 1 pair here
  // staged with every load in flight first (indices clamped into the round's items)
  constexpr int R = kEmitPairs / 256;
  uint32_t item[R], off[R];
  Rect rc[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t j = i0 + min(k * 256 + (int)threadIdx.x, m - 1);
    item[k] = sorted_ids[j];
    off[k] = ioff[j];
    rc[k] = srect[j];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int t = k * 256 + (int)threadIdx.x;
    if (t < m) {
      const uint32_t v = item[k] / (uint32_t)n;  // item ids are below 2^32
      s_off[t] = off[k];
      s_item[t] = item[k];
      s_rect[t] = rc[k];
      s_tb[t] = s_vtb[v];
      s_ntx[t] = s_vntx[v];
    }
  }
  __syncthreads();
  // each thread emits kEmitRun consecutive pairs: one search, then the rectangle is walked by
  // increments (row-major, columns wrapping at the seam), and one 16-byte store per array
  static_assert(kEmitPairs == 256 * kEmitRun && kEmitRun == 4, "four consecutive pairs per thread");
  const uint32_t q = p0 + (uint32_t)(kEmitRun * threadIdx.x);
  if (q >= p1) return;
  int lo = 0, hi = m;  // largest idx with s_off[idx] <= q
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (s_off[mid] <= q) lo = mid;
    else hi = mid;
  }
  Rect rr = s_rect[lo];
  uint32_t ntx = s_ntx[lo];
  // the rectangle walked: the item's 16x16 tiles, or the 32x32 tiles they fall in
  CoarseRect cr{(int)rr.col0, (int)rr.ncols, (int)rr.row0, (int)rr.nrows};
  if constexpr (COARSE) cr = coarse_rect(rr, (int)ntx);
  uint32_t local = q - s_off[lo];
  uint32_t r = local / (uint32_t)cr.nc, c = local - r * (uint32_t)cr.nc;
  uint32_t key[kEmitRun], val[kEmitRun];
#pragma unroll
  for (int j = 0; j < kEmitRun; ++j) {
    const uint32_t pj = q + (uint32_t)j;
    // next item once this one's pairs are used up (items without pairs here are skipped)
    while (lo + 1 < m && s_off[lo + 1] <= pj) {
      ++lo;
      rr = s_rect[lo];
      ntx = s_ntx[lo];
      cr = CoarseRect{(int)rr.col0, (int)rr.ncols, (int)rr.row0, (int)rr.nrows};
      if constexpr (COARSE) cr = coarse_rect(rr, (int)ntx);
      r = 0;
      c = 0;
    }
    const uint32_t cu = (uint32_t)cr.c0 + c;  // unwrapped column
    if constexpr (COARSE) {
      const uint32_t ntx32 = ntx >> 1;
      const uint32_t col = cu >= ntx32 ? cu - ntx32 : cu;
      key[j] = (s_tb[lo] + (uint32_t)(cr.r0 + (int)r) * ntx32 + col) |
               (coarse_mask(rr, (int)ntx, (int)cu, cr.r0 + (int)r) << kMaskShift);
    } else {
      const uint32_t col = cu >= ntx ? cu - ntx : cu;
      key[j] = s_tb[lo] + (uint32_t)(cr.r0 + (int)r) * ntx + col;
    }
    val[j] = s_item[lo];
    if (++c == (uint32_t)cr.nc) {
      c = 0;
      ++r;
    }
  }
#pragma unroll
  for (int j = 0; j < kEmitRun; ++j)
    if (q + (uint32_t)j < p1) atomicAdd(&hw[key[j] & dmask], 1u);
  if (q + kEmitRun <= p1) {
    *reinterpret_cast<uint4*>(pkey + q) = make_uint4(key[0], key[1], key[2], key[3]);
    *reinterpret_cast<uint4*>(pval + q) = make_uint4(val[0], val[1], val[2], val[3]);
  } else {
    for (int j = 0; j < kEmitRun && q + (uint32_t)j < p1; ++j) {
      pkey[q + j] = key[j];
      pval[q + j] = val[j];
    }
  }
}

template <bool COARSE, int BINS>
__global__ __launch_bounds__(256) void emit_pairs_kernel(const uint32_t* __restrict__ sorted_ids,
                                                         const uint32_t* __restrict__ ioff,
                                                         const Rect* __restrict__ srect,
                                                         const odgs_status* __restrict__ status,
                                                         const uint32_t* __restrict__ kept,
                                                         int64_t n, ViewTable vt, int tile, uint32_t* __restrict__ pkey,
                                                         uint32_t* __restrict__ pval, uint32_t* __restrict__ hist,
                                                         uint32_t dmask) {
  __shared__ uint32_t s_off[kEmitPairs + 1];
  __shared__ uint32_t s_item[kEmitPairs + 1];
  __shared__ Rect s_rect[kEmitPairs + 1];
  __shared__ uint32_t s_tb[kEmitPairs + 1];
  __shared__ uint16_t s_ntx[kEmitPairs + 1];
  __shared__ int64_t s_range[kEmitRounds][2];
  // digit counts, per wavefront when there are few digits
  constexpr int NH = BINS > 256 ? 1 : kSortThreads / kWave;
  __shared__ uint32_t h[NH][BINS];
  __shared__ uint32_t s_vtb[ODGS_MAX_VIEWS];  // per view: first global tile id (32x32 with coarse binning)
  __shared__ uint16_t s_vntx[ODGS_MAX_VIEWS];  // per view: tiles per row (16x16 with coarse binning)
  const int t = threadIdx.x;
  for (int k = t; k < NH * BINS; k += kSortThreads) (&h[0][0])[k] = 0;
  if (t < vt.n_views) {
    s_vtb[t] = (uint32_t)(COARSE ? vt.tile_base32[t] : vt.tile_base[t]);
    s_vntx[t] = (uint16_t)(vt.W[t] / tile);
  }
  const uint32_t np = (uint32_t)status->n_pairs_stored;
  const uint32_t b0 = blockIdx.x * (uint32_t)kSortBlockItems;
  if (b0 >= np) return;  // uniform: sort blocks past the pairs are neither scanned nor scattered
  const int64_t items = *kept;
  {
    // wavefront w finds the items holding the first and last pair of round w (all rounds' searches
    // at once: their dependent loads overlap)
    static_assert(kEmitRounds == kSortThreads / kWave, "one wavefront per round");
    const int w = t >> 6;
    const uint32_t p0 = b0 + (uint32_t)(w * kEmitPairs);
    if (p0 < np) {
      const uint32_t p1 = min(p0 + (uint32_t)kEmitPairs, np);
      const int64_t first = wave_last_le(ioff, items, p0);
      const int64_t last = wave_last_le(ioff, items, p1 - 1);
      if ((t & (kWave - 1)) == 0) {
        s_range[w][0] = first;
        s_range[w][1] = last;
      }
    }
  }
  for (int round = 0; round < kEmitRounds; ++round) {
    const uint32_t p0 = b0 + (uint32_t)(round * kEmitPairs);
    if (p0 >= np) break;  // uniform
    __syncthreads();  // the searches are done, the previous round's staging has been read
    emit_round<COARSE>(sorted_ids, ioff, srect, items, n, vt, tile, pkey, pval, p0,
                       min(p0 + (uint32_t)kEmitPairs, np), s_off, s_item, s_rect, s_tb, s_ntx, s_range[round],
                       h[NH > 1 ? t >> 6 : 0], dmask, s_vtb, s_vntx);
  }
  __syncthreads();
  for (int d = t; d < BINS; d += kSortThreads) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < NH; ++w) c += h[w][d];
    hist[(size_t)blockIdx.x * BINS + d] = c;
  }
}

// Tile ranges from the sorted keys: each thread scans eight consecutive keys (two 16-byte loads
// when the run is whole) and marks where a tile's run starts and ends.
constexpr int kRangeKeys = 8;

__global__ __launch_bounds__(256) void ranges_kernel(const uint32_t* __restrict__ keys,
                                                     const odgs_status* __restrict__ status, uint2* __restrict__ ranges) {
  const uint32_t n = (uint32_t)status->n_pairs_stored;
  const uint32_t j0 = (blockIdx.x * 256 + threadIdx.x) * (uint32_t)kRangeKeys;
  if (j0 >= n) return;
  uint32_t k[kRangeKeys];
  if (j0 + kRangeKeys <= n) {
    const uint4 a = *reinterpret_cast<const uint4*>(keys + j0);
    const uint4 b = *reinterpret_cast<const uint4*>(keys + j0 + 4);
    k[0] = a.x; k[1] = a.y; k[2] = a.z; k[3] = a.w;
    k[4] = b.x; k[5] = b.y; k[6] = b.z; k[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < kRangeKeys; ++i) k[i] = j0 + i < n ? keys[j0 + i] : 0u;
  }
  uint32_t prev = j0 > 0 ? keys[j0 - 1] : ~k[0];
  const uint32_t after = j0 + kRangeKeys < n ? keys[j0 + kRangeKeys] : 0u;
#pragma unroll
  for (int i = 0; i < kRangeKeys; ++i) {
    const uint32_t j = j0 + i;
    if (j < n) {
      if (prev != k[i]) ranges[k[i]].x = j;
      const bool last = j + 1 == n;
      const uint32_t next = i + 1 < kRangeKeys ? k[i + 1] : after;
      if (last || next != k[i]) ranges[k[i]].y = j + 1;
    }
    prev = k[i];
  }
}

// Refinement of the coarse lists (coarse binning): the sorted 32x32-tile list is split into the
// lists of the 16x16 tiles by the masks its keys carry.  The refined list has four regions, one per
// quadrant b of a 32x32 tile (b = 2*row + column): region b holds, in list order, every pair whose
// mask has bit b, so each 16x16 tile's list is one contiguous run in (depth, index) order.  A pair's
// position is the region's base plus the number of earlier pairs with bit b: four bit counts
// scanned over the whole list, chunk by chunk (the sort's blocks), with no per-tile work.  A chunk
// is four wavefronts of kRefineIters rounds of 64 consecutive pairs.
constexpr int kRefineWavePairs = kSortBlockItems / (kSortThreads / kWave);
constexpr int kRefineIters = kRefineWavePairs / kWave;

__device__ inline void coarse_tile_of(const ViewTable& vt, int T, int& v, int& cx, int& cy) {
  v = 0;
  while (T >= vt.tile_base32[v + 1]) ++v;
  const int ntx32 = vt.W[v] / 32, lt = T - vt.tile_base32[v];
  cx = lt % ntx32;
  cy = lt / ntx32;
}

// Per-chunk counts of the four mask bits.
__global__ __launch_bounds__(kSortThreads) void refine_count_kernel(const uint32_t* __restrict__ keys,
                                                                    const odgs_status* __restrict__ status,
                                                                    uint4* __restrict__ cnt) {
  __shared__ uint32_t wc[kSortThreads / kWave][4];
  const uint32_t n = (uint32_t)status->n_pairs_stored;
  const uint32_t base = blockIdx.x * (uint32_t)kSortBlockItems;
  if (base >= n) return;  // uniform per block
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const uint32_t wbase = base + (uint32_t)(w * kRefineWavePairs) + (uint32_t)lane;
  uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < kRefineIters; ++i) {
    const uint32_t j = wbase + (uint32_t)(i * kWave);
    const uint32_t kj = keys[min(j, n - 1)];  // unconditional loads stay in flight together
    const uint32_t m = j < n ? kj >> kMaskShift : 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) c[b] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((m >> b) & 1u));
  }
  if (lane == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) wc[w][b] = c[b];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < kSortThreads / kWave; ++q) s += wc[q][threadIdx.x];
    reinterpret_cast<uint32_t*>(cnt + blockIdx.x)[threadIdx.x] = s;
  }
}

// Exclusive scan of the chunk counts in place (one workgroup), the region bases and the coarse pair
// count into `meta` (words 0..3 and 4), and the refined pair total into the status record (the
// pair count and stored count of the 16x16 lists; overflow past the capacity as for the lists
// themselves).  When the coarse list itself overflowed, the refined count is of a truncated list:
// the pair count reported is then four times the coarse one, an upper bound of the true count (a
// coarse pair holds at most four 16x16 pairs).
__global__ __launch_bounds__(1024) void refine_scan_kernel(uint4* __restrict__ cnt, uint32_t* __restrict__ meta,
                                                           int64_t capacity, odgs_status* __restrict__ status) {
  __shared__ uint32_t wsum[1024 / kWave][4];
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t >> 6;
  const uint32_t n = (uint32_t)status->n_pairs_stored;
  const int chunks = (int)((n + (uint32_t)kSortBlockItems - 1) / (uint32_t)kSortBlockItems);
  constexpr int IPT = 4;                 // consecutive chunks per thread and round
  uint32_t carry[4] = {0u, 0u, 0u, 0u};  // each bit count is at most n < 2^31
  for (int base = 0; base < chunks; base += 1024 * IPT) {
    const int k0 = base + t * IPT;
    uint4 x[IPT];
    uint32_t s[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      x[j] = k0 + j < chunks ? cnt[k0 + j] : make_uint4(0u, 0u, 0u, 0u);
      s[0] += x[j].x;
      s[1] += x[j].y;
      s[2] += x[j].z;
      s[3] += x[j].w;
    }
    uint32_t incl[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      incl[b] = wave_incl_scan(s[b]);
      if (lane == kWave - 1) wsum[w][b] = incl[b];
    }
    __syncthreads();
    uint32_t ex[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      uint32_t pre = 0, total = 0;
      for (int q = 0; q < 1024 / kWave; ++q) {
        pre += q < w ? wsum[q][b] : 0u;
        total += wsum[q][b];
      }
      ex[b] = carry[b] + pre + incl[b] - s[b];
      carry[b] += total;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (k0 + j < chunks) cnt[k0 + j] = make_uint4(ex[0], ex[1], ex[2], ex[3]);
      ex[0] += x[j].x;
      ex[1] += x[j].y;
      ex[2] += x[j].z;
      ex[3] += x[j].w;
    }
  }
  __syncthreads();  // every thread has read the stored count
  if (t == 0) {
    int64_t r = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      meta[b] = (uint32_t)(r < capacity ? r : capacity);
      r += carry[b];
    }
    meta[4] = n;
    const bool truncated = (status->flags & ODGS_STATUS_OVERFLOW) != 0;
    status->n_pairs = truncated ? 4 * status->n_pairs : r;
    status->n_pairs_stored = (int32_t)(r < capacity ? r : capacity);
    if (r > capacity) status->flags |= ODGS_STATUS_OVERFLOW;
  }
}

// The writes: each wavefront recounts its pairs' bits before each round of 64 (ballots), so the
// pairs of one region that a round holds land in consecutive positions.  The pair that starts a
// 32x32 tile's run sets the starts of its four 16x16 tiles' ranges, the one that ends it the ends.
__global__ __launch_bounds__(kSortThreads) void refine_write_kernel(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, const uint4* __restrict__ pre,
    const uint32_t* __restrict__ meta, ViewTable vt, uint32_t capacity, uint32_t* __restrict__ out,
    uint2* __restrict__ ranges16) {
  __shared__ uint32_t wc[kSortThreads / kWave][4];
  const uint32_t n = meta[4];
  const uint32_t base = blockIdx.x * (uint32_t)kSortBlockItems;
  if (base >= n) return;  // uniform per block
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  const uint32_t wbase = base + (uint32_t)(w * kRefineWavePairs);
  uint32_t key[kRefineIters], val[kRefineIters];
  uint32_t c[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < kRefineIters; ++i) {
    const uint32_t j = wbase + (uint32_t)(i * kWave + lane);
    const uint32_t jc = min(j, n - 1);  // unconditional loads stay in flight together
    key[i] = keys[jc];
    val[i] = vals[jc];
    if (j >= n) key[i] = 0u;  // no mask bits past the list
    const uint32_t m = key[i] >> kMaskShift;
#pragma unroll
    for (int b = 0; b < 4; ++b) c[b] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((m >> b) & 1u));
  }
  if (lane == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) wc[w][b] = c[b];
  }
  __syncthreads();
  const uint4 p4 = pre[blockIdx.x];
  uint32_t run[4] = {meta[0] + p4.x, meta[1] + p4.y, meta[2] + p4.z, meta[3] + p4.w};
  for (int q = 0; q < w; ++q) {
#pragma unroll
    for (int b = 0; b < 4; ++b) run[b] += wc[q][b];
  }
  // tile of the pair before this lane's first one
  uint32_t last = wbase > 0 && wbase - 1 < n ? keys[wbase - 1] & kTileIdMask : 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < kRefineIters; ++i) {
    const uint32_t j = wbase + (uint32_t)(i * kWave + lane);
    const bool live = j < n;
    const uint32_t m = key[i] >> kMaskShift, t = key[i] & kTileIdMask;
    const uint32_t up = __shfl_up(t, 1);
    const uint32_t prev = lane == 0 ? last : up;
    // tile of the pair after this one (lane 63: the next round's first pair); none past the list
    const uint32_t down = __shfl_down(t, 1);
    const uint32_t first = i + 1 < kRefineIters ? __shfl(key[i + 1], 0) & kTileIdMask : 0u;
    uint32_t next = down;
    if (lane == kWave - 1)
      next = i + 1 < kRefineIters ? first : (j + 1 < n ? keys[j + 1] & kTileIdMask : 0xFFFFFFFFu);
    if (j + 1 >= n) next = 0xFFFFFFFFu;
    last = __shfl(t, kWave - 1);
    uint32_t g[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t bit = (m >> b) & 1u;
      const uint64_t bb = __builtin_amdgcn_ballot_w64(bit);
      g[b] = run[b] + (uint32_t)__popcll(bb & below);
      if (bit && g[b] < capacity) out[g[b]] = val[i];
      run[b] += (uint32_t)__popcll(bb);
    }
    const bool head = live && prev != t, tail = live && next != t;
    if (head || tail) {
      int v, cx, cy;
      coarse_tile_of(vt, (int)t, v, cx, cy);
      const int ntx16 = vt.W[v] / 16;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int tile16 = vt.tile_base[v] + (2 * cy + (b >> 1)) * ntx16 + 2 * cx + (b & 1);
        if (head) ranges16[tile16].x = min(g[b], capacity);
        if (tail) ranges16[tile16].y = min(g[b] + ((m >> b) & 1u), capacity);
      }
    }
  }
}

// Work queue of the compositors: every global tile id, in descending order of its list length
// (the tile's compositing cost), bucketed on a logarithmic scale with 32 buckets per octave (the
// order inside a bucket is arbitrary).  Three small launches: per-block bucket counts, one scan
// that turns them into per-(block, bucket) starts, and the scatter.
constexpr int kQueueBuckets = 1024;
constexpr int kQueueTiles = 4096;  // tiles per block of the count and scatter kernels (16 per thread)
// A list is split into quadrant tasks (for compositors that take them) when one wavefront alone would
// take long against the whole launch: when it holds at least 1 / kSplitShare of all pairs, or is one of
// the kSplitTop longest and holds half as much and kLongLen pairs; and at least kSplitLen pairs (with fewer
// than kSplitAllTiles tiles the device has wavefront slots to spare, and no list is too short).  At most split_tile_cap(tiles)
// lists are split.  Word 4 of the queue's header counts the long lists, those of 1 / kLongShare of all pairs
// and, from kSplitAllTiles tiles on, kLongLen pairs; word 6 the lists to split.
//
// An unsplit list of L pairs takes about 0.23 us L forward, a launch of P pairs at least 28 us P / 10^6, so
// a list sets the launch's length from L = P / 8200 on; a split list costs about half as much again in
// staging and culling, which is free only while wavefront slots are.  Forward / reverse us with lists
// split from 1 / 2730, 1 / 4096, 1 / 8192, 1 / 16384 of the pairs: 60k on a cube map and panoramas
// (0.57M pairs) 105 / 142, 107 / 145, 107 / 144, 107 / 147 (unsplit 214 / 306); 300k, 2048x1024, 1.8M
// pairs, forward 193, 175, 175, 175 (unsplit 219); 500k, 4096x2048, 8.4M pairs 261 / 463, 258 / 462,
// 276 / 513, 294 / 574; 500k, 8 views, 25.8M pairs 735 / 1293, 740 / 1306, 744 / 1316, 776 / 1376; 300k,
// mixed sizes, 20.8M pairs 957 / 1314, 928 / 1308, 778 / 1356.  The last one's few lists between the two
// shares are what kSplitTop is for: 772 / 1352, and 500k on 4096x2048 stays at 260 / 469.  Forward us with
// none, 32, 128 and 512 of them (reverse the same within 2%), on scenes drawn elsewise: mixed sizes, 14.9M
// pairs 831, 828, 678, 639 and 21.8M 868, 806, 798, 801; 200k on 4 of 2048x1024, 5.8M 313, 312, 312, 281; 400k
// on 4096x2048 and 6 of 1024x512, 16.6M 833, 830, 831, 586; 250k on 4096x2048, 2 of 2048x1024 and 5 of 512x256,
// 11.7M 660, 654, 662, 493; 700k on 2 of 4096x2048, 19.6M 518, 515, 512, 517.  The spherical footprint, whose
// quadrant tasks take one entry at a time, is even at all four (6.4M pairs 582, 574, 576, 577; 4.0M 433, 428,
// 429, 441; below that no list lies between the shares).  So 128 loses nowhere; 512 would gain more.
constexpr uint32_t kSplitLen = 64;
constexpr uint32_t kSplitShare = 4096;
constexpr uint32_t kSplitTop = 128;
constexpr uint32_t kLongLen = 1024;
constexpr uint32_t kLongShare = 4096;
constexpr int kSplitAllTiles = 4096;
constexpr int kSplitCapMin = 1024;
// At 32x32 tiles, whose four parts are tasks of their own anyway, word 8: the lists of at least
// 1 / kFineShare of all pairs and kLongLen pairs take their parts' quadrants as tasks in the forward.
// 250k Gaussians on 4 views of 1920x960 (2.8M pairs, lists of up to 4,661), forward us: 434 with none,
// 412, 351 and 345 from 1 / 1024, 1 / 2048 and 1 / 4096 of the pairs on (there the most a sixteenth, then an
// eighth of the tiles); one of the views 371 -> 239.  The reverse, which puts such a part's masks together
// from four runs of bits, goes 479 -> 498.  With none and with the rule, forward: 300k on 4096x2048 and 4 of
// 1024x512 900 -> 460; 60k on 6 of 1024x512 275 -> 241; 100k on 2048x1024 231 -> 213; but 400k on 8 of
// 2048x1024, where a thousand lists of 2,050 pairs and more (8.4M in all) each are staged sixteen times,
// 663 -> 751.  There the rule reaches further than it should.
constexpr uint32_t kFineShare = 4096;
constexpr int kFineCapMin = 256;

__device__ inline uint32_t cost_bucket(uint32_t len) {
  // 0 for an empty list, else 1 + 32 log2(len) (exponent and top five mantissa bits; <= 993)
  return len == 0 ? 0u : 1u + ((__float_as_uint((float)len) - 0x3f800000u) >> 18);
}

// bstart[block][bucket] = number of the block's tiles in the bucket (every entry written).
__global__ __launch_bounds__(256) void queue_count_kernel(const uint2* __restrict__ ranges, int tiles,
                                                          uint32_t* __restrict__ bstart) {
  __shared__ uint32_t h[kQueueBuckets];
  for (int b = threadIdx.x; b < kQueueBuckets; b += 256) h[b] = 0;
  __syncthreads();
  for (int k = 0; k < kQueueTiles / 256; ++k) {
    const int i = blockIdx.x * kQueueTiles + k * 256 + threadIdx.x;
    if (i < tiles) {
      const uint2 r = ranges[i];
      atomicAdd(&h[cost_bucket(r.y - r.x)], 1u);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kQueueBuckets; b += 256) bstart[(size_t)blockIdx.x * kQueueBuckets + b] = h[b];
}

// Header words 4, 6 and 8 from the scan over buckets, whose threads each name their bucket and the number
// of tiles in it or above.  (Word 4, the lists of 1 / kLongShare of the pairs and, from kSplitAllTiles tiles
// on, kLongLen, is for inspection: no kernel reads it.)  Contains a barrier; cut: two words of LDS.
__device__ inline void set_split(int bucket, uint32_t upto, uint32_t cap, bool split_all, uint32_t pairs, uint32_t* cut,
                                 uint32_t* __restrict__ header) {
  const uint32_t floor = split_all ? 1u : kSplitLen;
  if (bucket == (int)cost_bucket(max(split_all ? 1u : kLongLen, pairs / kLongShare))) header[4] = min(upto, cap);
  if (bucket == (int)cost_bucket(max(floor, pairs / kSplitShare))) cut[0] = upto;
  if (bucket == (int)cost_bucket(max(kLongLen, pairs / kFineShare))) header[8] = upto;
  if (bucket == (int)cost_bucket(max(kLongLen, pairs / (2 * kSplitShare)))) cut[1] = min(upto, kSplitTop);
  __syncthreads();
  if (threadIdx.x == 0) header[6] = min(max(cut[0], cut[1]), cap);
}

// Buckets in descending order, blocks in order: the counts become each (block, bucket)'s first
// queue position.  One workgroup; also clears the persistent launches' counters and records the
// numbers of long lists and of lists to split (set_split).
__global__ __launch_bounds__(kQueueBuckets) void queue_scan_kernel(uint32_t* __restrict__ bstart, int nblocks,
                                                                   uint32_t* __restrict__ ctr, uint32_t split_cap,
                                                                   bool split_all,
                                                                   const uint32_t* __restrict__ n_pairs) {
  __shared__ uint32_t wsum[kQueueBuckets / kWave], cut[2];
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t >> 6;
  const int bucket = kQueueBuckets - 1 - t;
  if (t < 4) ctr[t] = 0u;
  uint32_t c = 0;
  for (int b = 0; b < nblocks; ++b) c += bstart[(size_t)b * kQueueBuckets + bucket];
  const uint32_t incl = wave_incl_scan(c);
  if (lane == kWave - 1) wsum[w] = incl;
  __syncthreads();
  uint32_t run = incl - c;
  for (int k = 0; k < w; ++k) run += wsum[k];
  // tiles in this bucket or above: the first run + c queue entries
  set_split(bucket, run + c, split_cap, split_all, *n_pairs, cut, ctr);
  for (int b = 0; b < nblocks; ++b) {
    uint32_t* e = bstart + (size_t)b * kQueueBuckets + bucket;
    const uint32_t x = *e;
    *e = run;
    run += x;
  }
}

__global__ __launch_bounds__(256) void queue_scatter_kernel(const uint2* __restrict__ ranges, int tiles,
                                                            const uint32_t* __restrict__ bstart,
                                                            uint32_t* __restrict__ order) {
  __shared__ uint32_t cur[kQueueBuckets];
  for (int b = threadIdx.x; b < kQueueBuckets; b += 256) cur[b] = bstart[(size_t)blockIdx.x * kQueueBuckets + b];
  __syncthreads();
  for (int k = 0; k < kQueueTiles / 256; ++k) {
    const int i = blockIdx.x * kQueueTiles + k * 256 + threadIdx.x;
    if (i < tiles) {
      const uint2 r = ranges[i];
      order[atomicAdd(&cur[cost_bucket(r.y - r.x)], 1u)] = (uint32_t)i;
    }
  }
}

// The same queue of at most kQueueSmallTiles tiles by one workgroup (8,192 tiles: 7 us against 17 for the
// three launches; at 65,536 one workgroup takes 57 us against 23).
constexpr int kQueueSmallTiles = 8192;

__global__ __launch_bounds__(kQueueBuckets) void queue_small_kernel(const uint2* __restrict__ ranges, int tiles,
                                                                    uint32_t* __restrict__ queue, uint32_t split_cap,
                                                                    bool split_all,
                                                                    const uint32_t* __restrict__ n_pairs) {
  constexpr int TPT = kQueueSmallTiles / kQueueBuckets;
  __shared__ uint32_t h[kQueueBuckets];
  __shared__ uint32_t lds[kQueueBuckets / kWave], cut[2];
  const int t = threadIdx.x;
  h[t] = 0;
  if (t < 4) queue[t] = 0u;
  uint32_t b[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const uint2 r = ranges[min(k * kQueueBuckets + t, tiles - 1)];
    b[k] = cost_bucket(r.y - r.x);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < TPT; ++k)
    if (k * kQueueBuckets + t < tiles) atomicAdd(&h[b[k]], 1u);
  __syncthreads();
  const int bucket = kQueueBuckets - 1 - t;
  const uint32_t c = h[bucket];
  uint32_t total;
  const uint32_t incl = block_incl_scan<kQueueBuckets>(c, lds, total);
  set_split(bucket, incl, split_cap, split_all, *n_pairs, cut, queue);
  h[bucket] = incl - c;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const int i = k * kQueueBuckets + t;
    if (i < tiles) queue[16 + atomicAdd(&h[b[k]], 1u)] = (uint32_t)i;
  }
}

hipError_t launch_tile_queue(const uint2* ranges, int tiles, const uint32_t* n_pairs, uint32_t* bstart,
                             uint32_t* queue, hipStream_t st) {
  if (tiles <= kQueueSmallTiles) {
    hipLaunchKernelGGL(queue_small_kernel, dim3(1), dim3(kQueueBuckets), 0, st, ranges, tiles, queue,
                       (uint32_t)split_tile_cap(tiles), tiles < kSplitAllTiles, n_pairs);
    return hipGetLastError();
  }
  const int nb = (tiles + kQueueTiles - 1) / kQueueTiles;
  if (nb > 0) hipLaunchKernelGGL(queue_count_kernel, dim3(nb), dim3(256), 0, st, ranges, tiles, bstart);
  hipLaunchKernelGGL(queue_scan_kernel, dim3(1), dim3(kQueueBuckets), 0, st, bstart, nb, queue,
                     (uint32_t)split_tile_cap(tiles), tiles < kSplitAllTiles, n_pairs);
  if (nb > 0) hipLaunchKernelGGL(queue_scatter_kernel, dim3(nb), dim3(256), 0, st, ranges, tiles, bstart, queue + 16);
  return hipGetLastError();
}

__global__ void status_reset_kernel(odgs_status* st) {
  if (threadIdx.x == 0) {
    st->flags = 0;
    st->n_pairs_stored = 0;
    st->n_pairs = 0;
    st->n_visible = 0;
    st->n_culled = 0;
    st->n_nonfinite = 0;
    st->fwd_gen = ~st->bin_gen;  // bin_gen survives resets
  }
}

// Digit width of each pass over `bits` key bits: as many passes as 8-bit digits would take, the
// bits spread evenly over them (14 bits: two 7-bit passes, whose scatters write runs twice as long
// as an 8-bit digit's).
int sort_digit_bits(int bits) {
  const int passes = (bits + 7) / 8;
  return (bits + passes - 1) / passes;
}

// Threads of a scatter's workgroup, and the blocks per segment up to which its blocks sum the digit
// counts of earlier blocks themselves instead of leaving that to a scan launch.
constexpr int kScatterThreads = 512;
constexpr int kFoldBlocks = 32;

template <bool DROP>
void launch_scatter(const ScatterArgs& a, int segs, hipStream_t st) {
  const dim3 grid((unsigned)(segs * a.nblocks));
  if (a.nblocks <= kFoldBlocks)
    hipLaunchKernelGGL((radix_scatter_kernel<kScatterThreads, 256, DROP, true>), grid, dim3(kScatterThreads), 0, st, a);
  else
    hipLaunchKernelGGL((radix_scatter_kernel<kScatterThreads, 256, DROP, false>), grid, dim3(kScatterThreads), 0, st, a);
}

// (many rows: narrower pieces of them, for more workgroups)
void launch_scan(const ScatterArgs& a, int segs, int bins, uint32_t* hist, uint32_t* tot, hipStream_t st) {
  if (a.nblocks > 512)
    hipLaunchKernelGGL(radix_scan_kernel<8>, dim3((unsigned)bins / 8, (unsigned)segs), dim3(1024), 0, st, hist, a.n_dev,
                       a.n_host, a.nblocks, bins, tot);
  else
    hipLaunchKernelGGL(radix_scan_kernel<32>, dim3((unsigned)bins / 32, (unsigned)segs), dim3(1024), 0, st, hist, a.n_dev,
                       a.n_host, a.nblocks, bins, tot);
}

// One digit pass: the histogram unless it is there already, its scan unless the scatter folds it, the
// scatter.
template <bool DROP>
void radix_pass(ScatterArgs a, int segs, bool have_hist, bool top, uint32_t* hist, uint32_t* tot, hipStream_t st) {
  const dim3 grid((unsigned)(segs * a.nblocks));
  if (!have_hist) {
    if (top)  // the top digit: few distinct values
      hipLaunchKernelGGL((radix_hist_kernel<DROP, true>), grid, dim3(kSortThreads), 0, st, a.kin, a.stride, a.n_dev,
                         a.n_host, a.nblocks, a.shift, a.dbits, hist);
    else
      hipLaunchKernelGGL((radix_hist_kernel<DROP, false>), grid, dim3(kSortThreads), 0, st, a.kin, a.stride, a.n_dev,
                         a.n_host, a.nblocks, a.shift, a.dbits, hist);
  }
  if (a.nblocks > kFoldBlocks) launch_scan(a, segs, 256, hist, tot, st);
  a.hist = hist;
  a.tot = tot;
  launch_scatter<DROP>(a, segs, st);
}

}  // namespace

int sort_passes(int bits) { return (bits + 7) / 8; }

// Pairs of up to 2^kWideBits tiles are sorted by one pass over the whole id, whose digit totals are
// the tile ranges (1,953 tiles, 200k pairs: 12 + 5 us against 2 x 13 for two scatters, 2 x 4.7 for their
// scans, 6 for the second histogram and 4 for the ranges); above, the histogram rows (and with more
// sort blocks their number) outgrow what the second pass costs.
constexpr int kWideBits = 11;
constexpr int kWideBlocks = 1024;
bool sort_wide(int bits, int pair_blocks) { return bits > 8 && bits <= kWideBits && pair_blocks <= kWideBlocks; }
size_t sort_hist_words(int64_t item_rows, int64_t pair_blocks, bool wide) {
  return (size_t)std::max<int64_t>(256 * item_rows, (wide ? 1 << kWideBits : 256) * pair_blocks);
}
// (the digit totals per view, or of the tile digits; then the kept items per view and in all)
size_t sort_tot_words(int32_t n_views) { return std::max<size_t>(256 * (size_t)n_views, 1 << kWideBits); }


bool sort_by_rank(const odgs_plan* p) { return p->n <= kRankItems && p->items * p->n <= kRankPairs; }
uint32_t* item_ranks(const odgs_plan* p, void* ws) { return ws_ptr<uint32_t>(ws, p->off_did[p->depth_final ^ 1]); }

hipError_t launch_status_reset(const odgs_plan* p, void* ws, hipStream_t st) {
  hipLaunchKernelGGL(status_reset_kernel, dim3(1), dim3(64), 0, st, ws_ptr<odgs_status>(ws, p->off_status));
  return hipGetLastError();
}

TileSched make_sched(const odgs_plan* p, void* ws, int which) {
  uint32_t* q = ws_ptr<uint32_t>(ws, p->off_queue);
  TileSched s{};
  s.status = ws_ptr<odgs_status>(ws, p->off_status);
  s.tiles = p->tile_base[p->n_views];
  s.order = (p->s.flags & ODGS_FLAG_SCHED_TILE_ID) ? nullptr : q + 16;  // after 64 bytes of counters
  s.ctr = (p->s.flags & ODGS_FLAG_SCHED_PERSISTENT) ? q + 2 * which : nullptr;
  s.split = q + 4;
  s.split_cap = 0;
  s.split_all = 0;
  s.fine_cap = 0;
  return s;
}

// A launch holds fewer than 2^32 threads, so fewer than 2^26 tasks of a wavefront each: with four per tile
// counted, what is left of them bounds the tiles that may take twelve more (from 12.2M tiles on).
int fine_tile_cap(int tiles) {
  const int64_t room = ((int64_t(1) << 26) - 1 - 4 * (int64_t)tiles) / 12;
  return (int)std::min<int64_t>(std::min(tiles, std::max(kFineCapMin, tiles / 8)), std::max<int64_t>(room, 0));
}
int split_tile_cap(int tiles) { return tiles < kSplitCapMin ? tiles : std::max(kSplitCapMin, tiles / 8); }

int sched_grid(const TileSched& s, int per_cu) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 1;
  const int64_t g = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
  return (int)(g < sched_tasks(s) ? g : sched_tasks(s));
}

hipError_t launch_fill_u32(uint32_t* ptr, uint32_t value, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ptr, value, n);
  return hipGetLastError();
}

hipError_t launch_bin_sort(const odgs_plan* p, void* ws, hipStream_t st) {
  odgs_status* status = ws_ptr<odgs_status>(ws, p->off_status);
  const int64_t items = p->items;
  uint32_t* hist = ws_ptr<uint32_t>(ws, p->off_hist);
  uint32_t* tot = ws_ptr<uint32_t>(ws, p->off_digit);
  uint32_t* live = tot + sort_tot_words(p->n_views);  // kept items per view
  uint32_t* kept = live + ODGS_MAX_VIEWS;             // and in all
  uint2* ranges = ws_ptr<uint2>(ws, p->off_ranges);
  const int tiles = p->tile_base[p->n_views];
  const bool coarse = p->coarse != 0;
  const int bits = coarse ? p->coarse_bits : p->tile_bits;
  const bool wide = !coarse && sort_wide(bits, p->pair_blocks);
  if (!wide || items == 0) {  // (the wide pass writes every tile's range)
    const hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(ranges), 0u, 2 * (int64_t)tiles, st);
    if (e != hipSuccess) return e;
  }
  uint32_t* queue = ws_ptr<uint32_t>(ws, p->off_queue);
  const uint32_t* n_dev = reinterpret_cast<const uint32_t*>(&status->n_pairs_stored);
  if (items == 0) return launch_tile_queue(ranges, tiles, n_dev, hist, queue, st);
  uint32_t* dk[2] = {ws_ptr<uint32_t>(ws, p->off_dkey[0]), ws_ptr<uint32_t>(ws, p->off_dkey[1])};
  uint32_t* di[2] = {ws_ptr<uint32_t>(ws, p->off_did[0]), ws_ptr<uint32_t>(ws, p->off_did[1])};
  const uint32_t* sorted_ids = di[p->depth_final];
  Rect* srect = ws_ptr<Rect>(ws, p->off_srect);
  uint32_t* ioff = dk[p->depth_final ^ 1];  // first pair positions (a free buffer by then)
  const Rect* rect = ws_ptr<Rect>(ws, p->off_rect);
  const ViewTable vt = make_view_table(p);
  if (sort_by_rank(p)) {
    // 1., 2. ranks (cleared by the preprocess) and placement
    uint32_t* rank = item_ranks(p, ws);
    const int n = (int)p->n;
    hipLaunchKernelGGL(depth_rank_kernel, dim3((n + kRankThreads - 1) / kRankThreads, (n + kRankKeys - 1) / kRankKeys,
                                              (unsigned)p->n_views),
                       dim3(kRankThreads), 0, st, dk[0], n, rank);
#define ODGS_PLACE(IPT)                                                                                              \
  hipLaunchKernelGGL(rank_place_kernel<IPT>, dim3((unsigned)p->n_views), dim3(kPlaceThreads), 0, st, dk[0], rect, n,   \
                     vt, coarse ? 1 : 0, p->pair_capacity, rank, di[p->depth_final], srect, ioff, kept, status)
    if (n <= 2 * kPlaceThreads)
      ODGS_PLACE(2);
    else if (n <= 4 * kPlaceThreads)
      ODGS_PLACE(4);
    else
      ODGS_PLACE(8);
#undef ODGS_PLACE
  } else {
    // 1. each view's items by depth; the first pass drops the culled ones, the last one closes the
    //    gaps between the views
    for (int pass = 0; pass < 4; ++pass) {
      ScatterArgs a{};
      a.kin = dk[pass & 1];
      a.vin = pass == 0 ? nullptr : di[pass & 1];
      a.kout = dk[(pass & 1) ^ 1];
      a.vout = di[(pass & 1) ^ 1];
      a.n_dev = pass == 0 ? nullptr : live;
      a.n_host = (uint32_t)p->n;
      a.stride = (uint32_t)p->n;
      a.nblocks = (int)((p->n + kSortBlockItems - 1) / kSortBlockItems);
      a.shift = 8 * pass;
      a.dbits = 8;
      a.live_out = live;
      a.packed_out = pass == 3 ? kept : nullptr;
      if (pass == 0)
        radix_pass<true>(a, p->n_views, false, false, hist, tot, st);
      else
        radix_pass<false>(a, p->n_views, false, pass == 3, hist, tot, st);
    }
    // 2. pair counts and offsets in (view, depth) order, and P
    const int sblocks = (int)((items + kScanBlockItems - 1) / kScanBlockItems);
    uint32_t* bsum = ws_ptr<uint32_t>(ws, p->off_blocksum);
    uint64_t* boff = reinterpret_cast<uint64_t*>(bsum + align_up((size_t)sblocks, 64));
    uint32_t* scnt = di[p->depth_final ^ 1];  // per-item pair counts (free id buffer)
    hipLaunchKernelGGL(count_reduce_kernel, dim3((unsigned)align_up((size_t)sblocks, 8)), dim3(256), 0, st, sorted_ids,
                       kept, rect, p->n, vt, coarse ? 1 : 0, srect, scnt, bsum);
    hipLaunchKernelGGL(count_top_kernel, dim3(1), dim3(256), 0, st, bsum, boff, kept, p->pair_capacity, status);
    hipLaunchKernelGGL(item_offsets_kernel, dim3(sblocks), dim3(256), 0, st, scnt, boff, kept, p->pair_capacity, ioff);
  }
  // 3. emit pairs
  uint32_t* pk[2] = {ws_ptr<uint32_t>(ws, p->off_pkey[0]), ws_ptr<uint32_t>(ws, p->off_pkey[1])};
  uint32_t* pv[2] = {ws_ptr<uint32_t>(ws, p->off_pval[0]), ws_ptr<uint32_t>(ws, p->off_pval[1])};
  const int dw = wide ? bits : sort_digit_bits(bits);  // the first tile pass's digit
#define ODGS_EMIT(C, BINS)                                                                                         \
  hipLaunchKernelGGL((emit_pairs_kernel<C, BINS>), dim3((unsigned)p->pair_blocks), dim3(kSortThreads), 0, st,        \
                     sorted_ids, ioff, srect, status, kept, p->n, vt, p->s.tile, pk[0], pv[0], hist, (1u << dw) - 1u)
  if (coarse)
    ODGS_EMIT(true, 256);
  else if (wide)
    ODGS_EMIT(false, 1 << kWideBits);
  else
    ODGS_EMIT(false, 256);
#undef ODGS_EMIT
  // 4. stable sort of the pairs by global tile (the first pass's histogram counted by the emission)
  int sorted = 0;  // the buffer pair holding the sorted list
  for (int shift = 0; shift < bits; shift += dw, sorted ^= 1) {
    ScatterArgs a{};
    a.kin = pk[sorted];
    a.vin = pv[sorted];
    a.kout = pk[sorted ^ 1];
    a.vout = pv[sorted ^ 1];
    a.n_dev = n_dev;
    a.n_host = (uint32_t)p->pair_capacity;
    a.nblocks = p->pair_blocks;
    a.shift = shift;
    a.dbits = std::min(dw, bits - shift);
    if (wide) {
      launch_scan(a, 1, 1 << kWideBits, hist, tot, st);
      a.hist = hist;
      a.tot = tot;
      a.ranges = ranges;
      a.tiles = tiles;
      hipLaunchKernelGGL((radix_scatter_kernel<kScatterThreads, 1 << kWideBits, false, false>),
                         dim3((unsigned)p->pair_blocks), dim3(kScatterThreads), 0, st, a);
    } else {
      radix_pass<false>(a, 1, shift == 0, shift + dw >= bits, hist, tot, st);
    }
  }
  if (!coarse) {
    // 5. tile ranges
    if (!wide)
      hipLaunchKernelGGL(ranges_kernel, dim3((unsigned)((p->pair_capacity + 256 * kRangeKeys - 1) / (256 * kRangeKeys))),
                         dim3(256), 0, st, pk[sorted], status, ranges);
  } else {
    // 5. the 32x32 tiles' list split into the 16x16 tiles' lists and ranges, in the other pair
    //    buffer (scratch: the free radix histograms)
    uint4* cnt = reinterpret_cast<uint4*>(hist);  // per chunk (sort block)
    uint32_t* meta = hist + align_up((size_t)p->pair_blocks * 4, 64);
    const unsigned cgrid = (unsigned)p->pair_blocks;
    hipLaunchKernelGGL(refine_count_kernel, dim3(cgrid), dim3(kSortThreads), 0, st, pk[sorted], status, cnt);
    hipLaunchKernelGGL(refine_scan_kernel, dim3(1), dim3(1024), 0, st, cnt, meta, p->pair_capacity, status);
    hipLaunchKernelGGL(refine_write_kernel, dim3(cgrid), dim3(kSortThreads), 0, st, pk[sorted], pv[sorted], cnt, meta,
                       vt, (uint32_t)p->pair_capacity, pv[sorted ^ 1], ranges);
  }
  // 6. the compositors' work queue, longest list first (its scratch: the free radix histograms)
  return launch_tile_queue(ranges, tiles, n_dev, hist, queue, st);
}

}  // namespace odgs
