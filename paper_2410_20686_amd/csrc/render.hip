// Compositing kernels of the omnidirectional rasterizer, gfx950.
//
// Pixels are grouped in 8x8 quadrants.  At tiles of 16 and 32 one 64-wide wavefront composites a
// 16x16 block, four pixels per lane (lane l holds pixel (l % 8, l / 8) of each quadrant): a whole
// 16x16 tile, one quadrant of a split tile, or one of the four blocks of a 32x32 tile (the tasks
// of TileSched).  At tiles of 8, and in the counting variants of the forward, one
// workgroup per (view, tile) with one pixel per lane, each wavefront owning one quadrant.  The
// tile's depth-ordered list is staged through LDS in batches; while the forward stages, each
// record gets a bit mask of the quadrants its footprint can reach, so a quadrant skips, with a
// uniform branch, every Gaussian that cannot reach any of its pixels.  (The mask is conservative: a
// skipped Gaussian has alpha < 1/255 at every pixel of the quadrant, so results are identical to
// testing every pixel.)  The forward stores the masks per list position and the backward loads
// them.
//
// Forward: front-to-back compositing (Eq. gaussian2d, Eq. alphablending) until a pixel's
// transmittance would drop below 1e-4; the workgroup stops loading batches once every pixel is
// done.  Backward: back to front from the last contributor, transmittance recovered by
// multiplying with 1/(1 - alpha); the nine per-pixel gradients of the 2D quantities are summed
// over each 16-lane row by a DPP butterfly that leaves one value per lane, over the four rows by
// the row-swap permutes, kept per wavefront in LDS, and reach global memory with one double atomic
// per (Gaussian, tile, quantity), so the totals do not depend on the order in which tiles finish.
// One launch covers all views of a step: the grid spans the global tile ids of every view.
#include <type_traits>
#include <utility>

#include "common.h"
#include "wave.h"

namespace odgs {
namespace {

constexpr float kAlphaMax = 0.99f;
constexpr float kTStop = 1e-4f;

// Nine per-lane values can be summed over each 16-lane row in four DPP exchange steps (pairs (i, 15-i),
// (i, 7-i), (i, 3-i), (i, i^1) inside the row).  Values 0..7 are transposed (each step halves the
// slots a lane holds: value index = lane bits 3,2,1 read as 4*b3 + 2*b2 + b1 on even lanes); value
// 8 is summed in place through the first three steps and takes the odd lanes in the last one.
// Lane i ends with the row sum of value kRowSlot[i % 16] (none where the table says 15; value 8,
// held by all eight odd lanes, is assigned to lane 1 only).  The kernels take the first two steps
// (quad_reduce9) and leave the last two to LDS; the table of all four is modelled by a host test.
constexpr uint64_t kRowSlot = 0xF7F6F5F4F3F2F180ull;  // nibble i = value index held by row lane i

// Sum of a value over the eight lanes of an aligned 8-lane group (every lane gets the sum).
__device__ inline float group8_sum(float x) {
  x += dpp_read<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp_read<0x4E>(x);   // quad_perm [2,3,0,1]
  return x + dpp_read<0x141>(x);  // row_half_mirror: the other quad of the 8-lane group
}

// Wavefront sum of one value, in every lane.
__device__ inline float wave_sum(float x) {
  x = group8_sum(x);
  x += dpp_read<0x140>(x);  // row_mirror: the other half of the 16-lane row
  return sum_rows(x);
}

// Nine per-lane values summed over the wavefront with most of the data movement in LDS.
// Values 0..7 go value-major into the wavefront's scratch red[8][kRedStride]; lane 8j+m later
// reads entries 8m..8m+7 of value j, adds them, and an 8-lane DPP sum completes the total
// (held by lane 8j).  The reads are issued one accepted entry later, so their latency overlaps
// that entry's arithmetic; value 8 is summed with DPP directly.  LDS executes one wavefront's
// operations in order, so only compiler reordering across the wave barriers must be prevented.
constexpr int kRedStride = 68;  // padded rows (16-byte aligned)

__device__ inline void red_write(float (&red)[8][kRedStride], const float (&g)[9], int lane) {
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int q = 0; q < 8; ++q) red[q][lane] = g[q];
  __builtin_amdgcn_wave_barrier();
}

__device__ inline void red_read(const float (&red)[8][kRedStride], int lane, float4& r0, float4& r1) {
  __builtin_amdgcn_wave_barrier();
  const int j = lane >> 3, m = lane & 7;
  r0 = *reinterpret_cast<const float4*>(&red[j][8 * m]);
  r1 = *reinterpret_cast<const float4*>(&red[j][8 * m + 4]);
  __builtin_amdgcn_wave_barrier();
}

__device__ inline float red_finish(const float4& r0, const float4& r1) {
  return group8_sum(((r0.x + r0.y) + (r0.z + r0.w)) + ((r1.x + r1.y) + (r1.z + r1.w)));
}

// The first two of the exchange steps above (quad_reduce9) fold pairs of values with DPP adds whose bank masks write one
// value's sum into half of the lanes and the other value's into the other half: two 4-cycle adds
// per pair, where a select per side and an add took about eleven (measured on the VALU: DPP add 4.1
// cycles per wavefront, select 2.8 to 4.2, plain add 2.5).  They sit in one block in an order that
// keeps two instructions between a write and a DPP read of it, as the hardware asks for.  They
// leave g[0], g[1] and g[8]: bank b (lanes 4b .. 4b + 3) of a row holds four partial sums of value
// 4 (b / 2) + 2 (b % 2) in g[0], of the next value in g[1], and of value 8 (every bank alike) in g[8].
__device__ inline void quad_reduce9(float (&g)[9]) {
  asm("s_nop 1\n"
      "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %3, %3, %3 row_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %4, %4, %4 row_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %0, %5, %5 row_mirror row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %1, %6, %6 row_mirror row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %2, %7, %7 row_mirror row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %3, %8, %8 row_mirror row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %4, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      : "+&v"(g[0]), "+&v"(g[1]), "+&v"(g[2]), "+&v"(g[3]), "+&v"(g[8])
      : "v"(g[4]), "v"(g[5]), "v"(g[6]), "v"(g[7]));
}

// Minimum over the rectangle [x0, x1] x [y0, y1] of f(x, y) = a x^2 + 2 b x y + c y^2 (positive
// definite), with nba = -b/a and nbc = -b/c precomputed.  f is convex with its minimum at the origin,
// so its minimum over the rectangle lies on the vertical edge nearest to the origin or on the
// horizontal one (a coordinate whose range holds 0 takes 0: with both, the origin itself).  Float;
// callers add a margin that covers its rounding.
__device__ inline float rect_min_quadratic(float a, float b, float c, float nba, float nbc, float x0, float x1,
                                           float y0, float y1) {
  const float xc = __builtin_amdgcn_fmed3f(0.0f, x0, x1), yc = __builtin_amdgcn_fmed3f(0.0f, y0, y1);
  const float y = __builtin_amdgcn_fmed3f(nbc * xc, y0, y1);  // best y on the vertical edge
  const float x = __builtin_amdgcn_fmed3f(nba * yc, x0, x1);  // best x on the horizontal edge
  const float b2 = 2.0f * b;
  return fminf(fmaf(a * xc, xc, y * fmaf(b2, xc, c * y)), fmaf(a * x, x, yc * fmaf(b2, x, c * yc)));
}

// Quadrants (8x8 pixel blocks) of a tile that can hold a pixel where the Gaussian reaches
// alpha >= 1/255.  First the padded rectangle u +- eu, v +- ev; then, for quadrants that pass,
// the minimum of the exponent's quadratic form over the quadrant's pixel-centre rectangle.  The
// margin exceeds, tenfold or more, both the compositor's float evaluation error of the exponent
// (rounding of products and of du, dv) and the rounding of this test, so no contributing pixel
// is ever skipped.  Quadrants whose horizontal span reaches the +-W/2 wrap point keep the
// rectangle test only.
template <int TILE>
__device__ inline uint32_t quadrant_mask(const Rec& r, int tx0, int ty0, float Wf, float half) {
  constexpr int QPR = TILE / 8;
  const float u = r.r0.x, v = r.r0.y, eu = r.r1.w, ev = r.r2.w;
  // inverse covariance [[a, b], [b, c]] = 2 L^T L of the stored factor
  const float l0 = r.r0.z, l1 = r.r0.w, l2 = r.r1.x;
  const float a = 2.0f * l0 * l0, b = 2.0f * l0 * l1, c = 2.0f * fmaf(l1, l1, l2 * l2);
  const float nba = -b * __builtin_amdgcn_rcpf(a), nbc = -b * __builtin_amdgcn_rcpf(c);
  const float aa = fabsf(a), ab = fabsf(b), ac = fabsf(c);
  const float k2 = -2.0f * r.r1.z;
  const bool all_cols = eu + 3.5f >= half;
  // Offsets of the quadrants' centres (one per column and per row of quadrants), and the margin at
  // the farthest pixel centre of the tile, which covers every quadrant's.
  float du[QPR], dy[QPR], xmax = 0.0f, ymax = 0.0f;
#pragma unroll
  for (int k = 0; k < QPR; ++k) {
    du[k] = (float)(tx0 + 8 * k + 4) - u;
    du[k] = du[k] >= half ? du[k] - Wf : (du[k] < -half ? du[k] + Wf : du[k]);
    dy[k] = (float)(ty0 + 8 * k + 4) - v;
    xmax = fmaxf(xmax, fabsf(du[k]));
    ymax = fmaxf(ymax, fabsf(dy[k]));
  }
  const float X = xmax + 3.5f, Y = ymax + 3.5f;
  const float tmax = fmaf(aa * X, X, Y * fmaf(2.0f * ab, X, ac * Y));
  const float gmax = 2.0f * fmaf(aa + ab, X, (ab + ac) * Y);
  const float lim = k2 + fmaf(1e-5f, tmax, fmaf(1e-2f, gmax, fmaf(1e-4f, k2, 1e-6f)));
  uint32_t mask = 0;
#pragma unroll
  for (int q = 0; q < QPR * QPR; ++q) {
    const float dx = du[q % QPR], dv = dy[q / QPR];
    const bool rect = fabsf(dv) <= ev + 3.5f && (all_cols || fabsf(dx) <= eu + 3.5f);
    const bool near = !(fabsf(dx) + 4.0f < half) ||
                      rect_min_quadratic(a, b, c, nba, nbc, dx - 3.5f, dx + 3.5f, dv - 3.5f, dv + 3.5f) <= lim;
    mask |= (rect & near) ? (1u << q) : 0u;
  }
  return mask;
}

// Horizontal offset wrapped into [-W/2, W/2) without branches.
__device__ inline float wrap_du(float du, float Wf, float half) {
  du = du >= half ? du - Wf : du;
  return du < -half ? du + Wf : du;
}

// Stage `cnt` records of a tile list into LDS (entry e <- list position first + dir * e) and
// build, for every wavefront (one per 8x8 quadrant, one pixel per lane), the order-preserving
// list of entries whose footprint reaches its pixels.  Counts per list are returned in nq[]
// (identical in every thread).
template <int TILE, int BATCH>
struct Stage {
  static constexpr int N = TILE * TILE;  // threads
  static constexpr int NQ = (TILE / 8) * (TILE / 8);  // lists = wavefronts
  static constexpr int NW = N / kWave;
  static_assert(NQ == NW, "one list per wavefront");
  float4 s0[BATCH];
  float4 s1[BATCH];
  float4 s2[BATCH];
  uint32_t sid[BATCH];
  float dep[BATCH];  // sort depths (staged only for the expected-depth output)
  uint8_t list[NQ][BATCH];
  uint32_t wcnt[NW][NQ];  // per-wavefront counts, then (in place) exclusive prefix over wavefronts
  uint32_t tot[NQ];
};

// The culling masks travel from the forward to the backward: the forward stores, per list position,
// the quadrants of the reverse compositor's task in which some of its pixels reached the entry (see
// s_used; narrower than the footprint's) into the pair buffer the sort leaves unused, and the
// backward loads them instead of evaluating the footprint again: one byte per position, in byte
// planes at 16x16 blocks (the task's plane, see task_block).  The mask is written after the forward
// walks each batch.  The backward reads only list positions before its tile's last contributor,
// all of which the forward staged.
enum QuadMaskMode { kMaskEval = 0, kMaskLoad = 2 };

// Returns whether the seam wrap is the identity for every staged entry (uniform).
template <int TILE, int BATCH, int QM = kMaskEval>
__device__ inline bool stage_batch(Stage<TILE, BATCH>& S, const uint32_t* __restrict__ pair_items,
                                   const Rec* __restrict__ rec, uint32_t first, int dir, int cnt, int tx0, int ty0,
                                   float Wf, float half, int (&nq)[Stage<TILE, BATCH>::NQ],
                                   const float* __restrict__ depth = nullptr,
                                   const uint8_t* __restrict__ qmask_in = nullptr) {
  using St = Stage<TILE, BATCH>;
  const int t = threadIdx.x, ln = t & (kWave - 1), wv = t >> 6;
  const uint64_t below = ln == 0 ? 0ull : (~0ull >> (kWave - ln));
#pragma unroll
  for (int q = 0; q < St::NQ; ++q) nq[q] = 0;
  bool nowrap = true, all_nowrap = true;
  for (int r0 = 0; r0 < cnt; r0 += St::N) {
    const int e = r0 + t;
    uint32_t m = 0;
    if (e < cnt) {
      const uint32_t pos = first + dir * e;
      const uint32_t item = pair_items[pos];
      const Rec r = rec[item];
      S.s0[e] = r.r0;
      // the fourth word (the half extent, needed only for the mask below) carries whether every
      // pixel centre of the tile lies within W/2 - 1 of u: the seam wrap is then the identity
      const float reach = fabsf((float)tx0 + 0.5f * (float)TILE - r.r0.x) + 0.5f * (float)TILE + 1.0f;
      nowrap = nowrap && reach < half;
      // staged as (l2, p_min, opacity, no-wrap flag): the accept test reads its two words with one
      // 8-byte LDS load at an immediate offset
      S.s1[e] = make_float4(r.r1.x, r.r1.z, r.r1.y, reach < half ? 1.0f : 0.0f);
      S.s2[e] = r.r2;
      S.sid[e] = item;
      if (depth) S.dep[e] = depth[item];
      if constexpr (QM == kMaskLoad) {
        m = qmask_in[pos];
      } else {
        m = quadrant_mask<TILE>(r, tx0, ty0, Wf, half);
      }
    }
    uint32_t within[St::NQ];
#pragma unroll
    for (int q = 0; q < St::NQ; ++q) {
      const uint64_t bq = __builtin_amdgcn_ballot_w64((m >> q) & 1u);
      within[q] = __popcll(bq & below);
      if (ln == 0) S.wcnt[wv][q] = __popcll(bq);
    }
    __syncthreads();
    if constexpr (St::NW > 1) {
      // thread q turns list q's per-wavefront counts into exclusive prefixes
      if (t < St::NQ) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < St::NW; ++w) {
          const uint32_t c = S.wcnt[w][t];
          S.wcnt[w][t] = run;
          run += c;
        }
        S.tot[t] = run;
      }
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < St::NQ; ++q) {
      const int pre = St::NW > 1 ? (int)S.wcnt[wv][q] : 0;
      const int tot = St::NW > 1 ? (int)S.tot[q] : (int)S.wcnt[0][q];
      if ((m >> q) & 1u) S.list[q][nq[q] + pre + (int)within[q]] = (uint8_t)e;
      nq[q] += tot;
    }
    all_nowrap = __syncthreads_and(nowrap) != 0;
  }
  return all_nowrap;
}

// COUNT: also record the per-pixel work counters read by odgs_debug_pixel_counts (a separate
// instantiation, so the production forward carries no counting instructions).
// DEPTH: also write the alpha-weighted sort depth sum_j alpha_j T_j d_j of every pixel.
template <int TILE, int BATCH, bool COUNT, bool DEPTH>
__global__ __launch_bounds__(TILE* TILE) void render_fwd_kernel(
    ViewTable vt, const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_items, const Rec* __restrict__ rec,
    float* __restrict__ out_rgb, float* __restrict__ out_T, float* __restrict__ ws_T, int32_t* __restrict__ ws_last,
    int32_t* __restrict__ ws_ncontrib, int32_t* __restrict__ ws_neval, int32_t* __restrict__ ws_lasteval, float bg0,
    float bg1, float bg2, const float* __restrict__ depth, float* __restrict__ out_depth, uint8_t* __restrict__ qmask,
    int64_t qplane, TileSched sc) {
  using St = Stage<TILE, BATCH>;
  constexpr int N = St::N;
  __shared__ St S;
  // s_used[q][e]: some still-compositing pixel of quadrant q reaches entry e of the batch being
  // walked.  For list positions before a pixel's last contributor, that test here and the
  // backward's are the same float decision, so these quadrants include every one whose pixels the
  // backward must visit the entry for (and little else); that mask, in the backward's
  // granularity, is what the backward loads.
  __shared__ uint8_t s_used[St::NQ][BATCH];
  mark_forward(sc);
  __shared__ uint32_t s_claim;
  uint32_t round = 0;
  for (int g; (g = claim_tile(sc, round, &s_claim)) >= 0;) {
    const int v = view_of_tile(vt, g);
    const int W = vt.W[v], H = vt.H[v];
    const int ntx = W / TILE;
    const int lt = g - vt.tile_base[v];
    const int tx0 = (lt % ntx) * TILE, ty0 = (lt / ntx) * TILE;
    int lx, ly;
    local_pixel<TILE>(threadIdx.x, lx, ly);
    const int x = tx0 + lx, y = ty0 + ly;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // this wavefront's quadrant (uniform)
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    const float Wf = (float)W, half = wrap_half(vt, v);  // no seam in pinhole views
    const uint2 rg = ranges[g];
    float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f;
    int last = 0, ncontrib = 0, nev = 0, lastev = 0;
    // 0 while the pixel composites, NaN once it has stopped: added to the exponent's sum of squares
    // it makes the accept compare itself false for every later Gaussian (with 0 the sum is the same
    // float), so the wavefront's ballots are of single compares
    float qstop = 0.0f;
    // writes the masks of the batch walked last (after a barrier) and clears s_used for the next
    auto flush_used = [&](uint32_t first, int n_walked) {
      for (int e = threadIdx.x; e < BATCH; e += N) {
        if (e < n_walked) {
          uint32_t mq = 0;
#pragma unroll
          for (int q = 0; q < St::NQ; ++q) mq |= s_used[q][e] ? (1u << q) : 0u;
          if constexpr (TILE >= 32) {
            // the reverse compositor takes each 16x16 block b = 2 by + bx of a 32x32 tile as a
            // task: its four quadrants' bits go to byte plane b
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const int q0 = 8 * (b >> 1) + 2 * (b & 1);  // quadrant (2 bx, 2 by) of the 4x4 grid
              qmask[(int64_t)b * qplane + first + e] =
                  (uint8_t)(((mq >> q0) & 3u) | (((mq >> (q0 + 4)) & 3u) << 2));
            }
          } else {
            qmask[first + e] = (uint8_t)mq;
          }
        }
#pragma unroll
        for (int q = 0; q < St::NQ; ++q) s_used[q][e] = 0;
      }
    };
    uint32_t walked_base = 0;
    int walked_cnt = 0;
    for (uint32_t base = rg.x; base < rg.y; base += BATCH) {
      const bool all_done = __syncthreads_count(!(qstop == 0.0f)) == N;
      flush_used(walked_base, walked_cnt);
      walked_cnt = 0;
      if (all_done) break;
      const int cnt = (int)min((uint32_t)BATCH, rg.y - base);
      int nq[St::NQ];
      const bool nowrap =
          stage_batch<TILE, BATCH>(S, pair_items, rec, base, 1, cnt, tx0, ty0, Wf, half, nq, DEPTH ? depth : nullptr);
      const int n = __builtin_amdgcn_readfirstlane(nq[wq]);
      // one list walk, instantiated without the seam wrap for batches where it is the identity
      auto walk = [&](auto wrapc) {
      for (int i = 0; i < n; ++i) {
        if (__builtin_amdgcn_ballot_w64(qstop == 0.0f) == 0ull) break;  // uniform: every pixel has finished
        const int k = S.list[wq][i];
        const float4 a = S.s0[k];
        const float4 b = S.s1[k];
        const float du = decltype(wrapc)::value ? wrap_du(px - a.x, Wf, half) : px - a.x;
        const float dv = py - a.y;
        const float t1 = fmaf(a.z, du, a.w * dv), t2 = b.x * dv;
        const float power = -fmaf(t1, t1, fmaf(t2, t2, qstop));
        if (COUNT) nev += qstop == 0.0f ? 1 : 0;
        // alpha >= 1/255 (power <= 0 always: a sum of squares; NaN once stopped)
        const bool ok = power >= b.y;
        if (__builtin_amdgcn_ballot_w64(ok) == 0ull) continue;  // uniform
        // some pixel of this quadrant reaches the entry (it is accepted there unless that pixel
        // stops at it, in which case the backward does not need it for that pixel: a superset)
        s_used[wq][k] = 1;
        const float alpha = fminf(b.z * __expf(power), kAlphaMax);
        const float Tn = T * (1.0f - alpha);
        const bool acc = ok && !(Tn < kTStop);
        qstop = ok != acc ? __builtin_nanf("") : qstop;  // stop: reached, but T would drop below 1e-4
        const float4 c = S.s2[k];
        const float w = (acc ? alpha : 0.0f) * T;  // (a select of the product compiles to a branch here)
        C0 = fmaf(w, c.x, C0);
        C1 = fmaf(w, c.y, C1);
        C2 = fmaf(w, c.z, C2);
        if (DEPTH) D = D + w * S.dep[k];
        T = acc ? Tn : T;
        last = acc ? (int)(base - rg.x) + k + 1 : last;
        if (COUNT) {
          lastev = acc ? nev : lastev;
          ncontrib += acc ? 1 : 0;
        }

      }
      };
      if (nowrap)
        walk(std::false_type{});
      else
        walk(std::true_type{});
      walked_base = base;
      walked_cnt = cnt;
    }
    __syncthreads();
    flush_used(walked_base, walked_cnt);
    const int64_t plane = (int64_t)W * H;
    const int64_t pix = (int64_t)y * W + x;
    float* img = out_rgb + 3 * vt.pix_base[v];
    img[pix] = fmaf(T, bg0, C0);
    img[plane + pix] = fmaf(T, bg1, C1);
    img[2 * plane + pix] = fmaf(T, bg2, C2);
    const int64_t gp = vt.pix_base[v] + pix;
    ws_T[gp] = T;
    ws_last[gp] = last;
    if (COUNT) {
      ws_ncontrib[gp] = ncontrib;
      ws_neval[gp] = nev;
      ws_lasteval[gp] = lastev;
    }
    if (DEPTH) out_depth[gp] = D;
    if (out_T) out_T[gp] = T;
  }
}

// Forward compositing of a 16x16 tile by one wavefront, four pixels per lane (lane l holds pixel
// (l % 8, l / 8) of each quadrant): the tile's list is staged once with each entry's quadrant mask
// (the footprint test of the one-pixel forward), and an entry is evaluated only for the quadrants
// it can reach and whose pixels still composite.  The quadrants in which some pixel reached an
// entry are handed to the backward as in the one-pixel forward.  A quadrant task of a split tile
// (see TileSched) runs the same code with its one quadrant selected, and hands its masks over in
// the byte plane of its quadrant (plane q at byte offset q * qplane; whole tiles use plane 0).
//
// Bound by VALU issue; at 500k Gaussians, 8 views of 2048x1024 it went 808 -> 730 us when the stop
// and clamp handling moved behind branches that are rarely taken (the accepted step: 58 instead of 66
// issue cycles), the list words and the quadrants used went into registers instead of LDS, and the
// footprint test took the two edges that face the centre instead of all four.
// The 16x16 pixel block a task composites: its origin (bx0, by0), its quadrants (`sel`, updated)
// and the byte plane of its culling masks.  BIN = 16: the tile, or one quadrant of a split tile
// (plane q); BIN = 32: part p of the tile, the 16x16 block p = 2 by + bx, with all four quadrants or, of
// a tile in sixteen tasks, one (plane p: four runs of bits in the bytes of the tile's list, see quadrant_masks).
template <int BIN>
__device__ inline void task_block(const ViewTable& vt, int v, int g, uint32_t& sel, int& bx0, int& by0, int& plane) {
  const int ntx = vt.W[v] / BIN;
  const int lt = g - vt.tile_base[v];
  bx0 = (lt % ntx) * BIN;
  by0 = (lt / ntx) * BIN;
  plane = sel == 0xFu ? 0 : __builtin_ctz(sel & 0xFu);
  if constexpr (BIN == 32) {
    bx0 += 16 * (plane & 1);
    by0 += 16 * (plane >> 1);
    sel = sel >> 4 != 0u ? sel >> 4 : 0xFu;
  } else {
    static_assert(BIN == 16, "blocks of 16x16 pixels in tiles of 16 or 32");
  }
}

template <int BATCH>
struct FwdStage4 {  // (one entry more for composite_quadrant)
  float4 s0[BATCH + 1];  // u, v, l0, l1
  float4 s1[BATCH + 1];  // l2, p_min, opacity, sort depth (with the depth output)
  float4 s2[BATCH + 1];  // r, g, b, unused
  uint16_t list[BATCH];  // entry index | quadrant mask << 8 | flags << 12
  uint8_t used[BATCH];
};

using vec4 = float __attribute__((ext_vector_type(4)));  // (kept in registers across a loop)

// `x`, the same in every lane, in a scalar register; and the number of `mask`'s bits below this lane.
__device__ inline float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
__device__ inline int bits_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Bit j if `mask` has a bit, in a scalar register.
__device__ inline int bit_if(uint64_t mask, int j) {
  int x;
  asm("s_cmp_lg_u64 %1, 0\n\ts_cselect_b32 %0, %2, 0" : "=s"(x) : "s"(mask), "s"(1 << j) : "scc");
  return x;
}

// Zero, formed where it is used: no register holds it before.
__device__ inline float zero_here() {
  float x;
  asm volatile("v_mov_b32 %0, 0" : "=v"(x));
  return x;
}

__device__ inline vec4 as_vec4(const float4& f) { return vec4{f.x, f.y, f.z, f.w}; }

// One quadrant of a split tile, one pixel per lane.  A split tile's list is long against the launch, so
// what counts is the time one wavefront takes per entry: it issues an instruction every four to five
// cycles whatever the rest of the device does.  kQuadRun entries are evaluated together: their records
// are read from LDS at once (the asm statements keep the compiler from waiting for each in turn), the
// stop test is one per run, wrap and clamp are one branch per run, the entries reached are bits of a
// scalar, and past the list's end the run reads an entry that nothing reaches, so it needs no bounds.
// The next batch's records are loaded while the current one is composited.  Each pixel's float operations
// and their order are those of the one-entry loop.  Run by a whole wavefront; S is its staging.
// 60k Gaussians on a cube map and a panorama (0.57M pairs, lists of up to 901): 214 us unsplit, 129 us
// split with the one-entry loop, 106 us with runs whose reads the compiler had put one behind another, 80 us
// with this; 6k on 512x256 (lists of up to 102) 16.4 us with the one-entry loop, 11.6 us with this.
constexpr int kQuadRun = 4;

// A quadrant task's culling masks are a byte per list entry at BIN = 16, whose planes it has to itself,
// and a bit per entry at BIN = 32, where the four quadrants of a part share a plane: quadrant q's bits start
// at q quarters of the list's bytes (an eighth of them each; the lists are long ones).  The reverse takes
// the part whole, so that its float sums do not depend on the forward's tasks, and puts its masks together.
template <int BIN>
__device__ inline uint8_t* quadrant_masks(uint8_t* plane, uint2 rg, int q) {
  return BIN == 32 ? plane + rg.x + (uint32_t)q * ((rg.y - rg.x) >> 2) : plane;
}
__device__ inline uint32_t part_mask(const uint8_t* __restrict__ plane, uint2 rg, uint32_t k) {
  const uint8_t* p = plane + rg.x + (k >> 3);
  const uint32_t step = (rg.y - rg.x) >> 2;
  uint32_t m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) m |= ((uint32_t)p[(uint32_t)q * step] >> (k & 7u) & 1u) << q;
  return m;
}

template <int BIN, int BATCH, bool DEPTH>
__device__ inline void composite_quadrant(FwdStage4<BATCH>& S, int q, uint2 rg, const uint32_t* __restrict__ pair_items,
                                          const Rec* __restrict__ rec, const float* __restrict__ depth, int tx0, int ty0,
                                          float Wf, float half, uint8_t* __restrict__ qm, float& T_out, float (&C)[3],
                                          float& D_out, int& last_out) {
  constexpr int NB = BATCH < kWave ? BATCH : kWave;
  const int lane = threadIdx.x;
  const float px = (float)(tx0 + 8 * (q & 1) + (lane & 7)) + 0.5f;
  const float py = (float)(ty0 + 8 * (q >> 1) + (lane >> 3)) + 0.5f;
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f, qstop = 0.0f;  // qstop: NaN once stopped
  int last = 0;
  if (lane == 0)  // the entry nothing reaches
    S.s0[NB] = make_float4(0, 0, 0, 0), S.s1[NB] = make_float4(0, __builtin_inff(), 0, 0), S.s2[NB] = S.s0[NB];
  if (rg.x < rg.y) {
    // records one batch ahead, items two (indices clamped into the list)
    uint32_t item = pair_items[min(rg.x + lane, rg.y - 1)];
    const vec4* recs = reinterpret_cast<const vec4*>(rec);  // three words per record
    vec4 r0 = recs[3 * (int64_t)item], r1 = recs[3 * (int64_t)item + 1], r2 = recs[3 * (int64_t)item + 2];
    float dep = DEPTH ? depth[item] : 0.0f;
    item = pair_items[min(rg.x + NB + lane, rg.y - 1)];
    for (uint32_t base = rg.x; base < rg.y; base += NB) {
      const int cnt = (int)min((uint32_t)NB, rg.y - base);
      uint32_t m = 0;
      if (lane < cnt) {
        S.s0[lane] = make_float4(r0.x, r0.y, r0.z, r0.w);
        const float reach = fabsf((float)tx0 + 8.0f - r0.x) + 8.0f + 1.0f;
        S.s1[lane] = make_float4(r1.x, r1.z, r1.y, dep);
        S.s2[lane] = make_float4(r2.x, r2.y, r2.z, r2.w);
        S.used[lane] = 0;
        const Rec r{make_float4(r0.x, r0.y, r0.z, r0.w), make_float4(r1.x, r1.y, r1.z, r1.w),
                    make_float4(r2.x, r2.y, r2.z, r2.w)};
        m = quadrant_mask<8>(r, tx0 + 8 * (q & 1), ty0 + 8 * (q >> 1), Wf, half);
        const bool rare = r1.y > kAlphaMax || fmaxf(fmaxf(r2.x, r2.y), r2.z) == __builtin_inff();
        if (m != 0u) m |= (reach < half ? 0 : kEntryWrap << 4) | (rare ? kEntryClamp << 4 : 0);
      }
      const uint64_t bl = __builtin_amdgcn_ballot_w64(m != 0u);
      if (m != 0u) S.list[bits_below(bl)] = (uint16_t)(lane | (m << 8));
      const int n = __popcll(bl);
      r0 = recs[3 * (int64_t)item];
      r1 = recs[3 * (int64_t)item + 1];
      r2 = recs[3 * (int64_t)item + 2];
      if (DEPTH) dep = depth[item];
      item = pair_items[min(base + 2 * NB + lane, rg.y - 1)];
      __syncthreads();
      const uint32_t words = lane < n ? S.list[lane] : NB;  // past the end: the entry nothing reaches
      uint64_t used = 0;
      for (int i0 = 0; i0 < n; i0 += kQuadRun) {
        float a[kQuadRun][4], b[kQuadRun][3];
        int at[kQuadRun];  // the entries' LDS word (uniform)
        uint32_t flags = 0;
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) {
          const uint32_t km = __builtin_amdgcn_readlane(words, i0 + j);
          flags |= km;
          at[j] = (int)(km & 0xFFu);
          const float4 s0 = S.s0[at[j]], s1 = S.s1[at[j]];
          a[j][0] = s0.x, a[j][1] = s0.y, a[j][2] = s0.z, a[j][3] = s0.w;
          b[j][0] = s1.x, b[j][1] = s1.y, b[j][2] = s1.z;
        }
        // every read is issued before the first is waited for
        static_assert(kQuadRun == 4, "the operands of the next lines");
        asm volatile("" : "+v"(b[0][0]), "+v"(b[1][0]), "+v"(b[2][0]), "+v"(b[3][0]), "+v"(a[3][0]), "+v"(a[2][0]), "+v"(a[1][0]), "+v"(a[0][0]));
        float du[kQuadRun], alpha[kQuadRun], t[kQuadRun + 1];
        bool ok[kQuadRun];
        int hit = 0;
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) du[j] = px - a[j][0];
        if (__builtin_expect(opaque((int)(flags >> 12 & kEntryWrap)), 0)) {  // uniform
#pragma unroll
          for (int j = 0; j < kQuadRun; ++j) {
            du[j] = wrap_du(du[j], Wf, half);  // (the identity where it is not needed)
            keep_branch(du[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) {
          const float dv = py - a[j][1];
          const float t1 = fmaf(a[j][2], du[j], a[j][3] * dv), t2 = b[j][0] * dv;
          const float power = -fmaf(t1, t1, fmaf(t2, t2, qstop));
          ok[j] = power >= b[j][1];  // alpha >= 1/255 (NaN once the pixel has stopped)
          alpha[j] = ok[j] ? b[j][2] * __expf(power) : 0.0f;
          hit |= bit_if(__builtin_amdgcn_ballot_w64(ok[j]), j);
        }
        if (hit == 0) continue;  // uniform
        if (__builtin_expect(opaque((int)(flags >> 12 & kEntryClamp)), 0)) {  // uniform
          const float zero = zero_here();
#pragma unroll
          for (int j = 0; j < kQuadRun; ++j) {
            alpha[j] = fminf(alpha[j], kAlphaMax);
            keep_branch(alpha[j]);
            // an entry that reaches no pixel: its colour, times a weight of zero, may be infinite
            if ((hit >> j & 1) == 0) S.s2[at[j]].x = S.s2[at[j]].y = S.s2[at[j]].z = zero;
          }
        }
        t[0] = T;
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) t[j + 1] = t[j] * (1.0f - alpha[j]);
        // T never rises, so a pixel stops within the run only if its last product is below the threshold
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(t[kQuadRun] < kTStop) != 0ull, 0)) {
          // entry by entry: a pixel stops at the entry that would take T below 1e-4, without it.  An entry
          // at which all the pixels it reaches stop is none of the backward's, which evaluates runs whole.
          hit = 0;
#pragma unroll
          for (int j = 0; j < kQuadRun; ++j) {
            qstop = t[j] * (1.0f - alpha[j]) < kTStop ? __builtin_nanf("") : qstop;
            ok[j] = ok[j] && qstop == 0.0f;
            hit |= bit_if(__builtin_amdgcn_ballot_w64(ok[j]), j);
            alpha[j] = ok[j] ? alpha[j] : 0.0f;
            t[j + 1] = t[j] * (1.0f - alpha[j]);
          }
        }
        used |= (uint64_t)(uint32_t)hit << i0;
        T = t[kQuadRun];
        float c[kQuadRun][3], d[kQuadRun];
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) {
          const float4 s2 = S.s2[at[j]];
          c[j][0] = s2.x, c[j][1] = s2.y, c[j][2] = s2.z;
          if constexpr (DEPTH) d[j] = S.s1[at[j]].w;
        }
        asm volatile("" : "+v"(c[0][0]), "+v"(c[1][0]), "+v"(c[2][0]), "+v"(c[3][0]));
        if constexpr (DEPTH) asm volatile("" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]));
#pragma unroll
        for (int j = 0; j < kQuadRun; ++j) {
          const float w = alpha[j] * t[j];
          C0 = fmaf(w, c[j][0], C0);
          C1 = fmaf(w, c[j][1], C1);
          C2 = fmaf(w, c[j][2], C2);
          if constexpr (DEPTH) D = D + w * d[j];
          last = ok[j] ? (int)(base - rg.x) + at[j] + 1 : last;
        }
      }
      if (lane < n) S.used[words & 0xFFu] = (uint8_t)((used >> lane & 1u) << q);
      __syncthreads();
      // the backward's masks for this batch: whether each entry contributed to some pixel
      if constexpr (BIN == 32) {
        const uint64_t reached = __builtin_amdgcn_ballot_w64(lane < cnt && S.used[lane] != 0);
        if (8 * lane < cnt) qm[((base - rg.x) >> 3) + lane] = (uint8_t)(reached >> (8 * lane));
      } else {
        if (lane < cnt) qm[base + lane] = S.used[lane];
      }
      __syncthreads();
      if (__builtin_amdgcn_ballot_w64(qstop == 0.0f) == 0ull) {  // every pixel has stopped
        if constexpr (BIN == 32)  // the reverse of the part may go further
          for (uint32_t k = ((base + NB - rg.x) >> 3) + lane; k < (rg.y - rg.x + 7) >> 3; k += kWave) qm[k] = 0;
        break;
      }
    }
  }
  T_out = T;
  C[0] = C0;
  C[1] = C1;
  C[2] = C2;
  D_out = D;
  last_out = last;
}

// (Seven wavefronts per SIMD, 72 registers: left to itself the compiler takes more with the quadrant path
// beside the loop: 814 against 778 us at 500k Gaussians, 8 views, many lists split, in <16, 64, false>, the
// one instance this was measured for.  The others of batches up to 64 but <16, 32, false> spill a few words
// at it: 20 bytes of scratch with depth at 16, 20 without and 36 with depth at 32.)
template <int BIN, int BATCH, bool DEPTH>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(BATCH > 64 ? 1 : 7))) void render_fwd4_kernel(
    ViewTable vt, const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_items, const Rec* __restrict__ rec,
    float* __restrict__ out_rgb, float* __restrict__ out_T, float* __restrict__ ws_T, int32_t* __restrict__ ws_last,
    float bg0, float bg1, float bg2, const float* __restrict__ depth, float* __restrict__ out_depth,
    uint8_t* __restrict__ qmask, int64_t qplane, TileSched sc) {
  constexpr int TILE = 16;
  __shared__ FwdStage4<BATCH> S;
  const int nsplit = forward_split(sc), nfine = BIN == 32 ? forward_fine(sc) : 0;
  mark_forward(sc, nsplit, nfine);
  __shared__ uint32_t s_claim;
  uint32_t round = 0, sel = 0;
  const int lane = threadIdx.x;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  for (int g; (g = claim_task(sc, nsplit, nfine, 0, round, &s_claim, sel)) >= 0;) {
    const int v = view_of_tile(vt, g);
    const int W = vt.W[v], H = vt.H[v];
    int tx0, ty0, pl;
    task_block<BIN>(vt, v, g, sel, tx0, ty0, pl);
    const int x = tx0 + (lane & 7), y = ty0 + (lane >> 3);
    const float px0 = (float)x + 0.5f, px1 = (float)(x + 8) + 0.5f;
    const float py0 = (float)y + 0.5f, py1 = (float)(y + 8) + 0.5f;
    const float Wf = (float)W, half = wrap_half(vt, v);
    const uint2 rg = ranges[g];
    uint8_t* qm = qmask + (int64_t)pl * qplane;
    if (sel != 0xFu) {  // uniform: a quadrant of a split tile
      const int q = __builtin_ctz(sel);
      float Tq, C[3], Dq;
      int lastq;
      composite_quadrant<BIN, BATCH, DEPTH>(S, q, rg, pair_items, rec, depth, tx0, ty0, uniform(Wf), uniform(half),
                                            quadrant_masks<BIN>(qm, rg, q), Tq, C, Dq, lastq);
      const int64_t plane = (int64_t)W * H, pix = (int64_t)(y + 8 * (q >> 1)) * W + x + 8 * (q & 1);
      const int64_t gp = vt.pix_base[v] + pix;
      float* img = out_rgb + 3 * vt.pix_base[v];
      img[pix] = fmaf(Tq, bg0, C[0]);
      img[plane + pix] = fmaf(Tq, bg1, C[1]);
      img[2 * plane + pix] = fmaf(Tq, bg2, C[2]);
      ws_T[gp] = Tq;
      ws_last[gp] = lastq;
      if constexpr (DEPTH) out_depth[gp] = Dq;
      if (out_T) out_T[gp] = Tq;
      continue;
    }
    float T[4], C0[4], C1[4], C2[4], D[4], qstop[4];  // qstop: 0 while compositing, NaN once stopped
    int last[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      T[q] = 1.0f;
      C0[q] = C1[q] = C2[q] = D[q] = 0.0f;
      qstop[q] = 0.0f;
      last[q] = 0;
    }
    uint32_t alive = 0xFu;  // quadrants with a pixel still compositing (uniform)
    for (uint32_t base = rg.x; base < rg.y && alive != 0u; base += BATCH) {
      const int cnt = (int)min((uint32_t)BATCH, rg.y - base);
      int n = 0;
      for (int r0 = 0; r0 < cnt; r0 += kWave) {
        const int e = r0 + lane;
        uint32_t m = 0;
        if (e < cnt) {
          const uint32_t item = pair_items[base + e];
          const Rec r = rec[item];
          S.s0[e] = r.r0;
          const float reach = fabsf((float)tx0 + 0.5f * (float)TILE - r.r0.x) + 0.5f * (float)TILE + 1.0f;
          S.s1[e] = make_float4(r.r1.x, r.r1.z, r.r1.y, DEPTH ? depth[item] : 0.0f);
          S.s2[e] = r.r2;
          S.used[e] = 0;
          m = quadrant_mask<TILE>(r, tx0, ty0, Wf, half);
          if (m != 0u) m |= (reach < half ? 0 : kEntryWrap << 4) | (r.r1.y > kAlphaMax ? kEntryClamp << 4 : 0);
        }
        const uint64_t bl = __builtin_amdgcn_ballot_w64(m != 0u);
        if (m != 0u) S.list[n + __popcll(bl & below)] = (uint16_t)(e | (m << 8));
        n += __popcll(bl);
      }
      __syncthreads();
      for (int i0 = 0; i0 < n; i0 += kWave) {
        // the list words of 64 entries, one per lane, and the quadrants used of each
        const uint32_t words = S.list[min(i0 + lane, n - 1)];
        uint32_t used_words = 0;
        const int m = min(kWave, n - i0);
        for (int i = 0; i < m; ++i) {
          const uint32_t km = __builtin_amdgcn_readlane(words, i);
          const int k = (int)(km & 0xFFu);
          const uint32_t mq = (km >> 8) & (alive | 0xF0u);
          if ((mq & 0xFu) == 0u) continue;  // uniform
          const float4 a = S.s0[k];
          const float4 b = S.s1[k];
          float du0 = px0 - a.x, du1 = px1 - a.x;
          if (mq & (kEntryWrap << 4)) {  // uniform
            du0 = wrap_du(du0, Wf, half);
            du1 = wrap_du(du1, Wf, half);
          }
          uint32_t used = 0;
          const float4 c = S.s2[k];  // once per entry, not per accepting quadrant: forward 0.81 -> 0.78 ms
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (!((mq >> q) & 1u)) continue;  // uniform
            const float dv = (q >> 1 ? py1 : py0) - a.y;
            const float du = q & 1 ? du1 : du0;
            const float t1 = fmaf(a.z, du, a.w * dv), t2 = b.x * dv;
            const float power = -fmaf(t1, t1, fmaf(t2, t2, qstop[q]));
            bool ok = power >= b.y;  // alpha >= 1/255 (NaN once the pixel has stopped)
            if (__builtin_amdgcn_ballot_w64(ok) == 0ull) continue;  // uniform
            used |= 1u << q;
            // alpha = 0 where the entry does not reach the pixel: T (1 - 0) = T exactly
            float alpha = ok ? b.z * __expf(power) : 0.0f;
            if (__builtin_expect(opaque((int)(mq & (kEntryClamp << 4))) != 0, 0)) {
              alpha = fminf(alpha, kAlphaMax);
              keep_branch(alpha);
            }
            float Tn = T[q] * (1.0f - alpha);
            // a pixel stops at the entry that would take T below 1e-4, without it (rare: once per
            // pixel; T itself never is below, so only reached pixels can)
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(Tn < kTStop) != 0ull, 0)) {
              const bool stop = Tn < kTStop;
              ok = ok && !stop;
              alpha = stop ? 0.0f : alpha;
              Tn = stop ? T[q] : Tn;
              qstop[q] = stop ? __builtin_nanf("") : qstop[q];
              keep_branch(qstop[q]);
            }
            const float w = alpha * T[q];
            C0[q] = fmaf(w, c.x, C0[q]);
            C1[q] = fmaf(w, c.y, C1[q]);
            C2[q] = fmaf(w, c.z, C2[q]);
            if constexpr (DEPTH) D[q] = D[q] + w * b.w;
            T[q] = Tn;
            last[q] = ok ? (int)(base - rg.x) + k + 1 : last[q];
          }
          set_lane(used_words, used, i);
        }
        if (lane < m) S.used[words & 0xFFu] = (uint8_t)used_words;
      }
      // quadrants whose pixels have all stopped (taken once per batch: within a batch a stopped
      // quadrant costs its test per entry, which no longer reaches any pixel)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (((alive >> q) & 1u) && __builtin_amdgcn_ballot_w64(qstop[q] == 0.0f) == 0ull) alive &= ~(1u << q);
      __syncthreads();
      // the backward's masks for this batch: the quadrants in which some pixel reached each entry
      for (int e = lane; e < cnt; e += kWave) qm[base + e] = S.used[e];
      __syncthreads();
    }
    // entries past the point where every pixel stopped were never reached: their masks stay as
    // the binning left them, and the backward (which stops at each tile's last contributor) never
    // reads them
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t pix = (int64_t)(y + 8 * (q >> 1)) * W + x + 8 * (q & 1);
      float* img = out_rgb + 3 * vt.pix_base[v];
      const int64_t plane = (int64_t)W * H;
      img[pix] = fmaf(T[q], bg0, C0[q]);
      img[plane + pix] = fmaf(T[q], bg1, C1[q]);
      img[2 * plane + pix] = fmaf(T[q], bg2, C2[q]);
      const int64_t gp = vt.pix_base[v] + pix;
      ws_T[gp] = T[q];
      ws_last[gp] = last[q];
      if constexpr (DEPTH) out_depth[gp] = D[q];
      if (out_T) out_T[gp] = T[q];
    }
  }
}

// Reverse compositing state of one pixel (back to front from its last contributor).
struct BwdPixel {
  float T, DS, dl0, dl1, dl2;  // DS = dL/dC . (colour of everything behind, incl. background)
  int last;
};

// Whether products of the pixel's gradients may leave the float range (kLarge).
__device__ inline bool pixel_is_large(const BwdPixel& P) { return is_large(magnitude(P.dl0, P.dl1, P.dl2) + fabsf(P.DS)); }

// The position and shape sums are taken in the footprint's whitened coordinates t = L d
// (t1 = l0 du + l1 dv, t2 = l2 dv, L = [[l0, l1], [0, l2]] the record's factor of Sigma^-1 / 2, so
// power = -|t|^2): per pixel dpow * t and dpow * t t^T, whose entries are all of the same order for
// any footprint shape.  With h = L^T t = Sigma^-1 d / 2, d power / d(u, v) = 2 h and
// d power / d Sigma_2D = 2 h h^T, so the per-tile sums S_t = sum dpow t and Z = sum dpow t t^T map
// exactly to g_(u,v) = 2 L^T S_t and g_Sigma = 2 L^T Z L.  That map is applied once per (Gaussian,
// tile) in double at the flush.  (Summing dpow h h^T directly in float loses the long axis of a
// needle-like footprint: there h lies almost along the short axis and the long-axis component of
// h h^T sits ~1e5 below the rounding of the short one.)
template <int NS, int B>
__device__ inline double acc_total(const float (&acc)[NS][9][B], int q, int t) {
  double s = (double)acc[0][q][t];
#pragma unroll
  for (int w = 1; w < NS; ++w) s += (double)acc[w][q][t];
  return s;
}

// Value q of an entry's 2D-gradient record (layout of g2d) from its per-wavefront sums; a, b: the
// entry's staged record words (l0 = a.z, l1 = a.w, l2 = b.x, opacity = b.z).
template <int NS, int B>
__device__ inline double g2d_flush_value(const float (&acc)[NS][9][B], int q, int t, const float4& a, const float4& b) {
  const double l0 = a.z, l1 = a.w, l2 = b.x;
  switch (q) {
    case 0: return 2.0 * l0 * acc_total(acc, 0, t);
    case 1: return 2.0 * (l1 * acc_total(acc, 0, t) + l2 * acc_total(acc, 1, t));
    case 2: return 2.0 * (l0 * l0) * acc_total(acc, 2, t);
    case 3: return 4.0 * l0 * (l1 * acc_total(acc, 2, t) + l2 * acc_total(acc, 3, t));
    case 4: {
      const double z11 = acc_total(acc, 2, t), z12 = acc_total(acc, 3, t), z22 = acc_total(acc, 4, t);
      return 2.0 * ((l1 * l1) * z11 + 2.0 * (l1 * l2) * z12 + (l2 * l2) * z22);
    }
    default: return acc_total(acc, q, t);
  }
}

// One pixel's contribution of a Gaussian to the nine per-tile sums (added to gq when ADD, else
// written; slots 0..4 in whitened coordinates as above), and the pixel's recursion step.  `ok`: the
// Gaussian contributed to this pixel; t1 = l0 du + l1 dv, t2 = l2 dv.  `rare` (uniform): the opacity
// is above 0.99, so that alpha may be clamped (else G <= 1 keeps it below), or an upstream gradient or
// a colour is large or not finite, so that dL/dalpha needs a select of its own where the Gaussian does not
// contribute (else its products with alpha = 0 and G = 0 are zero); two branches past an instruction or
// two (the whole step compiled for both cases copies the pixel state between them, which costs more than
// the branches, and the select in every step 2%: 1,126 -> 1,152 us at 500k Gaussians, 8 views).
template <bool ADD>
__device__ inline void bwd_pixel_step(BwdPixel& P, bool ok, int rare, float power, float t1, float t2, const float4& b,
                                      const float4& c, float (&gq)[9]) {
  const float G = ok ? __expf(power) : 0.0f;
  const float araw = b.z * G;
  // alpha = 0 where the Gaussian does not contribute, so its weight below is 0 without a select
  float alpha = araw;
  if (__builtin_expect(opaque(rare) != 0, 0)) {
    alpha = fminf(alpha, kAlphaMax);
    keep_branch(alpha);
  }
  const float inv_om = __builtin_amdgcn_rcpf(1.0f - alpha);
  // transmittance in front of this Gaussian; where it does not contribute alpha = 0 and the
  // reciprocal of 1 is exactly 1 (powers of two are exact), so T is unchanged without a select
  P.T = P.T * inv_om;
  const float wk = alpha * P.T;
  const float dc = fmaf(P.dl0, c.x, fmaf(P.dl1, c.y, P.dl2 * c.z));  // dL/dC . colour
  float dla = fmaf(dc, P.T, -P.DS * inv_om);  // dL/dalpha
  if (__builtin_expect(opaque(rare) != 0, 0)) {
    dla = !ok || araw > kAlphaMax ? 0.0f : dla;  // a clamped alpha does not depend on the inputs
    keep_branch(dla);
  }
  P.DS = fmaf(dc, wk, P.DS);
  const float dpow = dla * alpha;
  const float g0 = dpow * t1, g1 = dpow * t2;
  gq[0] = ADD ? gq[0] + g0 : g0;
  gq[1] = ADD ? gq[1] + g1 : g1;
  // values 2..8 are products x_q y_q (fused into the running sums when adding)
  const float x[7] = {g0, g0, g1, dla, wk, wk, wk}, y[7] = {t1, t2, t2, G, P.dl0, P.dl1, P.dl2};
#pragma unroll
  for (int q = 0; q < 7; ++q) gq[2 + q] = ADD ? fmaf(x[q], y[q], gq[2 + q]) : x[q] * y[q];
}

// g2d layout: [items][9] = d/du, d/dv, d/dS_uu, d/dS_uv, d/dS_vv, d/dopacity, d/dr, d/dg,
// d/db(colour), where Sigma_2D = [[S_uu, S_uv], [S_uv, S_vv]] (S_uv the shared off-diagonal),
// formed per (Gaussian, tile) from the whitened-coordinate sums (g2d_flush_value).
template <int TILE, int BATCH>
__global__ __launch_bounds__(TILE* TILE) void render_bwd_kernel(ViewTable vt, const uint2* __restrict__ ranges,
                                                                const uint32_t* __restrict__ pair_items,
                                                                const Rec* __restrict__ rec, const float* __restrict__ ws_T,
                                                                const int32_t* __restrict__ ws_last,
                                                                const float* __restrict__ dL_drgb, double* __restrict__ g2d,
                                                                int64_t items, float bg0, float bg1, float bg2,
                                                                const uint8_t* __restrict__ qmask, TileSched sc) {
  static_assert(TILE == 8, "tiles of 16 and 32 take the four-pixel kernel");
  using St = Stage<TILE, BATCH>;
  constexpr int N = St::N;
  // One wavefront per 8x8 tile, owning a slot per (value, entry).
  constexpr int NS = St::NW;
  __shared__ St S;
  __shared__ float acc[NS][9][BATCH + 1];  // padded rows: the nine slot writes hit nine banks
  __shared__ float red[NS][8][kRedStride];  // reduction scratch
  __shared__ int smax;
  if (forward_is_stale(sc)) return;  // uniform
  __shared__ uint32_t s_claim;
  uint32_t round = 0;
  for (int g; (g = claim_tile(sc, round, &s_claim)) >= 0;) {
    const int v = view_of_tile(vt, g);
    const int W = vt.W[v], H = vt.H[v];
    const int ntx = W / TILE;
    const int lt = g - vt.tile_base[v];
    const int tx0 = (lt % ntx) * TILE, ty0 = (lt / ntx) * TILE;
    int lx, ly;
    local_pixel<TILE>(threadIdx.x, lx, ly);
    const int x = tx0 + lx, y = ty0 + ly;
    const int lane = threadIdx.x & (kWave - 1);
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    const float Wf = (float)W, half = wrap_half(vt, v);  // no seam in pinhole views
    const uint2 rg = ranges[g];
    const int64_t plane = (int64_t)W * H;
    const int64_t pix = (int64_t)y * W + x;
    const int64_t gp = vt.pix_base[v] + pix;
    const float* dimg = dL_drgb + 3 * vt.pix_base[v];
    BwdPixel P;
    P.dl0 = dimg[pix], P.dl1 = dimg[plane + pix], P.dl2 = dimg[2 * plane + pix];
    P.T = ws_T[gp];
    P.last = ws_last[gp];
    // dL/dC . (colour of everything behind, incl. background): the only way the colour behind a
    // Gaussian enters its alpha gradient, so one scalar replaces the three channels
    P.DS = P.T * fmaf(P.dl0, bg0, fmaf(P.dl1, bg1, P.dl2 * bg2));
    // largest `last` of the wavefront (uniform) and of the workgroup
    int wmax = P.last;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wmax = max(wmax, __shfl_xor(wmax, off));
    wmax = __builtin_amdgcn_readfirstlane(wmax);
    if (threadIdx.x == 0) smax = 0;
    __syncthreads();
    if (lane == 0) atomicMax(&smax, wmax);
    __syncthreads();
    const int end_all = smax;
    for (int end = end_all; end > 0; end -= BATCH) {
      const int cnt = min(BATCH, end);
      for (int t = threadIdx.x; t < cnt; t += N) {
#pragma unroll
        for (int w = 0; w < NS; ++w)
#pragma unroll
          for (int q = 0; q < 9; ++q) acc[w][q][t] = 0.0f;
      }
      int nq[St::NQ];
      // entry e is list position end - 1 - e (back to front)
      stage_batch<TILE, BATCH, kMaskLoad>(S, pair_items, rec, rg.x + end - 1, -1, cnt, tx0, ty0, Wf, half, nq, nullptr,
                                             qmask);
      const int n = __builtin_amdgcn_readfirstlane(nq[wq]);
      bool pend = false;  // an accepted entry whose values 0..7 still wait in red (uniform)
      int pk = 0;
      // software pipeline: the next entry's list index and records are read while this one is
      // processed, taking two LDS round trips off each iteration's dependency chain
      int kn = n > 0 ? S.list[wq][0] : 0;  // entries 0..n-1 of the list are valid
      float4 an = S.s0[kn], bn = S.s1[kn];
      for (int i = 0; i < n; ++i) {
        const int k = __builtin_amdgcn_readfirstlane(kn);  // uniform entry index
        const float4 a = an, b = bn;
        kn = S.list[wq][min(i + 1, n - 1)];
        an = S.s0[kn];
        bn = S.s1[kn];
        const int jrel = end - 1 - k;
        if (jrel >= wmax) continue;  // uniform: behind every contributor of this wavefront
        const float du = wrap_du(px - a.x, Wf, half);
        const float dv = py - a.y;
        const float t1 = fmaf(a.z, du, a.w * dv), t2 = b.x * dv;
        const float power = -fmaf(t1, t1, t2 * t2);
        const bool ok = jrel < P.last && !(power > 0.0f || power < b.y);
        if (__builtin_amdgcn_ballot_w64(ok) == 0ull) continue;  // uniform
        float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0;
        if (pend) red_read(red[wq], lane, r0, r1);  // previous accepted entry's values
        const float4 c = S.s2[k];
        float gq[9];
        bwd_pixel_step<false>(P, ok, 1, power, t1, t2, b, c, gq);
        if (pend) {
          const float sj = red_finish(r0, r1);
          if ((lane & 7) == 0) acc[wq][lane >> 3][pk] = sj;
        }
        red_write(red[wq], gq, lane);
        const float s8 = wave_sum(gq[8]);
        if (lane == 1) acc[wq][8][k] = s8;
        pend = true;
        pk = k;
      }
      if (pend) {
        float4 r0, r1;
        red_read(red[wq], lane, r0, r1);
        const float sj = red_finish(r0, r1);
        if ((lane & 7) == 0) acc[wq][lane >> 3][pk] = sj;
      }
      __syncthreads();
      // nine consecutive lanes carry one entry's nine values, so one atomic instruction covers
      // about seven items' contiguous 72-byte gradient records instead of 64 scattered lines
      for (int x = threadIdx.x; x < 9 * cnt; x += N) {
        const int t = x / 9, q = x - 9 * t;
        const double s = g2d_flush_value(acc, q, t, S.s0[t], S.s1[t]);
        if (s != 0.0) unsafeAtomicAdd(&g2d[(int64_t)S.sid[t] * 9 + q], s);
      }
      __syncthreads();
    }
  }
}

// Reverse compositing of a 16x16 tile by one wavefront, four pixels per lane (lane l holds pixel
// (l % 8, l / 8) of each quadrant): the four quadrants' contributions to an entry are added in
// registers and reduced across lanes once, and a quadrant the forward's pixels did not reach
// (its bit in the staged mask) costs nothing for that entry.
//
// The nine sums are reduced across lanes by two DPP steps only (quad_reduce9); the sixteen partial
// sums that leaves of each value (four lanes in each of the four 16-lane rows) go to LDS, and a
// group of kRingEntries entries is finished at once, one lane per (entry, value): sixteen partials
// added per lane cost less than the selects, DPP adds and row swaps that would finish them entry by
// entry.  The map from the whitened sums to the gradient record has no branches: value q is
// u (x Sa + y Sb) + w Sc of three sums, with coefficients that are record words selected by q.
//
// Bound by VALU issue.  Measured at 500k Gaussians, 8 views of 2048x1024: 1,550 us with the sums
// finished entry by entry, a divergent map per value and every step clamping; 1,402 us with bank-
// masked folds, a branch-free map and the clamp only for entries that can need it; 1,350 us with the
// last two steps of the reduction left to the group and the list words read from one register.  LDS
// per wavefront counts too: 7,748 bytes took seven of its 1,280-byte granules and held a CU to 18
// wavefronts where the registers allow 20; with a group's sums over its partials, 7,540 bytes take six:
// 1,355 -> 1,290 us.
template <int BATCH>
struct Stage4 {  // (one entry more for reverse_quadrant)
  float4 s0[BATCH + 1];  // u, v, l0, l1
  float4 s1[BATCH + 1];  // l2, p_min, opacity, unused
  float4 s2[BATCH + 1];  // r, g, b, unused
  uint32_t sid[BATCH];
  uint16_t list[BATCH];  // entry index | quadrant mask << 8 | flags << 12
};

// Entries per flush: seven entries of nine values take 63 of the 64 lanes.
constexpr int kRingEntries = 7;
constexpr int kRingRow = 36;  // per 16-lane row: 16 words of g[0], 16 of g[1], 4 of g[8]
constexpr int kRingStride = 4 * kRingRow;

// This lane's part in a flush: its entry fe of the group, the first of its value's four rows of
// partials, and, in one word, the byte offsets of the sums its value is mapped from and its value fq.
struct FlushLane {
  int fe;
  uint32_t fw;  // sums fa | fb << 8 | fc << 16 (byte offsets) | fq << 24
  const float4* fin;
};

__device__ inline FlushLane flush_lane(const float* ring, int lane) {
  FlushLane f;
  const int fe = lane / 9, fq = lane - 9 * fe;
  const int fa = 9 * fe + (fq < 2 ? 0 : (fq < 5 ? 2 : fq));
  const int fb = fq == 1 ? 9 * fe + 1 : (fq == 3 || fq == 4 ? 9 * fe + 3 : kWave - 1);
  const int fc = fq == 4 ? 9 * fe + 4 : kWave - 1;
  f.fe = fe;
  f.fw = (uint32_t)(4 * fa | (4 * fb) << 8 | (4 * fc) << 16 | fq << 24);
  f.fin = reinterpret_cast<const float4*>(ring + fe * kRingStride + (fq < 8 ? 16 * (fq & 1) + 4 * (fq >> 1) : 32));
  return f;
}

// Adds the gradients of the group's m entries (list entries i0 on, their partials in the ring) to
// their records.
template <int BATCH>
__device__ inline void flush_group(const Stage4<BATCH>& S, const FlushLane& f, float* ring, int i0, int m,
                                   double* __restrict__ g2d) {
  float* const sums = ring;  // per (entry, value), over the partials; the last word is zero
  float total = 0.0f;
  __syncthreads();
  if (f.fe < m) {  // (never lane 63: fe = 7)
    float r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 p = f.fin[k * (kRingRow / 4)];
      r[k] = (p.x + p.y) + (p.z + p.w);
    }
    total = (r[0] + r[1]) + (r[2] + r[3]);
  }
  __syncthreads();
  sums[threadIdx.x] = total;
  __syncthreads();
  if (f.fe < m) {
    const int fq = (int)(f.fw >> 24), t = S.list[i0 + f.fe] & 0xFF;
    const float4 a = S.s0[t];
    const float l0 = a.z, l1 = a.w, l2 = S.s1[t].x;
    // value fq of the record, from the sums S0 .. S8:
    //   0: 2 (l0 S0)   1: 2 (l1 S0 + l2 S1)   2: 2 l0 (l0 S2)   3: 4 l0 (l1 S2 + l2 S3)
    //   4: 2 l1 (l1 S2 + 2 l2 S3) + 2 l2 (l2 S4)   5 to 8: Sq
    float x = fq < 5 ? l1 : 1.0f, u = fq < 2 ? 2.0f : 1.0f;
    x = fq == 0 || fq == 2 ? l0 : x;
    const float y = fq == 4 ? 2.0f * l2 : l2;
    u = fq == 2 ? 2.0f * l0 : u;
    u = fq == 3 ? 4.0f * l0 : u;
    u = fq == 4 ? 2.0f * l1 : u;
    const double w = (double)l2;
    auto sum = [&](uint32_t offset) {
      return (double)*reinterpret_cast<const float*>(reinterpret_cast<const char*>(sums) + offset);
    };
    const double d = fma((double)u, fma((double)x, sum(f.fw & 0xFFu), (double)y * sum((f.fw >> 8) & 0xFFu)),
                         (w + w) * (w * sum((f.fw >> 16) & 0xFFu)));
    if (d != 0.0) unsafeAtomicAdd(&g2d[(int64_t)S.sid[t] * 9 + fq], d);
  }
  __syncthreads();
}

// One quadrant of a split tile in reverse, one pixel per lane: as in composite_quadrant, a run of
// kQuadRunBwd entries is evaluated together and only T and DS stay chains; the culling masks, items and
// records of the next batches are loaded ahead.  The cases of composite_quadrant: 306 us unsplit, 186 us with
// the one-entry loop, 138 us with this (three entries together: 141), and 23.4 -> 18.9 us.
constexpr int kQuadRunBwd = 2;

template <int BATCH>
__device__ inline void reverse_quadrant(Stage4<BATCH>& S, float* ring, const FlushLane& fl, BwdPixel P,
                                        float px, float py, uint2 rg, int wmax, const uint32_t* __restrict__ pair_items,
                                        const Rec* __restrict__ rec, const uint8_t* __restrict__ qm, float tcx, float Wf,
                                        float half, double* __restrict__ g2d) {
  constexpr int NB = BATCH < kWave ? BATCH : kWave;
  const int lane = threadIdx.x;
  if (wmax <= 0) return;  // uniform
  if (lane == 0)
    S.s0[NB] = make_float4(0, 0, 0, 0), S.s1[NB] = make_float4(0, __builtin_inff(), 0, 0), S.s2[NB] = S.s0[NB];
  // entry e of the batch that ends at `end` is list position end - 1 - e (clamped into the list's start)
  float* const out01 = ring + (lane >> 4) * kRingRow + (lane & 15);
  float* const out8 = ring + (lane >> 4) * kRingRow + 32 + (lane & 3);
  uint32_t pos = rg.x + max(wmax - 1 - lane, 0);
  uint32_t mask = qm[pos], item = pair_items[pos];
  const vec4* recs = reinterpret_cast<const vec4*>(rec);  // three words per record
  vec4 r0 = recs[3 * (int64_t)item], r1 = recs[3 * (int64_t)item + 1], r2 = recs[3 * (int64_t)item + 2];
  pos = rg.x + max(wmax - NB - 1 - lane, 0);
  uint32_t mask1 = qm[pos], item1 = pair_items[pos];
  for (int end = wmax; end > 0; end -= NB) {
    const int cnt = min(NB, end);
    uint32_t w = 0;
    if (lane < cnt && mask != 0u) {  // records only of the entries the forward's pixels reached
      S.s0[lane] = make_float4(r0.x, r0.y, r0.z, r0.w);
      const float reach = fabsf(tcx - r0.x) + 9.0f;
      S.s1[lane] = make_float4(r1.x, r1.z, r1.y, 0.0f);
      S.sid[lane] = item;
      S.s2[lane] = make_float4(r2.x, r2.y, r2.z, 0.0f);
      w = 1u | (reach < half ? 0 : kEntryWrap << 4) | (r1.y > kAlphaMax ? kEntryClamp << 4 : 0);
    }
    const uint64_t bl = __builtin_amdgcn_ballot_w64(w != 0u);
    if (w != 0u) S.list[bits_below(bl)] = (uint16_t)(lane | (w << 8));
    const int n = __popcll(bl);
    mask = mask1;
    item = item1;
    // (of the entries not reached too: an unconditional load is issued ahead)
    r0 = recs[3 * (int64_t)item];
    r1 = recs[3 * (int64_t)item + 1];
    r2 = recs[3 * (int64_t)item + 2];
    pos = rg.x + max(end - 2 * NB - 1 - lane, 0);
    mask1 = qm[pos];
    item1 = pair_items[pos];
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += kRingEntries) {
      const int m = min(kRingEntries, n - i0);
      // the group's list words, one per lane; past its end the entry nothing reaches
      const uint32_t words = lane < m ? S.list[i0 + lane] : NB;
      for (int i = 0; i < m; i += kQuadRunBwd) {
        vec4 a[kQuadRunBwd], b[kQuadRunBwd], c[kQuadRunBwd];
        float du[kQuadRunBwd], t1[kQuadRunBwd], t2[kQuadRunBwd], G[kQuadRunBwd], alpha[kQuadRunBwd];
        float wk[kQuadRunBwd], dla[kQuadRunBwd];
        bool ok[kQuadRunBwd];
        int k[kQuadRunBwd];
        uint32_t flags = 0;
#pragma unroll
        for (int j = 0; j < kQuadRunBwd; ++j) {
          const uint32_t km = __builtin_amdgcn_readlane(words, i + j);
          flags |= km;
          k[j] = (int)(km & 0xFFu);
          a[j] = as_vec4(S.s0[k[j]]);
          b[j] = as_vec4(S.s1[k[j]]);
          c[j] = as_vec4(S.s2[k[j]]);
        }
        static_assert(kQuadRunBwd == 2, "the operands of the next line");
        // every read is issued before the first is waited for
        asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]), "+v"(c[0]), "+v"(c[1]));
#pragma unroll
        for (int j = 0; j < kQuadRunBwd; ++j) du[j] = px - a[j].x;
        if (__builtin_expect(opaque((int)(flags >> 12 & kEntryWrap)), 0)) {  // uniform
#pragma unroll
          for (int j = 0; j < kQuadRunBwd; ++j) {
            du[j] = wrap_du(du[j], Wf, half);
            keep_branch(du[j]);
          }
        }
        // the steps of bwd_pixel_step, both entries through each before the next
#pragma unroll
        for (int j = 0; j < kQuadRunBwd; ++j) {
          const float dv = py - a[j].y;
          t1[j] = fmaf(a[j].z, du[j], a[j].w * dv);
          t2[j] = b[j].x * dv;
          const float p = -fmaf(t1[j], t1[j], t2[j] * t2[j]);
          ok[j] = end - 1 - k[j] < P.last && !(p < b[j].y);
          G[j] = ok[j] ? __expf(p) : 0.0f;
          alpha[j] = b[j].z * G[j];
        }
        const int clamp = (int)(flags >> 12 & kEntryClamp);
        if (__builtin_expect(opaque(clamp) != 0, 0)) {  // uniform
#pragma unroll
          for (int j = 0; j < kQuadRunBwd; ++j) {
            alpha[j] = fminf(alpha[j], kAlphaMax);
            keep_branch(alpha[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < kQuadRunBwd; ++j) {
          const float inv_om = __builtin_amdgcn_rcpf(1.0f - alpha[j]);
          P.T = P.T * inv_om;
          wk[j] = alpha[j] * P.T;
          const float dc = fmaf(P.dl0, c[j].x, fmaf(P.dl1, c[j].y, P.dl2 * c[j].z));
          dla[j] = ok[j] ? fmaf(dc, P.T, -P.DS * inv_om) : 0.0f;  // (a select each costs less here than a flag)
          P.DS = fmaf(dc, wk[j], P.DS);
        }
        if (__builtin_expect(opaque(clamp) != 0, 0)) {  // uniform
#pragma unroll
          for (int j = 0; j < kQuadRunBwd; ++j) {
            dla[j] = b[j].z * G[j] > kAlphaMax ? 0.0f : dla[j];
            keep_branch(dla[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < kQuadRunBwd; ++j) {
          if (j > 0 && i + j >= m) break;  // uniform (past an odd group)
          const float dpow = dla[j] * alpha[j], g0 = dpow * t1[j], g1 = dpow * t2[j];
          float g[9] = {g0,            g1,            g0 * t1[j],    g0 * t2[j],   g1 * t2[j],
                        dla[j] * G[j], wk[j] * P.dl0, wk[j] * P.dl1, wk[j] * P.dl2};
          quad_reduce9(g);
          out01[(i + j) * kRingStride] = g[0];
          out01[(i + j) * kRingStride + 16] = g[1];
          out8[(i + j) * kRingStride] = g[8];  // (four lanes write the same value)
        }
      }
      flush_group<BATCH>(S, fl, ring, i0, m, g2d);
    }
  }
}

template <int BIN, int BATCH>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(BATCH > 64 ? 1 : 5))) void render_bwd4_kernel(
    ViewTable vt, const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_items, const Rec* __restrict__ rec,
    const float* __restrict__ ws_T, const int32_t* __restrict__ ws_last, const float* __restrict__ dL_drgb,
    double* __restrict__ g2d, int64_t items, float bg0, float bg1, float bg2, const uint8_t* __restrict__ qmask,
    int64_t qplane, TileSched sc) {
  constexpr int TILE = 16;
  __shared__ Stage4<BATCH> S;
  __shared__ __attribute__((aligned(16))) float ring[kRingEntries * kRingStride];
  if (forward_is_stale(sc)) return;  // uniform
  const int nsplit = reverse_split(sc), nfine = BIN == 32 ? reverse_fine(sc) : 0;
  __shared__ uint32_t s_claim;
  uint32_t round = 0, sel = 0;
  const int lane = threadIdx.x;
  // this lane's words of an entry's ring record
  float* const out01 = ring + (lane >> 4) * kRingRow + (lane & 15);
  float* const out8 = ring + (lane >> 4) * kRingRow + 32 + (lane & 3);
  const FlushLane fl = flush_lane(ring, lane);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  for (int g; (g = claim_task(sc, nsplit, 0, nfine, round, &s_claim, sel)) >= 0;) {
    const int v = view_of_tile(vt, g);
    const int W = vt.W[v], H = vt.H[v];
    int tx0, ty0, pl;
    const bool bits = BIN == 32 && (sel & 0x100u) != 0u;  // the part's masks are four runs of bits
    sel &= 0xFFu;
    task_block<BIN>(vt, v, g, sel, tx0, ty0, pl);
    const int x = tx0 + (lane & 7), y = ty0 + (lane >> 3);
    const float px0 = (float)x + 0.5f, px1 = (float)(x + 8) + 0.5f;
    const float py0 = (float)y + 0.5f, py1 = (float)(y + 8) + 0.5f;
    const float Wf = (float)W, half = wrap_half(vt, v);
    const uint2 rg = ranges[g];
    const int64_t plane = (int64_t)W * H;
    const float* dimg = dL_drgb + 3 * vt.pix_base[v];
    const uint8_t* qm = qmask + (int64_t)pl * qplane;
    auto load_pixel = [&](int q) {
      BwdPixel p;
      const int64_t pix = (int64_t)(y + 8 * (q >> 1)) * W + x + 8 * (q & 1);
      const int64_t gp = vt.pix_base[v] + pix;
      p.dl0 = dimg[pix], p.dl1 = dimg[plane + pix], p.dl2 = dimg[2 * plane + pix];
      p.T = ws_T[gp];
      p.last = ws_last[gp];
      p.DS = p.T * fmaf(p.dl0, bg0, fmaf(p.dl1, bg1, p.dl2 * bg2));
      return p;
    };
    auto wave_max = [](int x) {  // the same in every lane
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) x = max(x, __shfl_xor(x, off));
      return __builtin_amdgcn_readfirstlane(x);
    };
    if (BIN == 16 && sel != 0xFu) {  // uniform: a quadrant of a split tile
      const int q = __builtin_ctz(sel);
      const BwdPixel p = load_pixel(q);
      reverse_quadrant<BATCH>(S, ring, fl, p, q & 1 ? px1 : px0, q >> 1 ? py1 : py0, rg, wave_max(p.last), pair_items, rec,
                              qm, (float)tx0 + 8.0f, Wf, half, g2d);
      continue;
    }
    BwdPixel P[4];  // quadrant q = 2 * qy + qx
    int wmax = 0;
    bool some_large = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      P[q] = load_pixel(q);
      wmax = max(wmax, P[q].last);
      some_large = some_large || pixel_is_large(P[q]);
    }
    const uint32_t large = __builtin_amdgcn_ballot_w64(some_large) != 0ull ? kEntryClamp << 4 : 0;
    wmax = wave_max(wmax);
    for (int end = wmax; end > 0; end -= BATCH) {
      const int cnt = min(BATCH, end);
      // stage entries end - 1 - e (back to front) with their quadrant masks; list those reaching
      // any quadrant, in order
      int n = 0;
      for (int r0 = 0; r0 < cnt; r0 += kWave) {
        const int e = r0 + lane;
        uint32_t m = 0;
        if (e < cnt) {
          const uint32_t pos = rg.x + end - 1 - e;
          m = bits ? part_mask(qm, rg, end - 1 - e) : qm[pos];
          if (m != 0u) {  // records only of the entries the forward's pixels reached
            const uint32_t item = pair_items[pos];
            const Rec r = rec[item];
            S.s0[e] = r.r0;
            const float reach = fabsf((float)tx0 + 0.5f * (float)TILE - r.r0.x) + 0.5f * (float)TILE + 1.0f;
            m |= reach < half ? 0 : kEntryWrap << 4;
            if (r.r1.y > kAlphaMax || is_large(magnitude(r.r2.x, r.r2.y, r.r2.z))) m |= kEntryClamp << 4;
            S.s1[e] = make_float4(r.r1.x, r.r1.z, r.r1.y, 0.0f);
            S.sid[e] = item;
            S.s2[e] = r.r2;
          }
        }
        const uint64_t bl = __builtin_amdgcn_ballot_w64(m != 0u);
        if (m != 0u) S.list[n + __popcll(bl & below)] = (uint16_t)(e | (m << 8));
        n += __popcll(bl);
      }
      __syncthreads();
      for (int i0 = 0; i0 < n; i0 += kRingEntries) {
        const int m = min(kRingEntries, n - i0);
        const uint32_t words = S.list[min(i0 + lane, n - 1)];  // the group's list words, one per lane
        for (int i = 0; i < m; ++i) {
          const uint32_t km = __builtin_amdgcn_readlane(words, i);
          const int k = (int)(km & 0xFFu);
          const int jrel = end - 1 - k;
          const float4 a = S.s0[k];
          const float4 b = S.s1[k];
          const uint32_t mq = km >> 8 | large;
          float du0 = px0 - a.x, du1 = px1 - a.x;
          const float4 c = S.s2[k];
          float gq[9];
#pragma unroll
          for (int q = 0; q < 9; ++q) gq[q] = 0.0f;
          if (mq & (kEntryWrap << 4)) {  // uniform
            du0 = wrap_du(du0, Wf, half);
            du1 = wrap_du(du1, Wf, half);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (!((mq >> q) & 1u)) continue;  // uniform: no pixel of this quadrant reached the entry
            const float dv = (q >> 1 ? py1 : py0) - a.y;
            const float du = q & 1 ? du1 : du0;
            const float t1 = fmaf(a.z, du, a.w * dv), t2 = b.x * dv;
            const float p = -fmaf(t1, t1, t2 * t2);
            const bool ok = jrel < P[q].last && !(p < b.y);
            if (__builtin_amdgcn_ballot_w64(ok) == 0ull) continue;  // uniform
            // (quadrant 0 comes first, so it writes the sums)
            if (q == 0) bwd_pixel_step<false>(P[q], ok, (int)(mq & (kEntryClamp << 4)), p, t1, t2, b, c, gq);
            else bwd_pixel_step<true>(P[q], ok, (int)(mq & (kEntryClamp << 4)), p, t1, t2, b, c, gq);
          }
          quad_reduce9(gq);
          out01[i * kRingStride] = gq[0];
          out01[i * kRingStride + 16] = gq[1];
          if ((lane & 12) == 0) out8[i * kRingStride] = gq[8];
        }
        flush_group<BATCH>(S, fl, ring, i0, m, g2d);
      }
    }
  }
}

__global__ void debug_records_kernel(const Rec* __restrict__ rec, const float* __restrict__ depth,
                                     const uint32_t* __restrict__ count, int64_t items, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= items) return;
  const Rec r = rec[i];
  float* o = out + i * 12;
  o[0] = r.r0.x; o[1] = r.r0.y; o[2] = r.r0.z; o[3] = r.r0.w;
  o[4] = r.r1.x; o[5] = r.r1.y; o[6] = r.r1.z; o[7] = depth[i];
  o[8] = r.r2.x; o[9] = r.r2.y; o[10] = r.r2.z;
  o[11] = (float)count[i];
}

__global__ void debug_keys_kernel(const uint32_t* __restrict__ pkey, const uint32_t* __restrict__ pval,
                                  const float* __restrict__ depth, const odgs_status* __restrict__ status, int64_t cap,
                                  int64_t n, uint64_t* __restrict__ keys, uint32_t* __restrict__ gauss) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t m = min((int64_t)status->n_pairs_stored, cap);
  if (j >= m) return;
  const uint32_t item = pval[j];
  keys[j] = ((uint64_t)pkey[j] << 32) | (uint64_t)__float_as_uint(depth[item]);
  gauss[j] = (uint32_t)(item % n);
}

// Coarse binning: the 16x16 tiles' lists sit in the item buffer in four regions (by quadrant of the
// 32x32 tile); written out in global 16x16 tile order (one workgroup: a scan of the list lengths per
// 1024 tiles, then each wavefront copies whole lists).
__global__ __launch_bounds__(1024) void debug_keys_coarse_kernel(const uint2* __restrict__ ranges, int tiles,
                                                                 const uint32_t* __restrict__ items,
                                                                 const float* __restrict__ depth, int64_t cap,
                                                                 int64_t n, uint64_t* __restrict__ keys,
                                                                 uint32_t* __restrict__ gauss) {
  __shared__ uint32_t wsum[1024 / kWave];
  __shared__ uint32_t s_off[1024];
  __shared__ uint2 s_rg[1024];
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t >> 6;
  int64_t carry = 0;
  for (int base = 0; base < tiles; base += 1024) {
    const uint2 rg = base + t < tiles ? ranges[base + t] : make_uint2(0u, 0u);
    const uint32_t len = rg.y - rg.x;
    uint32_t incl = len;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t pre = 0, total = 0;
    for (int q = 0; q < 1024 / kWave; ++q) {
      pre += q < w ? wsum[q] : 0u;
      total += wsum[q];
    }
    s_off[t] = pre + incl - len;
    s_rg[t] = rg;
    __syncthreads();
    for (int k = w; k < 1024 && base + k < tiles; k += 1024 / kWave) {
      const uint2 r = s_rg[k];
      const int64_t o = carry + s_off[k];
      for (uint32_t j = lane; j < r.y - r.x; j += kWave) {
        const int64_t pos = o + j;
        if (pos < cap) {
          const uint32_t item = items[r.x + j];
          keys[pos] = ((uint64_t)(base + k) << 32) | (uint64_t)__float_as_uint(depth[item]);
          gauss[pos] = (uint32_t)(item % n);
        }
      }
    }
    carry += total;
    __syncthreads();
  }
}

__global__ void debug_pixel_counts_kernel(const int32_t* __restrict__ last, const int32_t* __restrict__ nc,
                                          const int32_t* __restrict__ ne, const int32_t* __restrict__ le,
                                          int64_t pixels, int32_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pixels) return;
  out[4 * i] = last[i];
  out[4 * i + 1] = nc[i];
  out[4 * i + 2] = ne[i];
  out[4 * i + 3] = le[i];
}

template <int TILE, int BATCH>
struct FwdRun {
  static void run(const odgs_plan* p, const TileSched& sc, const ViewTable& vt, const uint2* ranges,
                  const uint32_t* items, const Rec* rec, float* out_rgb, float* out_T, float* wT, int32_t* wl,
                  int32_t* wn, int32_t* we, int32_t* wle, const float* depth, float* out_depth, uint8_t* qmask,
                  hipStream_t st) {
    const bool count = (p->s.flags & ODGS_FLAG_COUNT_WORK) != 0;
#define ODGS_FWD1(C, D)                                                                                             \
  launch_sched(render_fwd_kernel<TILE, BATCH, C, D>, sc, TILE * TILE, st, vt, ranges, items, rec, out_rgb, out_T, wT, \
               wl, wn, we, wle, p->s.bg[0], p->s.bg[1], p->s.bg[2], depth, out_depth, qmask,                         \
               (int64_t)p->pair_capacity)
#define ODGS_FWD4(BIN, SCHED, D)                                                                                     \
  launch_sched(render_fwd4_kernel<BIN, BATCH, D>, SCHED, kWave, st, vt, ranges, items, rec, out_rgb, out_T, wT, wl,     \
               p->s.bg[0], p->s.bg[1], p->s.bg[2], depth, out_depth, qmask, (int64_t)p->pair_capacity)
    // the counting variants keep one pixel per lane (counters per 8x8 quadrant)
    if (count && out_depth)
      ODGS_FWD1(true, true);
    else if (count)
      ODGS_FWD1(true, false);
    else if constexpr (TILE == 8) {
      if (out_depth)
        ODGS_FWD1(false, true);
      else
        ODGS_FWD1(false, false);
    } else {
      const TileSched sc4 = TILE == 16 ? with_split(sc) : with_parts(sc);
      if (out_depth)
        ODGS_FWD4(TILE, sc4, true);
      else
        ODGS_FWD4(TILE, sc4, false);
    }
#undef ODGS_FWD4
#undef ODGS_FWD1
  }
};

template <int TILE, int BATCH>
struct BwdRun {
  static void run(const odgs_plan* p, const TileSched& sc, const ViewTable& vt, const uint2* ranges,
                  const uint32_t* items, const Rec* rec, const float* wT, const int32_t* wl, const float* dL, double* g2d,
                  const uint8_t* qmask, hipStream_t st) {
    // four pixels per lane in one wavefront per 16x16 block (split tiles as the forward split
    // them; 32x32 tiles as four blocks); an 8x8 tile has a single quadrant and keeps one pixel per
    // lane
    if constexpr (TILE == 16)
      launch_sched(render_bwd4_kernel<16, BATCH>, with_split(sc), kWave, st, vt, ranges, items, rec, wT, wl, dL, g2d,
                   p->items, p->s.bg[0], p->s.bg[1], p->s.bg[2], qmask, (int64_t)p->pair_capacity);
    else if constexpr (TILE == 32)
      launch_sched(render_bwd4_kernel<32, BATCH>, with_parts(sc), kWave, st, vt, ranges, items, rec, wT, wl, dL, g2d,
                   p->items, p->s.bg[0], p->s.bg[1], p->s.bg[2], qmask, (int64_t)p->pair_capacity);
    else
      launch_sched(render_bwd_kernel<TILE, BATCH>, sc, TILE * TILE, st, vt, ranges, items, rec, wT, wl, dL, g2d,
                   p->items, p->s.bg[0], p->s.bg[1], p->s.bg[2], qmask);
  }
};

// Dispatch over the supported (tile, batch) pairs; returns false for an unsupported pair.
template <template <int, int> class F, typename... Args>
bool dispatch(int tile, int batch, Args&&... args) {
#define ODGS_CASE(TT, BB)                        \
  if (tile == TT && batch == BB) {               \
    F<TT, BB>::run(std::forward<Args>(args)...); \
    return true;                                 \
  }
  ODGS_CASE(8, 32) ODGS_CASE(8, 64) ODGS_CASE(8, 128) ODGS_CASE(8, 256)
  ODGS_CASE(16, 32) ODGS_CASE(16, 64) ODGS_CASE(16, 128) ODGS_CASE(16, 256)
  ODGS_CASE(32, 64) ODGS_CASE(32, 128) ODGS_CASE(32, 256)
#undef ODGS_CASE
  return false;
}

}  // namespace

hipError_t launch_render_fwd(const odgs_plan* p, void* ws, float* out_rgb, float* out_T, float* out_depth,
                             hipStream_t st) {
  const ViewTable vt = make_view_table(p);
  const int tiles = p->tile_base[p->n_views];
  if (tiles == 0) return hipSuccess;
  const uint2* ranges = ws_ptr<uint2>(ws, p->off_ranges);
  const uint32_t* items = ws_ptr<uint32_t>(ws, p->off_pval[p->pair_final]);
  const Rec* rec = ws_ptr<Rec>(ws, p->off_rec);
  float* wT = ws_ptr<float>(ws, p->off_T);
  int32_t* wl = ws_ptr<int32_t>(ws, p->off_last);
  int32_t* wn = ws_ptr<int32_t>(ws, p->off_ncontrib);
  int32_t* we = ws_ptr<int32_t>(ws, p->off_neval);
  int32_t* wle = ws_ptr<int32_t>(ws, p->off_lasteval);
  const float* depth = ws_ptr<float>(ws, p->off_depth);
  uint8_t* qmask = ws_ptr<uint8_t>(ws, p->off_pval[p->pair_final ^ 1]);  // unused by the sort's result
  const TileSched sc = make_sched(p, ws, 0);
  if (!dispatch<FwdRun>(p->s.tile, p->s.batch, p, sc, vt, ranges, items, rec, out_rgb, out_T, wT, wl, wn, we, wle,
                        depth, out_depth, qmask, st))
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_render_bwd(const odgs_plan* p, void* ws, const float* dL_drgb, hipStream_t st) {
  const ViewTable vt = make_view_table(p);
  const int tiles = p->tile_base[p->n_views];
  if (tiles == 0) return hipSuccess;
  double* g2d = ws_ptr<double>(ws, p->off_g2d);
  const uint2* ranges = ws_ptr<uint2>(ws, p->off_ranges);
  const uint32_t* items = ws_ptr<uint32_t>(ws, p->off_pval[p->pair_final]);
  const Rec* rec = ws_ptr<Rec>(ws, p->off_rec);
  const float* wT = ws_ptr<float>(ws, p->off_T);
  const int32_t* wl = ws_ptr<int32_t>(ws, p->off_last);
  const uint8_t* qmask = ws_ptr<uint8_t>(ws, p->off_pval[p->pair_final ^ 1]);  // written by the forward
  const TileSched sc = make_sched(p, ws, 1);
  if (!dispatch<BwdRun>(p->s.tile, p->s.batch_bwd, p, sc, vt, ranges, items, rec, wT, wl, dL_drgb, g2d, qmask, st))
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_debug_records(const odgs_plan* p, const void* ws, float* out, hipStream_t st) {
  if (p->items == 0) return hipSuccess;
  hipLaunchKernelGGL(debug_records_kernel, dim3((unsigned)((p->items + 255) / 256)), dim3(256), 0, st,
                     ws_ptr<Rec>(ws, p->off_rec), ws_ptr<float>(ws, p->off_depth), ws_ptr<uint32_t>(ws, p->off_count),
                     p->items, out);
  return hipGetLastError();
}

__global__ void debug_copy_kernel(const double* __restrict__ src, int64_t n, double* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t launch_debug_g2d(const odgs_plan* p, const void* ws, double* out, hipStream_t st) {
  const int64_t n = (int64_t)p->g2d_stride * p->items;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(debug_copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     ws_ptr<double>(ws, p->off_g2d), n, out);
  return hipGetLastError();
}

hipError_t launch_debug_pixel_counts(const odgs_plan* p, const void* ws, int32_t* out, hipStream_t st) {
  const int64_t pixels = p->pix_base[p->n_views];
  if (pixels == 0) return hipSuccess;
  hipLaunchKernelGGL(debug_pixel_counts_kernel, dim3((unsigned)((pixels + 255) / 256)), dim3(256), 0, st,
                     ws_ptr<int32_t>(ws, p->off_last), ws_ptr<int32_t>(ws, p->off_ncontrib),
                     ws_ptr<int32_t>(ws, p->off_neval), ws_ptr<int32_t>(ws, p->off_lasteval), pixels, out);
  return hipGetLastError();
}

hipError_t launch_debug_keys(const odgs_plan* p, const void* ws, int64_t cap, uint64_t* keys, uint32_t* gauss,
                             hipStream_t st) {
  if (cap <= 0) return hipSuccess;
  if (p->coarse) {
    hipLaunchKernelGGL(debug_keys_coarse_kernel, dim3(1), dim3(1024), 0, st, ws_ptr<uint2>(ws, p->off_ranges),
                       p->tile_base[p->n_views], ws_ptr<uint32_t>(ws, p->off_pval[p->pair_final]),
                       ws_ptr<float>(ws, p->off_depth), cap, p->n, keys, gauss);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(debug_keys_kernel, dim3((unsigned)((cap + 255) / 256)), dim3(256), 0, st,
                     ws_ptr<uint32_t>(ws, p->off_pkey[p->pair_final]), ws_ptr<uint32_t>(ws, p->off_pval[p->pair_final]),
                     ws_ptr<float>(ws, p->off_depth), ws_ptr<odgs_status>(ws, p->off_status), cap, p->n, keys, gauss);
  return hipGetLastError();
}

}  // namespace odgs
