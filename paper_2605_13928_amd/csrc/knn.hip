// tsne_knn: exact k nearest neighbours by squared Euclidean distance
// (the kNN input of tree-accelerated t-SNE, van der Maaten 2014, Sec. 4.1),
// in two precisions:
//   FP32  -- distances as FP32 direct differences on the VALU;
//   BF16  -- distances between bf16-rounded points from MFMA tiles
//            (v_mfma_f32_16x16x32_bf16, FP32 accumulation; the norms ride
//            in spare K slots, so the tile output IS the distance), the
//            n_cand best per row kept, then re-ranked by FP32 direct
//            differences on the original points.
// Selection (both paths): every row owns a candidate buffer in global
// memory, a count and a threshold tau in registers of the wave that owns
// the row.  A candidate with d <= tau is appended, at a slot counted across
// the wave's lanes (no atomics).  Before a buffer could overflow, the owning
// wave bounds the k-th smallest distance by a radix select, keeps the keys
// up to the bound and makes it the new threshold.  The true k best always
// satisfy d <= tau, so nothing is lost; ties are resolved by index at the
// end (a wave-wide bitonic sort of the (d, j) keys).  Since the kept keys
// are the best ones whatever order the candidates arrive in, both paths
// sweep them in a locality order (points sorted by their nearest of up to 256
// pivots, each query block sweeping outward from its own queries),
// so that tau is tight after a few tiles and few candidates are appended,
// and skip the candidate tiles whose bounding box lies beyond every
// threshold of the block (a bound that leaves the results those of the full
// sweep).
#include <cfloat>
#include <type_traits>

#include "common.hpp"
#include "scan.hpp"

namespace tsne {

// ---------------------------------------------------------------------
// Candidate buffers.

// A row's buffer is only ever written and read by the wave that owns the
// row, so workgroup scope suffices: wait for this wave's stores, no cache
// write-back or invalidation beyond the CU.
__device__ __forceinline__ void wg_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

// base + the number of lanes below this one in the mask.
__device__ __forceinline__ int lane_prefix(uint64_t m, int base) {
  return int(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), uint32_t(base))));
}

// Inclusive prefix sum over the 64 lanes of a wave, in DPP: shifts by 1, 2,
// 4 and 8 within each row of 16 (lanes shifted in from outside the row add
// 0), then row 0's total into row 1 and row 2's into row 3 (row_bcast:15),
// then lane 31's running total into rows 2 and 3 (row_bcast:31).
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// One pass of a radix select over a wave's words v (those with `in` set),
// 8 bits from `shift` up, with a histogram in the wave's 256-entry LDS array
// `hist`: the bin that holds the k-th smallest (by the words' lower bits; the
// higher ones are equal), the number of words below that bin, and in it.
template <int EPL, class In, class Word>
__device__ __forceinline__ void select_pass(uint32_t* __restrict__ hist, int shift, int k, In in, Word word, int& bin,
                                            int& below, int& inside) {
  const int lane = lane_id();
  reinterpret_cast<uint4*>(hist)[lane] = make_uint4(0, 0, 0, 0);
#pragma unroll
  for (int t = 0; t < EPL; ++t)
    if (in(t)) atomicAdd(&hist[(word(t) >> shift) & 255u], 1u);
  const uint4 hv = reinterpret_cast<const uint4*>(hist)[lane];
  const int h[4] = {int(hv.x), int(hv.y), int(hv.z), int(hv.w)};
  const int own = h[0] + h[1] + h[2] + h[3];
  const int incl = wave_incl_scan(own), excl = incl - own;
  const uint64_t owner = __ballot(excl < k && k <= incl);  // exactly one lane
  const int L = __ffsll((unsigned long long)owner) - 1;
  // first bin of this lane whose cumulative count reaches k
  int b = lane * 4, run = excl, hb = h[0];
#pragma unroll
  for (int u = 1; u < 4; ++u) {
    const bool on = run + hb < k;
    b += on ? 1 : 0;
    run += on ? hb : 0;
    hb = on ? h[u] : hb;
  }
  bin = __builtin_amdgcn_readlane(b, L);
  below = __builtin_amdgcn_readlane(run, L);
  inside = __builtin_amdgcn_readlane(hb, L);
}

// Shrink a row's buffer of c keys to those whose distance is at most a bound
// no less than the keep-th smallest (so to the best `keep` by (d, j) and
// perhaps some more), and set tau to that bound.  The bound comes from a
// radix select on the distance bits from the highest bit in which the keys
// differ; it stops once at most `slack` keys more than `keep` lie at or below
// the bin's upper edge (usually after two passes; with slack 0 only an exact
// bound will do).  If ties would leave more than `limit` >= keep + slack
// keys, the tied ones are selected by index and exactly `keep` are kept.  No
// sort: its unrolled masks and code cost the callers registers and
// instruction cache.  The kept keys are written in lane order.  Returns the
// new count.  Called by the whole wave with uniform arguments, c > keep.
constexpr int SLACK = 32;
template <int EPL>
__device__ int compact_row(uint64_t* __restrict__ buf, int c, int keep, int slack, int limit, float& tau,
                           uint32_t* __restrict__ hist) {
  const int lane = lane_id();
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  wg_fence();  // earlier appends of this wave visible to the loads below
  uint64_t v[EPL];
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const int e = t * 64 + lane;
    v[t] = e < c ? buf[e] : KEY_MAX;
  }
  const uint32_t d0 = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v[0] >> 32))));
  uint32_t diff = 0;
#pragma unroll
  for (int t = 0; t < EPL; ++t) diff |= t * 64 + lane < c ? uint32_t(v[t] >> 32) ^ d0 : 0u;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) diff |= xor_lane(diff, m);
  diff = uint32_t(__builtin_amdgcn_readfirstlane(int(diff))) | 255u;
  const int hb = 31 - __builtin_clz(diff);
  int shift = hb - 7;
  uint32_t pmask = ~((2u << hb) - 1u), prefix = d0 & pmask;
  int k = keep, kept;
  for (;;) {
    int bin, below, inside;
    select_pass<EPL>(
        hist, shift, k, [&](int t) { return t * 64 + lane < c && (uint32_t(v[t] >> 32) & pmask) == prefix; },
        [&](int t) { return uint32_t(v[t] >> 32); }, bin, below, inside);
    prefix |= uint32_t(bin) << shift;
    pmask = ~((1u << shift) - 1u);
    k -= below;
    kept = (keep - k) + inside;  // keys with d & pmask <= prefix
    if (shift == 0 || (kept <= keep + slack && (prefix | ~pmask) < 0x7F800000u)) break;
    shift = shift > 8 ? shift - 8 : 0;
  }
  const uint32_t bound = prefix | ~pmask;
  uint32_t last = ~0u;  // largest index kept of the keys at the bound
  if (kept > limit) {   // (then the bound is exact)
    last = 0;
    uint32_t im = 0;
    for (shift = 24; shift >= 0; shift -= 8) {
      int bin, below, inside;
      select_pass<EPL>(
          hist, shift, k,
          [&](int t) {
            return t * 64 + lane < c && uint32_t(v[t] >> 32) == bound && (uint32_t(v[t]) & im) == last;
          },
          [&](int t) { return uint32_t(v[t]); }, bin, below, inside);
      last |= uint32_t(bin) << shift;
      im |= 255u << shift;
      k -= below;
    }
    kept = keep;
  }
  int base = 0;
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const uint32_t d = uint32_t(v[t] >> 32);
    const bool take = t * 64 + lane < c && (d < bound || (d == bound && uint32_t(v[t]) <= last));
    const uint64_t m = __ballot(take);
    if (take) buf[base + __popcll(m & lt)] = v[t];
    base += __popcll(m);
  }
  tau = __uint_as_float(bound);
  wg_fence();
  return kept;
}

// The indices of a row's `keep` best keys, in no order (fewer if it holds
// fewer, then -1): the selection of compact_row without the sort.
template <int EPL>
__device__ void emit_set(uint64_t* __restrict__ buf, int c, int keep, int32_t* __restrict__ oidx,
                         uint32_t* __restrict__ hist) {
  const int lane = lane_id();
  if (c > keep) {
    float tau;
    compact_row<EPL>(buf, c, keep, 0, keep, tau, hist);
  } else {
    wg_fence();
  }
  const int have = c < keep ? c : keep;
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const int e = t * 64 + lane;
    if (e < keep) oidx[e] = e < have ? key_index(buf[e]) : -1;
  }
}

// Sort a row's buffer and write its first `keep` keys out.
template <int EPL>
__device__ void emit_row(const uint64_t* __restrict__ buf, int c, int keep, int32_t* __restrict__ oidx,
                         float* __restrict__ od2) {
  const int lane = lane_id();
  wg_fence();
  uint64_t v[EPL];
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const int e = t * 64 + lane;
    v[t] = e < c ? buf[e] : KEY_MAX;
  }
  wave_sort<EPL>(v);
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const int e = t * 64 + lane;
    if (e < keep) {
      oidx[e] = key_index(v[t]);
      if (od2) od2[e] = key_dist(v[t]);
    }
  }
}

// ---------------------------------------------------------------------
// Tile skipping (both paths).  The points are put in a locality order
// (below), so that a tile of consecutive positions is narrow in the leading
// coordinates; a tile whose box is farther from the box of a wave's
// queries than every threshold of the wave can hold no candidate for it,
// so the wave skips it, and the block fetches only the tiles some wave
// needs.  Boxes span the leading BOX_D coordinates.
constexpr int BOX_D = 32;
// Tiles are tested a window at a time, with the thresholds of that moment.  The
// first window ends where the first compactions have made them finite (without
// that, 64 tiles of 128 columns were all evaluated: 41 % of 20,000 points);
// the next ones double up to the 64 lanes, as the thresholds settle.  Most
// windows end after the first coordinates (all tiles far): four 16-byte loads
// per lane and step, from boxes stored coordinates apart.
// FP32: before a window the rows with more than F_TIGHTEN keys over k are
// compacted, and if at least F_BY_ROW tiles of it stay, the test is repeated
// with each row in place of the box of the wave's rows (a wave that holds rows
// of two clusters has a box between them: 0.41 -> 0.30 ms at 20,011 points).
constexpr int F_WIN0 = 4, B_WIN0 = 8;
constexpr int64_t B_SMALL_N = 1 << 19;  // BF16: 16 queries a wave up to here, 32 above (knn_bf16_kernel)
constexpr int F_TIGHTEN = 64, F_BY_ROW = 2;
// The it-th tile of a sweep: outward from t0 on both sides in turn, cyclically
// (a bijection of [0, nt)).  (Swept upward only, the rows of a block that end
// the run of their cluster met their neighbours last, with thresholds from
// other clusters until then: 1,000,000 points in BF16, 68 -> 57 ms.)
__device__ __forceinline__ int outward(int t0, int it, int nt) {
  const int t = t0 + ((it & 1) ? -((it + 1) >> 1) : it >> 1);
  return t < 0 ? t + nt : (t < nt ? t : t - nt);
}
__device__ __forceinline__ int next_window(int w, int w0) { return w < w0 ? w0 : (w < 64 ? 2 * w : 64); }

// ---------------------------------------------------------------------
// FP32 exact path.  Block = 4 waves x 4 or 8 rows (fknn_few_rows); each step
// covers 128 columns, 2 per lane; the rows' coordinates are LDS broadcasts,
// the columns' are per-lane LDS reads, dimension chunks of 56.  Rows and
// columns are positions of the locality order (Xt = X in that order; perm
// maps a position to its point, which keys and outputs name); a block sweeps
// the column tiles outward from its own rows and skips those the box tests of
// its waves rule out.  What bounds it is the last block, whose rows have
// neighbours in many tiles; thresholds and counts are in one register each (a
// lane per row: arrays of them went to scratch), the next tile in registers
// while this one is consumed.  20,011 points x 50, 30 clusters, k = 90: 2.61
// -> 0.30 ms; 100,000: 24.9 -> 2.0 ms; 40,000 without clusters: 8.5 -> 5.9.

typedef float floatx4_t __attribute__((ext_vector_type(4)));
constexpr int F_COLS = 128;
constexpr int F_DC = 56;
constexpr int XJ_S = F_COLS + 4;  // LDS row strides: multiples of 4 floats keep the
                                  // 16-byte reads aligned and spread the stores' banks
// 4 rows per wave, so that no block is long and all CUs have several: 1,500
// points 0.22 -> 0.17 ms, 20,000 in 30 clusters of many sizes 1.12 -> 0.92
// (of one size 0.30 both ways).  8 rows above 32,768 points (50,000: 0.87
// against 0.90) and, where a tile takes several chunks of coordinates, which
// the rows of a block then re-read, above the 768 blocks of 16 rows that are
// resident at once (points x 200 without clusters: 12,000 2.95 with 4 rows,
// 3.6 with 8; 20,000 9.0, 6.4).
inline bool fknn_few_rows(int64_t n, int d) { return n <= (d <= F_DC ? 32768 : 12288); }

// The rows of the locality order by column tiles, transposed: coordinate c of
// position F_COLS u + r is Xt[(u d + c) F_COLS + r] (zeros past n), so that a
// sweep copies a tile to LDS with 16-byte loads and stores.  A block per
// tile; it also writes the tile's box: box[(c / 2) ntiles + u] holds (min,
// max) of coordinates c, c + 1 < BOX_D over the rows below n ((0, 0) past d;
// NaN left out), coordinates apart so that 64 consecutive tiles are read
// with whole lines.
constexpr int GT_DC = 64;
__global__ __launch_bounds__(256) void gather_tiles_kernel(const float* __restrict__ X, int64_t n, int d,
                                                           int64_t ntiles, const int32_t* __restrict__ perm,
                                                           float* __restrict__ Xt, float2* __restrict__ box) {
  static_assert(BOX_D == 32 && GT_DC >= BOX_D, "eight threads per coordinate of the box");
  __shared__ float t_s[GT_DC * (F_COLS + 1)];
  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int64_t u = blockIdx.x, r0 = u * F_COLS;
  const int rows = int(n - r0 < F_COLS ? n - r0 : F_COLS);
  for (int dc = 0; dc < d; dc += GT_DC) {
    const int dl = d - dc < GT_DC ? d - dc : GT_DC;
    if (dc > 0) __syncthreads();
    for (int r = w; r < F_COLS; r += 32) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int rr = r + 4 * e;
        v[e] = rr < rows && lane < dl ? X[int64_t(perm[r0 + rr]) * d + dc + lane] : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (lane < dl) t_s[lane * (F_COLS + 1) + r + 4 * e] = v[e];
    }
    __syncthreads();
    for (int e = tid; e < dl * F_COLS; e += 256)
      Xt[(u * d + dc) * F_COLS + e] = t_s[(e / F_COLS) * (F_COLS + 1) + e % F_COLS];
    if (dc == 0) {
      const int c = tid >> 3;
      float lo = INFINITY, hi = -INFINITY;
      if (c < d)
        for (int r = tid & 7; r < rows; r += 8) {
          const float v = t_s[c * (F_COLS + 1) + r];
          lo = fminf(lo, v);
          hi = fmaxf(hi, v);
        }
#pragma unroll
      for (int m = 1; m < 8; m <<= 1) {
        lo = fminf(lo, xor_lane_f(lo, m));
        hi = fmaxf(hi, xor_lane_f(hi, m));
      }
      if ((tid & 7) == 0) box[((c >> 1) * ntiles + u) * 2 + (c & 1)] = c < d ? make_float2(lo, hi) : make_float2(0.0f, 0.0f);
    }
  }
}

__device__ __forceinline__ int64_t xt_at(int64_t p, int d, int c) {
  return (p / F_COLS * d + c) * F_COLS + p % F_COLS;
}

// Skipping test of the FP32 path.  Its distance sums d non-negative terms
// (a rounded difference, squared and added by one FMA each), so it is at
// least (1 - (d + 2) u) >= 1 - 2^-15 of the exact one for d <= 256; the
// box bound LB (32 terms) is within 2^-18 of exact.  With the box of a
// wave's rows, LB (1 - 2^-12) > tau_max (the wave's largest threshold)
// therefore means every distance of the tile exceeds every threshold of
// the wave: it would append nothing for it, and skipping it leaves the
// buffers, and the outputs, as the full sweep makes them.  The block
// stages the tiles that some wave evaluates (the OR of the waves' window
// masks, exchanged through LDS).
template <int EPL, int F_RW>
__global__ __launch_bounds__(256, 3) void knn_fp32_kernel(const float* __restrict__ Xt, const int32_t* __restrict__ perm,
                                                       const float4* __restrict__ cbox4, int64_t n, int d, int k,
                                                       uint64_t* __restrict__ bufs, int32_t* __restrict__ out_idx,
                                                       float* __restrict__ out_d2) {
  static_assert(F_RW % 4 == 0 && F_COLS % (4 * F_RW) == 0, "whole 16-byte reads, blocks within a tile");
  constexpr int F_ROWS = 4 * F_RW;
  constexpr int F_UNROLL = F_RW == 8 ? 8 : 1;  // (8 rows: -1 to -3 %; 4 rows: +9 %)
  constexpr int XI_S = F_ROWS + 4;
  constexpr int CAP = 64 * EPL;
  __shared__ __attribute__((aligned(16))) float xi_s[F_DC * XI_S];
  __shared__ __attribute__((aligned(16))) float xj_s[F_DC * XJ_S];
  __shared__ alignas(16) uint32_t hist_s[4][256];  // per-wave radix-select histograms
  __shared__ int32_t pj_s[F_COLS];     // the points of the staged columns
  __shared__ float4 qbox[4][BOX_D / 2];  // box of each wave's rows: (lo, hi) of two coordinates each
  __shared__ uint64_t wmask_s[2][4];     // each wave's live positions, by window parity
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = int64_t(blockIdx.x) * F_ROWS;
  // lane r holds the state of the wave's row r: its threshold (rows past n
  // never accept; nor do the lanes past the rows) and its buffer count
  float tauv = lane < F_RW && row0 + w * F_RW + lane < n ? INFINITY : -INFINITY;
  int cntv = 0;
  auto tau_of = [&](int r) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tauv), r)); };
  auto count_of = [&](int r) { return __builtin_amdgcn_readlane(cntv, r); };
  const int64_t wrow0 = row0 + w * F_RW;  // this wave's rows
  const bool has_rows = wrow0 < n;
  {
    // this wave's box (rows past n left out)
    const int c = lane & 31, g = lane >> 5;
    float lo = INFINITY, hi = -INFINITY;
    if (c < d) {
      for (int r = g; r < F_RW && wrow0 + r < n; r += 2) {
        const float v = Xt[xt_at(wrow0 + r, d, c)];
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
      }
    }
    lo = fminf(lo, xor_lane_f(lo, 32));
    hi = fmaxf(hi, xor_lane_f(hi, 32));
    if (lane < BOX_D)
      reinterpret_cast<float2*>(qbox[w])[lane] = lane < d ? make_float2(lo, hi) : make_float2(0.0f, 0.0f);
  }
  // coordinates dc .. dc + dl - 1 of the block's rows (all in one tile)
  auto stage_rows = [&](int dc, int dl) __attribute__((always_inline)) {
    for (int e = tid; e < dl * F_ROWS; e += 256)
      xi_s[e / F_ROWS * XI_S + e % F_ROWS] = Xt[xt_at(row0 + e % F_ROWS, d, dc + e / F_ROWS)];
  };
  const bool one_chunk = d <= F_DC;
  if (one_chunk) stage_rows(0, d);
  const int ntc = int((n + F_COLS - 1) / F_COLS);
  const int tstart = int(row0 / F_COLS);
  auto tile_of = [&](int it) __attribute__((always_inline)) -> int { return outward(tstart, it, ntc); };
  // live positions of the window [p0, p0 + width): this wave's (returned) and
  // the block's (any wave's, in `blk`); called by all waves together
  int wpar = 0;
  auto window = [&](int p0, int width, uint64_t& blk) __attribute__((always_inline)) -> uint64_t {
    const float tm = -wave_min(-tauv);  // this wave's largest threshold now
    const int p = p0 + lane;
    bool live = has_rows && lane < width && p < ntc;
    if (tm < INFINITY) {
      const float4* tb = cbox4 + tile_of(live ? p : 0);
      float lb = 0.0f;
#pragma unroll 1
      for (int h0 = 0; h0 < BOX_D / 2 && __ballot(live); h0 += 4) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = tb[int64_t(h0 + u) * ntc];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 q = qbox[w][h0 + u];  // (lo, hi) of coordinates 2h and 2h + 1
          const float g0 = fmaxf(fmaxf(v[u].x - q.y, q.x - v[u].y), 0.0f);
          const float g1 = fmaxf(fmaxf(v[u].z - q.w, q.z - v[u].w), 0.0f);
          lb = fmaf(g0, g0, lb);
          lb = fmaf(g1, g1, lb);
        }
        live = live && !(lb * (1.0f - 1.0f / 4096.0f) > tm);
      }
      // the same row by row, where that can save more than it costs
      if (__popcll(__ballot(live)) >= F_BY_ROW) {
        float lr[F_RW];
#pragma unroll
        for (int r = 0; r < F_RW; ++r) lr[r] = 0.0f;
        const int dd = d < BOX_D ? d : BOX_D;
#pragma unroll 2
        for (int c = 0; c < dd; ++c) {
          const float2 v = reinterpret_cast<const float2*>(tb + int64_t(c >> 1) * ntc)[c & 1];
          const float4* xr = reinterpret_cast<const float4*>(Xt + xt_at(wrow0, d, c));
          float x[F_RW];
#pragma unroll
          for (int q4 = 0; q4 < F_RW / 4; ++q4) {
            const float4 xv = xr[q4];
            x[4 * q4] = xv.x;
            x[4 * q4 + 1] = xv.y;
            x[4 * q4 + 2] = xv.z;
            x[4 * q4 + 3] = xv.w;
          }
#pragma unroll
          for (int r = 0; r < F_RW; ++r) {
            const float g = fmaxf(fmaxf(v.x - x[r], x[r] - v.y), 0.0f);
            lr[r] = fmaf(g, g, lr[r]);
          }
        }
        bool any = false;
#pragma unroll
        for (int r = 0; r < F_RW; ++r) any |= !(lr[r] * (1.0f - 1.0f / 4096.0f) > tau_of(r));
        live = live && any;
      }
    }
    const uint64_t mine = __ballot(live);
    // two buffers: a wave may write the next window's mask while another
    // still reads this one's
    if (lane == 0) wmask_s[wpar][w] = mine;
    __syncthreads();
    blk = wmask_s[wpar][0] | wmask_s[wpar][1] | wmask_s[wpar][2] | wmask_s[wpar][3];
    wpar ^= 1;
    return mine;
  };
  // compaction of the rows with more than `above` keys
  auto compact_above = [&](int above) __attribute__((always_inline)) {
    uint64_t need = __ballot(cntv > above);
    while (need) {
      const int r = __builtin_ctzll(need);
      need &= need - 1;
      float nt;
      const int nc = compact_row<EPL>(bufs + (row0 + w * F_RW + r) * CAP, count_of(r), k, SLACK, CAP - F_COLS, nt,
                                      hist_s[w]);
      tauv = lane == r ? nt : tauv;
      cntv = lane == r ? nc : cntv;
    }
  };
  int wb = 0, ww = 0;  // first position and width of the current window (none yet)
  uint64_t win = 0, mine = 0;
  // the next position from p on that some wave evaluates (ntc if none)
  auto find = [&](int p, bool& is_mine) __attribute__((always_inline)) -> int {
    is_mine = false;
    while (p < ntc) {
      if (p >= wb + ww) {
        wb = p;
        ww = next_window(ww, F_WIN0);
        compact_above(k + F_TIGHTEN);
        mine = window(wb, ww, win);
      }
      const uint64_t m = win >> (p - wb);
      if (m) {
        p += __builtin_ctzll(m);
        is_mine = (mine >> (p - wb)) & 1;
        return p;
      }
      p = wb + ww;
    }
    return ntc;
  };
  // A step is a chunk of coordinates of a tile.  The next step's chunk is
  // loaded to registers while this one is consumed from LDS.
  constexpr int PRE = F_DC * F_COLS / 4 / 256;
  floatx4_t pre[PRE] = {};
  int32_t pre_j = -1;
  auto load = [&](int p, int dc) __attribute__((always_inline)) {
    const int64_t u = tile_of(p);
    const floatx4_t* src = reinterpret_cast<const floatx4_t*>(Xt + (u * d + dc) * F_COLS);
    const int len = (d - dc < F_DC ? d - dc : F_DC) * (F_COLS / 4);
#pragma unroll
    for (int e = 0; e < PRE; ++e)
      if (tid + 256 * e < len) pre[e] = src[tid + 256 * e];
    if (dc == 0 && tid < F_COLS) pre_j = u * F_COLS + tid < n ? perm[u * F_COLS + tid] : -1;
  };
  float acc[F_RW][2];
  bool pos_mine = false;
  int dc = 0, pos = find(0, pos_mine);
  if (pos < ntc) load(pos, 0);
  while (pos < ntc) {
    const int64_t c0 = int64_t(tile_of(pos)) * F_COLS;
    const int dl = (d - dc) < F_DC ? (d - dc) : F_DC;
    __syncthreads();  // every wave is done with the previous step
#pragma unroll
    for (int e = 0; e < PRE; ++e) {
      const int at = tid + 256 * e;
      if (at < dl * (F_COLS / 4))
        *reinterpret_cast<floatx4_t*>(&xj_s[at / (F_COLS / 4) * XJ_S + at % (F_COLS / 4) * 4]) = pre[e];
    }
    if (!one_chunk) stage_rows(dc, dl);
    if (dc == 0) {
      if (tid < F_COLS) pj_s[tid] = pre_j;
#pragma unroll
      for (int r = 0; r < F_RW; ++r) acc[r][0] = acc[r][1] = 0.0f;
    }
    int npos = pos, ndc = dc + F_DC;
    bool nmine = pos_mine;
    if (ndc >= d) {
      ndc = 0;
      npos = find(pos + 1, nmine);
    }
    if (npos < ntc) load(npos, ndc);
    __syncthreads();
    if (pos_mine) {  // else no distance of this tile can pass a threshold of this wave
#pragma unroll F_UNROLL
      for (int c = 0; c < dl; ++c) {
        const float4* ap = reinterpret_cast<const float4*>(&xi_s[c * XI_S + w * F_RW]);
        float a[F_RW];
#pragma unroll
        for (int q4 = 0; q4 < F_RW / 4; ++q4) {
          const float4 v = ap[q4];
          a[4 * q4] = v.x;
          a[4 * q4 + 1] = v.y;
          a[4 * q4 + 2] = v.z;
          a[4 * q4 + 3] = v.w;
        }
        const float2 b = *reinterpret_cast<const float2*>(&xj_s[c * XJ_S + lane * 2]);
#pragma unroll
        for (int r = 0; r < F_RW; ++r) {
          const float t0 = a[r] - b.x, t1 = a[r] - b.y;
          acc[r][0] = __builtin_fmaf(t0, t0, acc[r][0]);
          acc[r][1] = __builtin_fmaf(t1, t1, acc[r][1]);
        }
      }
    }
    // filter: one compare per candidate; the append path (and, only in the
    // tail step and the step holding the block's own rows, the index checks)
    // runs when some lane has a candidate at or below its row's threshold
    bool any = false;
#pragma unroll
    for (int r = 0; r < F_RW; ++r) any |= fminf(acc[r][0], acc[r][1]) <= tau_of(r);
    if (pos_mine && ndc == 0 && __ballot(any)) {
      const bool edge = (c0 + F_COLS > n) || (c0 < row0 + F_ROWS && row0 < c0 + F_COLS);
      const int64_t j0 = c0 + lane * 2;
      const int32_t pj0 = pj_s[lane * 2], pj1 = pj_s[lane * 2 + 1];
#pragma unroll
      for (int r = 0; r < F_RW; ++r) {
        const int64_t gi = row0 + w * F_RW + r;
        const float tr = tau_of(r);
        const bool p0 = acc[r][0] <= tr && (!edge || (j0 < n && j0 != gi));
        const bool p1 = acc[r][1] <= tr && (!edge || (j0 + 1 < n && j0 + 1 != gi));
        const uint64_t m0 = __ballot(p0), m1 = __ballot(p1);
        if (m0 | m1) {
          // slots by lane: the counts are wave-uniform, no atomics
          int slot = lane_prefix(m1, lane_prefix(m0, count_of(r)));
          uint64_t* buf = bufs + gi * CAP;
          if (p0) buf[slot++] = make_key(acc[r][0], pj0);
          if (p1) buf[slot] = make_key(acc[r][1], pj1);
          cntv += lane == r ? __popcll(m0) + __popcll(m1) : 0;
        }
      }
      // compaction of rows that could overflow in the next step
      compact_above(CAP - F_COLS);
    }
    pos = npos;
    dc = ndc;
    pos_mine = nmine;
  }
  for (int r = 0; r < F_RW; ++r) {
    const int64_t gi = row0 + w * F_RW + r;
    if (gi >= n) break;
    const int64_t pt = perm[gi];
    uint64_t* buf = bufs + gi * CAP;
    int c = count_of(r);
    // fewer keys to sort where the selection leaves at most 128
    if (c > 128 && k <= 128) {
      float t;
      c = compact_row<EPL>(buf, c, k, SLACK, CAP - F_COLS, t, hist_s[w]);
    }
    if (c <= 128 && k <= 128) emit_row<2>(buf, c, k, out_idx + pt * k, out_d2 + pt * k);
    else emit_row<EPL>(buf, c, k, out_idx + pt * k, out_d2 + pt * k);
  }
}

// ---------------------------------------------------------------------
// BF16 path.

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return uint16_t((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}
__device__ __forceinline__ float bf16_to_f(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

constexpr uint16_t BF16_ONE = 0x3F80;
constexpr uint16_t BF16_INF = 0x7F80;

// Locality order (both paths).  Points are counting-sorted by a 16-bit key:
// the rank of the nearest of up to 256 pivots (points taken at equal steps of
// the input), then a Morton key of two coordinates of the offset from that
// pivot, four bits each.  The cells of the pivots adapt to the clusters of the
// data and are narrow in every coordinate, cells that are near each other get
// near numbers (loc_rank_kernel), and the offsets divide them by the leading
// coordinates, the widest ones of PCA scores.  Position p of the sorted order
// holds point perm[p]; within a key the order is that of the scatter's atomics.
// Nothing downstream depends on any of it (the selection keeps the best keys
// (d, original index) whatever order they arrive in), so non-finite
// coordinates and ties may fall anywhere.
// The pivots alone against a Morton key of the points' first three coordinates,
// whose tiles mix the clusters that overlap in those: 3.6 % of the tiles
// evaluated in place of 42 % (200,000 points x 50 in 30 clusters of one size
// and shape), 6.0 % in place of 14 % (of many sizes, variances falling with the
// coordinate).  Points without clusters need the offsets: with the second
// nearest pivot in their place 1,000,000 normal points of deviations 1 / j took
// 107 ms against 82 with the Morton key, now 71; PCA scores of 10^6 cells
// without clusters 176, 166, 167; c5 at 10^6 points 39.5, 63.3, 35.0; 20,000
// to 32,000 points in uneven clusters 2 to 4 % more than with the second pivot
// or up to 13 % less.
constexpr int LOC_BINS = 1 << 16;
constexpr int LOC_PIV = 256;     // pivots, at most; 64 points per pivot at least
constexpr int LOC_CEN = 32;
constexpr int LOC_SUB = 2;       // coordinates of the offset from the pivot
// Few points keep their own order: at 1,500 x 50 the sweep of all tiles took
// 0.115 ms, the order and the sweep after it 0.17 (4,000: 0.25 and 0.29;
// 8,000: 0.46 and 0.19 to 0.44).
constexpr int64_t LOC_MIN_N = 4096;
inline int loc_kpad(int d) { return (d + 31) / 32 * 32; }
static_assert(LOC_MIN_N / 64 >= LOC_CEN, "at least a pivot per centre");
inline int loc_pivots(int64_t n) { return n / 64 < LOC_PIV ? int(n / 64) : LOC_PIV; }

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// The m <= 256 pivots, a wave each: the row in bf16, padded with zeros to kp
// (a multiple of 32), and its squared norm (infinite for the slots past m and
// for a pivot that is not finite, which are then nearest to nothing).
__global__ __launch_bounds__(256) void loc_pivot_kernel(const float* __restrict__ X, int64_t n, int d, int m, int kp,
                                                        uint16_t* __restrict__ piv, float* __restrict__ pnorm) {
  const int lane = lane_id(), p = blockIdx.x * 4 + (threadIdx.x >> 6);
  const float* row = X + (p < m ? int64_t(p) * n / m : 0) * d;
  float norm = 0.0f;
  for (int c = lane; c < d; c += 64) norm = fmaf(row[c], row[c], norm);
  norm = wave_sum(norm);
  const bool ok = p < m && isfinite(norm);
  for (int c = lane; c < kp; c += 64) piv[p * kp + c] = ok && c < d ? bf16_rne(row[c]) : uint16_t(0);
  if (lane == 0) pnorm[p] = ok ? norm : INFINITY;
}

// The pivots' ranks, one pivot per thread of one block, by their first 32
// coordinates.  Centres are taken among the pivots by farthest-first
// traversal (so every cluster far from the others has one, and all of its
// pivots belong to it), chained from the first to the nearest one not yet
// in the chain, and the pivots are ranked by the place of their centre in
// the chain, then by how much nearer they are to the centre before than to
// the one after it.  (Ranked by a Morton key of centres taken from the first
// 32 pivots, half of 30 equal clusters of 20,000 points fell into two runs,
// and the points of the shorter run were near their neighbours only at the
// far end of their sweep.)
__global__ __launch_bounds__(LOC_PIV) void loc_rank_kernel(const uint16_t* __restrict__ piv,
                                                           const float* __restrict__ pnorm, int kp,
                                                           int* __restrict__ rank, float* __restrict__ scale) {
  __shared__ float4 coord[LOC_PIV][9];  // 8 used: rows of an odd number of 16 bytes
  __shared__ float dist_s[LOC_CEN][LOC_CEN + 1];
  __shared__ int cen_s[LOC_CEN], chain_s[LOC_CEN], place_s[LOC_CEN];
  __shared__ float part_d[2][4];
  __shared__ int part_p[2][4];
  __shared__ ulonglong2 key[LOC_PIV / 2];
  const int p = threadIdx.x, lane = lane_id(), w = p >> 6;
  const bool ok = pnorm[p] < INFINITY;
  uint4 raw[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) raw[u] = reinterpret_cast<const uint4*>(piv + p * kp)[u];
  float x[32];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t h[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[8 * u + 2 * e] = bf16_to_f(uint16_t(h[e]));
      x[8 * u + 2 * e + 1] = bf16_to_f(uint16_t(h[e] >> 16));
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) coord[p][c] = make_float4(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
  __syncthreads();
  auto distance = [&](int q) {  // from this thread's pivot to pivot q
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float4 v = coord[q][c];
      const float u0 = x[4 * c] - v.x, u1 = x[4 * c + 1] - v.y, u2 = x[4 * c + 2] - v.z, u3 = x[4 * c + 3] - v.w;
      s = fmaf(u0, u0, fmaf(u1, u1, fmaf(u2, u2, fmaf(u3, u3, s))));
    }
    return s;
  };
  float near_d = INFINITY;
  int near = 0, cur = 0;
  for (int s = 0; s < LOC_CEN; ++s) {
    if (p == 0) cen_s[s] = cur;
    const float dist = distance(cur);
    if (dist < near_d) {
      near_d = dist;
      near = s;
    }
    // the pivot farthest from its centre (the lowest of several)
    const float v = ok ? near_d : -1.0f;
    const float top = -wave_min(-v);
    const uint64_t who = __ballot(v == top);
    if (lane == 0) {
      part_d[s & 1][w] = top;
      part_p[s & 1][w] = 64 * w + (who ? __builtin_ctzll(who) : 0);
    }
    __syncthreads();
    float best = -2.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (part_d[s & 1][u] > best) {
        best = part_d[s & 1][u];
        cur = part_p[s & 1][u];
      }
  }
  __syncthreads();
  // the offsets' unit: four deviations of the pivots about their centres
#pragma unroll
  for (int c = 0; c < LOC_SUB; ++c) {
    const float4 v = coord[cen_s[near]][0];
    const float r = ok ? x[c] - (c == 0 ? v.x : v.y) : 0.0f;
    const float q = wave_sum(r * r), m = wave_sum(ok ? 1.0f : 0.0f);
    if (lane == 0) {
      part_d[0][w] = q;
      part_d[1][w] = m;
    }
    __syncthreads();
    if (p == 0) {
      float sq = 0.0f, sm = 0.0f;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        sq += part_d[0][u];
        sm += part_d[1][u];
      }
      scale[c] = sq > 0.0f ? 0.25f * sqrtf(sm / sq) : 0.0f;
    }
    __syncthreads();
  }
  for (int e = p; e < LOC_CEN * LOC_CEN; e += LOC_PIV) {
    const int a = e / LOC_CEN, b = e % LOC_CEN;
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float4 v = coord[cen_s[a]][c], y = coord[cen_s[b]][c];
      const float u0 = v.x - y.x, u1 = v.y - y.y, u2 = v.z - y.z, u3 = v.w - y.w;
      s = fmaf(u0, u0, fmaf(u1, u1, fmaf(u2, u2, fmaf(u3, u3, s))));
    }
    dist_s[a][b] = s;
  }
  __syncthreads();
  if (w == 0) {
    int at = 0;
    bool open = lane < LOC_CEN;
    for (int s = 0; s < LOC_CEN; ++s) {
      if (lane == 0) {
        chain_s[s] = at;
        place_s[at] = s;
      }
      open = open && lane != at;
      const float v = open ? dist_s[at][lane & (LOC_CEN - 1)] : INFINITY;
      const float low = wave_min(v);  // (by all lanes)
      const uint64_t who = __ballot(open && v == low);
      // (none is left after the last; distances that are not finite leave the lowest open one)
      const uint64_t left = who ? who : __ballot(open);
      at = left ? __builtin_ctzll(left) : 0;
    }
  }
  __syncthreads();
  const int place = place_s[near];
  const int before = chain_s[place > 0 ? place - 1 : 0], after = chain_s[place + 1 < LOC_CEN ? place + 1 : LOC_CEN - 1];
  const uint32_t t = __float_as_uint(distance(cen_s[before]) - distance(cen_s[after]));
  const uint32_t ord = (t >> 31) ? ~t : t | 0x80000000u;
  // (distinct; the slots past m and pivots that are not finite come last)
  const uint64_t own = (ok ? (uint64_t(place) << 40) | (uint64_t(ord) << 8) : ~uint64_t(255)) | uint64_t(p);
  reinterpret_cast<uint64_t*>(key)[p] = own;
  __syncthreads();
  int r = 0;
#pragma unroll 16
  for (int u = 0; u < LOC_PIV / 2; ++u) {
    const ulonglong2 v = key[u];
    r += (v.x < own ? 1 : 0) + (v.y < own ? 1 : 0);
  }
  rank[p] = r;
}

// key[i] = (rank of the nearest pivot) << 8 | (Morton key of the offset), and
// its count in hist.  A wave takes 32 points against all pivots on the bf16
// matrix cores (the order needs no more precision): MFMA operands lane l,
// pivot or point l % 16, k elements 32 s + 8 (l / 16) .. + 7; result register
// r: pivot 4 (l / 16) + r of the tile, point l % 16.
__global__ __launch_bounds__(256) void loc_key_kernel(const float* __restrict__ X, int64_t n, int d, int m, int kp,
                                                      const uint16_t* __restrict__ piv,
                                                      const float* __restrict__ pnorm, const int* __restrict__ rank,
                                                      const float* __restrict__ scale, uint16_t* __restrict__ key,
                                                      int* __restrict__ hist) {
  constexpr int PT = 2;  // tiles of 16 points
  const int lane = lane_id(), q16 = lane & 15, g4 = lane >> 4;
  const int64_t i0 = (int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * (16 * PT);
  if (i0 >= n) return;
  float best[PT];
  int at[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    best[t] = INFINITY;
    at[t] = 0;
  }
  auto offer = [&](int t, float dist, int u) {
    at[t] = dist < best[t] ? u : at[t];
    best[t] = fminf(dist, best[t]);
  };
  auto point = [&](int t, int k0) {  // 8 coordinates from k0 + 8 g4
    const int64_t i = i0 + 16 * t + q16;
    const float* row = X + (i < n ? i : n - 1) * d;
    bf16x8_t v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = k0 + 8 * g4 + e;
      v[e] = __builtin_bit_cast(__bf16, bf16_rne(c < d ? row[c < d ? c : 0] : 0.0f));
    }
    return v;
  };
  const int tiles = (m + 15) / 16;
  if (kp <= 64) {
    bf16x8_t x[PT][2];
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
      for (int s = 0; s < 2; ++s) x[t][s] = point(t, 32 * s);
    for (int u = 0; u < tiles; ++u) {
      const uint4* pr = reinterpret_cast<const uint4*>(piv + (16 * u + q16) * kp + 8 * g4);
      const bf16x8_t a0 = __builtin_bit_cast(bf16x8_t, pr[0]);
      const bf16x8_t a1 = __builtin_bit_cast(bf16x8_t, kp > 32 ? pr[4] : make_uint4(0, 0, 0, 0));
      const float4 nv = reinterpret_cast<const float4*>(pnorm)[4 * u + g4];
      const float nr[4] = {nv.x, nv.y, nv.z, nv.w};
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        floatx4_t acc = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, x[t][0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, x[t][1], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) offer(t, fmaf(-2.0f, acc[r], nr[r]), 16 * u + 4 * g4 + r);
      }
    }
  } else {
    for (int u = 0; u < tiles; ++u) {
      const float4 nv = reinterpret_cast<const float4*>(pnorm)[4 * u + g4];
      const float nr[4] = {nv.x, nv.y, nv.z, nv.w};
      floatx4_t acc[PT];
#pragma unroll
      for (int t = 0; t < PT; ++t) acc[t] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
      for (int k0 = 0; k0 < kp; k0 += 32) {
        const bf16x8_t a = __builtin_bit_cast(
            bf16x8_t, *reinterpret_cast<const uint4*>(piv + (16 * u + q16) * kp + k0 + 8 * g4));
#pragma unroll
        for (int t = 0; t < PT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, point(t, k0), acc[t], 0, 0, 0);
      }
#pragma unroll
      for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) offer(t, fmaf(-2.0f, acc[t][r], nr[r]), 16 * u + 4 * g4 + r);
    }
  }
  // the four lanes of a point
#pragma unroll
  for (int t = 0; t < PT; ++t) {
#pragma unroll
    for (int s = 16; s < 64; s <<= 1) offer(t, xor_lane_f(best[t], s), int(xor_lane(uint32_t(at[t]), s)));
    const int64_t i = i0 + 16 * t + q16;
    if (g4 == t && i < n) {
      uint32_t q[LOC_SUB], k = uint32_t(rank[at[t]]);
#pragma unroll
      for (int c = 0; c < LOC_SUB; ++c) {
        const float o = c < d ? X[i * d + c] - bf16_to_f(piv[at[t] * kp + c]) : 0.0f;
        q[c] = uint32_t(fminf(fmaxf(fmaf(o, scale[c], 0.5f) * 16.0f, 0.0f), 15.0f));  // (NaN: 0)
      }
#pragma unroll
      for (int b = 3; b >= 0; --b)
#pragma unroll
        for (int c = 0; c < LOC_SUB; ++c) k = k << 1 | ((q[c] >> b) & 1u);
      key[i] = uint16_t(k);
      atomicAdd(&hist[k], 1);
    }
  }
}

__global__ __launch_bounds__(256) void loc_identity_kernel(int64_t n, int32_t* __restrict__ perm) {
  const int64_t i = gtid();
  if (i < n) perm[i] = int32_t(i);
}

// perm[off[key] + rank among the points of that key] = i.
__global__ __launch_bounds__(256) void loc_scatter_kernel(const uint16_t* __restrict__ key, int64_t n,
                                                          const int64_t* __restrict__ off, int* __restrict__ cur,
                                                          int32_t* __restrict__ perm) {
  for (int64_t i = gtid(); i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const uint32_t k = key[i];
    perm[off[k] + atomicAdd(&cur[k], 1)] = int32_t(i);
  }
}

// One wave per position p of the locality order, for point perm[p].
// Query row:      [x~ (d), nh, nm, nl, 1, 1, 1, 0 ...]
// candidate row:  [-2 x~ (d), 1, 1, 1, nh, nm, nl, 0 ...]
// so that <query_i, candidate_j> = |x~_i|^2 + |x~_j|^2 - 2 <x~_i, x~_j>, the
// squared distance of the rounded points; |x~|^2 (FP32) is carried as the
// sum nh + nm + nl of three bf16 parts.  Candidate rows n .. nrows - 1
// (nrows = n + 1 rounded up to a whole tile) are points at infinite
// distance from every query ([0 ..., inf at d + 3, 0 ...]): the last tile
// is filled with them, so the tile loads need no bounds test.
__global__ __launch_bounds__(256) void bf16_prep_kernel(const float* __restrict__ X, int64_t n, int64_t nrows, int d,
                                                        const int32_t* __restrict__ perm, uint16_t* __restrict__ Xq,
                                                        uint16_t* __restrict__ Xc) {
  const int lane = lane_id();
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= nrows) return;
  if (row >= n) {
    Xc[row * 64 + lane] = lane == d + 3 ? BF16_INF : uint16_t(0);
    return;
  }
  const int64_t src = perm[row];
  const bool has = lane < d;
  const uint16_t h = has ? bf16_rne(X[src * d + lane]) : uint16_t(0);
  const float xr = bf16_to_f(h);
  const float nrm = wave_sum(xr * xr);
  const uint16_t nh = bf16_rne(nrm);
  const float r1 = nrm - bf16_to_f(nh);
  const uint16_t nm = bf16_rne(r1);
  const float r2 = r1 - bf16_to_f(nm);
  const uint16_t nl = bf16_rne(r2);
  uint16_t q = 0, c = 0;
  if (has) {
    q = h;
    c = bf16_rne(-2.0f * xr);  // exact: scaling by -2 keeps the 8-bit significand
  } else if (lane < d + 3) {
    const int t = lane - d;
    q = t == 0 ? nh : (t == 1 ? nm : nl);
    c = BF16_ONE;
  } else if (lane < d + 6) {
    const int t = lane - d - 3;
    q = BF16_ONE;
    c = t == 0 ? nh : (t == 1 ? nm : nl);
  }
  Xq[row * 64 + lane] = q;
  Xc[row * 64 + lane] = c;
}

constexpr int B_TJ = 64;  // candidates per LDS tile

// candidate rows: the n points and at least one infinite row, up to a
// whole number of tiles
__host__ __device__ constexpr int64_t bf16_rows(int64_t n) { return (n + B_TJ) / B_TJ * B_TJ; }

// Tile boxes for skipping candidate tiles.  Tile u holds rows
// 64 u .. 64 u + 63 of the locality order (those below n); box[u][c] is
// the (min, max) of the rounded coordinate c over them for c < BOX_D
// ((0, 0) past d), and tnrm[u] bounds their squared norms from above: the
// leading bf16 part nh of a row's FP32 norm is within 2^-9 of it
// (round to nearest), so max nh (1 + 2^-7) bounds the norm.  NaN values
// are left out of the box and of the bound; such a row's distances are
// NaN and never pass a threshold.
__global__ __launch_bounds__(256) void bf16_box_kernel(const uint16_t* __restrict__ Xq, int64_t n, int d,
                                                       int64_t ntiles, float2* __restrict__ box,
                                                       float* __restrict__ tnrm) {
  const int lane = lane_id();
  const int64_t u = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (u >= ntiles) return;
  const int64_t r0 = u * B_TJ;
  const int rows = int(n - r0 < B_TJ ? n - r0 : B_TJ);
  float lo = INFINITY, hi = -INFINITY;
  for (int r = 0; r < rows; ++r) {
    const float v = bf16_to_f(Xq[(r0 + r) * 64 + lane]);
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
  }
  if (lane < BOX_D) box[((lane >> 1) * ntiles + u) * 2 + (lane & 1)] = lane < d ? make_float2(lo, hi) : make_float2(0.0f, 0.0f);
  if (lane == d) tnrm[u] = hi * (1.0f + 1.0f / 128.0f);
}

// LDS tile of B_TJ candidate rows, 8 chunks of 16 bytes each; chunk c of
// row r is stored at r * 8 + (c ^ (r & 7)) so that 16 lanes reading chunk c
// of 16 consecutive rows hit distinct banks.
__device__ __forceinline__ int tile_slot(int r, int c) { return r * 8 + (c ^ (r & 7)); }

// LDS reads that the compiler does not see: it takes every LDS read after a
// direct-to-LDS load for a read of what that load brings and waits for all
// outstanding memory operations first, the prefetch of the other buffer
// included.  The caller has waited for the data; the block waits for the
// reads' results itself.
typedef int intx4_t __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ uint32_t lds_address(const T* p) {
  return uint32_t(uintptr_t((__attribute__((address_space(3))) const T*)p));
}
__device__ __forceinline__ void lds_read_b128(uint32_t at, intx4_t& v) {
  asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(at) : "memory");
}
__device__ __forceinline__ void lds_read2_b128(uint32_t at0, uint32_t at1, bf16x8_t& v0, bf16x8_t& v1) {
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v0), "=&v"(v1)
               : "v"(at0), "v"(at1)
               : "memory");
}

// Block = 4 waves x 16 QT queries, positions of the locality order (Xq, Xc
// and the buffers are in that order; perm maps a position to its point, which
// is what keys and outputs name).  The candidate tiles are swept outward
// from the block's own.  Lane l works on queries 16 t + (l % 16), t < QT, of
// its wave and, per 16-candidate subtile, on candidates 4 (l / 16) .. + 3
// (the MFMA C layout).  A query's threshold and buffer count are held
// (identically) by its four lanes.
// QT = 1 up to B_SMALL_N points, 2 above: few queries a wave make a narrow
// box, little to wait for in the other waves of a block, five waves a SIMD
// and short last blocks; many share a tile's load.  Whole calls on the c5
// points, k = 90, QT = 1 / 2: 20,000 0.92 / 1.22 ms, 250,000 5.7 / 6.8, 600,000
// 18.4 / 17.8, 1,000,000 39 / 35; without clusters 200,000 18.0 / 17.6, 600,000
// 106 / 84.  (QT = 4: 1.4 to 2 times QT = 1 up to 100,000 points, 3 % more
// than QT = 2 at 1,000,000.)
// The kernel is bound by the instructions of the appends (half of a wave's
// time), the waits of its four waves for each other and the last blocks (the
// heaviest of 3907 took 0.75 of the kernel at QT = 4).  What else cost was
// found by clocks in a copy: the compiler's wait for the prefetch of the next
// tile before every LDS read (lds_read_b128), the code and masks of unrolled
// subtiles and sorts (instruction cache, spills), box tests with 64 lines per
// load.  This kernel alone, c5, k = 90: 55 -> 30 ms.
// Tile skipping.  A wave does not evaluate a tile in which no distance can
// pass the threshold of any of its queries, and the block does not
// fetch a tile that none of its waves evaluates.  With B the box of the
// wave's queries
// and T the candidate tile's (leading BOX_D coordinates), LB = sum_c
// gap_c(B, T)^2 is at most the squared distance of any of the queries to
// any candidate of the tile, and the MFMA's distance differs from the
// exact one of the rounded points by less than 2^-15 (N_q + N_c) (64
// products of exact bf16 pairs, FP32 accumulation; N the squared norms, a
// sum of absolute terms of at most 2 (N_q + N_c); the norm's bf16 parts
// add 2^-20 of it), so LB > tau_max + 2^-12 (N_q + N_c), with tau_max the
// wave's largest threshold, means every distance of the tile exceeds every
// threshold of the wave: the tile would append nothing for it, and
// skipping it changes no buffer.  The outputs are those of the full sweep,
// bit for bit, but where squared distances underflow: the matrix cores
// flush what is below 2^-126 to zero, the box test does not.  The test is
// taken for windows of B_WIN0 up to 64 sweep positions at a time (one
// position per lane, a ballot per wave, the four masks OR-ed through LDS),
// with the thresholds of that moment; they only decrease, so a window's
// stale value skips less, never wrongly.
template <int EPL, int QT>
__global__ __launch_bounds__(256, 5) void knn_bf16_kernel(const uint4* __restrict__ Xq, const uint4* __restrict__ Xc,
                                                       const int32_t* __restrict__ perm, const float4* __restrict__ box4,
                                                       const float* __restrict__ tnrm, int64_t n, int d, int ncand,
                                                       uint64_t* __restrict__ bufs, int32_t* __restrict__ cand) {
  static_assert(QT == 1 || QT == 2, "the selects of a query's count");
  constexpr int CAP = 64 * EPL;
  __shared__ uint4 tile[2][B_TJ * 8];  // double-buffered: 64 rows x 128 bytes each
  __shared__ int32_t ptile[2][B_TJ];    // the original indices of those rows
  __shared__ alignas(16) uint32_t hist_s[4][256];   // per-wave radix-select histograms
  __shared__ float4 qbox[4][BOX_D / 2];  // box of each wave's queries: (lo, hi) of two coordinates each
  __shared__ float qnrm_s[4];            // bound on the squared norms of each wave's queries
  __shared__ uint64_t wmask_s[2][4];     // each wave's live positions, by window parity
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q16 = lane & 15, g4 = lane >> 4;
  // indices are 32-bit (n < 2^31 is checked by the caller); products that
  // address memory are taken in 64 bits
  const int n32 = int(n);
  // (a variable: the host pass drops a kernel whose calls of device builtins
  // depend on its template parameters)
  int qpw = 16 * QT;  // queries per wave
  const int qblock = int(blockIdx.x) * 4 * qpw;
  const int qbase = qblock + w * qpw;
  int cnt[QT] = {};  // buffer count of query (t, q16), the same in its four lanes
  // query fragments: tile t, k-step s; lane holds query qbase + 16 t + q16,
  // k elements 32 s + 8 g4 ... + 7
  bf16x8_t bq[QT][2];
  float tau[QT];
  // the subtile filter compares raw bit patterns as signed integers: for a
  // non-negative threshold, d <= tau implies bits(d) <= bits(tau) (a
  // negative d has a negative pattern), so no candidate that passes is
  // filtered out; a negative threshold (the padding queries, or a row whose
  // best distances round below 0) lets every subtile through to the exact
  // per-candidate test
  int tau_key[QT];
  auto key_of = [](float t) { return t >= 0.0f ? __float_as_int(t) : INT_MAX; };
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int qi = qbase + t * 16 + q16;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (qi < n32) v = Xq[int64_t(qi) * 8 + s * 4 + g4];
      bq[t][s] = __builtin_bit_cast(bf16x8_t, v);
    }
    // queries past n never accept; the others accept any finite distance
    // until their buffer is first compacted (the padding rows are infinite)
    tau[t] = qi < n32 ? FLT_MAX : -INFINITY;
    tau_key[t] = key_of(tau[t]);
  }
  // Tiles go from global memory straight to LDS (global_load_lds_dwordx4:
  // lane l of a wave writes the 16 bytes at the wave's LDS base + 16 l), so
  // the swizzle is applied on the global side: LDS slot u holds chunk
  // (u % 8) ^ (row % 8) of row u / 8.  Rows past n are the infinite rows.
  // Thread tid loads slots u = tid and tid + 256: a per-thread source
  // offset fixed for the whole sweep, and a wave-uniform LDS base.
  uint32_t soff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int u = tid + 256 * h;
    const int r = u >> 3;
    soff[h] = uint32_t(r * 8 + ((u & 7) ^ (r & 7)));
  }
  // Wave 0 also brings the tile's 64 entries of perm (padded to whole
  // tiles), so an append reads its candidate's index from LDS.
  auto load_tile = [&](int c0, int b) {
    const uint4* base = Xc + int64_t(c0) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) __builtin_amdgcn_global_load_lds(base + soff[h], tile[b] + 64 * w + 256 * h, 16, 0, 0);
    // (the LDS operand as an explicit element pointer: an array operand is
    // taken by value by this builtin)
    if (w == 0) __builtin_amdgcn_global_load_lds(perm + c0 + lane, &ptile[b][0], 4, 0, 0);
  };
  const int ntiles = (n32 + B_TJ - 1) / B_TJ;
  int t0 = (qblock + 2 * qpw) / B_TJ;  // the block's middle
  t0 = t0 < ntiles ? t0 : ntiles - 1;
  auto tile_of = [&](int it) -> int { return outward(t0, it, ntiles); };
  auto tile_c0 = [&](int it) -> int { return tile_of(it) * B_TJ; };
  // each wave's query box (rows past n repeat the last); the norms' bound is
  // that of the candidate tile they lie in
  const int qt = qbase / B_TJ;
  const bool has_q = qt < ntiles;  // else the wave holds only padding queries
  if (has_q) {
    const int c = lane & 31;
    float lo = INFINITY, hi = -INFINITY;
    for (int r = lane >> 5; r < qpw; r += 2) {
      const int qi = qbase + r < n32 ? qbase + r : n32 - 1;
      const float v = bf16_to_f(reinterpret_cast<const uint16_t*>(Xq)[int64_t(qi) * 64 + c]);
      lo = fminf(lo, v);
      hi = fmaxf(hi, v);
    }
    lo = fminf(lo, xor_lane_f(lo, 32));
    hi = fmaxf(hi, xor_lane_f(hi, 32));
    if (lane < BOX_D)
      reinterpret_cast<float2*>(qbox[w])[lane] = lane < d ? make_float2(lo, hi) : make_float2(0.0f, 0.0f);
    if (lane == 0) qnrm_s[w] = tnrm[qt];
  }
  __syncthreads();
  // live positions of the window [p0, p0 + width): this wave's (returned) and
  // the block's (any wave's, in `blk`); called by all waves together
  int wpar = 0;
  auto window = [&](int p0, int width, uint64_t& blk) -> uint64_t {
    // this wave's largest threshold now (padding queries hold -inf)
    float m4 = tau[0];
#pragma unroll
    for (int t = 1; t < QT; ++t) m4 = fmaxf(m4, tau[t]);
    const float tm = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(-wave_min(-m4))));
    const int p = p0 + lane;
    bool live = has_q && lane < width && p < ntiles;
    if (tm < FLT_MAX) {
      const int t = tile_of(live ? p : 0);
      const float4* tb = box4 + t;
      const float bound = tm + (qnrm_s[w] + tnrm[t]) * (1.0f / 4096.0f);
      float lb = 0.0f;
#pragma unroll 1
      for (int h0 = 0; h0 < BOX_D / 2 && __ballot(live); h0 += 4) {  // (most windows end after the first coordinates)
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = tb[int64_t(h0 + u) * ntiles];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 q = qbox[w][h0 + u];  // (lo, hi) of coordinates 2h and 2h + 1
          const float g0 = fmaxf(fmaxf(v[u].x - q.y, q.x - v[u].y), 0.0f);
          const float g1 = fmaxf(fmaxf(v[u].z - q.w, q.z - v[u].w), 0.0f);
          lb = fmaf(g0, g0, lb);
          lb = fmaf(g1, g1, lb);
        }
        live = live && !(lb > bound);
      }
    }
    const uint64_t mine = __ballot(live);
    // two buffers: a wave may write the next window's mask while another
    // still reads this one's
    if (lane == 0) wmask_s[wpar][w] = mine;
    __syncthreads();
    blk = wmask_s[wpar][0] | wmask_s[wpar][1] | wmask_s[wpar][2] | wmask_s[wpar][3];
    wpar ^= 1;
    return mine;
  };
  int wb = 0, ww = B_WIN0;  // first position and width of the current window
  uint64_t win = 0;
  uint64_t mine = window(0, ww, win);
  int pos = 0, buf = 0;
  bool cur_mine = mine & 1;  // position 0 is live for every wave with queries
  load_tile(tile_c0(0), 0);
  char* const wbuf = reinterpret_cast<char*>(bufs + int64_t(qbase) * CAP);  // the wave's buffers
  const uint32_t q16_off = uint32_t(q16 * CAP * 8);
  while (pos < ntiles) {
    const int c0 = tile_c0(pos);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part of the tile has landed
    __syncthreads();                // ... and every wave's; the other buffer is free
    // the next position some wave evaluates
    int nxt = pos + 1;
    bool nxt_mine = false;
    while (nxt < ntiles) {
      if (nxt >= wb + ww) {
        wb = nxt;
        ww = next_window(ww, B_WIN0);
        mine = window(wb, ww, win);
      }
      const uint64_t m = win >> (nxt - wb);
      if (m) {
        nxt += __builtin_ctzll(m);
        nxt_mine = (mine >> (nxt - wb)) & 1;
        break;
      }
      nxt = wb + ww;
    }
    // fetch the next tile while this one is consumed
    if (nxt < ntiles) load_tile(tile_c0(nxt), buf ^ 1);
    const uint4* tl = tile[buf];
    const int32_t* pt = ptile[buf];
    // tiles that hold some of this block's queries exclude the self pairs;
    // the others need only the threshold test
    auto sweep = [&](auto edge_c) {
      constexpr bool EDGE = decltype(edge_c)::value;
#pragma unroll 1
      for (int sub = 0; sub < B_TJ / 16; ++sub) {
        const int rloc = sub * 16 + q16;
        bf16x8_t a0, a1;
        lds_read2_b128(lds_address(tl + tile_slot(rloc, g4)), lds_address(tl + tile_slot(rloc, 4 + g4)), a0, a1);
        floatx4_t acc[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          acc[t] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bq[t][0], acc[t], 0, 0, 0);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bq[t][1], acc[t], 0, 0, 0);
        }
        // acc[t][r] = distance(query qbase + 16 t + q16, candidate c0 + 16 sub + 4 g4 + r)
        bool any = false;
#pragma unroll
        for (int t = 0; t < QT; ++t)
          any |= min(min(__float_as_int(acc[t][0]), __float_as_int(acc[t][1])),
                     min(__float_as_int(acc[t][2]), __float_as_int(acc[t][3]))) <= tau_key[t];
        if (__ballot(any)) {
          const int jb = c0 + sub * 16 + 4 * g4;
          intx4_t pj;  // perm[jb .. jb + 3]
          lds_read_b128(lds_address(pt + sub * 16 + 4 * g4), pj);
          const int pjr[4] = {pj[0], pj[1], pj[2], pj[3]};
#pragma unroll
          for (int t = 0; t < QT; ++t) {
            const int qi = qbase + t * 16 + q16;
            bool p[4];
            int c = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              p[r] = acc[t][r] <= tau[t] && (!EDGE || jb + r != qi);
              c += int(p[r]);
            }
            if (__ballot(c != 0) == 0) continue;
            // slots of query qi over its four lanes (rows g4 of 16 lanes):
            // exclusive prefix and total of c across the rows, by a 16-lane
            // and a 32-lane permute (no atomics, no memory)
            const auto r16 = __builtin_amdgcn_permlane16_swap(uint32_t(c), uint32_t(c), false, false);
            const int lo = int(r16[0]), hi = int(r16[1]);  // c of rows g4 & ~1 and g4 | 1
            const auto r32 = __builtin_amdgcn_permlane32_swap(uint32_t(lo + hi), uint32_t(lo + hi), false, false);
            const int s01 = int(r32[0]), s23 = int(r32[1]);  // c of rows 0 + 1 and 2 + 3
            int pos = cnt[t] + ((g4 & 1) ? lo : 0) + ((g4 & 2) ? s01 : 0);
            cnt[t] += s01 + s23;
            // byte offset of the next slot from the wave's buffers: a
            // wave-uniform base and a small per-lane offset (no 64-bit
            // pointer per query and t)
            uint32_t at = uint32_t(pos) * 8u + (q16_off + uint32_t(t * 16 * CAP * 8));
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (p[r]) {
                // (a negative distance counts as 0)
                const uint32_t hi = uint32_t(max(__float_as_int(acc[t][r]), 0));
                *reinterpret_cast<uint2*>(wbuf + at) = make_uint2(uint32_t(pjr[r]), hi);
                at += 8u;
              }
          }
        }
      }
    };
    if (cur_mine) {
      if (c0 < qblock + 4 * qpw && qblock < c0 + B_TJ) sweep(std::true_type{});
      else sweep(std::false_type{});
    }
    // compaction of queries that could overflow in the next tile; lanes
    // 0..15 speak for queries 16 t + lane
    uint64_t need = 0;
#pragma unroll
    for (int t = 0; t < QT; ++t) need |= (__ballot(cnt[t] > CAP - B_TJ) & 0xFFFFull) << (16 * t);
    while (need) {
      const int r = __ffsll((unsigned long long)need) - 1;
      need &= need - 1;
      const int t = r >> 4, q = r & 15;
      const int c = __builtin_amdgcn_readlane(t == 0 ? cnt[0] : cnt[QT - 1], q);
      float nt;
      const int nc = compact_row<EPL>(bufs + int64_t(qbase + r) * CAP, c, ncand, SLACK, CAP - B_TJ, nt, hist_s[w]);
#pragma unroll
      for (int tt = 0; tt < QT; ++tt)
        if (tt == t && q16 == q) {
          cnt[tt] = nc;
          tau[tt] = nt;
          tau_key[tt] = key_of(nt);
        }
    }
    buf ^= 1;
    pos = nxt;
    cur_mine = nxt_mine;
  }
  for (int r = 0; r < qpw; ++r) {
    const int qi = qbase + r;
    if (qi >= n32) break;
    const int t = r >> 4;
    const int c = __builtin_amdgcn_readlane(t == 0 ? cnt[0] : cnt[QT - 1], r & 15);
    emit_set<EPL>(bufs + int64_t(qi) * CAP, c, ncand, cand + int64_t(perm[qi]) * ncand, hist_s[w]);
  }
}

// Rows of X padded to dp = d rounded up to 4 (zeros past d), 16-byte
// aligned, for the re-rank's gathers: one wave per row.
__global__ __launch_bounds__(256) void pad_rows_kernel(const float* __restrict__ X, int64_t n, int d, int dp,
                                                       float* __restrict__ Xp) {
  const int64_t i = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int c = lane_id();
  if (i >= n || c >= dp) return;
  Xp[i * dp + c] = c < d ? X[i * d + c] : 0.0f;
}

// Re-rank: one wave per row; FP32 direct differences (same arithmetic as the
// FP32 path: squares accumulated in dimension order) of the row's
// candidates, sorted by (d, j); best k written.  Rows are taken in the
// locality order (wave w re-ranks row perm[w]), so the waves resident at one
// time gather overlapping candidate rows from the caches.  The query row is
// read with uniform (scalar) loads.  The gather of the padded rows Xp (dp <=
// DP floats each) is bound by the 128-byte lines that cross from L2 to L1:
// 64 candidates go straight to LDS, 7 chunks of 16 bytes of each per pass,
// with neighbouring lanes on neighbouring chunks, so that a line crosses
// once (a lane per candidate reads 16 bytes of 64 lines at a time, and they
// are evicted before the next 16 bytes); an odd number of chunks keeps the
// reads of a chunk of 16 rows on distinct banks.  Chunks past dp re-read the
// row's last (in bounds); coordinates past d add an exact 0.
constexpr int RR_C = 7;
template <int DP, bool FULL>
__global__ __launch_bounds__(256) void rerank_kernel(const float* __restrict__ Xp, int64_t n, int dpv,
                                                     const int32_t* __restrict__ perm, const int32_t* __restrict__ cand,
                                                     int ncand, int k, int32_t* __restrict__ out_idx,
                                                     float* __restrict__ out_d2) {
  static_assert(DP % 4 == 0, "whole float4 loads");
  __shared__ float4 rows_s[4][64 * RR_C];
  static_assert(sizeof(rows_s[0]) >= 256 * 8 + 256 * 4, "the keys and the histogram reuse it");
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int64_t pos = int64_t(blockIdx.x) * 4 + w;
  if (pos >= n) return;
  const int64_t row = int64_t(__builtin_amdgcn_readfirstlane(perm[pos]));
  const int dp = FULL ? DP : dpv, last = dp / 4 - 1;
  float4 xi[DP / 4];
#pragma unroll
  for (int u = 0; u < DP / 4; ++u) xi[u] = reinterpret_cast<const float4*>(Xp + row * dp)[u < last ? u : last];
  uint64_t v[4];
  int c = 0;  // candidates (a row short of them, with non-finite input, holds -1 past its own)
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    v[t] = KEY_MAX;
    if (t * 64 >= ncand) continue;
    const int e = t * 64 + lane;
    const int32_t j = e < ncand ? cand[row * ncand + e] : -1;
    const bool valid = j >= 0 && j < n;
    c += __popcll(__ballot(valid));
    const int js = valid ? j : 0;
    int64_t src[RR_C];  // the rows that this lane brings chunks of
#pragma unroll
    for (int u = 0; u < RR_C; ++u)
      src[u] = int64_t(__builtin_amdgcn_ds_bpermute((u * 64 + lane) / RR_C * 4, js)) * (dp / 4);
    float s2 = 0.0f;
#pragma unroll
    for (int c0 = 0; c0 < DP / 4; c0 += RR_C) {
      // the reads of what this overwrites have returned
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
#pragma unroll
      for (int u = 0; u < RR_C; ++u) {
        const int ch = c0 + (u * 64 + lane) % RR_C;
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const float4*>(Xp) + src[u] + (ch < last ? ch : last),
                                         &rows_s[w][u * 64], 16, 0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < RR_C && c0 + u < DP / 4; ++u) {
        const float4 q = rows_s[w][lane * RR_C + u], x = xi[c0 + u];
        if (!FULL && c0 + u > last) break;
        const float u0 = x.x - q.x, u1 = x.y - q.y, u2 = x.z - q.z, u3 = x.w - q.w;
        s2 = __builtin_fmaf(u0, u0, s2);
        s2 = __builtin_fmaf(u1, u1, s2);
        s2 = __builtin_fmaf(u2, u2, s2);
        s2 = __builtin_fmaf(u3, u3, s2);
      }
    }
    if (valid) v[t] = make_key(s2, j);
  }
  // at most 128 keys to sort where that is enough for k
  if (k <= 128) {
    uint64_t* keys = reinterpret_cast<uint64_t*>(rows_s[w]);
    if (c > 128) {
      wg_fence();
#pragma unroll
      for (int t = 0; t < 4; ++t) keys[t * 64 + lane] = v[t];
      float tau;
      c = compact_row<4>(keys, c, k, 128 - k, 128, tau, reinterpret_cast<uint32_t*>(keys + 256));
#pragma unroll
      for (int t = 0; t < 2; ++t) v[t] = t * 64 + lane < c ? keys[t * 64 + lane] : KEY_MAX;
    }
    uint64_t s[2] = {v[0], v[1]};
    wave_sort<2>(s);
    v[0] = s[0];
    v[1] = s[1];
  } else {
    wave_sort<4>(v);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int e = t * 64 + lane;
    if (e < k) {
      out_idx[row * k + e] = key_index(v[t]);
      out_d2[row * k + e] = key_dist(v[t]);
    }
  }
}

// Adds to *out the number of non-finite values among a[0, count): each wave
// sums its lanes' counts and, if any, adds them with one integer atomic.
__global__ __launch_bounds__(256) void count_nonfinite_kernel(const float* __restrict__ a, int64_t count,
                                                              unsigned long long* __restrict__ out) {
  int c = 0;
  for (int64_t i = gtid(); i < count; i += int64_t(gridDim.x) * blockDim.x) c += !isfinite(a[i]);
  c = wave_sum_i(c);
  if (__lane_id() == 0 && c) atomicAdd(out, static_cast<unsigned long long>(c));
}

struct KnnLayout {
  int epl;
  size_t o_buf, o_xq, o_xc, o_xs, o_xp, o_cand, o_perm, o_key, o_piv, o_pnorm, o_prank, o_scale, o_hist, o_cur, o_off, o_bsum, o_box, o_tnrm,
      bytes;
  static KnnLayout make(int64_t n, int d, int precision, int ncand) {
    KnnLayout L;
    Carve c;
    L.epl = 8;  // capacity 512: room for 384 (FP32) or 448 (BF16) appends between compactions
    L.o_buf = c.take(sizeof(uint64_t) * size_t(n) * size_t(64 * L.epl));
    // the locality order (both paths)
    L.o_perm = c.take(sizeof(int32_t) * size_t(bf16_rows(n)));  // padded like the BF16 candidate rows
    L.o_key = c.take(sizeof(uint16_t) * size_t(n));
    L.o_piv = c.take(sizeof(uint16_t) * size_t(loc_kpad(d)) * LOC_PIV);
    L.o_pnorm = c.take(sizeof(float) * LOC_PIV);
    L.o_prank = c.take(sizeof(int) * LOC_PIV);
    L.o_scale = c.take(sizeof(float) * LOC_SUB);
    L.o_hist = c.take(sizeof(int) * LOC_BINS);
    L.o_cur = c.take(sizeof(int) * LOC_BINS);
    L.o_off = c.take(sizeof(int64_t) * (LOC_BINS + 1));
    L.o_bsum = c.take(sizeof(int64_t) * (size_t(ceil_div(LOC_BINS + 1, SCAN_CHUNK)) + 1));
    if (precision == TSNE_KNN_FP32) {
      L.o_xs = c.take(sizeof(float) * size_t(ceil_div(n, F_COLS) * F_COLS) * size_t(d));  // X by column tiles
      L.o_xq = L.o_xc = L.o_cand = L.o_tnrm = L.o_xp = 0;
      L.o_box = c.take(sizeof(float2) * BOX_D * size_t(ceil_div(n, F_COLS)));
    } else {
      L.o_xs = 0;
      L.o_xp = c.take(sizeof(float) * size_t(n) * size_t((d + 3) / 4 * 4));  // X padded, for the re-rank
      L.o_xq = c.take(sizeof(uint16_t) * size_t(n) * 64);
      L.o_xc = c.take(sizeof(uint16_t) * size_t(bf16_rows(n)) * 64);  // + the infinite rows
      L.o_cand = c.take(sizeof(int32_t) * size_t(n) * size_t(ncand));
      L.o_box = c.take(sizeof(float2) * BOX_D * size_t(ceil_div(n, B_TJ)));
      L.o_tnrm = c.take(sizeof(float) * size_t(ceil_div(n, B_TJ)));
    }
    L.bytes = c.off;
    return L;
  }
};

}  // namespace tsne

extern "C" int tsne_knn(const float* X, int64_t n, int32_t d, int32_t k, int32_t precision, int32_t n_cand,
                        int32_t* nbr_idx, float* nbr_d2, int64_t* nonfinite, void* workspace, size_t* workspace_bytes,
                        void* stream) {
  using namespace tsne;
  if (!X || !nbr_idx || !nbr_d2 || n < 2 || d < 1 || k < 1 || k >= n) return TSNE_ERR_INVALID_ARG;
  if (precision != TSNE_KNN_FP32 && precision != TSNE_KNN_BF16) return TSNE_ERR_INVALID_ARG;
  if (precision == TSNE_KNN_BF16 && (n_cand < k || n_cand >= n)) return TSNE_ERR_INVALID_ARG;
  if (k > TSNE_MAX_K || d > TSNE_MAX_D) return TSNE_ERR_UNSUPPORTED;
  if (precision == TSNE_KNN_BF16 && (n_cand > TSNE_MAX_K || d > TSNE_MAX_D_BF16)) return TSNE_ERR_UNSUPPORTED;
  if (n > (int64_t(1) << 31) - 1) return TSNE_ERR_UNSUPPORTED;
  const KnnLayout L = KnnLayout::make(n, d, precision, n_cand);
  int rc = workspace_protocol(workspace, workspace_bytes, L.bytes);
  if (rc >= 0) return rc;
  TSNE_REQUIRE_GFX950();
  char* ws = static_cast<char*>(workspace);
  uint64_t* bufs = reinterpret_cast<uint64_t*>(ws + L.o_buf);
  hipStream_t s = as_stream(stream);
  if (nonfinite) {
    unsigned long long* nf = reinterpret_cast<unsigned long long*>(nonfinite);
    if ((rc = launch_fill<unsigned long long>(nf, 1, 0ull, s))) return rc;
    const int64_t cnt = n * int64_t(d);
    const int64_t blocks = ceil_div(cnt, 256) < 2048 ? ceil_div(cnt, 256) : 2048;
    hipLaunchKernelGGL(count_nonfinite_kernel, dim3(unsigned(blocks)), dim3(256), 0, s, X, cnt, nf);
    TSNE_CHECK_LAUNCH();
  }
  // locality order (both paths): pivots, keys and their counts, offsets,
  // scatter; the input's own order for few points
  uint16_t* piv = reinterpret_cast<uint16_t*>(ws + L.o_piv);
  float* pnorm = reinterpret_cast<float*>(ws + L.o_pnorm);
  int* prank = reinterpret_cast<int*>(ws + L.o_prank);
  float* scale = reinterpret_cast<float*>(ws + L.o_scale);
  uint16_t* key = reinterpret_cast<uint16_t*>(ws + L.o_key);
  int* hist = reinterpret_cast<int*>(ws + L.o_hist);
  int* cur = reinterpret_cast<int*>(ws + L.o_cur);
  int64_t* off = reinterpret_cast<int64_t*>(ws + L.o_off);
  int64_t* bsum = reinterpret_cast<int64_t*>(ws + L.o_bsum);
  int32_t* perm = reinterpret_cast<int32_t*>(ws + L.o_perm);
  if (n <= LOC_MIN_N) {
    hipLaunchKernelGGL(loc_identity_kernel, dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, s, n, perm);
    TSNE_CHECK_LAUNCH();
  } else {
    // (hist and cur are adjacent)
    if ((rc = launch_fill<int>(hist, 2 * LOC_BINS, 0, s))) return rc;
    const dim3 lgrid(unsigned(ceil_div(n, 256) < 2048 ? ceil_div(n, 256) : 2048));
    const int m = loc_pivots(n), kp = loc_kpad(d);
    hipLaunchKernelGGL(loc_pivot_kernel, dim3(LOC_PIV / 4), dim3(256), 0, s, X, n, d, m, kp, piv, pnorm);
    TSNE_CHECK_LAUNCH();
    hipLaunchKernelGGL(loc_rank_kernel, dim3(1), dim3(LOC_PIV), 0, s, piv, pnorm, kp, prank, scale);
    TSNE_CHECK_LAUNCH();
    hipLaunchKernelGGL(loc_key_kernel, dim3(unsigned(ceil_div(n, 128))), dim3(256), 0, s, X, n, d, m, kp, piv, pnorm,
                       prank, scale, key, hist);
    TSNE_CHECK_LAUNCH();
    if ((rc = exclusive_scan<int>(hist, LOC_BINS, off, bsum, s))) return rc;
    hipLaunchKernelGGL(loc_scatter_kernel, lgrid, dim3(256), 0, s, key, n, off, cur, perm);
    TSNE_CHECK_LAUNCH();
  }
  if (precision == TSNE_KNN_FP32) {
    float* Xs = reinterpret_cast<float*>(ws + L.o_xs);
    float2* box = reinterpret_cast<float2*>(ws + L.o_box);
    const int64_t ntc = ceil_div(n, F_COLS);
    hipLaunchKernelGGL(gather_tiles_kernel, dim3(unsigned(ntc)), dim3(256), 0, s, X, n, d, ntc, perm, Xs, box);
    TSNE_CHECK_LAUNCH();
    const float4* box4 = reinterpret_cast<const float4*>(box);
    if (fknn_few_rows(n, d))
      hipLaunchKernelGGL((knn_fp32_kernel<8, 4>), dim3(unsigned(ceil_div(n, 16))), dim3(256), 0, s, Xs, perm, box4, n, d,
                         k, bufs, nbr_idx, nbr_d2);
    else
      hipLaunchKernelGGL((knn_fp32_kernel<8, 8>), dim3(unsigned(ceil_div(n, 32))), dim3(256), 0, s, Xs, perm, box4, n, d,
                         k, bufs, nbr_idx, nbr_d2);
    TSNE_CHECK_LAUNCH();
    return TSNE_OK;
  }
  uint16_t* Xq = reinterpret_cast<uint16_t*>(ws + L.o_xq);
  uint16_t* Xc = reinterpret_cast<uint16_t*>(ws + L.o_xc);
  int32_t* cand = reinterpret_cast<int32_t*>(ws + L.o_cand);
  // the padding of perm (the infinite candidate rows) names point 0; such a
  // candidate never passes a threshold, so the value is never used
  if ((rc = launch_fill<int32_t>(perm + n, bf16_rows(n) - n, 0, s))) return rc;
  hipLaunchKernelGGL(bf16_prep_kernel, dim3(unsigned(ceil_div(bf16_rows(n), 4))), dim3(256), 0, s, X, n, bf16_rows(n),
                     d, perm, Xq, Xc);
  TSNE_CHECK_LAUNCH();
  const int64_t ntiles = ceil_div(n, B_TJ);
  float2* box = reinterpret_cast<float2*>(ws + L.o_box);
  float* tnrm = reinterpret_cast<float*>(ws + L.o_tnrm);
  hipLaunchKernelGGL(bf16_box_kernel, dim3(unsigned(ceil_div(ntiles, 4))), dim3(256), 0, s, Xq, n, d, ntiles, box, tnrm);
  TSNE_CHECK_LAUNCH();
  const uint4 *Xq4 = reinterpret_cast<const uint4*>(Xq), *Xc4 = reinterpret_cast<const uint4*>(Xc);
  const float4* box4 = reinterpret_cast<const float4*>(box);
  if (n <= B_SMALL_N)
    hipLaunchKernelGGL((knn_bf16_kernel<8, 1>), dim3(unsigned(ceil_div(n, 64))), dim3(256), 0, s, Xq4, Xc4, perm, box4,
                       tnrm, n, d, n_cand, bufs, cand);
  else
    hipLaunchKernelGGL((knn_bf16_kernel<8, 2>), dim3(unsigned(ceil_div(n, 128))), dim3(256), 0, s, Xq4, Xc4, perm, box4,
                       tnrm, n, d, n_cand, bufs, cand);
  TSNE_CHECK_LAUNCH();
  const int dp = (d + 3) / 4 * 4;
  float* Xp = reinterpret_cast<float*>(ws + L.o_xp);
  hipLaunchKernelGGL(pad_rows_kernel, dim3(unsigned(ceil_div(n, 4))), dim3(256), 0, s, X, n, d, dp, Xp);
  TSNE_CHECK_LAUNCH();
  // the exact width for the common 50-coordinate input, else the largest
  if (dp == 52)
    hipLaunchKernelGGL((rerank_kernel<52, true>), dim3(unsigned(ceil_div(n, 4))), dim3(256), 0, s, Xp, n, dp, perm, cand,
                       n_cand, k, nbr_idx, nbr_d2);
  else
    hipLaunchKernelGGL((rerank_kernel<(TSNE_MAX_D_BF16 + 3) / 4 * 4, false>), dim3(unsigned(ceil_div(n, 4))), dim3(256), 0, s,
                       Xp, n, dp, perm, cand, n_cand, k, nbr_idx, nbr_d2);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}
