// tsne_kl_grad_fft: t-SNE gradient (van der Maaten & Hinton 2008, eq. 5)
// with the repulsive sums and Z approximated by FFT-accelerated polynomial
// interpolation (Linderman, Rachh, Hoskins, Steinerberger & Kluger 2019,
// Nat. Methods 16, 243-245); the attraction stays exact over the CSR rows.
//
// Per call, all on the stream, no host synchronisation:
//   bbox_kernel / params_kernel  the square domain [lo, lo + B h]^2, B boxes
//                                of side h per axis, p x p nodes per box at
//                                local positions (k + 1/2) / p, so N = p B
//                                equispaced nodes (spacing h / p) per axis;
//                                FFT size F = smallest power of two >= 2 N.
//   count / scan / scatter       the points sorted by box (counting sort).
//   accum_kernel                 16 lanes per box sum its points' charges
//                                1, z_x, z_y (z = y - centre) times the
//                                tensor Lagrange weights into the box's
//                                p x p nodes, in 64-bit fixed point (exact,
//                                so independent of the order the scatter
//                                leaves: deterministic), and writes them;
//                                every node belongs to exactly one box.
//   rows_fwd / cols / rows_inv   the 2-D circular convolution by FP64 FFTs
//                                (equal to the linear one for F >= 2N) of
//                                three complex grids: W0, W1 + i W2, and
//                                K1 + i K2 with K1 = 1 / (1 + r^2), K2 = K1^2
//                                at the node offsets.  The kernels are even,
//                                so their spectra are real: FFT(W0) (K1^ + i
//                                K2^) transforms back to phi1 + i phi2 and
//                                (W1^ + i W2^) K2^ to phi3x + i phi3y -- three
//                                forward and two inverse transforms.
//   gather_kernel                each point interpolates the four node
//                                potentials: R_i = z_i phi2 - (phi3x, phi3y),
//                                Z = sum_i phi1_i - n (the j = i terms).
//   finalize (klgrad.hip)        CSR attraction, g = 4 (alpha A - R / Z), KL.
// Every size is read from the parameters on the device; the launches and
// the workspace are sized for the largest FFT the caller allows.
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "klgrad.hpp"
#include "scan.hpp"

namespace tsne {

constexpr int FI_GRID = 512;    // blocks of the point passes (and Z partials)
constexpr int FI_MAX_P = 5;     // interpolation nodes per box and axis
constexpr int FI_MIN_FFT = 64;  // FFT sizes: powers of two in [64, 4096]
constexpr int FI_MAX_FFT = 4096;

struct FiParams {
  double lo, h, c, scale;  // domain origin, box side, centre, fixed-point scale
  int B, N, F, logF;
};

// --- domain ------------------------------------------------------------

__global__ __launch_bounds__(256) void fi_bbox_kernel(const float2* __restrict__ Y, int64_t n,
                                                      float* __restrict__ part) {
  float mn = INFINITY, mx = -INFINITY;
  for (int64_t i = gtid(); i < n; i += int64_t(gridDim.x) * 256) {
    const float2 y = Y[i];
    mn = fminf(mn, fminf(y.x, y.y));
    mx = fmaxf(mx, fmaxf(y.x, y.y));
  }
  __shared__ float smn[4], smx[4];
  mn = wave_min(mn);
  mx = -wave_min(-mx);
  if (lane_id() == 0) {
    smn[threadIdx.x >> 6] = mn;
    smx[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = fminf(fminf(smn[0], smn[1]), fminf(smn[2], smn[3]));
    part[2 * blockIdx.x + 1] = fmaxf(fmaxf(smx[0], smx[1]), fmaxf(smx[2], smx[3]));
  }
}

// One block: reduce the bounding box, fix the grid and fill the FFTs' twiddle
// table.  min and max are exact in any order; range and h are FP64
// operations on those floats.
__global__ __launch_bounds__(256) void fi_params_kernel(const float* __restrict__ part, int nb, int64_t n, int p,
                                                        int min_boxes, float max_box_width, int max_fft,
                                                        FiParams* __restrict__ out, double2* __restrict__ tw,
                                                        int* __restrict__ nheavy) {
  __shared__ int size;
  float mn = INFINITY, mx = -INFINITY;
  for (int b = threadIdx.x; b < nb; b += 256) {
    mn = fminf(mn, part[2 * b]);
    mx = fmaxf(mx, part[2 * b + 1]);
  }
  __shared__ float smn[4], smx[4];
  mn = wave_min(mn);
  mx = -wave_min(-mx);
  if (lane_id() == 0) {
    smn[threadIdx.x >> 6] = mn;
    smx[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double lo = double(fminf(fminf(smn[0], smn[1]), fminf(smn[2], smn[3])));
    const double hi = double(fmaxf(fmaxf(smx[0], smx[1]), fmaxf(smx[2], smx[3])));
    double rng = hi - lo;
    if (!isfinite(lo) || !isfinite(rng)) {  // non-finite input: any valid grid (results are not finite)
      lo = 0.0;
      rng = 1e-3;
    }
    if (!(rng > 0.0)) rng = 1e-3;
    double Bd = ceil(rng / double(max_box_width));
    Bd = fmax(Bd, double(min_boxes));
    Bd = fmin(Bd, double(max_fft / (2 * p)));
    const int B = int(Bd);
    const int N = p * B;
    int F = FI_MIN_FFT, logF = 6;
    while (F < 2 * N) {
      F <<= 1;
      ++logF;
    }
    FiParams P;
    P.lo = lo;
    P.h = rng / double(B);
    P.c = lo + 0.5 * rng;
    // fixed point: every node sum is at most n (|z| + 1) times the square of
    // the largest Lagrange weight on [0, 1] (1.5, 1.88, 2.19, 3.28 for
    // p = 2 .. 5: squared < 16); keep it below 2^62
    const double bound = double(n) * (0.5 * rng + 1.0) * 16.0;
    P.scale = exp2(floor(log2(4.611686018427388e18 / bound)));
    P.B = B;
    P.N = N;
    P.F = F;
    P.logF = logF;
    *out = P;
    *nheavy = 0;
    size = F;
  }
  __syncthreads();
  // the FFTs' twiddles exp(-2 pi i k / F)
  for (int k = threadIdx.x; k < size; k += 256) {
    double sn, cs;
    sincospi(-2.0 * double(k) / double(size), &sn, &cs);
    tw[k] = make_double2(cs, sn);
  }
}

// 1 / prod_{m != k} (t_k - t_m) of the nodes t_k = (k + 1/2) / P: the
// Lagrange weights as products without divisions.
template <int P>
__device__ __forceinline__ constexpr double fi_denom(int k) {
  double d = 1.0;
  for (int m = 0; m < P; ++m)
    if (m != k) d *= double(k - m);
  double pw = 1.0;
  for (int m = 1; m < P; ++m) pw *= double(P);
  return pw / d;
}

// Box index and Lagrange weights of one coordinate (t = (y - lo) / h, b =
// floor(t) clamped, as in the definition).
template <int P>
__device__ __forceinline__ int fi_weights(float y, const FiParams& g, double (&L)[P]) {
  const double t = (double(y) - g.lo) / g.h;
  const double bd = fmin(fmax(floor(t), 0.0), double(g.B - 1));
  const double u = t - bd;
#pragma unroll
  for (int k = 0; k < P; ++k) {
    double v = fi_denom<P>(k);
#pragma unroll
    for (int m = 0; m < P; ++m)
      if (m != k) v *= u - (double(m) + 0.5) / double(P);
    L[k] = v;
  }
  return int(bd);
}

// --- spread ------------------------------------------------------------

// Box of a point (the same clamped FP64 floor as fi_weights).
__device__ __forceinline__ int fi_box(float y, const FiParams& g) {
  const double t = (double(y) - g.lo) / g.h;
  return int(fmin(fmax(floor(t), 0.0), double(g.B - 1)));
}

// Counting sort of the points by box, with the counts gathered per block: a
// block counts its FI_CPTS points in an LDS table (open addressing, at most
// FI_PROBE probes; a key that finds no slot is counted in global memory
// directly) and adds each distinct box once.  When most points fall in a few
// boxes (a compact or clustered embedding) this replaces the contended
// global atomics on those boxes' counters by one per block.  The atomics
// return each point's rank within its box, so that the scatter after the
// prefix sum is a plain pass (counting and hashing a second time there took
// 75 us at 10^6 points).
constexpr int FI_CPPT = 4;              // points per thread
constexpr int FI_CPTS = 256 * FI_CPPT;  // points per block
constexpr int FI_TBL = 2048;            // LDS slots per block
constexpr int FI_PROBE = 8;

__device__ __forceinline__ int fi_tbl_find(int* tkey, int key) {
  const uint32_t h = uint32_t(key) * 2654435761u;
  for (int q = 0; q < FI_PROBE; ++q) {
    const int slot = int((h + uint32_t(q)) & (FI_TBL - 1));
    const int prev = atomicCAS(&tkey[slot], -1, key);
    if (prev == key || prev == -1) return slot;
  }
  return -1;
}

__global__ __launch_bounds__(256) void fi_count_kernel(const float2* __restrict__ Y, int64_t n,
                                                       const FiParams* __restrict__ gp, int* __restrict__ cnt,
                                                       int2* __restrict__ where) {
  __shared__ int tkey[FI_TBL], tcnt[FI_TBL];
  const FiParams g = *gp;
  for (int q = threadIdx.x; q < FI_TBL; q += 256) {
    tkey[q] = -1;
    tcnt[q] = 0;
  }
  const int64_t i0 = int64_t(blockIdx.x) * FI_CPTS + threadIdx.x;
  float2 y[FI_CPPT];
#pragma unroll
  for (int u = 0; u < FI_CPPT; ++u) y[u] = Y[i0 + 256 * u < n ? i0 + 256 * u : n - 1];
  __syncthreads();
  int box[FI_CPPT], slot[FI_CPPT], rank[FI_CPPT];
#pragma unroll
  for (int u = 0; u < FI_CPPT; ++u) {
    if (i0 + 256 * u >= n) continue;
    box[u] = fi_box(y[u].x, g) * g.B + fi_box(y[u].y, g);
    slot[u] = fi_tbl_find(tkey, box[u]);
    rank[u] = slot[u] >= 0 ? atomicAdd(&tcnt[slot[u]], 1) : atomicAdd(&cnt[box[u]], 1);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < FI_TBL; q += 256)
    if (tcnt[q]) tcnt[q] = atomicAdd(&cnt[tkey[q]], tcnt[q]);  // the block's start within the box
  __syncthreads();
#pragma unroll
  for (int u = 0; u < FI_CPPT; ++u)
    if (i0 + 256 * u < n) where[i0 + 256 * u] = make_int2(box[u], rank[u] + (slot[u] >= 0 ? tcnt[slot[u]] : 0));
}

__global__ __launch_bounds__(256) void fi_scatter_kernel(int64_t n, const int2* __restrict__ where,
                                                         const int64_t* __restrict__ off,
                                                         int32_t* __restrict__ order) {
  const int64_t i = gtid();
  if (i >= n) return;
  const int2 w = where[i];
  order[off[w.x] + w.y] = int32_t(i);
}

// Node sums.  16 lanes (a DPP row) share a box: each adds its points'
// charges 1, z_x, z_y times the tensor Lagrange weights in registers, 64-bit
// fixed point, then the 16 sums are added by row rotations (integers: exact
// in any order).  A box of more than FI_HEAVY points (a compact or clustered
// embedding can put most points in a few boxes) is cut into chunks of
// FI_HEAVY points, listed by the pass over the boxes and added by a second
// kernel.  One thread per box (64-point chunks) took 183 + 97 us at 10^6
// points in 13,000 boxes and 78 us at 70,000: a thread walked its 8 to 64
// points one dependent gather after another, on a third of the chip's
// wavefronts; 16 lanes take 32 + 19 us and 9 us.
constexpr int FI_HEAVY = 256;
constexpr int FI_BATCH = 4;  // points of a lane in flight

template <int P>
__device__ __forceinline__ void fi_accum_point(float2 y, const FiParams& g, long long (&acc)[3][P][P]) {
  double Lx[P], Ly[P];
  fi_weights<P>(y.x, g, Lx);
  fi_weights<P>(y.y, g, Ly);
  const double zx = double(y.x) - g.c, zy = double(y.y) - g.c;
#pragma unroll
  for (int kx = 0; kx < P; ++kx) {
#pragma unroll
    for (int ky = 0; ky < P; ++ky) {
      const double w = Lx[kx] * Ly[ky] * g.scale;
      acc[0][kx][ky] += __double2ll_rn(w);
      acc[1][kx][ky] += __double2ll_rn(w * zx);
      acc[2][kx][ky] += __double2ll_rn(w * zy);
    }
  }
}

// Sums over the sorted points [e0, e1) of one box by the 16 lanes of a row;
// every lane ends with the total.
template <int P>
__device__ __forceinline__ void fi_accum_range(const float2* __restrict__ Y, const FiParams& g,
                                               const int32_t* __restrict__ order, int64_t e0, int64_t e1,
                                               long long (&acc)[3][P][P]) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int kx = 0; kx < P; ++kx)
#pragma unroll
      for (int ky = 0; ky < P; ++ky) acc[c][kx][ky] = 0;
  for (int64_t e = e0 + (lane_id() & 15); e < e1; e += 16 * FI_BATCH) {
    int32_t ix[FI_BATCH];
    float2 yv[FI_BATCH];
#pragma unroll
    for (int u = 0; u < FI_BATCH; ++u) ix[u] = order[e + 16 * u < e1 ? e + 16 * u : e];
#pragma unroll
    for (int u = 0; u < FI_BATCH; ++u) yv[u] = Y[ix[u]];
#pragma unroll
    for (int u = 0; u < FI_BATCH; ++u)
      if (e + 16 * u < e1) fi_accum_point<P>(yv[u], g, acc);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int kx = 0; kx < P; ++kx)
#pragma unroll
      for (int ky = 0; ky < P; ++ky) {
        uint64_t v = uint64_t(acc[c][kx][ky]);
        auto rot = [&](auto ctrl) {
          constexpr int C = decltype(ctrl)::value;
          v += (uint64_t(uint32_t(dpp_i<C>(int(uint32_t(v >> 32))))) << 32) | uint32_t(dpp_i<C>(int(uint32_t(v))));
        };
        rot(std::integral_constant<int, 0x128>{});
        rot(std::integral_constant<int, 0x124>{});
        rot(std::integral_constant<int, 0x122>{});
        rot(std::integral_constant<int, 0x121>{});
        acc[c][kx][ky] = (long long)v;
      }
}

// Node sums of every box: channel c at G + c N^2, node (gx, gy) at gx N +
// gy.  A heavy box gets zeros here and its chunks in `heavy` (box and chunk
// number; their order follows the counter's atomics and reaches no result).
template <int P>
__global__ __launch_bounds__(256) void fi_accum_kernel(const float2* __restrict__ Y,
                                                       const FiParams* __restrict__ gp,
                                                       const int64_t* __restrict__ off,
                                                       const int32_t* __restrict__ order,
                                                       unsigned long long* __restrict__ G, int* __restrict__ nheavy,
                                                       int2* __restrict__ heavy) {
  const FiParams g = *gp;
  const int nb = g.B * g.B;
  const int64_t NN = int64_t(g.N) * g.N;
  const int sl = lane_id() & 15;
  // whole rows of 16 lanes run or stop together
  for (int b = int(gtid() >> 4); b < nb; b += int(gridDim.x) * 16) {
    const int64_t e0 = off[b], e1 = off[b + 1];
    const bool light = e1 - e0 <= FI_HEAVY;
    if (!light && sl == 0) {
      const int nc = int((e1 - e0 + FI_HEAVY - 1) / FI_HEAVY);
      const int at = atomicAdd(nheavy, nc);
      for (int c = 0; c < nc; ++c) heavy[at + c] = make_int2(b, c);
    }
    long long acc[3][P][P];
    fi_accum_range<P>(Y, g, order, e0, light ? e1 : e0, acc);
    const int bx = b / g.B, by = b % g.B;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int kx = 0; kx < P; ++kx)
#pragma unroll
        for (int ky = 0; ky < P; ++ky)
          if (sl == (c * P * P + kx * P + ky) % 16)
            G[c * NN + int64_t(P * bx + kx) * g.N + (P * by + ky)] = (unsigned long long)acc[c][kx][ky];
  }
}

// The listed chunks, 16 lanes each, added to the nodes their box zeroed.
// The four rows of a wave add their sums first when they share the box.
template <int P>
__global__ __launch_bounds__(256) void fi_accum_heavy_kernel(const float2* __restrict__ Y,
                                                             const FiParams* __restrict__ gp,
                                                             const int64_t* __restrict__ off,
                                                             const int32_t* __restrict__ order,
                                                             const int* __restrict__ nheavy,
                                                             const int2* __restrict__ heavy,
                                                             unsigned long long* __restrict__ G) {
  const FiParams g = *gp;
  const int H = *nheavy;
  const int64_t NN = int64_t(g.N) * g.N;
  const int lane = lane_id(), sl = lane & 15;
  for (int c0 = int(gtid() >> 6) * 4; c0 < H; c0 += int(gridDim.x) * 16) {  // whole waves
    const int c = c0 + (lane >> 4);
    const bool act = c < H;
    const int2 hb = heavy[act ? c : c0];
    const int64_t e0 = off[hb.x] + int64_t(FI_HEAVY) * hb.y;
    const int64_t e1 = e0 + FI_HEAVY < off[hb.x + 1] ? e0 + FI_HEAVY : off[hb.x + 1];
    long long acc[3][P][P];
    fi_accum_range<P>(Y, g, order, e0, act ? e1 : e0, acc);
    const bool one = __ballot(hb.x == __builtin_amdgcn_readfirstlane(hb.x)) == ~uint64_t(0);
    const int bx = hb.x / g.B, by = hb.x % g.B;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int kx = 0; kx < P; ++kx)
#pragma unroll
        for (int ky = 0; ky < P; ++ky) {
          uint64_t v = uint64_t(acc[q][kx][ky]);
          if (one) {  // wave-uniform
            v += shfl_xor_u64(v, 16);
            v += shfl_xor_u64(v, 32);
          }
          if ((one ? lane : sl) == (q * P * P + kx * P + ky) % 16 && act)
            atomicAdd(&G[q * NN + int64_t(P * bx + kx) * g.N + (P * by + ky)], (unsigned long long)v);
        }
  }
}

// --- FFT ---------------------------------------------------------------

// 2-D circular convolution on the F x F grid in three passes, with no
// transposes and no work on the zero padding (N <= F / 2 of F rows and
// columns hold data):
//   fi_rows_fwd_kernel  length-F FFTs of the N nonzero rows of W0, W1 + i W2
//                       and K1 + i K2, their elements taken from the node
//                       sums and the kernel's definition on the way in;
//   fi_cols_kernel      per column: the three column FFTs (K's rows mirrored:
//                       it is even), the products W0^ (K1^ + i K2^) and
//                       (W1^ + i W2^) K2^ (K1^, K2^ are real), and the two
//                       inverse column FFTs, of which N rows are kept;
//   fi_rows_inv_kernel  the inverse row FFTs of those N rows, of which N
//                       columns are kept (the only ones the gather reads).
// What bounds it: latency and LDS round trips, the data (3 N F complex
// numbers, 17 MB at F = 1024) staying in L2 / MALL.  A block of T threads
// works on 8 T complex numbers in LDS (T = 256: 32 KB, for transforms up to
// 2048; T = 512 for 4096), L = 8 T / F lines together, and a thread holds 8
// elements in registers: radix 8, the factor 2 or 4 that is left over first
// in the forward and last in the inverse direction, so that a column's
// spectrum goes from the forward FFT's last pass to the inverse's first in
// registers.  (16 elements per thread halve the wavefronts and spilled the
// column pass: 46 us.)  Twiddles: one table of exp(-2 pi i k /
// F) per call, the powers 2 .. 7 by multiplication.
// Measured at F = 1024 (70,001 and 10^6 points): 11 + 31 + 11 us for the
// three passes, against 250 us for radix-2 row passes with a sincospi per
// butterfly over all F rows, transposes, a load and a product pass (eight
// launches).

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmuli(double2 a) { return make_double2(a.y, -a.x); }  // -i a

// Forward DFTs of length 2, 4 and 8 in natural order.
__device__ __forceinline__ void dft2(double2& a, double2& b) {
  const double2 t = b;
  b = csub(a, t);
  a = cadd(a, t);
}
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
  dft2(a, c);
  dft2(b, d);
  d = cmuli(d);
  dft2(a, b);
  dft2(c, d);
  const double2 t = b;
  b = c;
  c = t;
}
__device__ __forceinline__ void dft8(double2* v) {
  constexpr double H = 0.70710678118654752440;
  dft4(v[0], v[2], v[4], v[6]);
  dft4(v[1], v[3], v[5], v[7]);
  // v[0 2 4 6] = even bins 0..3, v[1 3 5 7] = odd bins 0..3
  v[3] = make_double2(H * (v[3].x + v[3].y), H * (v[3].y - v[3].x));
  v[5] = cmuli(v[5]);
  v[7] = make_double2(H * (v[7].y - v[7].x), -H * (v[7].x + v[7].y));
  double2 o[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[k] = cadd(v[2 * k], v[2 * k + 1]);
    o[k + 4] = csub(v[2 * k], v[2 * k + 1]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = o[k];
}

// A block's lines of F complex numbers.  Butterfly q of a radix-R pass is
// number q / L of line q % L (neighbouring lanes take neighbouring lines,
// then neighbouring elements).  In LDS element i of a line sits at i with its
// low three bits changed by the next three and by the line, so that 8
// lanes (16 bytes each, one LDS cycle) never share a bank.
struct FiLines {
  int logF, logL, lsh;
  double2* s;
  const double2* tw;
  __device__ __forceinline__ int at(int line, int i) const {
    return (line << logF) + (i ^ ((i >> 3) & 7) ^ ((line << lsh) & 7));
  }
  __device__ __forceinline__ int line(int q) const { return q & ((1 << logL) - 1); }
  __device__ __forceinline__ int num(int q) const { return q >> logL; }
};
__device__ __forceinline__ FiLines fi_lines(int logPts, int logF, double2* s, const double2* tw) {
  const int logL = logPts - logF;
  return FiLines{logF, logL, logL < 3 ? 3 - logL : 0, s, tw};
}

// threadIdx.x, opaque at every use: the LDS addresses of a pass are then
// formed where they are used (kept across the passes, the dozens of them
// spilled).
__device__ __forceinline__ int fi_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Pass of radix R over the 8 elements a thread holds, v[u R + r] = element
// num + r F / R of butterfly u (q = tid + T u): twiddles for sub-transforms
// of length Ns = 2^logNs, then the length-R DFTs.
template <int T, int R>
__device__ __forceinline__ void fi_pass(const FiLines& f, double2 (&v)[8], int logNs) {
  constexpr int logR = R == 8 ? 3 : (R == 4 ? 2 : 1);
  const int t = fi_tid();
#pragma unroll
  for (int u = 0; u < 8 / R; ++u) {
    double2* w = v + u * R;
    if (logNs > 0) {
      const int k = f.num(t + T * u) & ((1 << logNs) - 1);
      const double2 w1 = f.tw[k << (f.logF - logR - logNs)];
      double2 p = w1;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        w[r] = cmul(w[r], p);
        if (r + 1 < R) p = cmul(p, w1);
      }
    }
    if constexpr (R == 8) dft8(w);
    else if constexpr (R == 4) dft4(w[0], w[1], w[2], w[3]);
    else dft2(w[0], w[1]);
    if (R > 2) __builtin_amdgcn_sched_barrier(0);  // one butterfly's temporaries at a time
  }
}
// The pass's outputs to LDS (Stockham order), and the next pass's inputs.
template <int T, int R>
__device__ __forceinline__ void fi_store(const FiLines& f, const double2 (&v)[8], int logNs) {
  const int t = fi_tid();
#pragma unroll
  for (int u = 0; u < 8 / R; ++u) {
    const int q = t + T * u, ln = f.line(q), j = f.num(q);
    const int k = j & ((1 << logNs) - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) f.s[f.at(ln, (j - k) * R + k + (r << logNs))] = v[u * R + r];
  }
}
template <int T, int R>
__device__ __forceinline__ void fi_fetch(const FiLines& f, double2 (&v)[8]) {
  constexpr int logR = R == 8 ? 3 : (R == 4 ? 2 : 1);
  const int t = fi_tid();
#pragma unroll
  for (int u = 0; u < 8 / R; ++u) {
    const int q = t + T * u, ln = f.line(q), j = f.num(q);
#pragma unroll
    for (int r = 0; r < R; ++r) v[u * R + r] = f.s[f.at(ln, j + (r << (f.logF - logR)))];
  }
}

// Forward FFT of the elements get(line, i), which go through LDS first (in
// registers from the start, their addresses made the kernels spill); the
// result is left in registers: v[8 u + r] = bin num + r F / 8 of butterfly u.
template <int T, typename Get>
__device__ __forceinline__ void fi_forward(const FiLines& f, double2 (&v)[8], Get get) {
#pragma unroll 4
  for (int e = threadIdx.x; e < 8 * T; e += T) f.s[f.at(f.line(e), f.num(e))] = get(f.line(e), f.num(e));
  __syncthreads();
  const int rem = f.logF % 3;
  int logNs = 0;
  if (rem == 1) {
    fi_fetch<T, 2>(f, v);
    fi_pass<T, 2>(f, v, 0);
    __syncthreads();
    fi_store<T, 2>(f, v, 0);
    __syncthreads();
    logNs = 1;
  } else if (rem == 2) {
    fi_fetch<T, 4>(f, v);
    fi_pass<T, 4>(f, v, 0);
    __syncthreads();
    fi_store<T, 4>(f, v, 0);
    __syncthreads();
    logNs = 2;
  }
#pragma unroll 1
  for (;;) {
    fi_fetch<T, 8>(f, v);
    __syncthreads();  // every element read
    fi_pass<T, 8>(f, v, logNs);
    if (logNs + 3 >= f.logF) break;
    fi_store<T, 8>(f, v, logNs);
    __syncthreads();
    logNs += 3;
  }
}

// Inverse FFT (unnormalised) of the spectrum in registers, laid out as
// fi_forward leaves it; put(line, i, value) takes the results, from LDS.
// Taken as the conjugate of the forward FFT of the conjugate.
template <int T, typename Put>
__device__ __forceinline__ void fi_inverse(const FiLines& f, double2 (&v)[8], Put put) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e].y = -v[e].y;
  const int rem = f.logF % 3;
  int logNs = 0;
#pragma unroll 1
  for (;;) {
    fi_pass<T, 8>(f, v, logNs);
    if (logNs + 3 >= f.logF) break;
    fi_store<T, 8>(f, v, logNs);
    __syncthreads();
    logNs += 3;
    if (logNs + rem == f.logF && rem != 0) break;
    fi_fetch<T, 8>(f, v);
    __syncthreads();
  }
  if (rem == 0) {
    fi_store<T, 8>(f, v, f.logF - 3);
  } else if (rem == 1) {
    fi_fetch<T, 2>(f, v);
    __syncthreads();
    fi_pass<T, 2>(f, v, f.logF - 1);
    fi_store<T, 2>(f, v, f.logF - 1);
  } else {
    fi_fetch<T, 4>(f, v);
    __syncthreads();
    fi_pass<T, 4>(f, v, f.logF - 2);
    fi_store<T, 4>(f, v, f.logF - 2);
  }
  __syncthreads();
#pragma unroll 4
  for (int e = threadIdx.x; e < 8 * T; e += T) {
    const double2 z = f.s[f.at(f.line(e), f.num(e))];
    put(f.line(e), f.num(e), make_double2(z.x, -z.y));
  }
  __syncthreads();
}

// Row FFTs: plane ch at Cg + ch * plane, rows 0 .. N - 1 with row stride F.
template <int T>
__global__ __launch_bounds__(T, 4) void fi_rows_fwd_kernel(const unsigned long long* __restrict__ G,
                                                             const FiParams* __restrict__ gp, int p,
                                                             const double2* __restrict__ tw,
                                                             double2* __restrict__ Cg, int64_t plane) {
  __shared__ double2 s[8 * T];
  const FiParams g = *gp;
  const FiLines f = fi_lines(T == 256 ? 11 : 12, g.logF, s, tw);
  const int F = g.F, N = g.N;
  const int64_t NN = int64_t(N) * N;
  const int groups = (N + (1 << f.logL) - 1) >> f.logL;  // groups of L rows, per plane
  const double inv = 1.0 / g.scale;
  const double delta = g.h / double(p);
  for (int w = blockIdx.x; w < 3 * groups; w += gridDim.x) {
    const int ch = w / groups, r0 = (w - ch * groups) << f.logL;
    double2* Cp = Cg + ch * plane;
    double2 v[8];
    fi_forward<T>(f, v, [&](int ln, int i) {
      const int row = r0 + ln;
      double2 z = make_double2(0.0, 0.0);
      if (row >= N) return z;
      if (ch < 2) {
        if (i < N) {
          const int node = row * N + i;
          if (ch == 0) z.x = double((long long)G[node]) * inv;
          else z = make_double2(double((long long)G[NN + node]) * inv, double((long long)G[2 * NN + node]) * inv);
        }
      } else if (i < N || i > F - N) {
        const double dx = delta * double(row), dy = delta * double(i < N ? i : i - F);
        const double k1 = 1.0 / (1.0 + dx * dx + dy * dy);
        z = make_double2(k1, k1 * k1);
      }
      return z;
    });
    const int row = r0 + f.line(threadIdx.x), j = f.num(threadIdx.x);
    if (row < N) {
#pragma unroll
      for (int r = 0; r < 8; ++r) Cp[row * F + j + (r << (f.logF - 3))] = v[r];
    }
  }
}

template <int T>
__global__ __launch_bounds__(T, 3) void fi_cols_kernel(const FiParams* __restrict__ gp,
                                                         const double2* __restrict__ tw, double2* __restrict__ Cg,
                                                         int64_t plane) {
  __shared__ double2 s[8 * T];
  const FiLines f = fi_lines(T == 256 ? 11 : 12, gp->logF, s, tw);
  const int F = gp->F, N = gp->N;
  const int groups = (F + (1 << f.logL) - 1) >> f.logL;
  for (int w = blockIdx.x; w < groups; w += gridDim.x) {
    // groups that share lines of memory on one XCD (workgroups are dealt to
    // the 8 of them round-robin)
    const int c0 = (groups % 8 == 0 ? w % 8 * (groups / 8) + w / 8 : w) << f.logL;
    double2 kh[8], v[8];
    const double2* Kp = Cg + 2 * plane + c0;
    fi_forward<T>(f, kh, [&](int ln, int i) {
      const int row = i < N ? i : F - i;
      return row < N ? Kp[row * F + ln] : make_double2(0.0, 0.0);
    });
#pragma unroll 1
    for (int ch = 0; ch < 2; ++ch) {
      double2* Cp = Cg + ch * plane + c0;
      fi_forward<T>(f, v, [&](int ln, int i) {
        return i < N ? Cp[i * F + ln] : make_double2(0.0, 0.0);
      });
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[e] = ch == 0 ? cmul(v[e], kh[e]) : make_double2(v[e].x * kh[e].y, v[e].y * kh[e].y);
      fi_inverse<T>(f, v, [&](int ln, int i, double2 z) {
        if (i < N) Cp[i * F + ln] = z;
      });
    }
  }
}

template <int T>
__global__ __launch_bounds__(T, 4) void fi_rows_inv_kernel(const FiParams* __restrict__ gp,
                                                             const double2* __restrict__ tw,
                                                             double2* __restrict__ Cg, int64_t plane) {
  __shared__ double2 s[8 * T];
  const FiLines f = fi_lines(T == 256 ? 11 : 12, gp->logF, s, tw);
  const int F = gp->F, N = gp->N;
  const int groups = (N + (1 << f.logL) - 1) >> f.logL;
  for (int w = blockIdx.x; w < 2 * groups; w += gridDim.x) {
    const int ch = w / groups, r0 = (w - ch * groups) << f.logL;
    double2* Cp = Cg + ch * plane;
    double2 v[8];
    const int row = r0 + f.line(threadIdx.x), j = f.num(threadIdx.x);
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = row < N ? Cp[row * F + j + (r << (f.logF - 3))] : make_double2(0.0, 0.0);
    fi_inverse<T>(f, v, [&](int ln, int i, double2 z) {
      if (i < N && r0 + ln < N) Cp[(r0 + ln) * F + i] = z;
    });
  }
}

// --- gather ------------------------------------------------------------

// Point values of the potentials (divided by F^2): phi1 + i phi2 from
// plane 0, phi3x + i phi3y from plane 1.  R_i = z_i phi2 - phi3;
// Z partials per block in FP64 (block 0 also subtracts the n self terms).
template <int P>
__global__ __launch_bounds__(256) void fi_gather_kernel(const float2* __restrict__ Y, int64_t n,
                                                        const FiParams* __restrict__ gp,
                                                        const double2* __restrict__ Cg, int64_t plane,
                                                        float2* __restrict__ R, double* __restrict__ Zblock) {
  __shared__ double red[4];
  const FiParams g = *gp;
  const double norm = 1.0 / (double(g.F) * double(g.F));
  double zacc = 0.0;
  for (int64_t i = gtid(); i < n; i += int64_t(gridDim.x) * 256) {
    const float2 y = Y[i];
    double Lx[P], Ly[P];
    const int bx = fi_weights<P>(y.x, g, Lx);
    const int by = fi_weights<P>(y.y, g, Ly);
    double f1 = 0.0, f2 = 0.0, f3x = 0.0, f3y = 0.0;
#pragma unroll
    for (int kx = 0; kx < P; ++kx) {
#pragma unroll
      for (int ky = 0; ky < P; ++ky) {
        const double w = Lx[kx] * Ly[ky];
        const int64_t t = int64_t(P * bx + kx) * g.F + (P * by + ky);
        const double2 a = Cg[t], b = Cg[plane + t];
        f1 += w * a.x;
        f2 += w * a.y;
        f3x += w * b.x;
        f3y += w * b.y;
      }
    }
    f1 *= norm;
    f2 *= norm;
    f3x *= norm;
    f3y *= norm;
    const double zx = double(y.x) - g.c, zy = double(y.y) - g.c;
    R[i] = make_float2(float(zx * f2 - f3x), float(zy * f2 - f3y));
    zacc += f1;
  }
  const double bz = block_sum_d(zacc, red);
  if (threadIdx.x == 0) Zblock[blockIdx.x] = bz - (blockIdx.x == 0 ? double(n) : 0.0);
}

struct FiPlan {
  size_t o_part, o_par, o_tw, o_G, o_C, o_R, o_Zb, o_kl, o_cnt, o_where, o_off, o_bsum, o_ord, o_nheavy, o_heavy, bytes;
  int64_t plane, nbox;  // nbox: boxes of the largest grid (B <= max_fft / 4)
};

FiPlan fi_plan(int64_t n, int max_fft) {
  FiPlan L;
  Carve c;
  const int64_t Nmax = max_fft / 2;
  const int64_t Bmax = max_fft / 4;  // p >= 2
  L.plane = Nmax * max_fft;  // rows past N <= F / 2 hold no data
  L.nbox = Bmax * Bmax;
  L.o_part = c.take(sizeof(float) * 2 * FI_GRID);
  L.o_par = c.take(sizeof(FiParams));
  L.o_tw = c.take(sizeof(double2) * size_t(max_fft));
  L.o_cnt = c.take(sizeof(int) * size_t(L.nbox));
  L.o_where = c.take(sizeof(int2) * size_t(n));
  L.o_off = c.take(sizeof(int64_t) * size_t(L.nbox + 1));
  L.o_bsum = c.take(sizeof(int64_t) * (size_t(ceil_div(L.nbox + 1, SCAN_CHUNK)) + 1));
  L.o_ord = c.take(sizeof(int32_t) * size_t(n));
  L.o_nheavy = c.take(sizeof(int));
  // a heavy box of m > FI_HEAVY points has fewer than 2 m / FI_HEAVY chunks
  L.o_heavy = c.take(sizeof(int2) * size_t(2 * ceil_div(n, FI_HEAVY)));
  L.o_G = c.take(sizeof(unsigned long long) * 3 * size_t(Nmax) * size_t(Nmax));
  // three half planes are used; the size stays the 48 max_fft^2 bytes that the
  // interface states, which callers may have laid out
  L.o_C = c.take(sizeof(double2) * 3 * size_t(max_fft) * size_t(max_fft));
  L.o_R = c.take(sizeof(float2) * size_t(n));
  L.o_Zb = c.take(sizeof(double) * FI_GRID);
  L.o_kl = c.take(finalize_kl_bytes(n));
  L.bytes = c.off;
  return L;
}

template <int P>
int fi_spread(const float2* Y, int64_t n, const FiParams* par, const int64_t* off, const int32_t* order,
              int64_t nbox, int* nheavy, int2* heavy, unsigned long long* G, hipStream_t s) {
  const int64_t blocks = ceil_div(nbox, 16);
  hipLaunchKernelGGL(fi_accum_kernel<P>, dim3(unsigned(blocks < 2048 ? blocks : 2048)), dim3(256), 0, s, Y, par, off,
                     order, G, nheavy, heavy);
  TSNE_CHECK_LAUNCH();
  const int64_t hblocks = ceil_div(2 * ceil_div(n, FI_HEAVY), 16);
  hipLaunchKernelGGL(fi_accum_heavy_kernel<P>, dim3(unsigned(hblocks < 2048 ? hblocks : 2048)), dim3(256), 0, s, Y,
                     par, off, order, nheavy, heavy, G);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

template <int P>
int fi_collect(const float2* Y, int64_t n, const FiParams* par, const double2* Cg, int64_t plane, float2* R,
               double* Zb, hipStream_t s) {
  hipLaunchKernelGGL(fi_gather_kernel<P>, dim3(FI_GRID), dim3(256), 0, s, Y, n, par, Cg, plane, R, Zb);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// The convolution: G to the potentials' planes 0 and 1 of Cg.  The grids
// cover the largest transform; the kernels stop at the sizes in par.
template <int T>
int fi_convolve(const unsigned long long* G, const FiParams* par, int p, const double2* tw, double2* Cg,
                int64_t plane, int max_fft, hipStream_t s) {
  auto blocks = [](int64_t b) { return dim3(unsigned(b < 2048 ? b : 2048)); };
  const int64_t rows = ceil_div(int64_t(max_fft) * (max_fft / 2), 8 * T);  // groups of rows of a plane
  hipLaunchKernelGGL(fi_rows_fwd_kernel<T>, blocks(3 * rows), dim3(T), 0, s, G, par, p, tw, Cg, plane);
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(fi_cols_kernel<T>, blocks(2 * rows), dim3(T), 0, s, par, tw, Cg, plane);
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(fi_rows_inv_kernel<T>, blocks(2 * rows), dim3(T), 0, s, par, tw, Cg, plane);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

}  // namespace tsne

extern "C" int tsne_kl_grad_fft(const float* Y, int64_t n, const int64_t* row_ptr, const int32_t* col,
                                const float* val, float exaggeration, int32_t n_interp, int32_t min_boxes,
                                float max_box_width, int32_t max_fft, float* grad, double* Z, double* kl,
                                int64_t* nonfinite, void* workspace, size_t* workspace_bytes, void* stream) {
  using namespace tsne;
  if (!Y || !row_ptr || !col || !val || !grad || n < 2) return TSNE_ERR_INVALID_ARG;
  if (!(exaggeration > 0.0f) || !(exaggeration < INFINITY)) return TSNE_ERR_INVALID_ARG;
  if (n_interp < 2 || n_interp > FI_MAX_P || min_boxes < 1) return TSNE_ERR_INVALID_ARG;
  if (!(max_box_width > 0.0f) || !(max_box_width < INFINITY)) return TSNE_ERR_INVALID_ARG;
  if (max_fft < FI_MIN_FFT || max_fft > FI_MAX_FFT || (max_fft & (max_fft - 1))) return TSNE_ERR_INVALID_ARG;
  if (2 * int64_t(n_interp) * min_boxes > max_fft) return TSNE_ERR_INVALID_ARG;
  if (n > (int64_t(1) << 31)) return TSNE_ERR_UNSUPPORTED;
  const FiPlan L = fi_plan(n, max_fft);
  int rc = workspace_protocol(workspace, workspace_bytes, L.bytes);
  if (rc >= 0) return rc;
  TSNE_REQUIRE_GFX950();
  char* ws = static_cast<char*>(workspace);
  hipStream_t s = as_stream(stream);
  unsigned long long* nf = reinterpret_cast<unsigned long long*>(nonfinite);
  if (nf && (rc = launch_fill<unsigned long long>(nf, 1, 0ull, s))) return rc;
  const float2* Y2 = reinterpret_cast<const float2*>(Y);
  float* part = reinterpret_cast<float*>(ws + L.o_part);
  FiParams* par = reinterpret_cast<FiParams*>(ws + L.o_par);
  unsigned long long* G = reinterpret_cast<unsigned long long*>(ws + L.o_G);
  double2* Cg = reinterpret_cast<double2*>(ws + L.o_C);
  float2* R = reinterpret_cast<float2*>(ws + L.o_R);
  double* Zb = reinterpret_cast<double*>(ws + L.o_Zb);
  double* klp = reinterpret_cast<double*>(ws + L.o_kl);
  int* cnt = reinterpret_cast<int*>(ws + L.o_cnt);
  int2* where = reinterpret_cast<int2*>(ws + L.o_where);
  int64_t* off = reinterpret_cast<int64_t*>(ws + L.o_off);
  int64_t* bsum = reinterpret_cast<int64_t*>(ws + L.o_bsum);
  int32_t* order = reinterpret_cast<int32_t*>(ws + L.o_ord);
  double2* tw = reinterpret_cast<double2*>(ws + L.o_tw);
  int* nheavy = reinterpret_cast<int*>(ws + L.o_nheavy);
  int2* heavy = reinterpret_cast<int2*>(ws + L.o_heavy);

  hipLaunchKernelGGL(fi_bbox_kernel, dim3(FI_GRID), dim3(256), 0, s, Y2, n, part);
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(fi_params_kernel, dim3(1), dim3(256), 0, s, part, FI_GRID, n, n_interp, min_boxes,
                     max_box_width, max_fft, par, tw, nheavy);
  TSNE_CHECK_LAUNCH();
  // counting sort of the points by box, then the per-box node sums
  if ((rc = launch_fill<int>(cnt, L.nbox, 0, s))) return rc;
  hipLaunchKernelGGL(fi_count_kernel, dim3(unsigned(ceil_div(n, FI_CPTS))), dim3(256), 0, s, Y2, n, par, cnt, where);
  TSNE_CHECK_LAUNCH();
  if ((rc = exclusive_scan<int>(cnt, L.nbox, off, bsum, s))) return rc;
  hipLaunchKernelGGL(fi_scatter_kernel, dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, s, n, where, off, order);
  TSNE_CHECK_LAUNCH();
  switch (n_interp) {
    case 2: rc = fi_spread<2>(Y2, n, par, off, order, L.nbox, nheavy, heavy, G, s); break;
    case 3: rc = fi_spread<3>(Y2, n, par, off, order, L.nbox, nheavy, heavy, G, s); break;
    case 4: rc = fi_spread<4>(Y2, n, par, off, order, L.nbox, nheavy, heavy, G, s); break;
    default: rc = fi_spread<5>(Y2, n, par, off, order, L.nbox, nheavy, heavy, G, s);
  }
  if (rc) return rc;
  rc = max_fft <= 2048 ? fi_convolve<256>(G, par, n_interp, tw, Cg, L.plane, max_fft, s)
                       : fi_convolve<512>(G, par, n_interp, tw, Cg, L.plane, max_fft, s);
  if (rc) return rc;
  switch (n_interp) {
    case 2: rc = fi_collect<2>(Y2, n, par, Cg, L.plane, R, Zb, s); break;
    case 3: rc = fi_collect<3>(Y2, n, par, Cg, L.plane, R, Zb, s); break;
    case 4: rc = fi_collect<4>(Y2, n, par, Cg, L.plane, R, Zb, s); break;
    default: rc = fi_collect<5>(Y2, n, par, Cg, L.plane, R, Zb, s);
  }
  if (rc) return rc;
  // the attraction takes the rows in box order (a spatial order of Y: rows
  // that share P-neighbours run together, so their y_j gathers hit L2); the
  // order within a box follows the scatter's atomics, so a requested KL, whose
  // per-block sums would follow it, takes the rows in index order instead
  return finalize_csr_launch(Y, n, row_ptr, col, val, exaggeration, reinterpret_cast<const float*>(R), Zb, FI_GRID,
                             grad, Z, kl, klp, nf, s, kl ? nullptr : order);
}
