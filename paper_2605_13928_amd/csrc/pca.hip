// tsne_pca: principal components of X (n x g, row-major FP32) by randomized
// truncated SVD of the column-centred matrix: randomized subspace iteration
// with re-orthonormalisation and the direct SVD of the projected matrix
// (Halko, Martinsson & Tropp 2011, SIAM Review 53, Algorithm 4.4 and
// Algorithm 5.1), with a subspace of l = 64 columns:
//   Q = orth((X - 1 mu^T) Omega);  q times: Q~ = orth(Xc^T Q), Q = orth(Xc Q~)
//   Z = Xc^T Q (= B^T),  Z^T Z = U diag(s^2) U^T,
//   components V = Z U diag(1/s),  scores = Q U diag(s).
// The two products with X -- Xc W (n x 64) and Xc^T Q (g x 64) -- run on the
// FP32 matrix cores (v_mfma_f32_16x16x4_f32), X centred on the fly as it is
// staged in LDS (no cancellation against the mean).  orth() is a CholeskyQR
// pass, two for the last Q (Gram matrix in FP64, Cholesky + triangular
// inverse in one FP64 block, the first pass shifted), the 64 x 64 symmetric
// eigenproblem a one-sided Jacobi method in FP64 (32 disjoint rotations per
// step).  Sums over rows are per-chunk partials added in a fixed order:
// the result is bitwise reproducible.
#include <math.h>

#include <type_traits>

#include "common.hpp"

namespace tsne {

constexpr int PCA_L = 64;       // subspace width = one 64-column MFMA tile row
constexpr int PCA_RC = 2048;    // rows per partial of the column sums and X^T Q, at most
constexpr int PCA_RMIN = 64;    // ... and at least
constexpr int PCA_BM = 128;     // rows of a block of the product with W
// columns of X staged at a time there (32: four blocks per CU; 64, two blocks,
// took 590 instead of 525 us at 200,000 x 2,000)
constexpr int PCA_KC = 32;
constexpr int PCA_GRC = 64;     // rows per partial of a Gram matrix (the least, where m allows)
constexpr int PCA_GMAX = 768;   // partials of a Gram matrix (at most: three blocks on each of 256 CUs)

typedef float floatx4_t __attribute__((ext_vector_type(4)));

// --- column means ---------------------------------------------------------

// part[r][j] = sum of X[i][j] over the rc rows i of chunk r = blockIdx.y
// (FP64, eight independent partial sums per thread, added in a fixed order).
__global__ __launch_bounds__(256) void pca_colsum_kernel(const float* __restrict__ X, int64_t n, int g, int rc,
                                                         double* __restrict__ part) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= g) return;
  const int64_t r0 = int64_t(blockIdx.y) * rc;
  const int64_t r1 = r0 + rc < n ? r0 + rc : n;
  double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int64_t i = r0;
  for (; i + 8 <= r1; i += 8)
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += double(X[(i + u) * g + j]);
  for (; i < r1; ++i) s[0] += double(X[i * g + j]);
  part[int64_t(blockIdx.y) * g + j] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// The chunks' sums of 64 columns per block, wave w of 16 a sixteenth of the
// chunks, the waves' sums added in order.
__global__ __launch_bounds__(1024) void pca_colmean_kernel(const double* __restrict__ part, int64_t nchunk, int g,
                                                           int64_t n, float* __restrict__ mean) {
  __shared__ double sum[16][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = blockIdx.x * 64 + lane;
  const int64_t per = (nchunk + 15) / 16;
  const int64_t r0 = w * per, r1 = r0 + per < nchunk ? r0 + per : nchunk;
  double s = 0.0;
  if (j < g)
    for (int64_t r = r0; r < r1; ++r) s += part[r * g + j];
  sum[w][lane] = s;
  __syncthreads();
  if (w == 0 && j < g) {
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) t += sum[u][lane];
    mean[j] = float(t / double(n));
  }
}

// --- C = (A - 1 mu^T) W  (M x K times K x 64; the first ncols columns stored) --

// Block: 128 rows of A, 4 waves x 32 rows; the columns [kper y, kper (y + 1))
// of A for blockIdx.y = y, whose product goes to C + y M ldc (with more than
// one y: partials, added by pca_reduce_kernel), in chunks of PCA_KC staged in
// LDS, the next chunk loaded into registers while the current one is used (VEC:
// 16-byte loads, K a multiple of 4).  The loads are unconditional, their
// addresses clamped into the matrices, so that none waits inside a branch:
// rows past M and columns past K are zeroed, and the mean subtracted, when
// the registers are written to LDS.  MFMA 16x16x4 operands: lane l holds
// A[l % 16][l / 16] and W[l / 16][l % 16]; the result tile
// D[4 (l / 16) + r][l % 16] in register r.
template <bool CENTER, bool VEC>
__global__ __launch_bounds__(256, 4) void pca_gemm_tall_kernel(const float* __restrict__ A, int64_t M, int K,
                                                            const float* __restrict__ mu,
                                                            const float* __restrict__ W, float* __restrict__ C,
                                                            int ldc, int ncols, int kper) {
  constexpr int BM = PCA_BM, KC = PCA_KC, SA = KC + 4, SW = PCA_L + 16;
  constexpr int AE = VEC ? (BM * KC) / (4 * 256) : (BM * KC) / 256;  // loads per thread
  constexpr int CT = VEC ? KC / 4 : KC;                              // threads across a row of the chunk
  constexpr int RSTEP = 256 / CT;                                    // rows between a thread's loads
  constexpr int WE = KC / 16;
  __shared__ __attribute__((aligned(16))) float As[BM * SA];
  __shared__ __attribute__((aligned(16))) float Ws[KC * SW];
  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t m0 = int64_t(blockIdx.x) * BM;
  // this thread's A column offset within a chunk and first row within the block
  const int ac = (VEC ? 4 : 1) * (tid % CT);
  const int ar = tid / CT;
  const int kb = int(blockIdx.y) * kper, ke = kb + kper < K ? kb + kper : K;
  floatx4_t acc[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float4 ra[VEC ? AE : 1];
  float rs[VEC ? 1 : AE];
  float4 rm = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float4 rw[WE];
  auto load = [&](int k0) {
    const int c = k0 + ac < ke ? k0 + ac : kb;
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const int64_t row = m0 + ar + RSTEP * e;
      const float* src = A + (row < M ? row : M - 1) * K + c;
      if (VEC) ra[VEC ? e : 0] = *reinterpret_cast<const float4*>(src);
      else rs[VEC ? 0 : e] = *src;
    }
    if (CENTER) {
      if (VEC) rm = *reinterpret_cast<const float4*>(mu + c);
      else rm.x = mu[c];
    }
#pragma unroll
    for (int e = 0; e < WE; ++e) {
      const int r = k0 + (tid >> 4) + 16 * e;
      rw[e] = *reinterpret_cast<const float4*>(W + int64_t(r < ke ? r : ke - 1) * PCA_L + 4 * (tid & 15));
    }
  };
  load(kb);
  for (int k0 = kb; k0 < ke; k0 += KC) {
    const bool cok = k0 + ac < ke;
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const bool ok = cok && m0 + ar + RSTEP * e < M;
      float* dst = As + (ar + RSTEP * e) * SA + ac;
      if (VEC) {
        float4 v = ra[VEC ? e : 0];
        if (CENTER) {
          v.x -= rm.x;
          v.y -= rm.y;
          v.z -= rm.z;
          v.w -= rm.w;
        }
        *reinterpret_cast<float4*>(dst) = ok ? v : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      } else {
        const float v = CENTER ? rs[VEC ? 0 : e] - rm.x : rs[VEC ? 0 : e];
        *dst = ok ? v : 0.0f;
      }
    }
#pragma unroll
    for (int e = 0; e < WE; ++e) {
      const int r = (tid >> 4) + 16 * e;
      *reinterpret_cast<float4*>(Ws + r * SW + 4 * (tid & 15)) =
          k0 + r < ke ? rw[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    __syncthreads();
    if (k0 + KC < ke) load(k0 + KC);  // in flight during the products below
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      float av[2], bv[4];
#pragma unroll
      for (int a = 0; a < 2; ++a) av[a] = As[(w * 32 + 16 * a + li) * SA + kk + lk];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = Ws[(kk + lk) * SW + 16 * b + li];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = m0 + w * 32 + 16 * a + 4 * lk + r;
        const int col = 16 * b + li;
        if (row < M && col < ncols) C[(int64_t(blockIdx.y) * M + row) * ldc + col] = acc[a][b][r];
      }
}

// --- part[r] = (A - 1 mu^T)^T Bm over the rows of chunk r  (K x 64 each) -----

// Block (256 columns of A from c0 = 256 blockIdx.x, row chunk r = blockIdx.y
// of rc rows); wave w owns columns c0 + 64 w .. + 63 (4 tiles of 16)
// against all 64 columns of Bm (4 tiles); rows staged 32 at a time, the
// next stage loaded into registers while the current one is used.  As in
// the tall product, the loads are unconditional (clamped addresses) and the
// zeroing and centring happen on the way to LDS.
template <bool CENTER, bool VEC>
__global__ __launch_bounds__(256) void pca_gemm_red_kernel(const float* __restrict__ A, int64_t M, int K,
                                                           const float* __restrict__ mu,
                                                           const float* __restrict__ Bm, int rc,
                                                           float* __restrict__ part) {
  constexpr int MS = 32, NB = 256, SA = NB + 16, SB = PCA_L + 16;
  constexpr int AE = VEC ? (MS * NB) / (4 * 256) : (MS * NB) / 256;
  constexpr int RSTEP = VEC ? 4 : 1;  // rows between a thread's loads
  __shared__ __attribute__((aligned(16))) float At[MS * SA];
  __shared__ __attribute__((aligned(16))) float Bt[MS * SB];
  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int c0 = blockIdx.x * NB;
  const int64_t r0 = int64_t(blockIdx.y) * rc;
  const int64_t r1 = r0 + rc < M ? r0 + rc : M;
  // this thread's column of A (fixed for the block) and first row of a stage
  const int ac = VEC ? 4 * (tid & 63) : tid;
  const int ar = VEC ? (tid >> 6) : 0;
  const bool cok = c0 + ac < K;
  const int c = cok ? c0 + ac : 0;
  float4 rm = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (CENTER) {
    if (VEC) rm = *reinterpret_cast<const float4*>(mu + c);
    else rm.x = mu[c];
  }
  floatx4_t acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float4 ra[VEC ? AE : 1];
  float rs[VEC ? 1 : AE];
  float4 rb[2];
  auto load = [&](int64_t ms) {
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const int64_t row = ms + ar + RSTEP * e;
      const float* src = A + (row < r1 ? row : r1 - 1) * K + c;
      if (VEC) ra[VEC ? e : 0] = *reinterpret_cast<const float4*>(src);
      else rs[VEC ? 0 : e] = *src;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t row = ms + (tid >> 4) + 16 * e;
      rb[e] = *reinterpret_cast<const float4*>(Bm + (row < r1 ? row : r1 - 1) * PCA_L + 4 * (tid & 15));
    }
  };
  load(r0);
  for (int64_t ms = r0; ms < r1; ms += MS) {
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const bool ok = cok && ms + ar + RSTEP * e < r1;
      float* dst = At + (ar + RSTEP * e) * SA + ac;
      if (VEC) {
        float4 v = ra[VEC ? e : 0];
        if (CENTER) {
          v.x -= rm.x;
          v.y -= rm.y;
          v.z -= rm.z;
          v.w -= rm.w;
        }
        *reinterpret_cast<float4*>(dst) = ok ? v : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      } else {
        const float v = CENTER ? rs[VEC ? 0 : e] - rm.x : rs[VEC ? 0 : e];
        *dst = ok ? v : 0.0f;
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = (tid >> 4) + 16 * e;
      *reinterpret_cast<float4*>(Bt + r * SB + 4 * (tid & 15)) =
          ms + r < r1 ? rb[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    __syncthreads();
    if (ms + MS < r1) load(ms + MS);
#pragma unroll
    for (int kk = 0; kk < MS; kk += 4) {
      float av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = At[(kk + lk) * SA + 64 * w + 16 * a + li];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = Bt[(kk + lk) * SB + 16 * b + li];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();
  }
  float* out = part + int64_t(blockIdx.y) * K * PCA_L;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = c0 + 64 * w + 16 * a + 4 * lk + r;
        if (col < K) out[int64_t(col) * PCA_L + 16 * b + li] = acc[a][b][r];
      }
}

// out[t] = sum over chunks r (in order) of part[r][t], as float; sixteen
// chunks' loads in flight.
__global__ __launch_bounds__(256) void pca_reduce_kernel(const float* __restrict__ part, int64_t nchunk,
                                                         int64_t count, float* __restrict__ out) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= count) return;
  double s = 0.0;
  for (int64_t r = 0; r < nchunk; r += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(r + u < nchunk ? r + u : nchunk - 1) * count + t];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += r + u < nchunk ? double(v[u]) : 0.0;
  }
  out[t] = float(s);
}

// --- Gram matrix Y^T Y of an m x 64 factor, FP64 -------------------------

// Block r sums rows [r rpb, (r + 1) rpb) of Y (rpb a multiple of 32).  Rows
// are staged 32 at a time in LDS as doubles, the next stage loaded into
// registers (clamped addresses, rows past the end zeroed on the way to LDS)
// while the current one is used; wave w takes rows w, w + 4, ... of a stage
// and lane l accumulates the 8 x 8 entries (8 (l / 8) + i, 8 (l % 8) + j).
// The four waves' sums are added in wave order.
__global__ __launch_bounds__(256) void pca_gram_kernel(const float* __restrict__ Y, int64_t m, int64_t rpb,
                                                       double* __restrict__ part) {
  constexpr int RS = 32;
  __shared__ __attribute__((aligned(16))) double ys[RS * PCA_L];
  __shared__ double sum[PCA_L * PCA_L];
  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int ia = 8 * (lane >> 3), ib = 8 * (lane & 7);
  const int64_t r0 = int64_t(blockIdx.x) * rpb;
  const int64_t r1 = r0 + rpb < m ? r0 + rpb : m;
  double acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = 0.0;
  float4 rv[2];
  auto load = [&](int64_t s) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t row = s + (tid >> 4) + 16 * e;
      rv[e] = *reinterpret_cast<const float4*>(Y + (row < r1 ? row : r1 - 1) * PCA_L + 4 * (tid & 15));
    }
  };
  load(r0);
  for (int64_t s = r0; s < r1; s += RS) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = (tid >> 4) + 16 * e;
      const bool ok = s + r < r1;
      double* d = ys + r * PCA_L + 4 * (tid & 15);
      d[0] = ok ? double(rv[e].x) : 0.0;
      d[1] = ok ? double(rv[e].y) : 0.0;
      d[2] = ok ? double(rv[e].z) : 0.0;
      d[3] = ok ? double(rv[e].w) : 0.0;
    }
    __syncthreads();
    if (s + RS < r1) load(s + RS);
#pragma unroll 2
    for (int t = 0; t < RS / 4; ++t) {
      const double* yr = ys + (w + 4 * t) * PCA_L;
      double av[8], bv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        av[i] = yr[ia + i];
        bv[i] = yr[ib + i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = fma(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
  for (int v = 0; v < 4; ++v) {
    if (w == v) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          double& o = sum[(ia + i) * PCA_L + ib + j];
          o = v == 0 ? acc[i][j] : o + acc[i][j];
        }
    }
    __syncthreads();
  }
  double* out = part + int64_t(blockIdx.x) * PCA_L * PCA_L;
  for (int e = tid; e < PCA_L * PCA_L; e += 256) out[e] = sum[e];
}

// G[e] = sum over the nchunk partials, e < 64 x 64: block b takes the entries
// 64 b .., wave w of its 16 a sixteenth of the partials (eight loads in
// flight), the waves' sums are added in order.
__global__ __launch_bounds__(1024) void pca_gram_reduce_kernel(const double* __restrict__ part, int64_t nchunk,
                                                               double* __restrict__ G) {
  __shared__ double sum[16][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int e = blockIdx.x * 64 + lane;
  const int64_t per = (nchunk + 15) / 16;
  const int64_t r0 = w * per, r1 = r0 + per < nchunk ? r0 + per : nchunk;
  double s = 0.0;
  for (int64_t r = r0; r < r1; r += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(r + u < r1 ? r + u : r1 - 1) * PCA_L * PCA_L + e];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += r + u < r1 ? v[u] : 0.0;
  }
  sum[w][lane] = s;
  __syncthreads();
  if (w == 0) {
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) t += sum[u][lane];
    G[e] = t;
  }
}

// 1 / sqrt(x) for x > 0 in FP64: the hardware's estimate and two Newton steps
// (a third of the dependent operations of 1.0 / sqrt(x)).
__device__ __forceinline__ double rsqrt_d(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * (1.5 - 0.5 * x * y * y);
  return y * (1.5 - 0.5 * x * y * y);
}

__device__ __forceinline__ double readlane_d(double v, int src) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(b), src);
  const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(b >> 32), src);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// --- Cholesky G = R^T R (upper R) and R^-1, one block, FP64 ------------------

// shift > 0 adds shift * trace / 64 to the diagonal (the first, shifted pass
// of CholeskyQR2).  Right-looking, one row of R per step.  The inverse comes
// from the same pass: the row operations that take G to R (row i minus
// R[j][i] times the scaled row j, row j divided by R[j][j]) form the matrix E
// with E G = R, i.e. E = R^-T; applied to X = I alongside, they leave X =
// R^-T (lower triangular).  Rinv = X^T (float, 64 x 64 row-major) is the W of
// the next product Q = Y Rinv.
// Pivots are taken as at least `lim`: where the columns of Y are dependent (a
// constant X, fewer than 64 distinct rows) they are zero or rounding errors of
// either sign, whose roots would scale such a column to infinity or to one
// that is not orthogonal to the others.  After the shifted pass the squared
// norms of a basis are 0.2 to 1 and what is left of dependent columns some
// 1e-4 and less: a limit of 1e-6 of the mean keeps it below 1e-3 of a basis
// vector, or orthogonal to 6e-5.
// What bounds it: a chain of 64 pivots.  Lane c holds column c of A and X in
// registers, wave w the rows 16 u + 4 w .. + 3 (u < 4).  A step takes the four
// rows of one wave: its pivots one after another, their effect on the four
// rows by lane reads, then one LDS write, one barrier, and the update of the
// rows below from the four rows' broadcast.  With both matrices in LDS and
// one row per step a launch took 87 us (48 LDS reads, a root and two divisions
// per step); one row per step in registers 39; now 26 to 38.  Entries of A left of
// the current columns are not kept and reach no result.
__global__ __launch_bounds__(256, 1) void pca_cholinv_kernel(const double* __restrict__ Gin, double shift,
                                                          float* __restrict__ Rinv) {
  __shared__ __attribute__((aligned(16))) double rowR[2][PCA_L][4], rowX[2][PCA_L][4];  // [buffer][column][row]
  const int w = threadIdx.x >> 6, c = threadIdx.x & 63;
  const double mean = wave_sum_d(Gin[c * (PCA_L + 1)]) / PCA_L;
  const double add = shift * mean;
  const double lim = readlane_d(mean > 0.0 ? (shift > 0.0 ? 1e-300 : 1e-6 * mean) : 1.0, 0);
  double a[4][4], x[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * u + 4 * w + r;
      a[u][r] = Gin[i * PCA_L + c] + (i == c ? add : 0.0);
      x[u][r] = i == c ? 1.0 : 0.0;
    }
#pragma unroll
  for (int u0 = 0; u0 < 4; ++u0) {
    for (int w0 = 0; w0 < 4; ++w0) {
      const int j = 16 * u0 + 4 * w0, b = w0 & 1;
      if (w == w0) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const double d = readlane_d(a[u0][p], j + p);
          const double ri = rsqrt_d(d > lim ? d : lim);
          a[u0][p] *= ri;
          x[u0][p] *= ri;
#pragma unroll
          for (int r = p + 1; r < 4; ++r) {
            const double f = readlane_d(a[u0][p], j + r);
            a[u0][r] -= f * a[u0][p];
            x[u0][r] -= f * x[u0][p];
          }
          rowR[b][c][p] = a[u0][p];
          rowX[b][c][p] = x[u0][p];
        }
      }
      __syncthreads();  // (two buffers: a step's rows are read before the next but one's are written)
      double rc[4], xc[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        rc[p] = rowR[b][c][p];
        xc[p] = rowX[b][c][p];
      }
#pragma unroll
      for (int u = u0; u < 4; ++u) {
        if (u == u0 && w <= w0) continue;  // wave-uniform
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const double f = rowR[b][16 * u + 4 * w + r][p];
            a[u][r] -= f * rc[p];
            x[u][r] -= f * xc[p];
          }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) Rinv[c * PCA_L + 16 * u + 4 * w + r] = float(x[u][r]);
}

// --- symmetric eigenproblem of the 64 x 64 Gram matrix, one block, FP64 -------

// One-sided Jacobi (Hestenes) on G: rotations of column pairs until all
// columns are orthogonal, G J = W; J is orthogonal and G symmetric positive
// semidefinite, so the columns of W are the eigenvectors times their
// eigenvalues.  A sweep takes the pairs (c, c ^ s), s = 1 .. 63 in Gray-code
// order: every pair once, and in each step all 32 pairs are disjoint.  Outputs the eigenvalues
// in descending order (lam) and the matching eigenvectors as the columns of U
// (row-major 64 x 64, FP64; zero for an eigenvalue of zero).
// What bounds it: a chain of 63 steps per sweep, 6 to 7 sweeps for the graded
// matrices of a PCA.  Wave w holds rows 16 w .. 16 w + 15 in registers, lane c
// column c and its partner's column.  Both lanes of a pair rotate both columns
// (the same operations on the same bits), so the next step's partner, whose s
// differs in one bit, comes from the lane that differs in that bit: register
// moves within a wave (DPP, permlane swaps), no LDS.  The only exchange between
// waves is the pairs' inner products (one LDS write, one barrier, four reads),
// the squared norms being carried along.  The two-sided method with both
// matrices in LDS took 600 us, fetching the partner by permutes through the
// LDS unit 270, this one 230.
__global__ __launch_bounds__(256, 1) void pca_jacobi_kernel(const double* __restrict__ Gin, double* __restrict__ lam,
                                                         double* __restrict__ U) {
  constexpr int NR = PCA_L / 4;
  __shared__ double part[2][4][PCA_L];
  const int w = threadIdx.x >> 6, c = threadIdx.x & 63;
  // scaled by a power of two to a largest diagonal entry near 1 (the squares
  // below then stay in range)
  double top = Gin[c * (PCA_L + 1)];
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) top = fmax(top, shfl_xor_d(top, m));
  const int ex = top > 0.0 && top < INFINITY ? ilogb(top) : 0;
  double a[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) a[r] = ldexp(Gin[(NR * w + r) * PCA_L + c], -ex);
  int buf = 0;
  // sum over the waves, in their order
  auto total = [&](double v) {
    part[buf][w][c] = v;
    __syncthreads();
    const double t = (part[buf][0][c] + part[buf][1][c]) + (part[buf][2][c] + part[buf][3][c]);
    buf ^= 1;
    return t;
  };
  auto norm2 = [&]() {
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) v = fma(a[r], a[r], v);
    return total(v);
  };
  for (int sweep = 0; sweep < 40; ++sweep) {
    double nr = norm2();
    double o[NR], onr = nr;  // the partner's column and norm (s = 0: its own)
#pragma unroll
    for (int r = 0; r < NR; ++r) o[r] = a[r];
    bool rough = false;  // a pair whose cosine was above 1e-8: another sweep is needed
    for (int k = 1; k < PCA_L; ++k) {
      const int st = k ^ (k >> 1);
      auto swap = [&](auto mc) {
        constexpr int M = decltype(mc)::value;
        auto move = [](double v) {
          const uint64_t q = __builtin_bit_cast(uint64_t, v);
          return __builtin_bit_cast(double, (uint64_t(xor_lane<M>(uint32_t(q >> 32))) << 32) | xor_lane<M>(uint32_t(q)));
        };
#pragma unroll
        for (int r = 0; r < NR; ++r) o[r] = move(o[r]);
        onr = move(onr);
      };
      switch (__builtin_ctz(unsigned(k))) {  // the bit in which this s differs from the last
        case 0: swap(std::integral_constant<int, 1>{}); break;
        case 1: swap(std::integral_constant<int, 2>{}); break;
        case 2: swap(std::integral_constant<int, 4>{}); break;
        case 3: swap(std::integral_constant<int, 8>{}); break;
        case 4: swap(std::integral_constant<int, 16>{}); break;
        default: swap(std::integral_constant<int, 32>{});
      }
      double v0 = 0.0, v1 = 0.0;
#pragma unroll
      for (int r = 0; r < NR; r += 2) {
        v0 = fma(a[r], o[r], v0);
        v1 = fma(a[r + 1], o[r + 1], v1);
      }
      const double apq = total(v0 + v1);
      const bool first = c < (c ^ st);
      const double app = first ? nr : onr, aqq = first ? onr : nr;
      const double lim = app * aqq, sq = apq * apq;
      const bool act = sq > 1e-28 * lim;
      if (__ballot(act) == 0) continue;  // the same in every wave
      rough |= __ballot(sq > 1e-16 * lim) != 0;
      // the rotation (of the smaller angle) that makes the columns orthogonal:
      // with d = aqq - app, e = 2 apq, cos 2theta = |d| / sqrt(d^2 + e^2)
      const double d = aqq - app, e = d < 0.0 ? -2.0 * apq : 2.0 * apq;
      const double h2 = fma(d, d, e * e);
      const double ih = rsqrt_d(h2 > 1e-300 ? h2 : 1e-300);
      const double c2 = fma(0.5 * fabs(d), ih, 0.5);
      const double rc = rsqrt_d(c2), si = 0.5 * e * ih * rc;
      const bool turn = act && h2 > 1e-300;
      const double cs = turn ? c2 * rc : 1.0;
      const double sn = turn ? (first ? -si : si) : 0.0;
      const double dn = sn * rc * apq;  // tan theta apq
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double x = a[r];
        a[r] = fma(cs, x, sn * o[r]);
        o[r] = fma(cs, o[r], -sn * x);
      }
      nr += dn;
      onr -= dn;
    }
    if (!rough) break;
  }
  const double l = sqrt(norm2());
  // place of this column in descending order, a NaN after all numbers: the
  // places are a permutation whatever the input
  const double key = l >= 0.0 ? l : -1.0;
  int rank = 0;
  for (int q = 0; q < PCA_L; ++q) {
    const double kq = readlane_d(key, q);
    rank += kq > key || (kq == key && q < c) ? 1 : 0;
  }
  if (w == 0) lam[rank] = ldexp(l, ex);
  const double inv = l > 0.0 ? 1.0 / l : 0.0;
#pragma unroll
  for (int r = 0; r < NR; ++r) U[(NR * w + r) * PCA_L + rank] = a[r] * inv;
}

// W1 = U diag(1/s) (float), s = sqrt(lam); 0 for s = 0.
__global__ __launch_bounds__(256) void pca_post_eig_kernel(const double* __restrict__ lam,
                                                           const double* __restrict__ U, float* __restrict__ W1) {
  for (int e = threadIdx.x; e < PCA_L * PCA_L; e += 256) {
    const double s = sqrt(lam[e % PCA_L]);  // (lam >= 0, or NaN)
    W1[e] = float(s == 0.0 ? 0.0 : U[e] / s);
  }
}

// Sign of each of the first k components (the entry of largest magnitude
// positive, the first on ties), the components out (k x g, signed), the
// singular values, and W2 = U diag(s sign) for the scores.  One block per
// component c < k (blockIdx.x), V = g x 64.
__global__ __launch_bounds__(256) void pca_sign_kernel(const float* __restrict__ V, int g, int k,
                                                       const double* __restrict__ lam, const double* __restrict__ U,
                                                       float* __restrict__ comps, double* __restrict__ sv,
                                                       float* __restrict__ W2) {
  __shared__ float bv[256];
  __shared__ int bi[256];
  const int c = blockIdx.x, tid = threadIdx.x;
  float best = -1.0f;
  int bidx = tid < g ? tid : 0;  // a row of V whatever the comparisons say (of NaN they are all false)
  for (int j = tid; j < g; j += 256) {
    const float a = fabsf(V[int64_t(j) * PCA_L + c]);
    if (a > best) {  // j increases per thread: keeps the first maximum
      best = a;
      bidx = j;
    }
  }
  bv[tid] = best;
  bi[tid] = bidx;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) {
      const float o = bv[tid + h];
      const int oi = bi[tid + h];
      if (o > bv[tid] || (o == bv[tid] && oi < bi[tid])) {
        bv[tid] = o;
        bi[tid] = oi;
      }
    }
    __syncthreads();
  }
  const float sign = V[int64_t(bi[0]) * PCA_L + c] < 0.0f ? -1.0f : 1.0f;
  for (int j = tid; j < g; j += 256) comps[int64_t(c) * g + j] = sign * V[int64_t(j) * PCA_L + c];
  const double s = sqrt(lam[c]);
  if (tid == 0) sv[c] = s;
  if (tid < PCA_L) W2[tid * PCA_L + c] = float(U[tid * PCA_L + c] * s * double(sign));
}

struct PcaPlan {
  size_t o_mpart, o_Ya, o_Yb, o_Za, o_Zb, o_part, o_gpart, o_G, o_Rinv, o_lam, o_U, o_W1, o_W2, bytes;
  int64_t nchunk, gchunk_max;
  int rc;  // rows per chunk of the column sums and of X^T Q
};

// Row blocks of a Gram matrix over m rows: at most PCA_GMAX blocks, each a
// multiple of 32 rows and at least PCA_GRC rows where m allows.
struct GramSplit {
  int64_t nblk, rpb;
};
GramSplit gram_split(int64_t m) {
  int64_t nblk = ceil_div(m, PCA_GRC);
  if (nblk > PCA_GMAX) nblk = PCA_GMAX;
  const int64_t rpb = ceil_div(ceil_div(m, nblk), 32) * 32;
  return {ceil_div(m, rpb), rpb};
}

// Rows of X W in whole tiles without a split of the columns (head), and the
// split of the columns for the rest (see pca_tall).
struct PcaSplit {
  int64_t head;
  int parts, kper;
};
PcaSplit pca_split(int64_t M, int K, bool centred) {
  const int64_t tiles = ceil_div(M, PCA_BM), rest = tiles % 512;
  if (!centred || rest == 0 || rest > 256) return {M, 1, K};
  int64_t parts = 512 / rest;
  const int64_t chunks = ceil_div(K, PCA_KC);
  if (parts > chunks) parts = chunks;
  const int kper = int(ceil_div(chunks, parts)) * PCA_KC;
  return {(tiles - rest) * PCA_BM, int(ceil_div(K, kper)), kper};
}

PcaPlan pca_plan(int64_t n, int g) {
  PcaPlan L;
  Carve c;
  // chunks of X's rows: enough for three blocks (the reduction's occupancy)
  // on each of the 256 CUs, of 64 to 2048 rows (the sums within a chunk are
  // FP32), in whole rounds of 768 blocks
  const int64_t cols = ceil_div(g, 256);
  const int64_t rounds = ceil_div(ceil_div(n, PCA_RC) * cols, 768);
  int64_t want = 768 * rounds / cols;
  if (want < 1) want = 1;
  if (want > 65535) want = 65535;  // grid.y
  int64_t rc = ceil_div(ceil_div(n, want), 32) * 32;
  rc = rc < PCA_RMIN ? PCA_RMIN : (rc > PCA_RC ? PCA_RC : rc);
  L.rc = int(rc);
  L.nchunk = ceil_div(n, rc);
  const int64_t gn = gram_split(n).nblk, gg = gram_split(g).nblk;
  L.gchunk_max = gn > gg ? gn : gg;
  L.o_mpart = c.take(sizeof(double) * size_t(L.nchunk) * size_t(g));
  L.o_Ya = c.take(sizeof(float) * size_t(n) * PCA_L);
  L.o_Yb = c.take(sizeof(float) * size_t(n) * PCA_L);
  L.o_Za = c.take(sizeof(float) * size_t(g) * PCA_L);
  L.o_Zb = c.take(sizeof(float) * size_t(g) * PCA_L);
  const PcaSplit sp = pca_split(n, g, true);
  const int64_t red = L.nchunk * int64_t(g), tall = sp.parts * (n - sp.head);
  L.o_part = c.take(sizeof(float) * size_t(red > tall ? red : tall) * PCA_L);
  L.o_gpart = c.take(sizeof(double) * size_t(L.gchunk_max) * PCA_L * PCA_L);
  L.o_G = c.take(sizeof(double) * PCA_L * PCA_L);
  L.o_Rinv = c.take(sizeof(float) * PCA_L * PCA_L);
  L.o_lam = c.take(sizeof(double) * PCA_L);
  L.o_U = c.take(sizeof(double) * PCA_L * PCA_L);
  L.o_W1 = c.take(sizeof(float) * PCA_L * PCA_L);
  L.o_W2 = c.take(sizeof(float) * PCA_L * PCA_L);
  L.bytes = c.off;
  return L;
}

struct PcaCtx {
  const PcaPlan& L;
  char* ws;
  hipStream_t s;
  template <typename T>
  T* at(size_t o) const {
    return reinterpret_cast<T*>(ws + o);
  }
};

// The product of rows [0, M) of A with W, the columns in `parts` ranges of
// kper: to C, or (parts > 1) M x 64 partials to C.
int pca_tall_launch(const PcaCtx& x, const float* A, int64_t M, int K, const float* mu, const float* W, float* C,
                    int ldc, int ncols, int parts, int kper) {
  const dim3 grid(unsigned(ceil_div(M, PCA_BM)), unsigned(parts));
  const bool vec = K % 4 == 0;
  if (mu && vec)
    hipLaunchKernelGGL((pca_gemm_tall_kernel<true, true>), grid, dim3(256), 0, x.s, A, M, K, mu, W, C, ldc, ncols, kper);
  else if (mu)
    hipLaunchKernelGGL((pca_gemm_tall_kernel<true, false>), grid, dim3(256), 0, x.s, A, M, K, mu, W, C, ldc, ncols, kper);
  else
    hipLaunchKernelGGL((pca_gemm_tall_kernel<false, true>), grid, dim3(256), 0, x.s, A, M, K, mu, W, C, ldc, ncols, kper);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// C (M x ncols, ldc) = (A - mu) W, A is M x K (mu nullable: no centring, K =
// 64).  The rows that do not fill a round of 512 blocks of 128 rows (two per
// CU; four fit, but a lone pair runs twice as fast) to a half (all rows of a small matrix, the last
// few tiles of a large one) split the columns as well, into enough ranges to
// fill the round, and their partials are added in order: 2,700 x 1,838 (22
// blocks) 91 -> 20 us, 200,000 x 2,000 (1,563 blocks, 27 past three rounds)
// 540 -> 525 us.
int pca_tall(const PcaCtx& x, const float* A, int64_t M, int K, const float* mu, const float* W, float* C, int ldc,
             int ncols) {
  const PcaSplit sp = pca_split(M, K, mu != nullptr);
  int rc;
  if (sp.head > 0 && (rc = pca_tall_launch(x, A, sp.head, K, mu, W, C, ldc, ncols, 1, K))) return rc;
  if (sp.head == M) return TSNE_OK;
  float* part = x.at<float>(x.L.o_part);
  const int64_t tail = M - sp.head;
  if ((rc = pca_tall_launch(x, A + sp.head * K, tail, K, mu, W, part, PCA_L, PCA_L, sp.parts, sp.kper))) return rc;
  hipLaunchKernelGGL(pca_reduce_kernel, dim3(unsigned(ceil_div(tail * PCA_L, 256))), dim3(256), 0, x.s, part,
                     int64_t(sp.parts), tail * PCA_L, C + sp.head * PCA_L);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// out (K x 64) = (A - mu)^T Bm, A is M x K
int pca_red(const PcaCtx& x, const float* A, int64_t M, int K, const float* mu, const float* Bm, float* out) {
  float* part = x.at<float>(x.L.o_part);
  const int64_t nchunk = x.L.nchunk;
  const int rc = x.L.rc;
  const dim3 grid(unsigned(ceil_div(K, 256)), unsigned(nchunk));
  if (K % 4 == 0) hipLaunchKernelGGL((pca_gemm_red_kernel<true, true>), grid, dim3(256), 0, x.s, A, M, K, mu, Bm, rc, part);
  else hipLaunchKernelGGL((pca_gemm_red_kernel<true, false>), grid, dim3(256), 0, x.s, A, M, K, mu, Bm, rc, part);
  TSNE_CHECK_LAUNCH();
  const int64_t count = int64_t(K) * PCA_L;
  hipLaunchKernelGGL(pca_reduce_kernel, dim3(unsigned(ceil_div(count, 256))), dim3(256), 0, x.s, part, nchunk, count,
                     out);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// G (64 x 64, FP64, in the workspace) = Y^T Y
int pca_gram(const PcaCtx& x, const float* Y, int64_t m) {
  const GramSplit sp = gram_split(m);
  hipLaunchKernelGGL(pca_gram_kernel, dim3(unsigned(sp.nblk)), dim3(256), 0, x.s, Y, m, sp.rpb,
                     x.at<double>(x.L.o_gpart));
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(pca_gram_reduce_kernel, dim3(PCA_L * PCA_L / 64), dim3(1024), 0, x.s, x.at<double>(x.L.o_gpart),
                     sp.nblk, x.at<double>(x.L.o_G));
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// One shifted CholeskyQR pass of the m x 64 factor a: b = a R^-1.
int pca_orth(const PcaCtx& x, const float* a, float* b, int64_t m, double shift) {
  int rc;
  float* Rinv = x.at<float>(x.L.o_Rinv);
  if ((rc = pca_gram(x, a, m))) return rc;
  hipLaunchKernelGGL(pca_cholinv_kernel, dim3(1), dim3(256), 0, x.s, x.at<double>(x.L.o_G), shift, Rinv);
  TSNE_CHECK_LAUNCH();
  return pca_tall(x, a, m, PCA_L, nullptr, Rinv, b, PCA_L, PCA_L);
}

}  // namespace tsne

extern "C" int tsne_pca(const float* X, int64_t n, int32_t g, int32_t k, int32_t q, const float* omega,
                        float* scores, float* components, double* singular_values, float* mean, void* workspace,
                        size_t* workspace_bytes, void* stream) {
  using namespace tsne;
  if (!X || !omega || !scores || !components || !singular_values || !mean) return TSNE_ERR_INVALID_ARG;
  if (n < PCA_L || g < PCA_L || k < 1 || k > PCA_L || q < 0 || q > 16) return TSNE_ERR_INVALID_ARG;
  if (n > int64_t(65535) * PCA_RC || g > (1 << 20)) return TSNE_ERR_UNSUPPORTED;  // row chunks index grid.y
  const PcaPlan L = pca_plan(n, g);
  int rc = workspace_protocol(workspace, workspace_bytes, L.bytes);
  if (rc >= 0) return rc;
  TSNE_REQUIRE_GFX950();
  const PcaCtx x{L, static_cast<char*>(workspace), as_stream(stream)};
  float* Ya = x.at<float>(L.o_Ya);
  float* Yb = x.at<float>(L.o_Yb);
  float* Za = x.at<float>(L.o_Za);
  float* Zb = x.at<float>(L.o_Zb);
  // column means
  hipLaunchKernelGGL(pca_colsum_kernel, dim3(unsigned(ceil_div(g, 256)), unsigned(L.nchunk)), dim3(256), 0, x.s,
                     X, n, g, L.rc, x.at<double>(L.o_mpart));
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(pca_colmean_kernel, dim3(unsigned(ceil_div(g, 64))), dim3(1024), 0, x.s,
                     x.at<double>(L.o_mpart), L.nchunk, g, n, mean);
  TSNE_CHECK_LAUNCH();
  // range finder with power iterations.  Only the last Q has to be
  // orthonormal (B = Q^T Xc below), so only it takes both passes of
  // CholeskyQR2; before that one pass keeps the span and a basis with a
  // condition number near 1, which is all the next product needs.  (The
  // second pass multiplies by a matrix near I: it cannot mend what rounding
  // did to the span in the first.)
  if ((rc = pca_tall(x, X, n, g, mean, omega, Ya, PCA_L, PCA_L))) return rc;
  if ((rc = pca_orth(x, Ya, Yb, n, 1e-12))) return rc;
  for (int it = 0; it < q; ++it) {
    if ((rc = pca_red(x, X, n, g, mean, Yb, Za))) return rc;
    if ((rc = pca_orth(x, Za, Zb, g, 1e-12))) return rc;
    if ((rc = pca_tall(x, X, n, g, mean, Zb, Ya, PCA_L, PCA_L))) return rc;
    if ((rc = pca_orth(x, Ya, Yb, n, 1e-12))) return rc;
  }
  if ((rc = pca_orth(x, Yb, Ya, n, 0.0))) return rc;
  // Z = Xc^T Q = B^T; Z^T Z = U diag(s^2) U^T
  if ((rc = pca_red(x, X, n, g, mean, Ya, Za))) return rc;
  if ((rc = pca_gram(x, Za, g))) return rc;
  double* lam = x.at<double>(L.o_lam);
  double* U = x.at<double>(L.o_U);
  hipLaunchKernelGGL(pca_jacobi_kernel, dim3(1), dim3(256), 0, x.s, x.at<double>(L.o_G), lam, U);
  TSNE_CHECK_LAUNCH();
  float* W1 = x.at<float>(L.o_W1);
  float* W2 = x.at<float>(L.o_W2);
  hipLaunchKernelGGL(pca_post_eig_kernel, dim3(1), dim3(256), 0, x.s, lam, U, W1);
  TSNE_CHECK_LAUNCH();
  // components V = Z U diag(1/s) (g x 64, in Zb), signs, outputs
  if ((rc = pca_tall(x, Za, g, PCA_L, nullptr, W1, Zb, PCA_L, PCA_L))) return rc;
  if ((rc = launch_fill<float>(W2, PCA_L * PCA_L, 0.0f, x.s))) return rc;
  hipLaunchKernelGGL(pca_sign_kernel, dim3(unsigned(k)), dim3(256), 0, x.s, Zb, g, k, lam, U, components,
                     singular_values, W2);
  TSNE_CHECK_LAUNCH();
  // scores = Q U diag(s sign): the first k columns, straight into the output
  return pca_tall(x, Ya, n, PCA_L, nullptr, W2, scores, k, k);
}
