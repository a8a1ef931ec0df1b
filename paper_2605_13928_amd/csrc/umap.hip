// UMAP on a kNN graph (McInnes, Healy & Melville 2018, arXiv:1802.03426):
// the smoothed kNN weights of the local fuzzy simplicial sets (Sec. 3.1),
// the a, b fit of the low-dimensional similarity (Sec. 3.2) and the layout
// epochs (Sec. 3.2, SGD with negative sampling).  The fuzzy union itself is
// tsne_umap_fuzzy_union in symmetrize.hip.
//
// Data-parallel epoch: every step of epoch t is evaluated at the positions
// Y_t and the steps are summed, Y_{t+1} = Y_t + sum.  Each step is rounded
// to 64-bit fixed point (2^-32) before it is added, so the sums are exact
// whatever order the atomics take and an epoch is bitwise reproducible.
// The integer decisions are the same on every implementation of this
// reading: the schedule in FP32 (entry e sampled in epoch t when
// floor((t + 1) r_e) > floor(t r_e), r_e = w_e / w_max), the negatives from
// SplitMix64 (Steele, Lea & Flood 2014) on the counter
// (t nnz + e) neg_rate + p, vertex ((z >> 32) n) >> 32.
#include <math.h>

#include <type_traits>

#include "common.hpp"

namespace tsne {

constexpr float UMAP_CLIP = 4.0f;
constexpr float UMAP_EPS = 1e-3f;        // added to the squared distance of a repulsive step
constexpr float UMAP_FX = 4294967296.0f;  // 2^32: fixed-point scale of the summed steps
constexpr int UMAP_MAX_NEG = 64;
constexpr int UMAP_RED_BLOCKS = 256;

// --- smoothed kNN weights ------------------------------------------------------

// 16 lanes (a DPP row) per row: d_j = sqrt(d2_j) (FP64 from the FP32 squared
// distances), rho = the smallest positive d_j (0 if none), sigma the FP64
// root of f(sigma) = sum_j exp(-max(0, d_j - rho) / sigma) = log2(k) above
// floor = 1e-3 mean(d) (1e-3 when all d are 0; sigma stays there when the
// floor already meets the target), w_j = exp(-max(0, d_j - rho) / sigma).
// What bounds it: FP64 exponentials.  In t = 1 / sigma, ln f is convex and
// decreasing, so Newton steps in t from 0 rise to the root without passing it;
// they take 6 to 9 evaluations of f to the last bit, where a bisection by one
// thread per row took 55 (15.2 ms for 700,000 rows of 30, now 0.64).  A
// row that they do not settle (non-finite distances) is bisected as before.
constexpr int UMAP_NEWTON = 60;

__device__ __forceinline__ double row16_sum_d(double v) {
  auto add = [&](auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    const uint64_t q = __builtin_bit_cast(uint64_t, v);
    const uint64_t o = (uint64_t(uint32_t(dpp_i<C>(int(uint32_t(q >> 32))))) << 32) | uint32_t(dpp_i<C>(int(uint32_t(q))));
    v += __builtin_bit_cast(double, o);
  };
  add(std::integral_constant<int, 0x128>{});
  add(std::integral_constant<int, 0x124>{});
  add(std::integral_constant<int, 0x122>{});
  add(std::integral_constant<int, 0x121>{});
  return v;
}

template <int KPL>  // distances per lane
__global__ __launch_bounds__(256) void umap_weights_kernel(const float* __restrict__ d2, int64_t n, int k,
                                                           float* __restrict__ rho_out, float* __restrict__ sigma_out,
                                                           float* __restrict__ w) {
  const int64_t i = gtid() >> 4;
  const int sl = lane_id() & 15;
  if (i >= n) return;  // whole rows of 16 lanes
  const float* r = d2 + i * k;
  const double target = log2(double(k));
  double x[KPL];
  double rho = INFINITY, sum = 0.0;
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    const int j = sl + 16 * u;
    x[u] = j < k ? sqrt(double(r[j])) : 0.0;
    sum += x[u];
    if (x[u] > 0.0 && x[u] < rho) rho = x[u];
  }
  sum = row16_sum_d(sum);
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    const double o = shfl_xor_d(rho, m);
    rho = o < rho ? o : rho;
  }
  bool any = false;  // a positive distance (rho may be infinite itself)
#pragma unroll
  for (int u = 0; u < KPL; ++u) any |= x[u] > 0.0;
  any = (__ballot(any) >> (lane_id() & 48) & 0xFFFFull) != 0;
  if (!any) rho = 0.0;
  double xmax = 0.0;
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    const double v = x[u] - rho;
    x[u] = v > 0.0 ? v : 0.0;
    xmax = x[u] > xmax ? x[u] : xmax;
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    const double o = shfl_xor_d(xmax, m);
    xmax = o > xmax ? o : xmax;
  }
  auto f = [&](double s) {
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < KPL; ++u)
      if (sl + 16 * u < k) acc += exp(-x[u] / s);
    return row16_sum_d(acc);
  };
  const double mean = sum / k;
  const double floor_s = mean > 0.0 ? 1e-3 * mean : 1e-3;
  double s = floor_s;
  if (f(floor_s) < target) {
    double sx = 0.0;
#pragma unroll
    for (int u = 0; u < KPL; ++u) sx += x[u];
    sx = row16_sum_d(sx);
    const double lt = log(target);
    double t = log(double(k) / target) * double(k) / sx;  // the step from t = 0
    bool settled = false;
    for (int it = 0; it < UMAP_NEWTON && t > 0.0 && t < INFINITY; ++it) {
      double a = 0.0, b = 0.0;
#pragma unroll
      for (int u = 0; u < KPL; ++u) {
        const double e = sl + 16 * u < k ? exp(-x[u] * t) : 0.0;
        a += e;
        b += e * x[u];
      }
      a = row16_sum_d(a);
      b = row16_sum_d(b);
      const double tn = t + (log(a) - lt) * a / b;
      // at the root the steps are rounding, of either sign
      settled = tn <= t * (1.0 + 4e-16);
      if (!(tn > t)) break;
      t = tn;
      if (settled) break;
    }
    s = 1.0 / t;
    if (!settled || !(s > floor_s)) {
      double lo = floor_s, hi = fmax(2.0 * floor_s, xmax > 0.0 ? xmax : 1.0);
      for (int it = 0; it < 2100 && f(hi) < target; ++it) hi *= 2.0;
      for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (f(mid) < target) lo = mid;
        else hi = mid;
      }
      s = 0.5 * (lo + hi);
    }
  }
  if (sl == 0) {
    rho_out[i] = float(rho);
    sigma_out[i] = float(s);
  }
#pragma unroll
  for (int u = 0; u < KPL; ++u)
    if (sl + 16 * u < k) w[i * k + sl + 16 * u] = float(exp(-x[u] / s));
}

// --- layout ----------------------------------------------------------------------

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t ctr) {
  uint64_t z = seed + (ctr + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ float umap_clip(float v) { return fminf(fmaxf(v, -UMAP_CLIP), UMAP_CLIP); }

__device__ __forceinline__ long long umap_fx(float v) { return __float2ll_rn(v * UMAP_FX); }

// Largest stored weight: block maxima, then one block over them (max is
// exact in any order).
__global__ __launch_bounds__(256) void umap_wmax_kernel(const float* __restrict__ val, int64_t nnz,
                                                        float* __restrict__ part) {
  __shared__ float red[256];
  float m = 0.0f;
  const int64_t step = int64_t(gridDim.x) * 256;
  int64_t e = gtid();
  for (; e + 7 * step < nnz; e += 8 * step) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = val[e + u * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
  }
  for (; e < nnz; e += step) m = fmaxf(m, val[e]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (int(threadIdx.x) < h) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void umap_wmax_final_kernel(float* __restrict__ part, int nb,
                                                              float* __restrict__ wmax) {
  __shared__ float red[256];
  red[threadIdx.x] = int(threadIdx.x) < nb ? part[threadIdx.x] : 0.0f;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (int(threadIdx.x) < h) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *wmax = red[0];
}

// An epoch by blocks of UMAP_ROWS rows of the CSR graph.  The block's stored
// entries, one contiguous range, are taken UMAP_CHUNK at a time: all threads
// read them, test the schedule and put the sampled ones in a list in LDS;
// then a thread per listed entry does its attractive and repulsive steps,
// added to its row's sums in LDS.  The steps are summed in 64-bit fixed point,
// so neither the order of the list nor that of the LDS atomics changes a bit.
// What bounds it: an epoch samples about 0.3 of the entries and each sample
// has 1 + neg_rate random reads of Y and as many powers.  With a thread per
// row and a step per entry, a wave ran a step's ~1,000 instructions whenever
// one of its 64 rows had sampled that entry: VALU-bound, 1.24 ms per epoch at
// 10^6 points (25 M entries); with the lists 0.46 ms.
constexpr int UMAP_ROWS = 128;
constexpr int UMAP_EPT = 8;  // entries per thread and chunk
constexpr int UMAP_CHUNK = 256 * UMAP_EPT;
constexpr int UMAP_NB = 5;   // negatives whose positions are in flight together

// The neg_rate repulsive steps of sampled entry e of row i (counter base
// (t nnz + e) neg_rate), added to (ax, ay).
__device__ __forceinline__ void umap_negatives(const float2* __restrict__ Y, int64_t n, int64_t i, float2 yi,
                                               uint64_t seed, uint64_t base, int neg_rate, float a, float b,
                                               float alpha, long long& ax, long long& ay) {
  const float c2b = 2.0f * b;
  for (int p0 = 0; p0 < neg_rate; p0 += UMAP_NB) {
    int64_t c[UMAP_NB];
    float2 yc[UMAP_NB];
#pragma unroll
    for (int u = 0; u < UMAP_NB; ++u) {
      const int p = p0 + u;
      const uint64_t z = splitmix64(seed, base + uint64_t(p));
      // slots past neg_rate stand on i itself and are skipped like a draw of i
      c[u] = p < neg_rate ? int64_t(((z >> 32) * uint64_t(n)) >> 32) : i;
    }
#pragma unroll
    for (int u = 0; u < UMAP_NB; ++u) yc[u] = Y[c[u]];
#pragma unroll
    for (int u = 0; u < UMAP_NB; ++u) {
      if (c[u] == i) continue;
      const float ex = yi.x - yc[u].x, ey = yi.y - yc[u].y;
      const float q2 = ex * ex + ey * ey;
      if (q2 > 0.0f) {
        const float cr = c2b / ((UMAP_EPS + q2) * (1.0f + a * powf(q2, b)));
        ax += umap_fx(alpha * umap_clip(cr * ex));
        ay += umap_fx(alpha * umap_clip(cr * ey));
      }
    }
  }
}

// Epoch t: for every entry (i, j) sampled in this epoch, the attractive step
// alpha clip(c_a (y_i - y_j)) added to y_i and subtracted from y_j; then
// neg_rate repulsive steps alpha clip(c_r (y_i - y_c)) added to y_i; c_a =
// -2ab d2^(b-1) / (1 + a d2^b), c_r = 2b / ((eps + d2)(1 + a d2^b)), no step
// at d2 = 0 or for a draw c = i.
// SYM: a symmetric graph (pattern and values, as the fuzzy union writes
// them): entries (i, j) and (j, i) hold the same FP32 value, so they are
// sampled in the same epochs, and the step that entry (j, i) applies to y_i
// is bitwise equal to y_i's own step for (i, j) (the squared distance is the
// same, c_a is symmetric, and clip is odd).  Each vertex therefore takes
// twice its own attractive steps plus its negatives, nothing is scattered, and
// the block writes its rows' new positions to Yout: the same bits.
// Otherwise the steps into y_j go to D with 64-bit integer atomics, and so
// does each row's own sum (umap_apply_kernel takes the step).
template <bool SYM>
__global__ __launch_bounds__(256) void umap_epoch_kernel(const float2* __restrict__ Y, float2* __restrict__ Yout,
                                                         int64_t n, const int64_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col,
                                                         const float* __restrict__ val, int64_t nnz,
                                                         const float* __restrict__ wmax, float a, float b,
                                                         float alpha, int neg_rate, uint64_t seed, int t,
                                                         unsigned long long* __restrict__ D) {
  __shared__ int64_t rp[UMAP_ROWS + 1];
  __shared__ float2 yrow[UMAP_ROWS];
  __shared__ unsigned long long sx[UMAP_ROWS], sy[UMAP_ROWS];
  __shared__ int32_t lcol[UMAP_CHUNK];
  __shared__ uint16_t lent[UMAP_CHUNK];  // the entry's place in the chunk
  __shared__ int count;
  const int tid = threadIdx.x, lane = lane_id();
  const int64_t r0 = int64_t(blockIdx.x) * UMAP_ROWS;
  const int rows = int(n - r0 < UMAP_ROWS ? n - r0 : UMAP_ROWS);
  if (tid <= UMAP_ROWS) rp[tid] = row_ptr[r0 + (tid < rows ? tid : rows)];
  if (tid < UMAP_ROWS) {
    yrow[tid] = Y[r0 + (tid < rows ? tid : rows - 1)];
    sx[tid] = 0ull;
    sy[tid] = 0ull;
  }
  if (tid == 0) count = 0;
  const float rmax = *wmax;
  const float t0 = float(t), t1 = float(t + 1);
  const float cab = -2.0f * a * b;
  __syncthreads();
  const int64_t E1 = rp[UMAP_ROWS];
  for (int64_t c0 = rp[0]; c0 < E1; c0 += UMAP_CHUNK) {
    float v[UMAP_EPT];
    int32_t cj[UMAP_EPT];
#pragma unroll
    for (int u = 0; u < UMAP_EPT; ++u) {
      const int64_t e = c0 + tid + 256 * u;
      v[u] = e < E1 ? __builtin_nontemporal_load(val + e) : 0.0f;
      cj[u] = e < E1 ? __builtin_nontemporal_load(col + e) : 0;
    }
#pragma unroll
    for (int u = 0; u < UMAP_EPT; ++u) {
      const float r = __fdiv_rn(v[u], rmax);  // correctly rounded, as the schedule requires
      const bool smp = c0 + tid + 256 * u < E1 && floorf(t1 * r) > floorf(t0 * r);
      const uint64_t m = __ballot(smp);
      int base = 0;
      if (lane == 0 && m) base = atomicAdd(&count, __popcll(m));
      base = __builtin_amdgcn_readfirstlane(base);
      if (smp) {
        const int at = base + __popcll(m & ((uint64_t(1) << lane) - 1));
        lcol[at] = cj[u];
        lent[at] = uint16_t(tid + 256 * u);
      }
    }
    __syncthreads();
    const int L = count;
    for (int q = tid; q < L; q += 256) {
      const int64_t e = c0 + lent[q];
      const int64_t j = lcol[q];
      const float2 yj = Y[j];
      int lo = 0, hi = UMAP_ROWS;  // row: rp[lo] <= e < rp[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (rp[mid] <= e) lo = mid;
        else hi = mid;
      }
      const float2 yi = yrow[lo];
      long long ax = 0, ay = 0;
      umap_negatives(Y, n, r0 + lo, yi, seed, (uint64_t(t) * uint64_t(nnz) + uint64_t(e)) * uint64_t(neg_rate),
                     neg_rate, a, b, alpha, ax, ay);
      const float dx = yi.x - yj.x, dy = yi.y - yj.y;
      const float d2 = dx * dx + dy * dy;
      if (d2 > 0.0f) {
        const float pb = powf(d2, b);
        const float c = cab * (pb / d2) / (1.0f + a * pb);
        const long long fx = umap_fx(alpha * umap_clip(c * dx)), fy = umap_fx(alpha * umap_clip(c * dy));
        ax += SYM ? 2 * fx : fx;
        ay += SYM ? 2 * fy : fy;
        if (!SYM) {
          atomicAdd(&D[2 * j], static_cast<unsigned long long>(-fx));
          atomicAdd(&D[2 * j + 1], static_cast<unsigned long long>(-fy));
        }
      }
      atomicAdd(&sx[lo], static_cast<unsigned long long>(ax));
      atomicAdd(&sy[lo], static_cast<unsigned long long>(ay));
    }
    __syncthreads();  // the list is read, the sums are complete
    if (tid == 0) count = 0;
    if (c0 + UMAP_CHUNK < E1) __syncthreads();
  }
  if (tid < rows) {
    if (SYM) {
      float2 y = yrow[tid];
      y.x += float(double(static_cast<long long>(sx[tid])) * (1.0 / 4294967296.0));
      y.y += float(double(static_cast<long long>(sy[tid])) * (1.0 / 4294967296.0));
      Yout[r0 + tid] = y;
    } else {
      if (sx[tid]) atomicAdd(&D[2 * (r0 + tid)], sx[tid]);
      if (sy[tid]) atomicAdd(&D[2 * (r0 + tid) + 1], sy[tid]);
    }
  }
}

// Y_{t+1} = Y_t + D 2^-32 (FP32), D cleared for the next epoch.
__global__ __launch_bounds__(256) void umap_apply_kernel(float2* __restrict__ Y, int64_t n,
                                                         unsigned long long* __restrict__ D) {
  const int64_t i = gtid();
  if (i >= n) return;
  const long long dx = static_cast<long long>(D[2 * i]), dy = static_cast<long long>(D[2 * i + 1]);
  float2 y = Y[i];
  y.x += float(double(dx) * (1.0 / 4294967296.0));
  y.y += float(double(dy) * (1.0 / 4294967296.0));
  Y[i] = y;
  D[2 * i] = 0ull;
  D[2 * i + 1] = 0ull;
}

__global__ __launch_bounds__(256) void umap_copy_kernel(const float2* __restrict__ src, float2* __restrict__ dst,
                                                        int64_t n) {
  const int64_t i = gtid();
  if (i < n) dst[i] = src[i];
}

struct UmapLayout {
  size_t o_part, o_wmax, o_D, o_Y, bytes;
  static UmapLayout make(int64_t n) {
    UmapLayout L;
    Carve c;
    L.o_part = c.take(sizeof(float) * UMAP_RED_BLOCKS);
    L.o_wmax = c.take(sizeof(float));
    L.o_D = c.take(sizeof(unsigned long long) * 2 * size_t(n));
    L.o_Y = c.take(sizeof(float2) * size_t(n));
    L.bytes = c.off;
    return L;
  }
};

// --- a, b of Phi(d) = 1 / (1 + a d^2b): least squares against Psi ------------------

// Levenberg-Marquardt (Marquardt's diagonal scaling) from (1, 1) over the 300
// points d = 3 m / 299; a step is taken only if it lowers the sum of squares
// and keeps a > 0.
struct FitAB {
  double x[300], y[300];
  explicit FitAB(double min_dist) {
    for (int m = 0; m < 300; ++m) {
      x[m] = 3.0 * m / 299.0;
      y[m] = x[m] <= min_dist ? 1.0 : exp(-(x[m] - min_dist));
    }
  }
  double cost(double a, double b) const {
    double s = 0.0;
    for (int m = 0; m < 300; ++m) {
      const double r = 1.0 / (1.0 + a * pow(x[m], 2.0 * b)) - y[m];
      s += r * r;
    }
    return s;
  }
};

}  // namespace tsne

extern "C" int tsne_umap_fit_ab(double min_dist, double* a_out, double* b_out) {
  using namespace tsne;
  if (!a_out || !b_out || !(min_dist >= 0.0) || !(min_dist < 3.0)) return TSNE_ERR_INVALID_ARG;
  const FitAB F(min_dist);
  double a = 1.0, b = 1.0, lam = 1e-3, c0 = F.cost(a, b);
  for (int it = 0; it < 2000 && lam < 1e20; ++it) {
    double h00 = 0.0, h01 = 0.0, h11 = 0.0, g0 = 0.0, g1 = 0.0;
    for (int m = 0; m < 300; ++m) {
      const double xm = F.x[m];
      const double p = xm > 0.0 ? pow(xm, 2.0 * b) : 0.0;
      const double phi = 1.0 / (1.0 + a * p);
      const double r = phi - F.y[m];
      const double ja = -p * phi * phi;
      const double jb = xm > 0.0 ? -a * p * 2.0 * log(xm) * phi * phi : 0.0;
      h00 += ja * ja;
      h01 += ja * jb;
      h11 += jb * jb;
      g0 += ja * r;
      g1 += jb * r;
    }
    const double m00 = h00 * (1.0 + lam), m11 = h11 * (1.0 + lam);
    const double det = m00 * m11 - h01 * h01;
    if (!(det > 0.0)) {
      lam *= 10.0;
      continue;
    }
    const double da = -(m11 * g0 - h01 * g1) / det, db = -(m00 * g1 - h01 * g0) / det;
    const double an = a + da, bn = b + db;
    const double c1 = an > 0.0 ? F.cost(an, bn) : INFINITY;
    if (c1 < c0) {
      const bool tiny = fabs(da) <= 1e-15 * fabs(a) && fabs(db) <= 1e-15 * fabs(b);
      a = an;
      b = bn;
      c0 = c1;
      lam = fmax(lam * 0.1, 1e-12);
      if (tiny) break;
    } else {
      lam *= 10.0;
    }
  }
  *a_out = a;
  *b_out = b;
  return TSNE_OK;
}

extern "C" int tsne_umap_weights(const float* nbr_d2, int64_t n, int32_t k, float* rho, float* sigma, float* w,
                                 void* stream) {
  using namespace tsne;
  if (!nbr_d2 || !rho || !sigma || !w || n < 1 || k < 1) return TSNE_ERR_INVALID_ARG;
  if (k > TSNE_MAX_K) return TSNE_ERR_UNSUPPORTED;
  TSNE_REQUIRE_GFX950();
  auto kern = k <= 16   ? umap_weights_kernel<1>
              : k <= 32 ? umap_weights_kernel<2>
              : k <= 64 ? umap_weights_kernel<4>
              : k <= 128 ? umap_weights_kernel<8>
                         : umap_weights_kernel<16>;
  hipLaunchKernelGGL(kern, dim3(unsigned(ceil_div(n, 16))), dim3(256), 0, as_stream(stream), nbr_d2, n, int(k), rho,
                     sigma, w);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

extern "C" int tsne_umap_layout(float* Y, int64_t n, const int64_t* row_ptr, const int32_t* col, const float* val,
                                int64_t nnz, int32_t symmetric, double a, double b, double alpha0, int32_t neg_rate,
                                int32_t n_epochs, int32_t epoch_begin, int32_t epoch_end, uint64_t seed,
                                void* workspace, size_t* workspace_bytes, void* stream) {
  using namespace tsne;
  if (!Y || !row_ptr || !col || !val || n < 2 || nnz < 1) return TSNE_ERR_INVALID_ARG;
  if (!(a > 0.0) || !(b > 0.0) || !(alpha0 >= 0.0) || neg_rate < 0 || neg_rate > UMAP_MAX_NEG) return TSNE_ERR_INVALID_ARG;
  if (n_epochs < 1 || epoch_begin < 0 || epoch_begin > epoch_end || epoch_end > n_epochs) return TSNE_ERR_INVALID_ARG;
  if (symmetric != 0 && symmetric != 1) return TSNE_ERR_INVALID_ARG;
  if (n >= (int64_t(1) << 31)) return TSNE_ERR_UNSUPPORTED;
  const UmapLayout L = UmapLayout::make(n);
  int rc = workspace_protocol(workspace, workspace_bytes, L.bytes);
  if (rc >= 0) return rc;
  TSNE_REQUIRE_GFX950();
  char* ws = static_cast<char*>(workspace);
  float* part = reinterpret_cast<float*>(ws + L.o_part);
  float* wmax = reinterpret_cast<float*>(ws + L.o_wmax);
  unsigned long long* D = reinterpret_cast<unsigned long long*>(ws + L.o_D);
  float2* Yb = reinterpret_cast<float2*>(ws + L.o_Y);
  hipStream_t s = as_stream(stream);
  if (!symmetric && (rc = launch_fill<unsigned long long>(D, 2 * n, 0ull, s))) return rc;
  const int64_t nbk = ceil_div(nnz, 256);
  const int nb = int(nbk < UMAP_RED_BLOCKS ? nbk : UMAP_RED_BLOCKS);
  hipLaunchKernelGGL(umap_wmax_kernel, dim3(unsigned(nb)), dim3(256), 0, s, val, nnz, part);
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(umap_wmax_final_kernel, dim3(1), dim3(256), 0, s, part, nb, wmax);
  TSNE_CHECK_LAUNCH();
  const dim3 grid(unsigned(ceil_div(n, 256))), egrid(unsigned(ceil_div(n, UMAP_ROWS)));
  float2* Y2 = reinterpret_cast<float2*>(Y);
  float2* cur = Y2;
  float2* nxt = Yb;
  for (int t = epoch_begin; t < epoch_end; ++t) {
    const float alpha = float(alpha0 * (1.0 - double(t) / double(n_epochs)));
    if (symmetric) {
      hipLaunchKernelGGL(umap_epoch_kernel<true>, egrid, dim3(256), 0, s, cur, nxt, n, row_ptr, col, val, nnz, wmax,
                         float(a), float(b), alpha, int(neg_rate), seed, int(t),
                         static_cast<unsigned long long*>(nullptr));
      TSNE_CHECK_LAUNCH();
      float2* tmp = cur;
      cur = nxt;
      nxt = tmp;
    } else {
      hipLaunchKernelGGL(umap_epoch_kernel<false>, egrid, dim3(256), 0, s, Y2, static_cast<float2*>(nullptr), n,
                         row_ptr, col, val, nnz, wmax, float(a), float(b), alpha, int(neg_rate), seed, int(t), D);
      TSNE_CHECK_LAUNCH();
      hipLaunchKernelGGL(umap_apply_kernel, grid, dim3(256), 0, s, Y2, n, D);
      TSNE_CHECK_LAUNCH();
    }
  }
  if (cur != Y2) {
    hipLaunchKernelGGL(umap_copy_kernel, grid, dim3(256), 0, s, cur, Y2, n);
    TSNE_CHECK_LAUNCH();
  }
  return TSNE_OK;
}
