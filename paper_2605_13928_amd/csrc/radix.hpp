// Stable least-significant-digit radix sort of items with a 32-bit key and up
// to two 32-bit payloads, by the low `bits` bits of the keys in passes of at
// most RS_BITS bits.  A pass counts the digits of each block of RS_ITEMS items
// (LDS integer atomics), takes one exclusive scan over the counts laid out
// digit-major (so every (digit, block) gets its global start), and scatters.
// Equal keys keep their input order, and nothing depends on timing, so the
// result is deterministic.
//
// What bounds it: memory.  A block's items are therefore first put in digit
// order in LDS (one component after another through the same 16 KB), so that
// the stores to a digit's range are runs of consecutive items (32 of them with
// 128 digits, a line of 128 bytes); storing from the input order instead,
// 2048 items over 256 digits, took 1.55 ms per pass of 90 M (key, value)
// pairs.  The digits of a pass are as few as the number of passes allows (20
// bits: 7 + 7 + 6).  The first pass takes its items from a functor and the
// last one can leave the keys out, so neither needs a pass of its own.
#pragma once

#include "common.hpp"
#include "scan.hpp"

namespace tsne {

constexpr int RS_BITS = 8;  // digit bits of a pass, at most
constexpr int RS_BINS = 1 << RS_BITS;
constexpr int RS_ROUNDS = 16;
constexpr int RS_ITEMS = 256 * RS_ROUNDS;  // items per block

// Items of a pass after the first: arrays (b unused with one payload).
struct RsArrays {
  const uint32_t *key, *a, *b;
  __device__ __forceinline__ uint32_t get_key(int64_t i) const { return key[i]; }
  __device__ __forceinline__ uint32_t get_a(int64_t i) const { return a[i]; }
  __device__ __forceinline__ uint32_t get_b(int64_t i) const { return b[i]; }
};

// Number of items: *count on the device when given, else n.
__device__ __forceinline__ int64_t rs_total(int64_t n, const int64_t* count) { return count ? *count : n; }

// cnt[d * nblk + b] = items of block b whose digit is d.
template <typename In>
__global__ __launch_bounds__(256) void rs_count_kernel(In in, int64_t n_max, const int64_t* __restrict__ count,
                                                       int shift, int bins, int64_t nblk,
                                                       uint32_t* __restrict__ cnt) {
  __shared__ uint32_t h[RS_BINS];
  const int tid = threadIdx.x;
  h[tid] = 0u;
  __syncthreads();
  const int64_t n = rs_total(n_max, count);
  const int64_t base = int64_t(blockIdx.x) * RS_ITEMS + tid;
  uint32_t k[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) k[r] = base + r * 256 < n ? in.get_key(base + r * 256) : 0u;
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r)
    if (base + r * 256 < n) atomicAdd(&h[(k[r] >> shift) & uint32_t(bins - 1)], 1u);
  __syncthreads();
  if (tid < bins) cnt[int64_t(tid) * nblk + blockIdx.x] = h[tid];
}

// Items of block b to off[d * nblk + b] + (their rank among the block's
// items of digit d, in input order); NPAY payloads, the keys with KEYS.
template <typename In, int NPAY, bool KEYS>
__global__ __launch_bounds__(256) void rs_scatter_kernel(In in, int64_t n_max, const int64_t* __restrict__ count,
                                                         int shift, int bits, int64_t nblk,
                                                         const int64_t* __restrict__ off,
                                                         uint32_t* __restrict__ kout, uint32_t* __restrict__ aout,
                                                         uint32_t* __restrict__ bout) {
  __shared__ uint32_t stage[RS_ITEMS];
  __shared__ uint32_t wc[4][RS_BINS];  // digit counts per wave, then the wave's local starts
  __shared__ int64_t gbase[RS_BINS];   // global position of local position 0 of each digit
  __shared__ uint32_t wtot[4];
  const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int64_t n = rs_total(n_max, count);
  const int64_t b0 = int64_t(blockIdx.x) * RS_ITEMS;
  if (b0 >= n) return;
  const int items = n - b0 < RS_ITEMS ? int(n - b0) : RS_ITEMS;
  const uint32_t mask = (1u << bits) - 1u;
  // wave w holds the block's items [1024 w, 1024 (w + 1)), lane l those at l,
  // 64 + l, ...
  const int first = w * (RS_ITEMS / 4) + lane;
  uint32_t key[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) key[r] = first + 64 * r < items ? in.get_key(b0 + first + 64 * r) : 0u;
  uint32_t pa[NPAY > 0 ? RS_ROUNDS : 1];  // in flight while the ranks are formed
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r)
    if (NPAY > 0) pa[NPAY > 0 ? r : 0] = first + 64 * r < items ? in.get_a(b0 + first + 64 * r) : 0u;
#pragma unroll
  for (int u = 0; u < 4; ++u) wc[u][tid] = 0u;
  const int64_t goff = tid <= int(mask) ? off[int64_t(tid) * nblk + blockIdx.x] : 0;
  __syncthreads();
  // rank of each item among the wave's earlier items of its digit: the lanes
  // that hold the digit from a ballot per bit, the earlier rounds from the
  // wave's counters (LDS executes a wave's accesses in order)
  volatile uint32_t* cw = wc[w];
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  uint32_t pos[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = first + 64 * r < items;
    const uint32_t d = (key[r] >> shift) & mask;
    const uint64_t act = __ballot(valid);
    uint32_t mlo = uint32_t(act), mhi = uint32_t(act >> 32);
    for (int b = 0; b < bits; ++b) {
      const uint32_t t = 0u - ((d >> b) & 1u);  // all ones where the bit is set
      const uint64_t bb = __ballot(t != 0u);
      mlo &= ~(uint32_t(bb) ^ t);
      mhi &= ~(uint32_t(bb >> 32) ^ t);
    }
    const uint64_t m = (uint64_t(mhi) << 32) | mlo;
    const uint32_t before = uint32_t(__popcll(m & lt));
    const uint32_t pre = valid ? cw[d] : 0u;
    __builtin_amdgcn_wave_barrier();
    if (valid && before == 0) cw[d] = pre + uint32_t(__popcll(m));
    __builtin_amdgcn_wave_barrier();
    pos[r] = pre + before;
  }
  __syncthreads();
  // local starts: exclusive sum over the digits, and over the waves within one
  {
    const uint32_t c0 = wc[0][tid], c1 = wc[1][tid], c2 = wc[2][tid], c3 = wc[3][tid];
    uint32_t s = c0 + c1 + c2 + c3;
    const uint32_t own = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = uint32_t(__shfl_up(int(s), o));
      if (lane >= o) s += v;
    }
    if (lane == 63) wtot[w] = s;
    __syncthreads();
    uint32_t start = s - own;
    for (int u = 0; u < w; ++u) start += wtot[u];
    wc[0][tid] = start;
    wc[1][tid] = start + c0;
    wc[2][tid] = start + c0 + c1;
    wc[3][tid] = start + c0 + c1 + c2;
    gbase[tid] = goff - int64_t(start);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    pos[r] += wc[w][(key[r] >> shift) & mask];
    if (first + 64 * r < items) stage[pos[r]] = key[r];
  }
  __syncthreads();
  // local position p = tid + 256 r goes to its digit's range
  uint32_t dst[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const int p = tid + 256 * r;
    if (p < items) {
      const uint32_t k = stage[p];
      dst[r] = uint32_t(gbase[(k >> shift) & mask] + p);
      if (KEYS) kout[dst[r]] = k;
    }
  }
  auto payload = [&](const uint32_t (&v)[NPAY > 0 ? RS_ROUNDS : 1], uint32_t* out) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
      if (first + 64 * r < items) stage[pos[r]] = v[NPAY > 0 ? r : 0];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
      if (tid + 256 * r < items) out[dst[r]] = stage[tid + 256 * r];
  };
  if (NPAY > 1) {
    uint32_t pb[NPAY > 0 ? RS_ROUNDS : 1];
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) pb[NPAY > 0 ? r : 0] = first + 64 * r < items ? in.get_b(b0 + first + 64 * r) : 0u;
    payload(pa, aout);
    payload(pb, bout);
  } else if (NPAY > 0) {
    payload(pa, aout);
  }
}

// Workspace of a sort of at most n items (n < 2^32): digit counts, their
// offsets and the scan's chunk sums.
struct RadixScratch {
  int64_t nblk, ncnt;
  size_t cnt_bytes, off_bytes, bsum_bytes;
  static RadixScratch make(int64_t n, int bits) {
    RadixScratch r;
    r.nblk = ceil_div(n, RS_ITEMS);
    r.ncnt = (int64_t(1) << digit_bits(bits)) * r.nblk;
    r.cnt_bytes = sizeof(uint32_t) * size_t(r.ncnt);
    r.off_bytes = sizeof(int64_t) * size_t(r.ncnt + 1);
    r.bsum_bytes = sizeof(int64_t) * (size_t(ceil_div(r.ncnt + 1, SCAN_CHUNK)) + 1);
    return r;
  }
  static int passes(int bits) { return (bits + RS_BITS - 1) / RS_BITS; }
  static int digit_bits(int bits) { return (bits + passes(bits) - 1) / passes(bits); }
};

struct RsBuffers {
  uint32_t *key, *a, *b;
};

// One pass of a sort: the items of `in` in the order of their digit at
// `shift`, to `out`.
template <typename In, int NPAY, bool KEYS>
inline int radix_pass(In in, int64_t n, const int64_t* count, int shift, int bits, const RadixScratch& R,
                      uint32_t* cnt, int64_t* off, int64_t* bsum, RsBuffers out, hipStream_t s) {
  const int bins = 1 << bits;
  hipLaunchKernelGGL((rs_count_kernel<In>), dim3(unsigned(R.nblk)), dim3(256), 0, s, in, n, count, shift, bins,
                     R.nblk, cnt);
  TSNE_CHECK_LAUNCH();
  int rc = exclusive_scan<uint32_t>(cnt, int64_t(bins) * R.nblk, off, bsum, s);
  if (rc) return rc;
  hipLaunchKernelGGL((rs_scatter_kernel<In, NPAY, KEYS>), dim3(unsigned(R.nblk)), dim3(256), 0, s, in, n, count,
                     shift, bits, R.nblk, off, out.key, out.a, out.b);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

// Sorts n >= 1 items (at most: *count of them when count is given) by the
// low `bits` bits of their keys.  The first pass reads them from `first`; the
// passes alternate between the buffers so that the last one writes `out`
// (with keys if KEYS); `tmp` and `tmp2` hold the passes before it (tmp2 with
// three passes or more; it may be `out` when out has room for keys).
template <typename In, int NPAY, bool KEYS>
inline int radix_sort(In first, int64_t n, const int64_t* count, int bits, const RadixScratch& R, uint32_t* cnt,
                      int64_t* off, int64_t* bsum, RsBuffers tmp, RsBuffers tmp2, RsBuffers out, hipStream_t s) {
  const int np = RadixScratch::passes(bits), db = RadixScratch::digit_bits(bits);
  RsBuffers src{};
  for (int p = 0; p < np; ++p) {
    const int shift = p * db, b = bits - shift < db ? bits - shift : db;
    const bool last = p == np - 1;
    // the pass before the last writes tmp, the one before that tmp2, ...
    const RsBuffers dst = last ? out : ((np - 1 - p) % 2 ? tmp : tmp2);
    const RsArrays arr{src.key, src.a, src.b};
    int rc;
    if (p == 0) {
      rc = last ? radix_pass<In, NPAY, KEYS>(first, n, count, shift, b, R, cnt, off, bsum, dst, s)
                : radix_pass<In, NPAY, true>(first, n, count, shift, b, R, cnt, off, bsum, dst, s);
    } else {
      rc = last ? radix_pass<RsArrays, NPAY, KEYS>(arr, n, count, shift, b, R, cnt, off, bsum, dst, s)
                : radix_pass<RsArrays, NPAY, true>(arr, n, count, shift, b, R, cnt, off, bsum, dst, s);
    }
    if (rc) return rc;
    src = dst;
  }
  return TSNE_OK;
}

}  // namespace tsne
