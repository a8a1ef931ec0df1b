// tsne_symmetrize: P = (C + C^T) / (2n) on the union of the kNN patterns
// (van der Maaten & Hinton 2008, Sec. 3.1; sparse pattern as in van der
// Maaten 2014, Sec. 4.1), as CSR with ascending columns plus the transpose
// positions.  HBM-bound integer work, deterministic:
//   1. the transposed lists: a stable radix sort (radix.hpp) of the directed
//      entries (i, j, p) by their target j, so each target's list holds its
//      sources in ascending order (the entries are numbered in source order);
//      invalid targets sort to a bucket n of their own and are reported
//      through err
//   2. in_ptr from the sorted targets (each boundary writes the starts of
//      the targets it passes), with a repeated (j, i) reported through err
//   3. union size per row (binary search of each out-entry in the in-list),
//      scan -> row_ptr
//   4. per row: the k out-entries sorted by column in registers, then the
//      merge by ranks: position of an element = its rank in its own list +
//      its rank in the other list - the shared entries before it
//   5. tpos: the entries (i, j), numbered in (i, j) order, stably sorted by j
//      are in the order of their transposes (j, i), and the pattern is
//      symmetric, so the number at place p is the position of the transpose
//      of entry p: a radix sort of the columns with their positions (few
//      entries search row col[e] instead)
// What bounds it: the passes over the n k directed and about 1.6 n k stored
// entries (about 15 GB at 10^6 points, k = 90).  The values travel with the
// sort (12 bytes per entry and pass): gathered afterwards by entry number,
// 4 random bytes moved a line each (1.9 ms); the sort of tpos replaces a
// binary search of row col[e] for every stored entry e (11.4 ms, a few
// random lines each).
// Entry values are (p_{j|i} + p_{i|j}) / (2n) in row i and
// (p_{i|j} + p_{j|i}) / (2n) in row j: the same FP32 sum, so P = P^T bitwise.
// tsne_umap_fuzzy_union runs the same steps with the probabilistic t-conorm
// b = (a + a') - a a' of the two directed weights in step 6 (McInnes, Healy &
// Melville 2018, Sec. 3.1), symmetric bitwise for the same reason.
#include "common.hpp"
#include "radix.hpp"
#include "scan.hpp"

namespace tsne {

__device__ __forceinline__ bool edge_ok(int64_t i, int32_t j, int64_t n) { return j >= 0 && j < n && j != i; }

// Directed entry e = (i, j = nbr[e]) as an item of the first sort: key its
// target, or n for an invalid target (out of range or i itself), which is
// reported; payloads its source and its value.
struct SymItems {
  const int32_t* nbr;
  const uint32_t* val;
  int64_t n;
  int k;
  int* err;
  __device__ __forceinline__ uint32_t get_key(int64_t e) const {
    const int32_t j = nbr[e];
    const bool ok = edge_ok(uint32_t(e) / uint32_t(k), j, n);  // n k < 2^30
    if (!ok) atomicOr(err, 1);
    return ok ? uint32_t(j) : uint32_t(n);
  }
  __device__ __forceinline__ uint32_t get_a(int64_t e) const { return uint32_t(e) / uint32_t(k); }
  __device__ __forceinline__ uint32_t get_b(int64_t e) const { return val[e]; }
};

// Stored entry e as an item of the second sort: key its column, payload e.
struct ColItems {
  const int32_t* col;
  __device__ __forceinline__ uint32_t get_key(int64_t e) const { return uint32_t(col[e]); }
  __device__ __forceinline__ uint32_t get_a(int64_t e) const { return uint32_t(e); }
  __device__ __forceinline__ uint32_t get_b(int64_t) const { return 0u; }
};

// in_ptr[j] = first position of target j in the sorted keys, j = 0 .. n
// (in_ptr[n] = the number of valid entries): position p writes the starts
// of the targets after key[p - 1] up to key[p].  A source repeated within one
// list (a row that names the same neighbour twice) is reported.
__global__ __launch_bounds__(256) void sym_inptr_kernel(const int32_t* __restrict__ skey,
                                                        const int32_t* __restrict__ ssrc, int64_t nk, int64_t n,
                                                        int64_t* __restrict__ in_ptr, int* __restrict__ err) {
  const int64_t p = gtid();
  if (p > nk) return;
  const int64_t prev = p > 0 ? int64_t(skey[p - 1]) : -1;
  const int64_t cur = p < nk ? int64_t(skey[p]) : n + 1;
  const int64_t hi = cur < n ? cur : n;
  for (int64_t j = prev + 1; j <= hi; ++j) in_ptr[j] = p;
  if (cur < n && prev == cur && ssrc[p - 1] == ssrc[p]) atomicOr(err, 1);
}

// First position in sorted[0..len) whose value is >= x (len the same in every
// lane: the halving is uniform).
template <typename Ptr>
__device__ __forceinline__ int lower_bound_i32(Ptr sorted, int len, int32_t x) {
  int lo = 0, m = len;
  while (m > 1) {
    const int half = m >> 1;
    lo = sorted[lo + half - 1] < x ? lo + half : lo;
    m -= half;
  }
  return m == 1 && sorted[lo] < x ? lo + 1 : lo;
}

// A row's in-list is searched by its wave from LDS when it has at most
// SYM_STAGE entries (a hub's longer one from memory).
constexpr int SYM_STAGE = 512;

__global__ __launch_bounds__(256) void sym_union_count_kernel(int64_t n, int k, const int32_t* __restrict__ nbr,
                                                              const int64_t* __restrict__ in_ptr,
                                                              const int32_t* __restrict__ s_src,
                                                              int64_t* __restrict__ ucount) {
  __shared__ int32_t st[4][SYM_STAGE];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t row = int64_t(blockIdx.x) * 4 + w;
  if (row >= n) return;
  const int32_t* in = s_src + in_ptr[row];
  const int len = int(in_ptr[row + 1] - in_ptr[row]);
  const bool staged = len <= SYM_STAGE;
  if (staged)
    for (int b = lane; b < len; b += 64) st[w][b] = in[b];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  int dups = 0;
  for (int a0 = 0; a0 < k; a0 += 64) {
    const int a = a0 + lane;
    const int32_t c = a < k ? nbr[row * k + a] : -1;
    bool dup;
    if (staged) {
      const int lb = lower_bound_i32(st[w], len, c);
      dup = lb < len && st[w][lb] == c;
    } else {
      const int lb = lower_bound_i32(in, len, c);
      dup = lb < len && in[lb] == c;
    }
    dups += __popcll(__ballot(dup && a < k));
  }
  if (lane == 0) ucount[row] = int64_t(k) + len - dups;
}

// Combined value of an entry from its out-weight u and in-weight v (0 when
// absent): MODE 0 the t-SNE average (u + v) / 2n, MODE 1 the fuzzy union.
template <int MODE>
__device__ __forceinline__ float sym_combine(float u, float v, float two_n) {
  if (MODE == 0) return (u + v) / two_n;
  return (u + v) - u * v;
}

// One wave per row, EPL * 64 >= k.  The out-entries are sorted as (column <<
// sb) | slot, 2^sb >= k (below 2 n k < 2^31; a column out of range, already
// reported, as column 0).
template <int MODE, int EPL>
__global__ __launch_bounds__(256) void sym_write_kernel(int64_t n, int k, int sb, const int32_t* __restrict__ nbr,
                                                        const float* __restrict__ Pc,
                                                        const int64_t* __restrict__ in_ptr,
                                                        const int32_t* __restrict__ s_src,
                                                        const float* __restrict__ s_val,
                                                        const int64_t* __restrict__ row_ptr, int32_t* __restrict__ col,
                                                        float* __restrict__ val) {
  __shared__ int32_t st[4][SYM_STAGE];
  __shared__ int32_t oc[4][EPL * 64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t row = int64_t(blockIdx.x) * 4 + w;
  if (row >= n) return;
  const float two_n = 2.0f * float(n);
  const int32_t* in = s_src + in_ptr[row];
  const float* inv = s_val + in_ptr[row];
  const int len = int(in_ptr[row + 1] - in_ptr[row]);
  const bool staged = len <= SYM_STAGE;
  const int64_t rp = row_ptr[row];
  uint32_t v[EPL];
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    const int a = 64 * t + lane;
    const int32_t c = a < k ? nbr[row * k + a] : 0;
    v[t] = a < k ? (uint32_t(c >= 0 && c < n ? c : 0) << sb) | uint32_t(a) : ~0u;
  }
  if (staged)
    for (int b = lane; b < len; b += 64) st[w][b] = in[b];
  wave_sort32<EPL>(v);
#pragma unroll
  for (int t = 0; t < EPL; ++t) oc[w][64 * t + lane] = int32_t(v[t] >> sb);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint64_t lt_mask = (uint64_t(1) << lane) - 1;
  // out-entries
  int run = 0;
#pragma unroll
  for (int t = 0; t < EPL; ++t) {
    if (64 * t >= k) break;
    const int a = 64 * t + lane;
    const int32_t c = a < k ? int32_t(v[t] >> sb) : 0;
    const float u = a < k ? Pc[row * k + (v[t] & ((1u << sb) - 1u))] : 0.0f;
    int lb;
    bool dup;
    if (staged) {
      lb = lower_bound_i32(st[w], len, c);
      dup = a < k && lb < len && st[w][lb] == c;
    } else {
      lb = lower_bound_i32(in, len, c);
      dup = a < k && lb < len && in[lb] == c;
    }
    const uint64_t m = __ballot(dup);
    if (a < k) {
      const int pos = a + lb - (run + __popcll(m & lt_mask));
      col[rp + pos] = c;
      val[rp + pos] = sym_combine<MODE>(u, dup ? inv[lb] : 0.0f, two_n);
    }
    run += __popcll(m);
  }
  // in-entries not shared with the out-list
  run = 0;
  for (int b0 = 0; b0 < len; b0 += 64) {
    const int b = b0 + lane;
    const int32_t c = b < len ? (staged ? st[w][b] : in[b]) : 0;
    const int lb = lower_bound_i32(oc[w], k, c);
    const bool dup = b < len && lb < k && oc[w][lb] == c;
    const uint64_t m = __ballot(dup);
    if (b < len && !dup) {
      const int pos = b + lb - (run + __popcll(m & lt_mask));
      col[rp + pos] = c;
      val[rp + pos] = sym_combine<MODE>(0.0f, inv[b], two_n);
    }
    run += __popcll(m);
  }
}

// tpos of few entries (2 n k at most SYM_SEARCH): a thread per stored entry e
// finds its row, then the row's number among the entries of row col[e].  The
// sort's launches take some 40 us however few the entries are, the searches
// as long as their random lines.  Whole call, sort / search: 1,000 x 15 113 /
// 78 us, 5,000 x 90 152 / 128, 20,000 x 30 168 / 151; 10,000 x 90 173 / 172,
// 20,000 x 90 211 / 273.
constexpr int64_t SYM_SEARCH = 1200000;
__global__ __launch_bounds__(256) void sym_tpos_kernel(int64_t n, const int64_t* __restrict__ row_ptr,
                                                       const int32_t* __restrict__ col, int32_t* __restrict__ tpos) {
  const int64_t e = gtid();
  if (e >= row_ptr[n]) return;
  int32_t row = 0;  // the last row that starts at or before e
  for (int32_t m = int32_t(n); m > 1;) {
    const int32_t half = m >> 1;
    row = row_ptr[row + half] <= e ? row + half : row;
    m -= half;
  }
  const int32_t j = col[e];
  int32_t t = -1;
  if (j >= 0 && j < n) {  // (else an input that is reported)
    const int64_t a = row_ptr[j];
    t = int32_t(a + lower_bound_i32(col + a, int(row_ptr[j + 1] - a), row));
  }
  tpos[e] = t;
}

__global__ void sym_nnz_kernel(const int64_t* __restrict__ row_ptr, int64_t n, const int* __restrict__ err,
                               int64_t* __restrict__ nnz) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *nnz = *err ? int64_t(-1) : row_ptr[n];
}

struct SymLayout {
  size_t o_err, o_inptr, o_buf, o_ucount, o_bsum, o_rcnt, o_roff, o_rbsum, bytes;
  RadixScratch R1, R2;  // of the directed entries, of the stored ones
  static SymLayout make(int64_t n, int k) {
    SymLayout L;
    const size_t nk = size_t(n) * size_t(k);
    const size_t nb = size_t(ceil_div(n + 1, SCAN_CHUNK)) + 1;
    L.R1 = RadixScratch::make(int64_t(nk), key_bits(n));
    L.R2 = RadixScratch::make(int64_t(2 * nk), key_bits(n - 1));
    auto most = [](size_t a, size_t b) { return a > b ? a : b; };
    Carve c;
    L.o_err = c.take(sizeof(int));
    L.o_inptr = c.take(sizeof(int64_t) * (size_t(n) + 1));
    // six arrays of n k (the two triples of the first sort), then three of
    // 2 n k (the second sort's; its fourth is tpos itself)
    L.o_buf = c.take(sizeof(uint32_t) * 6 * nk);
    L.o_ucount = c.take(sizeof(int64_t) * size_t(n));
    L.o_bsum = c.take(sizeof(int64_t) * nb);
    L.o_rcnt = c.take(most(L.R1.cnt_bytes, L.R2.cnt_bytes));
    L.o_roff = c.take(most(L.R1.off_bytes, L.R2.off_bytes));
    L.o_rbsum = c.take(most(L.R1.bsum_bytes, L.R2.bsum_bytes));
    L.bytes = c.off;
    return L;
  }
  // bits of a key 0 .. top
  static int key_bits(int64_t top) {
    int b = 1;
    while ((int64_t(1) << b) <= top) ++b;
    return b;
  }
};

// The union of the kNN patterns as CSR with the MODE combination of the two
// directed values (steps 1-5 above).
template <int MODE>
int symmetrize_impl(const int32_t* nbr_idx, const float* P_cond, int64_t n, int32_t k, int64_t* row_ptr,
                    int32_t* col, float* val, int32_t* tpos, int64_t* nnz, void* workspace, size_t* workspace_bytes,
                    void* stream) {
  if (!nbr_idx || !P_cond || !row_ptr || !col || !val || !nnz || n < 2 || k < 1 || k >= n) return TSNE_ERR_INVALID_ARG;
  if (k > TSNE_MAX_K) return TSNE_ERR_UNSUPPORTED;
  if (n > (int64_t(1) << 30)) return TSNE_ERR_UNSUPPORTED;  // 2 n k must fit int32 positions in tpos
  if (2 * n * int64_t(k) > (int64_t(1) << 31) - 1) return TSNE_ERR_UNSUPPORTED;
  const SymLayout L = SymLayout::make(n, k);
  int rc = workspace_protocol(workspace, workspace_bytes, L.bytes);
  if (rc >= 0) return rc;
  TSNE_REQUIRE_GFX950();
  char* ws = static_cast<char*>(workspace);
  int* err = reinterpret_cast<int*>(ws + L.o_err);
  int64_t* in_ptr = reinterpret_cast<int64_t*>(ws + L.o_inptr);
  uint32_t* buf = reinterpret_cast<uint32_t*>(ws + L.o_buf);
  int64_t* ucount = reinterpret_cast<int64_t*>(ws + L.o_ucount);
  int64_t* bsum = reinterpret_cast<int64_t*>(ws + L.o_bsum);
  uint32_t* rcnt = reinterpret_cast<uint32_t*>(ws + L.o_rcnt);
  int64_t* roff = reinterpret_cast<int64_t*>(ws + L.o_roff);
  int64_t* rbsum = reinterpret_cast<int64_t*>(ws + L.o_rbsum);
  hipStream_t s = as_stream(stream);
  const int64_t nk = n * k;
  const dim3 g_rows(unsigned(ceil_div(n, 4))), b(256);

  if ((rc = launch_fill<int>(err, 1, 0, s))) return rc;
  const RsBuffers lists{buf, buf + nk, buf + 2 * nk}, tmp{buf + 3 * nk, buf + 4 * nk, buf + 5 * nk};
  const SymItems items{nbr_idx, reinterpret_cast<const uint32_t*>(P_cond), n, int(k), err};
  if ((rc = radix_sort<SymItems, 2, true>(items, nk, nullptr, SymLayout::key_bits(n), L.R1, rcnt, roff, rbsum, tmp,
                                          lists, lists, s)))
    return rc;
  const int32_t* skey = reinterpret_cast<const int32_t*>(lists.key);
  const int32_t* s_src = reinterpret_cast<const int32_t*>(lists.a);
  const float* s_val = reinterpret_cast<const float*>(lists.b);
  hipLaunchKernelGGL(sym_inptr_kernel, dim3(unsigned(ceil_div(nk + 1, 256))), b, 0, s, skey, s_src, nk, n, in_ptr,
                     err);
  TSNE_CHECK_LAUNCH();
  hipLaunchKernelGGL(sym_union_count_kernel, g_rows, b, 0, s, n, k, nbr_idx, in_ptr, s_src, ucount);
  TSNE_CHECK_LAUNCH();
  if ((rc = exclusive_scan<int64_t>(ucount, n, row_ptr, bsum, s))) return rc;
  int sb = 0;
  while ((1 << sb) < k) ++sb;
  auto write = k <= 64 ? sym_write_kernel<MODE, 1> : (k <= 128 ? sym_write_kernel<MODE, 2> : sym_write_kernel<MODE, 4>);
  hipLaunchKernelGGL(write, g_rows, b, 0, s, n, int(k), sb, nbr_idx, P_cond, in_ptr, s_src, s_val, row_ptr, col, val);
  TSNE_CHECK_LAUNCH();
  if (tpos && 2 * nk <= SYM_SEARCH) {
    hipLaunchKernelGGL(sym_tpos_kernel, dim3(unsigned(ceil_div(2 * nk, 256))), b, 0, s, n, row_ptr, col, tpos);
    TSNE_CHECK_LAUNCH();
  } else if (tpos) {
    // the lists are no longer needed
    uint32_t* tp = reinterpret_cast<uint32_t*>(tpos);
    const RsBuffers t1{buf, buf + 2 * nk, nullptr}, t2{buf + 4 * nk, tp, nullptr};
    if ((rc = radix_sort<ColItems, 1, false>(ColItems{col}, 2 * nk, row_ptr + n, SymLayout::key_bits(n - 1), L.R2,
                                             rcnt, roff, rbsum, t1, t2, RsBuffers{nullptr, tp, nullptr}, s)))
      return rc;
  }
  hipLaunchKernelGGL(sym_nnz_kernel, dim3(1), dim3(64), 0, s, row_ptr, n, err, nnz);
  TSNE_CHECK_LAUNCH();
  return TSNE_OK;
}

}  // namespace tsne

extern "C" int tsne_symmetrize(const int32_t* nbr_idx, const float* P_cond, int64_t n, int32_t k, int64_t* row_ptr,
                               int32_t* col, float* val, int32_t* tpos, int64_t* nnz, void* workspace,
                               size_t* workspace_bytes, void* stream) {
  return tsne::symmetrize_impl<0>(nbr_idx, P_cond, n, k, row_ptr, col, val, tpos, nnz, workspace, workspace_bytes,
                                  stream);
}

extern "C" int tsne_umap_fuzzy_union(const int32_t* nbr_idx, const float* w, int64_t n, int32_t k, int64_t* row_ptr,
                                     int32_t* col, float* val, int32_t* tpos, int64_t* nnz, void* workspace,
                                     size_t* workspace_bytes, void* stream) {
  return tsne::symmetrize_impl<1>(nbr_idx, w, n, k, row_ptr, col, val, tpos, nnz, workspace, workspace_bytes, stream);
}
