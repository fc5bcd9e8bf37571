// Cross-tokenizer alignment kernels (Sec. 3.1 "Token Alignment"; App. B.1),
// producing the CSR span table described in heterofold.h.
//
// Integer-only.  Per receiver token, binary searches over the sender spans give
// the TA partner (sender token ending at the same character) and the number of
// overlapping sender tokens; an exclusive scan of the counts gives the entry
// offsets and a forward fill of the partners the fallback, after which each row
// writes its entries.  What bounds it is latency: the searches' chains of
// loads (the three of a row advance together), and the launches, about 6 us each
// whatever they do.  So:
//   * up to kOneBlockRows rows of a few sequences, unless they overlap many sender
//     tokens (one_block): one workgroup does everything (align_one_kernel);
//   * otherwise align_count writes each workgroup's totals, the counts and
//     partners are parked in row_ptr / den, and align_fill sums the totals of the
//     workgroups before its own.  Each receiver row is handled by the same thread
//     in both, and rows' parked values live in their own slots, so no launch
//     reads another workgroup's parked data;
//   * past kScanBlocks workgroups, where every workgroup summing all before it
//     would be quadratic, one workgroup scans the totals in between (align_scan).
// 178 rows: 9.8 us; 1,821 rows: 8.0 + 9.2 us; 7,300 rows: 9.6 + 10.4 us.  Three
// launches, with one search after the other, took 20, 28 and 34 us.
#include <hip/hip_runtime.h>
#include <limits.h>

#include "hf_internal.h"

namespace hf {
namespace {

constexpr int kScanThreads = 1024;
constexpr int kOneBlockRows = 1024;
constexpr int kOneBlockSeqs = 4;
constexpr int kScanBlocks = 1024;

// One binary search over a[0..n).
// A step is a load at a position that is inside whenever the array is not
// empty, then the comparison, so that the loads of several searches go out
// together.
struct Search {
  const int32_t* a;
  int lo, hi, n;
  __device__ __forceinline__ Search(const int32_t* a_, int n_, bool on)
      : a(a_), lo(0), hi(on ? n_ : 0), n(n_) {}
  __device__ __forceinline__ int probe() const { return a[min((lo + hi) >> 1, n - 1)]; }
  __device__ __forceinline__ void advance(bool right_of_mid) {
    const int mid = (lo + hi) >> 1;
    const bool open = lo < hi;
    hi = open && !right_of_mid ? mid : hi;
    lo = open && right_of_mid ? mid + 1 : lo;
  }
};

struct Plus {
  __device__ long long operator()(long long a, long long b) const { return a + b; }
};
struct LastValid {  // keeps the right operand unless it is "none" (negative)
  __device__ long long operator()(long long a, long long b) const { return b >= 0 ? b : a; }
};
struct Max {
  __device__ long long operator()(long long a, long long b) const { return b > a ? b : a; }
};
struct Min {
  __device__ long long operator()(long long a, long long b) const { return b < a ? b : a; }
};

template <typename Op>
__device__ __forceinline__ long long wave_inclusive_scan(long long v, Op op) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    long long o = __shfl_up(v, d, 64);
    if (lane >= d) v = op(o, v);
  }
  return v;
}

// Inclusive scan over the workgroup (threads in order); also returns the
// workgroup total.  smem: NT/64 entries.  All threads must call it.
template <int NT, typename Op>
__device__ long long block_inclusive_scan(long long v, Op op, long long identity,
                                          long long* smem, long long& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_inclusive_scan(v, op);
  if (lane == 63) smem[wid] = v;
  __syncthreads();
  long long prefix = identity, tot = identity;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wid) prefix = op(prefix, smem[w]);
    tot = op(tot, smem[w]);
  }
  __syncthreads();
  total = tot;
  return op(prefix, v);
}

__device__ __forceinline__ int seq_of_block(const AlignArgs& p, int blk) {
  int b = 0;
  while (b + 1 < p.B && p.blk_start[b + 1] <= blk) ++b;
  return b;
}

// TA partner of receiver token j (or -1) and, in overlap mode, the number of
// sender tokens sharing at least one character with it (0 if none).
struct RowInfo {
  int partner;
  int count;
  int lo, hi;  // overlap candidate range [lo, hi)
};

__device__ __forceinline__ RowInfo row_info(const AlignArgs& p, const int32_t* sb,
                                            const int32_t* se, int Ts, int rb, int re) {
  RowInfo r;
  r.partner = -1;
  r.count = 1;
  r.lo = r.hi = 0;
  const bool overlap = p.mode == HF_ALIGN_OVERLAP;
  // the last sender token ending at or before re; in overlap mode the first one
  // ending after rb and the first one starting at or after re
  Search past(se, Ts, rb < re), first(se, Ts, overlap), end(sb, Ts, overlap);
  if (overlap) {
    for (int n = Ts; n > 0; n >>= 1) {
      const int v0 = past.probe(), v1 = first.probe(), v2 = end.probe();
      past.advance(!(v0 > re));
      first.advance(!(v1 > rb));
      end.advance(!(v2 >= re));
    }
  } else {
    for (int n = Ts; n > 0; n >>= 1) past.advance(!(past.probe() > re));
  }
  if (rb < re) {
    int i = past.lo - 1;
    while (i >= 0 && se[i] == re && !(sb[i] < se[i])) --i;  // skip empty tokens at re
    if (i >= 0 && se[i] == re && sb[i] < se[i]) r.partner = i;
  }
  if (overlap) {
    r.lo = first.lo;
    r.hi = end.lo;
    int c = 0;
    for (int i = r.lo; i < r.hi; ++i) {
      int o = min(se[i], re) - max(sb[i], rb);
      c += (o > 0);
    }
    r.count = c;
  }
  return r;
}

// Row g's offset, entries and denominator: entries from `off`, the fallback (its
// own TA partner, or the one filled forward) `a`.
__device__ __forceinline__ void write_row(const AlignArgs& p, int g, long long off, int a,
                                          const RowInfo& r, const int32_t* sb, const int32_t* se,
                                          int rb, int re) {
  p.row_ptr[g] = (int32_t)(off < p.cap ? off : p.cap);
  if (p.mode == HF_ALIGN_TA || r.count == 0) {
    if (off < p.cap) {
      p.col[off] = a;
      p.num[off] = 1;
    }
    p.den[g] = 1;
    return;
  }
  int total = 0;
  long long e = off;
  for (int i = r.lo; i < r.hi; ++i) {
    int o = min(se[i], re) - max(sb[i], rb);
    if (o > 0) {
      if (e < p.cap) {
        p.col[e] = i;
        p.num[e] = o;
      }
      ++e;
      total += o;
    }
  }
  p.den[g] = total;
}

// First nonempty token of sb / se [0, Ts), 0 if there is none, by a workgroup of
// NT threads (all must call it).
template <int NT>
__device__ int first_nonempty(const int32_t* sb, const int32_t* se, int Ts, long long* smem) {
  for (int base = 0; base < Ts; base += NT) {
    const int i = base + (int)threadIdx.x;
    long long cand = LLONG_MAX;
    if (i < Ts && sb[i] < se[i]) cand = i;
    long long m;
    block_inclusive_scan<NT>(cand, Min(), LLONG_MAX, smem, m);
    if (m != LLONG_MAX) return (int)m;
  }
  return 0;
}

// The whole alignment of up to kOneBlockRows receiver rows, one per thread.
__global__ __launch_bounds__(kOneBlockRows) void align_one_kernel(const AlignArgs p) {
  __shared__ long long red[kOneBlockRows / 64];
  __shared__ int need[kOneBlockSeqs];
  __shared__ int first[kOneBlockSeqs];
  const int g = threadIdx.x;
  const bool valid = g < p.total_rows;
  int b = 0;
  while (b + 1 < p.B && p.r0[b + 1] <= g) ++b;
  const int32_t* sb = p.s_beg + p.s0[b];
  const int32_t* se = p.s_end + p.s0[b];
  if (g < kOneBlockSeqs) need[g] = 0;
  RowInfo r{-1, 0, 0, 0};
  int rb = 0, re = 0;
  long long cnt = 0, part = -1;
  if (valid) {
    rb = p.r_beg[g];
    re = p.r_end[g];
    r = row_info(p, sb, se, p.Ts[b], rb, re);
    cnt = r.count > 0 ? r.count : 1;
    // tagged with the sequence, so that a fill never crosses sequences
    if (r.partner >= 0) part = ((long long)b << 32) | r.partner;
  }
  long long tot, tl;
  const long long off = block_inclusive_scan<kOneBlockRows>(cnt, Plus(), 0, red, tot) - cnt;
  const long long fill = block_inclusive_scan<kOneBlockRows>(part, LastValid(), -1, red, tl);
  const bool none = valid && !(fill >= 0 && (int)(fill >> 32) == b);
  if (none) need[b] = 1;
  __syncthreads();
  for (int q = 0; q < p.B; ++q) {
    if (!need[q]) continue;
    const int f = first_nonempty<kOneBlockRows>(p.s_beg + p.s0[q], p.s_end + p.s0[q], p.Ts[q], red);
    if (g == 0) first[q] = f;
  }
  __syncthreads();
  if (valid) write_row(p, g, off, none ? first[b] : (int)(fill & 0xffffffffLL), r, sb, se, rb, re);
  if (g == 0) p.row_ptr[p.total_rows] = (int32_t)(tot < p.cap ? tot : p.cap);
}

__global__ __launch_bounds__(kAlignBlock) void align_count_kernel(const AlignArgs p) {
  __shared__ long long red[kAlignBlock / 64];
  const int blk = blockIdx.x;
  const int b = seq_of_block(p, blk);
  const int j = (blk - p.blk_start[b]) * kAlignBlock + threadIdx.x;
  const bool valid = j < p.Tr[b];
  const int32_t* sb = p.s_beg + p.s0[b];
  const int32_t* se = p.s_end + p.s0[b];
  long long cnt = 0, part = -1;
  if (valid) {
    const int g = p.r0[b] + j;
    RowInfo r = row_info(p, sb, se, p.Ts[b], p.r_beg[g], p.r_end[g]);
    int c = (p.mode == HF_ALIGN_OVERLAP) ? (r.count > 0 ? r.count : 1) : 1;
    p.row_ptr[g] = c;          // parked: entry count of row g
    p.den[g] = r.partner;      // parked: TA partner of row g
    cnt = c;
    part = r.partner;
  }
  long long tot_cnt, tot_part;
  block_inclusive_scan<kAlignBlock>(cnt, Plus(), 0, red, tot_cnt);
  block_inclusive_scan<kAlignBlock>(part, LastValid(), -1, red, tot_part);
  if (threadIdx.x == 0) {
    p.blk_sum[blk] = tot_cnt;
    p.blk_last[blk] = (int32_t)tot_part;
  }
}

__global__ __launch_bounds__(kScanThreads) void align_scan_kernel(const AlignArgs p) {
  __shared__ long long red[kScanThreads / 64];
  __shared__ long long incl_last[kScanThreads];
  __shared__ int first_ne[HF_MAX_BATCH];
  const int tid = threadIdx.x;

  // First nonempty sender token of each sequence (0 if there is none).
  for (int b = 0; b < p.B; ++b) {
    const int f = first_nonempty<kScanThreads>(p.s_beg + p.s0[b], p.s_end + p.s0[b], p.Ts[b], red);
    if (tid == 0) first_ne[b] = f;
  }
  __syncthreads();

  long long sum_carry = 0, last_carry = -1;
  for (int base = 0; base < p.nblk; base += kScanThreads) {
    const int k = base + tid;
    const bool valid = k < p.nblk;
    const int bs = valid ? seq_of_block(p, k) : 0;
    long long s = valid ? p.blk_sum[k] : 0;
    // Tag partners with their sequence so a carry never crosses sequences.
    long long lv = (valid && p.blk_last[k] >= 0) ? (((long long)bs << 32) | p.blk_last[k]) : -1;
    long long tot_s, tot_l;
    long long incl_s = block_inclusive_scan<kScanThreads>(s, Plus(), 0, red, tot_s);
    long long incl_l = block_inclusive_scan<kScanThreads>(lv, LastValid(), -1, red, tot_l);
    incl_last[tid] = incl_l;
    __syncthreads();
    if (valid) {
      p.blk_off[k] = sum_carry + incl_s - s;
      long long before = tid > 0 ? LastValid()(last_carry, incl_last[tid - 1]) : last_carry;
      p.blk_carry[k] = (before >= 0 && (before >> 32) == bs) ? (int32_t)(before & 0xffffffffLL)
                                                             : first_ne[bs];
    }
    sum_carry += tot_s;
    last_carry = LastValid()(last_carry, tot_l);
    __syncthreads();
  }
  if (tid == 0) p.row_ptr[p.total_rows] = (int32_t)(sum_carry < p.cap ? sum_carry : p.cap);
}

// SCANNED: align_scan has left each workgroup's offset and carried partner.
template <bool SCANNED>
__global__ __launch_bounds__(kAlignBlock) void align_fill_kernel(const AlignArgs p) {
  __shared__ long long red[kAlignBlock / 64];
  const int blk = blockIdx.x;
  const int b = seq_of_block(p, blk);
  const int j = (blk - p.blk_start[b]) * kAlignBlock + threadIdx.x;
  const bool valid = j < p.Tr[b];
  const int g = p.r0[b] + j;
  const int32_t* sb = p.s_beg + p.s0[b];
  const int32_t* se = p.s_end + p.s0[b];
  long long cnt = valid ? p.row_ptr[g] : 0;
  long long part = valid ? p.den[g] : -1;
  const int rb = valid ? p.r_beg[g] : 0, re = valid ? p.r_end[g] : 0;
  RowInfo r{-1, 1, 0, 0};
  if (valid && p.mode == HF_ALIGN_OVERLAP) r = row_info(p, sb, se, p.Ts[b], rb, re);
  long long tot;
  long long base, carry;
  if (SCANNED) {
    base = p.blk_off[blk];
    carry = p.blk_carry[blk];
  } else {  // the totals of the workgroups before this one
    long long sum = 0, last = -1;
    for (int k = threadIdx.x; k < blk; k += kAlignBlock) {
      sum += p.blk_sum[k];
      if (k >= p.blk_start[b] && p.blk_last[k] >= 0) last = ((long long)k << 32) | p.blk_last[k];
    }
    block_inclusive_scan<kAlignBlock>(sum, Plus(), 0, red, base);
    block_inclusive_scan<kAlignBlock>(last, Max(), -1, red, tot);
    carry = tot >= 0 ? (tot & 0xffffffffLL) : -1;
  }
  const long long off = block_inclusive_scan<kAlignBlock>(cnt, Plus(), 0, red, tot) - cnt + base;
  if (!SCANNED && blk == p.nblk - 1 && threadIdx.x == 0)
    p.row_ptr[p.total_rows] = (int32_t)(base + tot < p.cap ? base + tot : p.cap);
  const long long fill = block_inclusive_scan<kAlignBlock>(part, LastValid(), -1, red, tot);
  if (!SCANNED && carry < 0 && __syncthreads_or(valid && fill < 0))
    carry = first_nonempty<kAlignBlock>(sb, se, p.Ts[b], red);
  if (!valid) return;
  write_row(p, g, off, fill >= 0 ? (int)fill : (int)carry, r, sb, se, rb, re);
}

}  // namespace

size_t align_workspace_bytes(int nblk) {
  size_t n = (size_t)(nblk > 0 ? nblk : 1);
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  return 2 * up(n * sizeof(long long)) + 2 * up(n * sizeof(int32_t));
}

// Whether one workgroup aligns the batch.  It looks for a fallback one sequence after
// the other: us of one workgroup and of two launches at 1,024 rows, 2 sequences
// 13.8/17.3, 4 16.7/17.2, 6 22/17, 16 39/18, 64 124/21.  And it walks the overlaps on one
// CU: 900 rows of 1, 9, 16 and 99 sender tokens each 13.6/17.5, 25/20, 49/30, 302/139;
// 500 rows 13.9/17.3, 17/20, 31/30, 177/136.  Up to kAlignBlock rows the two launches
// have no more than one workgroup a sequence either (250 rows of 98: 100/131).
static bool one_block(const AlignArgs& a) {
  if (a.total_rows < 1 || a.total_rows > kOneBlockRows || a.B > kOneBlockSeqs) return false;
  const long long senders = a.s0[a.B - 1] + a.Ts[a.B - 1];
  return a.mode == HF_ALIGN_TA || a.total_rows <= kAlignBlock ||
         senders * a.total_rows <= 4LL << 20;
}

hipError_t launch_alignment(const AlignArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)a.nblk), block(kAlignBlock);
  if (one_block(a)) {
    hipLaunchKernelGGL(align_one_kernel, dim3(1), dim3(kOneBlockRows), 0, s, a);
    return hipGetLastError();
  }
  if (a.nblk > 0) hipLaunchKernelGGL(align_count_kernel, grid, block, 0, s, a);
  if (a.nblk > 0 && a.nblk <= kScanBlocks) {
    hipLaunchKernelGGL(align_fill_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(align_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, a);
  if (a.nblk > 0) hipLaunchKernelGGL(align_fill_kernel<true>, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace hf
