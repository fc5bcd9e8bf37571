// Offline construction of the folded affine maps on the GPU, in fp64:
//   * weighted sender RMS (Eq. 3), means and the joint covariance of [x/r | y]
//     (Sec. 3.2) -- one weighted, centred Gram product over all samples;
//   * Recolor (Eq. 4-5): symmetric roots of the covariances and the Procrustes
//     factor R* = U Q^T of the whitened cross-covariance, by Newton-Schulz
//     iterations (matrix products only; R* is the polar factor of that matrix);
//   * the fold of the low-rank correction into the map (Eq. 9).
//
// Every product runs on one fp64 matrix-core GEMM kernel
// (v_mfma_f64_16x16x4f64).  The iterations run without host synchronization:
// a small state record in device memory tells the remaining launches of a
// converged iteration to do nothing.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "hf_internal.h"

namespace hf {
namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kBN = 64, kBK = 16;  // a tile is 128 x 64 or 64 x 64
constexpr int kPad = 4;            // padding of the LDS rows, doubles
constexpr int kGemmThreads = 256;
constexpr int kGemmResident = 768;  // workgroups resident at once (3 per CU: 51 KB of LDS each)
// Products with fewer 128 x 64 tiles than this (two per CU) run on 64 x 64 tiles.
constexpr int kGemmSmallTiles = 512;
constexpr int kRedThreads = 256;
constexpr int kMaxRedBlocks = 1024;

// Newton-Schulz convergence: once the residual |I - P|_F falls below this, the
// error contracts as e' = 3/4 e^2 + e^3/4, so three more steps reach rounding --
// which for P = Z Y of the roots grows with the condition number of S (last residual
// at 150 x 150: 5e-14 at 1e4, 3e-12 at 1e8, 2e-10 at 1e12).
constexpr double kNsSwitch = 1e-3;
constexpr int kNsExtra = 2;
// Scaling of the steps (ns_update): the smallest singular value assumed at the
// start, for the roots and for the polar factor, and the largest squared scale.
// Roots: a low bound takes fewer steps where S is badly conditioned (13, 22, 34 against
// 14, 25, 36 at condition numbers 1e4, 1e8, 1e12) and 13 instead of 10 where it is not.
// The eigenvalues' mean square over their squared mean tells: kNsSpread comes out
// at condition numbers of some 1e3 to 1e4 if they are spread evenly on a log scale.
constexpr double kNsFloorAlike = 3e-2;
constexpr double kNsFloorSpread = 3e-3;
constexpr double kNsSpread = 4.0;
constexpr double kNsFloorPolar = 1e-2;
constexpr double kNsMaxScale2 = 2.25;
constexpr int kNsRestart = 20;

struct NsState {
  int done;       // 1 once the iteration has converged and its last step is taken
  int extra;      // steps still to take after the switch (-1 before it)
  int iters;      // steps taken: the iterate is in ping-pong buffer iters & 1
  int arrived;    // workgroups that have left their share of the residual
  double res;     // last residual |I - P|_F
  double low;     // assumed lower bound of the iterate's singular values
  double again;   // the bound when the scaling starts over (1: it does not)
  double alpha;   // this step is X' = beta X + alpha X P
  double beta;
};

__device__ inline double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  return s;  // valid in thread 0
}

// Fixed-order sum of partials other workgroups of this launch wrote.
__device__ inline double sum_partials(const double* partial, long long n, double* red) {
  double s = 0.0;
  for (long long i = threadIdx.x; i < n; i += blockDim.x)
    s += __hip_atomic_load(partial + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return block_sum(s, red);
}

// Whether this workgroup is the last of n to leave its share (thread 0 has
// written it).  No workgroup waits for another; the last one finds all shares.
__device__ inline bool last_arrival(int* arrived, long long n) {
  __shared__ int last;
  if (threadIdx.x == 0) {
    __threadfence();
    last = atomicAdd(arrived, 1) == (int)(n - 1);
  }
  __syncthreads();
  const bool mine = last != 0;
  __syncthreads();
  if (mine) {
    __threadfence();
    if (threadIdx.x == 0) *arrived = 0;
  }
  return mine;
}

// The step after the residual |I - P|_F of the current iterate is known (one
// thread).  A plain step x <- x (3 - x^2) / 2 takes a small singular value up by
// 3/2 only.  The step on mu x, with mu^2 = 3 / (1 + l + l^2), maps [l, 1] into
// [l', 1], l' = mu l (3 - mu^2 l^2) / 2, and takes small values up by 3 mu / 2
// (Chen and Chow's scaling of the Newton-Schulz sign iteration); values
// below l also grow and stay positive, so a bound assumed too high costs steps
// and nothing else: where values are still small after kNsRestart steps, the
// scaling of the polar iteration starts over.  That of the roots does not: values
// that have converged shrink by 3/8 in a scaled step and grow back, and the coupled
// iterates do not correct the rounding of that (in fp64 on the host the error of
// S^{1/2} is 2 to 3 times larger at condition numbers of 1e10 and more).
// mu^2 <= 2.25 keeps the factor (3 - mu^2) / 2 that the largest values meet at 3/8
// or more, away from cancellation, for one more step in a dozen.  mu = 1 exactly
// once the residual shows convergence.
__device__ inline void ns_update(NsState* st, double res) {
  st->res = res;
  if (st->extra == 0) {
    st->done = 1;
    return;
  }
  if (st->extra > 0)
    st->extra -= 1;
  else if (res <= kNsSwitch)
    st->extra = kNsExtra;
  st->iters += 1;
  double l = st->low;
  if (res < 0.3) l = 1.0;
  else if (l > 0.9) l = st->iters >= kNsRestart ? st->again : 1.0;
  const double mu2 = fmin(kNsMaxScale2, 3.0 / (1.0 + l + l * l)), mu = sqrt(mu2);
  st->alpha = -0.5 * mu * mu2;
  st->beta = 1.5 * mu;
  st->low = 0.5 * mu * l * (3.0 - mu2 * l * l);
}

// One product D = alpha op(A) op(B) + beta C + gamma I of a launch.
enum JobKind {
  kPlain = 0,
  kStep,     // D = st->alpha op(A) op(B) + st->beta C
  kGram,     // P = op(A) op(B) with the residual |I - P|_F
  kGramSym   // the same with a symmetric result: upper tiles, mirrored
};
struct GemmJob {
  int m, n;
  long long k;
  const double* A;
  long long lda;
  const double* B;
  long long ldb;
  const double* C;  // read when beta != 0 (may alias D)
  long long ldc;
  double* D;
  long long ldd;
  double alpha, beta, gamma;
  const double* ratio_num;  // alpha *= sqrt(num / den), or nullptr
  const double* ratio_den;
  int kind;
  int a_kmajor, b_kmajor;  // op(A)(i, kk) at A[kk lda + i], else A[i lda + kk]; op(B) likewise
  int fast;  // inner tiles may read both operands 16 bytes at a time, in whole slices
  NsState* st;         // step kinds: the iteration; nothing is done once it is done
  double* partial;     // kGram: residual shares, one per tile
  const NsState* a_sel;  // A (B) is A1 (B1) where this iteration took an odd number of steps
  const double* A1;
  const NsState* b_sel;
  const double* B1;
};
constexpr int kMaxJobs = 4;
struct GemmBatch {
  int n_jobs;
  int bm;                         // tile height: 128 or 64
  long long first[kMaxJobs + 1];  // first tile of each job
  GemmJob job[kMaxJobs];
};

typedef double double2_t __attribute__((ext_vector_type(2)));

// One thread's 4 elements of each kBK x 64 slice of an operand: element (i, kk) at
// P[kk ld + i] (KM) or P[i ld + kk].  FAST: the tile lies inside the operand and its
// rows are 16-byte aligned.  Otherwise rows past the edge repeat the last one; what
// they give is not stored.  Nothing looks at a loaded value before gemm_store: with
// elements selected in every slice (each waits for its load) a 333 x 777 x 555 product
// took 80 us and 2000 x 2000 x 2000 440 to 500, now 33 and 300; a last slice that k cuts
// goes through gemm_tail.
template <bool KM, bool FAST>
struct GemmSrc {
  const double* q;  // this thread's elements of slice 0
  int off[4];       // KM, not FAST: its columns

  __device__ inline GemmSrc(const double* P, long long ld, int rows, int i0, int tid) {
    const int i = KM ? i0 + (tid & 15) * 4 : i0 + (tid & 63);
    if (KM) q = P + (tid >> 4) * ld + (FAST ? i : 0);
    else q = P + (long long)(FAST ? i : min(i, rows - 1)) * ld + (tid >> 6) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) off[e] = KM ? min(i + e, rows - 1) : e;
  }
  // FAST: of the rows `down` below
  __device__ inline void load(long long ld, long long kt, double (&r)[4], int down = 0) const {
    const double* z = q + (KM ? kt * kBK * ld + down : kt * kBK + down * ld);
    if (FAST) {
      const double2_t a = *reinterpret_cast<const double2_t*>(z);
      const double2_t b = *reinterpret_cast<const double2_t*>(z + 2);
      r[0] = a.x; r[1] = a.y; r[2] = b.x; r[3] = b.y;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = z[off[e]];
    }
  }
};

// The same elements of a slice from k0 that reaches past k: inputs past the end read
// the last one and count as zero.
template <bool KM>
__device__ inline void gemm_tail(const double* P, long long ld, int rows, long long k, int i0,
                                 long long k0, int tid, double (&r)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = min(KM ? i0 + (tid & 15) * 4 + e : i0 + (tid & 63), rows - 1);
    const long long kk = KM ? k0 + (tid >> 4) : k0 + (tid >> 6) * 4 + e;
    const long long in = kk < k ? kk : k - 1;
    const double v = KM ? P[in * ld + i] : P[(long long)i * ld + in];
    r[e] = kk < k ? v : 0.0;
  }
}

template <bool KM, int LD>
__device__ inline void gemm_store(double (*S)[LD], int c0, int tid, const double (&r)[4]) {
  if (KM) {
    double* q = &S[tid >> 4][c0 + (tid & 15) * 4];
    *reinterpret_cast<double2_t*>(q) = double2_t{r[0], r[1]};
    *reinterpret_cast<double2_t*>(q + 2) = double2_t{r[2], r[3]};
  } else {
    const int i = c0 + (tid & 63), k4 = (tid >> 6) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) S[k4 + e][i] = r[e];
  }
}

template <int BM>
struct GemmLds {
  __attribute__((aligned(16))) double A[2][kBK][BM + kPad];
  __attribute__((aligned(16))) double B[2][kBK][kBN + kPad];
};

// One thread's share of a slice of both operands.
template <int BM>
struct GemmRegs {
  double a[BM / 64][4], b[4];
};

// The k-loop of one tile, for one pair of layouts.  PF slices load while one is
// multiplied: one for the tall tile, whose three workgroups per CU hide each
// other's loads, two for the small one, which runs where a CU has one workgroup;
// one again for short products on small tiles (Batch::launch).
template <int BM, int PF, bool AK, bool BK, bool FAST>
__device__ inline void gemm_tile(const GemmJob& g, const double* A, const double* B, int m0, int n0,
                                 GemmLds<BM>& L, double4_t (&acc)[BM / 32][2]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lk = lane >> 4;
  const long long nk = g.k / kBK;  // whole slices
  GemmRegs<BM> r[PF];
  const GemmSrc<AK, FAST> srcA(A, g.lda, g.m, m0, tid);
  const GemmSrc<AK, FAST> srcA1(A, g.lda, g.m, m0 + (BM > 64 ? 64 : 0), tid);
  const GemmSrc<BK, FAST> srcB(B, g.ldb, g.n, n0, tid);
  auto load = [&](GemmRegs<BM>& z, long long kt) {
    srcA.load(g.lda, kt, z.a[0]);
    if (BM > 64) {
      if (FAST) srcA.load(g.lda, kt, z.a[BM / 64 - 1], 64);
      else srcA1.load(g.lda, kt, z.a[BM / 64 - 1]);
    }
    srcB.load(g.ldb, kt, z.b);
  };
  auto store = [&](const GemmRegs<BM>& z, int buf) {
#pragma unroll
    for (int h = 0; h < BM / 64; ++h) gemm_store<AK>(L.A[buf], 64 * h, tid, z.a[h]);
    gemm_store<BK>(L.B[buf], 0, tid, z.b);
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < kBK / 4; ++ks) {
      double a[BM / 32], b[2];
#pragma unroll
      for (int x = 0; x < BM / 32; ++x) a[x] = L.A[buf][ks * 4 + lk][wm * (BM / 2) + x * 16 + li];
#pragma unroll
      for (int y = 0; y < 2; ++y) b[y] = L.B[buf][ks * 4 + lk][wn * 32 + y * 16 + li];
#pragma unroll
      for (int x = 0; x < BM / 32; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
    }
  };
  // slice kt + PF loads into the registers that slice kt has left
  if (nk > 0) {
    load(r[0], 0);
    store(r[0], 0);
    if (PF == 2 && nk > 1) load(r[1], 1);
    __syncthreads();
    long long kt = 0;
    if (PF == 1) {
      for (; kt + 1 < nk; ++kt) {
        load(r[0], kt + 1);
        multiply((int)(kt & 1));
        store(r[0], (int)((kt + 1) & 1));
        __syncthreads();
      }
    } else {
      for (; kt + 3 < nk; kt += 2) {
        load(r[0], kt + 2);
        multiply(0);
        store(r[PF - 1], 1);
        __syncthreads();
        load(r[PF - 1], kt + 3);
        multiply(1);
        store(r[0], 0);
        __syncthreads();
      }
      // at most three slices left: kt in LDS buffer 0, kt + 1 in r[1]
      if (kt + 2 < nk) load(r[0], kt + 2);
      if (kt + 1 < nk) {
        multiply(0);
        store(r[PF - 1], 1);
        __syncthreads();
        ++kt;
        if (kt + 1 < nk) {
          multiply(1);
          store(r[0], 0);
          __syncthreads();
          ++kt;
        }
      }
    }
    multiply((int)(kt & 1));
    __syncthreads();
  }
  if (!FAST && g.k % kBK != 0) {
#pragma unroll
    for (int h = 0; h < BM / 64; ++h)
      gemm_tail<AK>(A, g.lda, g.m, g.k, m0 + 64 * h, nk * kBK, tid, r[0].a[h]);
    gemm_tail<BK>(B, g.ldb, g.n, g.k, n0, nk * kBK, tid, r[0].b);
    store(r[0], 0);
    __syncthreads();
    multiply(0);
    __syncthreads();
  }
}

// The fp64 products.  A launch runs the BM x 64 tiles of up to four products
// (the two root iterations run side by side); 4 waves in a 2 x 2 grid own
// BM/2 x 32 each as matrix-core tiles of 16 x 16.  The fp64 MFMA reads
// op(A)(i, k) from lane i + 16 k and op(B)(k, j) from lane j + 16 k, and leaves
// D(lane / 16 + 4 v, lane % 16) in element v of each lane (rows interleaved).
// X^T X of the polar iteration, which is symmetric whatever X holds, has only the
// tiles that reach its upper triangle computed, and mirrored.
//
// What bounds it: the fp64 matrix cores (78.6 TFLOP/s; the library reaches 72).
// A 3072 x 3072 product takes 0.97 to 1.10 ms from one card to another (53 to 60
// TFLOP/s; on the same cards 1.09 to 1.30 ms with 64 x 64 tiles and loads under
// conditions).  64 x 32 per wave reads 6 fragments from LDS for 8
// matrix instructions (32 x 32: 4 for 4); 128 x 128 tiles would leave the 576
// of them 0.75 of three rounds.  Three workgroups per CU (1.10 ms) hide
// the loads and the barrier better than two (1.18).  A workgroup takes every
// gridDim.x-th tile, so the launches of an iteration that is already done are
// 768 workgroups and not thousands.
template <int BM, int PF>
__device__ __forceinline__ void gemm_batch(const GemmBatch& gb) {
  __shared__ GemmLds<BM> L;
  __shared__ double red[kGemmThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lk = lane >> 4;

  const long long total = gb.first[gb.n_jobs];
  for (long long t0 = blockIdx.x; t0 < total; t0 += gridDim.x) {
    int ji = 0;
    while (ji + 1 < gb.n_jobs && gb.first[ji + 1] <= t0) ++ji;
    const GemmJob& g = gb.job[ji];
    if (g.st && g.st->done) continue;
    const bool sym = g.kind == kGramSym;
    const long long t = t0 - gb.first[ji];
    const int ntn = (g.n + kBN - 1) / kBN;
    int tm, tn;
    if (sym) {  // row block tm has the column blocks tm BM / 64 .. ntn - 1
      long long rem = t;
      tm = 0;
      while (rem >= ntn - tm * (BM / kBN)) {
        rem -= ntn - tm * (BM / kBN);
        ++tm;
      }
      tn = tm * (BM / kBN) + (int)rem;
    } else {
      tm = (int)(t / ntn);
      tn = (int)(t - (long long)tm * ntn);
    }
    const int m0 = tm * BM, n0 = tn * kBN;
    const double* A = g.a_sel && (g.a_sel->iters & 1) ? g.A1 : g.A;
    const double* B = g.b_sel && (g.b_sel->iters & 1) ? g.B1 : g.B;
    const bool fast = g.fast && m0 + BM <= g.m && n0 + kBN <= g.n;

    double4_t acc[BM / 32][2];
#pragma unroll
    for (int a = 0; a < BM / 32; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = double4_t{0.0, 0.0, 0.0, 0.0};
    if (g.a_kmajor && g.b_kmajor) {
      if (fast) gemm_tile<BM, PF, true, true, true>(g, A, B, m0, n0, L, acc);
      else gemm_tile<BM, PF, true, true, false>(g, A, B, m0, n0, L, acc);
    } else if (g.a_kmajor) {
      if (fast) gemm_tile<BM, PF, true, false, true>(g, A, B, m0, n0, L, acc);
      else gemm_tile<BM, PF, true, false, false>(g, A, B, m0, n0, L, acc);
    } else if (g.b_kmajor) {
      if (fast) gemm_tile<BM, PF, false, true, true>(g, A, B, m0, n0, L, acc);
      else gemm_tile<BM, PF, false, true, false>(g, A, B, m0, n0, L, acc);
    } else {
      if (fast) gemm_tile<BM, PF, false, false, true>(g, A, B, m0, n0, L, acc);
      else gemm_tile<BM, PF, false, false, false>(g, A, B, m0, n0, L, acc);
    }

    double alpha = g.alpha, beta = g.beta;
    if (g.kind == kStep) {
      alpha = g.st->alpha;
      beta = g.st->beta;
    } else if (g.ratio_num) {
      alpha *= sqrt(*g.ratio_num / *g.ratio_den);
    }
    const bool gram = g.kind == kGram || g.kind == kGramSym;
    double res = 0.0;
#pragma unroll
    for (int x = 0; x < BM / 32; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = m0 + wm * (BM / 2) + x * 16 + lk + 4 * v;
          const int j = n0 + wn * 32 + y * 16 + li;
          if (i >= g.m || j >= g.n || (sym && i > j)) continue;
          double val = alpha * acc[x][y][v];
          if (beta != 0.0) val += beta * g.C[(long long)i * g.ldc + j];
          if (i == j) val += g.gamma;
          g.D[(long long)i * g.ldd + j] = val;
          if (sym && i != j) g.D[(long long)j * g.ldd + i] = val;
          if (gram) res += i == j ? (val - 1.0) * (val - 1.0) : (sym ? 2.0 : 1.0) * val * val;
        }
    if (gram) {
      const double share = block_sum(res, red);
      if (tid == 0) g.partial[t] = share;
      const long long n_tiles = gb.first[ji + 1] - gb.first[ji];
      if (last_arrival(&g.st->arrived, n_tiles)) {
        const double s = sum_partials(g.partial, n_tiles, red);
        if (tid == 0) ns_update(g.st, sqrt(s));
      }
    }
  }
}

template <int BM, int PF>
__global__ __launch_bounds__(kGemmThreads, BM == 64 && PF == 1 ? 4 : 3) void gemm_f64_kernel(
    const GemmBatch gb) {
  gemm_batch<BM, PF>(gb);
}

// The products of one step of an iteration, described once in the workspace:
// the hundreds of launches of the iterations then pass one pointer each instead of
// 800 bytes of arguments (5 us of host time each on a 100 x 37 solve).
template <int BM>
__global__ __launch_bounds__(kGemmThreads, 3) void gemm_f64_planned_kernel(
    const GemmBatch* __restrict__ gb) {
  gemm_batch<BM, BM == 64 ? 2 : 1>(*gb);
}

constexpr int kPlanPart = 4;  // descriptions per launch of the kernel that stores them
struct PlanPart {
  GemmBatch g[kPlanPart];
};
static_assert(sizeof(PlanPart) <= 4096, "kernel argument size");
__global__ __launch_bounds__(256) void store_plan_kernel(const PlanPart part, GemmBatch* dst, int n) {
  const uint32_t* src = reinterpret_cast<const uint32_t*>(part.g);
  uint32_t* out = reinterpret_cast<uint32_t*>(dst);
  for (unsigned i = threadIdx.x; i < n * sizeof(GemmBatch) / 4; i += 256) out[i] = src[i];
}

// ---------------------------------------------------------------------------
// Weighted, centred Gram product of the samples V = [X | Y] (n rows, m = p + q
// columns): G = (V - 1 shift^T)^T diag(w) (V - 1 shift^T), upper 128 x 128
// tiles only, the rows split into `splits` ranges whose partial tiles a second
// kernel adds up in a fixed order.  Work item = (split, tile), split-major, so
// the workgroups resident together stream the same rows.
// ---------------------------------------------------------------------------
constexpr int kCT = 128;   // tile edge
constexpr int kCK = 16;    // rows per step
constexpr int kCPad = 16;
constexpr int kCovResident = 512;  // workgroups resident at once (2 per CU)

struct CovArgs {
  long long n;
  int p, m;
  const void* X;
  long long ldx;
  const void* Y;
  long long ldy;
  const float* w;
  const double* shift;  // [m]
  int nt;               // tiles per edge
  int n_tiles;          // nt (nt + 1) / 2
  long long rows_per_split;
  double* partial;      // [splits][n_tiles][kCT][kCT]
};

// Four consecutive samples as fp32 (bf16 widened exactly).
__device__ inline void load4(const float* p, float (&v)[4]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}
__device__ inline void load4(const uint16_t* p, float (&v)[4]) {
  const uint2 a = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(a.x << 16);
  v[1] = __uint_as_float(a.x & 0xffff0000u);
  v[2] = __uint_as_float(a.y << 16);
  v[3] = __uint_as_float(a.y & 0xffff0000u);
}
__device__ inline float load1(const float* p) { return *p; }
__device__ inline float load1(const uint16_t* p) { return __uint_as_float(((uint32_t)*p) << 16); }
__device__ inline double load_elem(const float* p, long long i) { return (double)p[i]; }
__device__ inline double load_elem(const uint16_t* p, long long i) {
  return (double)__uint_as_float(((uint32_t)p[i]) << 16);
}

// 256 threads = 4 waves in a 2 x 2 grid, each owning 64 x 64 as 4 x 4 MFMA tiles.
// A thread stages columns (tid % 16) 4 + {0, 64} .. +3 of row tid / 16 of each
// operand, so that 16 threads write a whole LDS row without bank conflicts.
// VEC: groups of 4 columns are aligned and lie in X or in Y whole, so a thread
// walks fixed pointers down the rows with one load each and no branch between
// them (branches made the compiler wait for each load before the next).
// Columns past m read earlier ones again; their results are not used.
// What bounds it: the fp64 matrix cores.  2^18 x 4096 samples: 70.2 ms, 64.6 TFLOP/s
// (77.2 ms with loads behind the branches; 62.9 without loads and staging).
template <typename T, bool VEC>
__global__ __launch_bounds__(256, 2) void cov_kernel(CovArgs g) {
  __shared__ __attribute__((aligned(16))) double As[2][kCK][kCT + kCPad];
  __shared__ __attribute__((aligned(16))) double Bs[2][kCK][kCT + kCPad];
  const int item = blockIdx.x;
  const int split = item / g.n_tiles, tile = item - split * g.n_tiles;
  int tm = 0, rem = tile;
  while (rem >= g.nt - tm) {
    rem -= g.nt - tm;
    ++tm;
  }
  const int tn = tm + rem;
  const long long r_beg = (long long)split * g.rows_per_split;
  const long long r_end = r_beg + g.rows_per_split < g.n ? r_beg + g.rows_per_split : g.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lk = lane >> 4;
  const T* X = static_cast<const T*>(g.X);
  const T* Y = static_cast<const T*>(g.Y);

  // staging role: group o of columns: 0, 1 of operand A, 2, 3 of operand B
  const int kk = tid >> 4, c4 = (tid & 15) * 4;
  int col[4];
  double sh[4][4];
  const T* at[4];    // VEC: the group in this thread's row
  long long by[4];   // VEC: kCK rows further down
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    col[o] = (o < 2 ? tm : tn) * kCT + (o & 1) * 64 + c4;
#pragma unroll
    for (int e = 0; e < 4; ++e) sh[o][e] = col[o] + e < g.m ? g.shift[col[o] + e] : 0.0;
    if (VEC) {
      const int c = col[o] < g.m ? col[o] : g.m - 4;
      const long long r = r_beg + kk < r_end ? r_beg + kk : r_end - 1;
      at[o] = c < g.p ? X + r * g.ldx + c : Y + r * g.ldy + (c - g.p);
      by[o] = kCK * (c < g.p ? g.ldx : g.ldy);
    }
  }

  double4_t acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = double4_t{0.0, 0.0, 0.0, 0.0};

  float v[4][4];
  float wr = 1.f;
  auto fetch = [&](long long k0) {
    // rows past the range read an earlier one again and are staged as zeros
    const bool in = k0 + kk < r_end;
    const long long r = in ? k0 + kk : r_end - 1;
    if (g.w) wr = g.w[r];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      if (VEC) {
        load4(at[o], v[o]);
        if (k0 + kCK + kk < r_end) at[o] += by[o];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = col[o] + e < g.m ? col[o] + e : g.m - 1;
          v[o][e] = load1(c < g.p ? X + r * g.ldx + c : Y + r * g.ldy + (c - g.p));
        }
      }
    }
  };
  auto stage = [&](int buf, long long k0) {
    const double wd = (double)wr;
    const bool in = k0 + kk < r_end;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      double d[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d[e] = (double)v[o][e] - sh[o][e];
        if (o < 2) d[e] *= wd;
        // rows past the range count as zero, rows of weight 0 as absent if finite (an
        // Inf or NaN sample reaches the result whatever its weight, here and in the means)
        if (!in || (o >= 2 && wr == 0.f)) d[e] = 0.0;
      }
      double* q = (o < 2 ? As : Bs)[buf][kk] + (o & 1) * 64 + c4;
      *reinterpret_cast<double2_t*>(q) = double2_t{d[0], d[1]};
      *reinterpret_cast<double2_t*>(q + 2) = double2_t{d[2], d[3]};
    }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < kCK / 4; ++ks) {
      double a[4], b[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        a[x] = As[buf][ks * 4 + lk][wm * 64 + x * 16 + li];
        b[x] = Bs[buf][ks * 4 + lk][wn * 64 + x * 16 + li];
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
    }
  };

  const long long nk = r_end > r_beg ? (r_end - r_beg + kCK - 1) / kCK : 0;
  if (nk > 0) {
    fetch(r_beg);
    stage(0, r_beg);
    __syncthreads();
    for (long long kt = 0; kt + 1 < nk; ++kt) {
      const int cur = (int)(kt & 1);
      fetch(r_beg + (kt + 1) * kCK);
      multiply(cur);
      stage(cur ^ 1, r_beg + (kt + 1) * kCK);
      __syncthreads();
    }
    multiply((int)((nk - 1) & 1));
  }

  double* out = g.partial + ((long long)split * g.n_tiles + tile) * (kCT * kCT);
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        out[(wm * 64 + x * 16 + lk + 4 * u) * kCT + wn * 64 + y * 16 + li] = acc[x][y][u];
}

// cov[i][j] = scale_i scale_j / W * sum over splits of the (min, max) entry:
// both triangles from the upper tiles, so the result is exactly symmetric.  A
// workgroup sums one 32 x 32 block of an upper tile, writes it, and writes it
// transposed through LDS, so that every partial is read once, in whole lines
// (4096 columns, 16 splits: 2350 us with the lower triangle read down the columns).
constexpr int kRB = 32;
__global__ __launch_bounds__(256) void cov_reduce_kernel(const double* partial, int splits,
                                                          int n_tiles, int nt, int m,
                                                          const double* scale,
                                                          const double* inv_w, double* cov) {
  __shared__ double t[kRB][kRB + 1];
  constexpr int per = kCT / kRB;
  const int tile = blockIdx.x / (per * per), blk = blockIdx.x - tile * (per * per);
  int tm = 0, rem = tile;
  while (rem >= nt - tm) {
    rem -= nt - tm;
    ++tm;
  }
  const int bi = (blk / per) * kRB, bj = (blk % per) * kRB;  // inside the tile
  const int i0 = tm * kCT + bi, j0 = (tm + rem) * kCT + bj;
  const int c = threadIdx.x & (kRB - 1), r = threadIdx.x / kRB;
  if (i0 >= m || j0 >= m || j0 + kRB <= i0) return;  // nothing on or above the diagonal
  const double iw = *inv_w;
  const long long step = (long long)n_tiles * (kCT * kCT);
  const double* src = partial + (long long)tile * (kCT * kCT) + bi * kCT + bj + c;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < splits; ++k)
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += src[k * step + (r + 8 * u) * kCT];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = i0 + r + 8 * u, j = j0 + c;
    double v = 0.0;
    if (i < m && j < m && i <= j) {
      v = s[u] * scale[i] * scale[j] * iw;
      cov[(long long)i * m + j] = v;
    }
    t[r + 8 * u][c] = v;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = j0 + r + 8 * u, i = i0 + c;  // row j, column i of the lower triangle
    if (j < m && i < m && i < j) cov[(long long)j * m + i] = t[c][r + 8 * u];
  }
}

// ---------------------------------------------------------------------------
// Elementwise and reduction kernels of the solve (fixed order: block tree, then
// the last workgroup over the partials).  blockIdx.y is the root iteration.
// ---------------------------------------------------------------------------
struct NsProblem {
  const double* M;  // rows x cols block, leading dimension ld
  long long ld;
  int rows, cols;
  double* lam;      // absolute ridge, or nullptr
  double* norm;     // |M + lam I|_F
  double* Y;        // first iterate
  double* Z1;       // the second iterate's other factor
  NsState* st;
  double* partial;
  double* trace;    // trace of M + lam I (nullptr: the polar iteration)
};
struct NsPair {
  NsProblem q[2];
};

// The singular value the scaled steps of a root start from: by the spread of the d
// eigenvalues of S, or what the ridge assures where that is more.  c = |S|_F.
__device__ inline double ns_root_bound(int d, double trace, double c, double lam) {
  const double floor = d * c * c >= kNsSpread * trace * trace ? kNsFloorSpread : kNsFloorAlike;
  return fmin(1.0, fmax(floor, sqrt(fmax(0.0, lam / c))));
}

__device__ inline NsState ns_initial(double again) {
  NsState z;
  z.done = 0;
  z.extra = -1;
  z.iters = 0;
  z.arrived = 0;
  z.res = -1.0;
  z.low = 1.0;
  z.again = again;
  z.alpha = -0.5;
  z.beta = 1.5;
  return z;
}

// Reset the iteration; *lam = ridge * trace(M) / rows.
__global__ __launch_bounds__(kRedThreads) void ns_start_kernel(const NsPair pr, double ridge,
                                                               NsState* polar) {
  __shared__ double red[kRedThreads / 64];
  const NsProblem& q = pr.q[blockIdx.x];
  double s = 0.0;
  for (int i = threadIdx.x; i < q.rows; i += blockDim.x) s += q.M[(long long)i * q.ld + i];
  s = block_sum(s, red);
  if (threadIdx.x != 0) return;
  *q.lam = ridge * s / q.rows;
  *q.trace = s + ridge * s;
  *q.st = ns_initial(1.0);
  if (blockIdx.x == 0) *polar = ns_initial(kNsFloorPolar);
}

// *norm = |M + lam I|_F, and the singular value the scaled steps start from.
__global__ __launch_bounds__(kRedThreads) void ns_norm_kernel(const NsPair pr) {
  __shared__ double red[kRedThreads / 64];
  const NsProblem& q = pr.q[blockIdx.y];
  const double add = q.lam ? *q.lam : 0.0;
  const long long total = (long long)q.rows * q.cols;
  double s = 0.0;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(e / q.cols), j = (int)(e - (long long)i * q.cols);
    const double v = q.M[(long long)i * q.ld + j] + (i == j ? add : 0.0);
    s += v * v;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) q.partial[blockIdx.x] = s;
  if (!last_arrival(&q.st->arrived, gridDim.x)) return;
  const double c = sqrt(sum_partials(q.partial, gridDim.x, red));
  if (threadIdx.x == 0) {
    *q.norm = c;
    q.st->low = q.trace ? ns_root_bound(q.rows, *q.trace, c, add) : kNsFloorPolar;
  }
}

// Y0 = (M + lam I) / c with Z0 = I: P0 = Y0, whose residual decides the first step.
__global__ __launch_bounds__(kRedThreads) void ns_root_init_kernel(const NsPair pr) {
  __shared__ double red[kRedThreads / 64];
  const NsProblem& q = pr.q[blockIdx.y];
  const int d = q.rows;
  const long long total = (long long)d * d;
  const double inv = 1.0 / *q.norm, lam = *q.lam;
  double s = 0.0;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(e / d), j = (int)(e - (long long)i * d);
    const double v = (q.M[(long long)i * q.ld + j] + (i == j ? lam : 0.0)) * inv;
    q.Y[e] = v;
    const double o = v - (i == j ? 1.0 : 0.0);
    s += o * o;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) q.partial[blockIdx.x] = s;
  if (!last_arrival(&q.st->arrived, gridDim.x)) return;
  const double t = sum_partials(q.partial, gridDim.x, red);
  if (threadIdx.x == 0) ns_update(q.st, sqrt(t));
}

// Z1 = beta I + alpha Y0 (the first step of Z0 = I).
__global__ __launch_bounds__(kRedThreads) void ns_root_first_kernel(const NsPair pr) {
  const NsProblem& q = pr.q[blockIdx.y];
  const int d = q.rows;
  const long long total = (long long)d * d;
  const double alpha = q.st->alpha, beta = q.st->beta;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(e / d), j = (int)(e - (long long)i * d);
    q.Z1[e] = alpha * q.Y[e] + (i == j ? beta : 0.0);
  }
}

// X *= 1 / *nrm
__global__ void scale_kernel(double* X, long long total, const double* nrm) {
  const double inv = 1.0 / *nrm;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x)
    X[e] *= inv;
}

// out[i] = alpha sum_k M(i, k) x[k] + beta c[i], M(i, k) at M[i * si + k * sk]:
// one wave per output.
__global__ __launch_bounds__(64) void matvec_kernel(int rows, int k, const double* M, long long si,
                                                    long long sk, const double* x, double alpha,
                                                    double beta, const double* c, double* out) {
  const int i = blockIdx.x;
  double s = 0.0;
  for (int kk = threadIdx.x; kk < k; kk += 64) s += M[i * si + kk * sk] * x[kk];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) out[i] = alpha * s + (beta != 0.0 ? beta * c[i] : 0.0);
}

__global__ void info_kernel(const NsState* st, hf_recolor_info* info) {
  const int i = threadIdx.x;
  if (i < 3) {
    info->iterations[i] = st[i].iters;
    info->converged[i] = st[i].done;
    info->residual[i] = st[i].res;
  }
}

// ---------------------------------------------------------------------------
// The solve for p, q <= kSmallDim in two launches: one workgroup of 8 waves per
// root iteration, then one for the rest.  Within a workgroup an iteration
// ends when it has converged, where the launches of the general path
// go on, and most of them find nothing to do.
// What bounds it: one CU's matrix cores and the latency of its loads.  us here and on
// the general path: 32 x 32 265/1033, 64 x 64 520/1134, 80 x 80 1151/1250, 96 x 16
// 765/994, 96 x 48 877/1055; 96 x 96 1449/1320, 100 x 37 with 10 steps 1064/1106, with 13
// 1358/1227, 104 x 104 1924/1413, 128 x 16 1398/1048, 128 x 128 2779/1443: past 96 the
// products outgrow one CU.
// ---------------------------------------------------------------------------
constexpr int kSmallDim = 96;
constexpr int kSmallThreads = 512;

struct SmallProduct {
  int m, n, k;
  const double* A;
  int lda;
  bool ak;
  const double* B;
  int ldb;
  bool bk;
  const double* C;
  int ldc;
  double* D;
  int ldd;
  double alpha, beta;
  bool sym;  // upper blocks only, mirrored
};

// One 32 x 32 block of a product by one wave, operands straight from global
// memory (L1 and L2: a workgroup's matrices are at most 128 KB each), 16 inputs
// loading while 16 are multiplied.  Returns this lane's share of |I - D|_F^2.
__device__ inline double small_block(const SmallProduct& g, int m0, int n0) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int sa = g.ak ? g.lda : 1, sb = g.bk ? g.ldb : 1;
  int oa[2], ob[2];  // element offsets of this lane's row / column at input lk
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    // rows and columns past the edge repeat the last one and are not stored
    const int i = min(m0 + 16 * x + li, g.m - 1), j = min(n0 + 16 * x + li, g.n - 1);
    oa[x] = (g.ak ? i : i * g.lda) + lk * sa;
    ob[x] = (g.bk ? j : j * g.ldb) + lk * sb;
  }
  double4_t acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = double4_t{0.0, 0.0, 0.0, 0.0};
  double a[2][2][4], b[2][2][4];
  const int whole = g.k / 16, steps = (g.k + 15) / 16;
  auto load = [&](int buf, int t) {
    if (t < whole) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          a[buf][x][u] = g.A[oa[x] + (16 * t + 4 * u) * sa];
          b[buf][x][u] = g.B[ob[x] + (16 * t + 4 * u) * sb];
        }
    } else if (t < steps) {  // inputs past the end count as zero
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 16 * t + 4 * u, over = max(k + lk - (g.k - 1), 0);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const double v = g.A[oa[x] + (k - over) * sa];
          a[buf][x][u] = over ? 0.0 : v;
          b[buf][x][u] = g.B[ob[x] + (k - over) * sb];
        }
      }
    }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[buf][x][u], b[buf][y][u], acc[x][y], 0, 0, 0);
  };
  load(0, 0);
  for (int t = 0; t < steps; t += 2) {
    load(1, t + 1);
    multiply(0);
    if (t + 1 < steps) {
      load(0, t + 2);
      multiply(1);
    }
  }
  double res = 0.0;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = m0 + 16 * x + lk + 4 * v, j = n0 + 16 * y + li;
        if (i >= g.m || j >= g.n || (g.sym && i > j)) continue;
        double val = g.alpha * acc[x][y][v];
        if (g.C) val += g.beta * g.C[i * g.ldc + j];
        g.D[i * g.ldd + j] = val;
        if (g.sym && i != j) g.D[j * g.ldd + i] = val;
        res += i == j ? (val - 1.0) * (val - 1.0) : (g.sym ? 2.0 : 1.0) * val * val;
      }
  return res;
}

__device__ inline int small_blocks(const SmallProduct& g) {
  const int nm = (g.m + 31) / 32, nn = (g.n + 31) / 32;
  return g.sym ? nn * (nn + 1) / 2 : nm * nn;
}

// Blocks wave, wave + 8, ... of the products g[0..n) taken together.
template <int N>
__device__ inline double small_products(const SmallProduct (&g)[N]) {
  double res = 0.0;
  int first = 0;
#pragma unroll
  for (int z = 0; z < N; ++z) {
    const int nn = (g[z].n + 31) / 32, nb = small_blocks(g[z]);
    for (int t = (int)(threadIdx.x >> 6); t < first + nb; t += kSmallThreads / 64) {
      if (t < first) continue;
      int rem = t - first, bm = 0;
      while (rem >= (g[z].sym ? nn - bm : nn)) {
        rem -= g[z].sym ? nn - bm : nn;
        ++bm;
      }
      const int bn = (g[z].sym ? bm : 0) + rem;
      res += small_block(g[z], 32 * bm, 32 * bn);
    }
    first += nb;
  }
  __syncthreads();  // the results are there for the whole workgroup
  return res;
}

__device__ inline SmallProduct small_product(int m, int n, int k, const double* A, int lda, bool ak,
                                             const double* B, int ldb, bool bk, double* D, int ldd) {
  return SmallProduct{m, n, k, A, lda, ak, B, ldb, bk, nullptr, 0, D, ldd, 1.0, 0.0, false};
}

// A root iteration (blockIdx.x) from start to end, as ns_roots runs it.
__global__ __launch_bounds__(kSmallThreads) void small_roots_kernel(const NsPair pr, double ridge,
                                                                   double* Y1z, double* Z0z,
                                                                   double* Pz, double* Y1y,
                                                                   double* Z0y, double* Py, int most) {
  __shared__ double red[kSmallThreads / 64];
  __shared__ NsState st;
  __shared__ double bc;
  const NsProblem& q = pr.q[blockIdx.x];
  double* Y[2] = {q.Y, blockIdx.x ? Y1y : Y1z};
  double* Z[2] = {blockIdx.x ? Z0y : Z0z, q.Z1};
  double* P = blockIdx.x ? Py : Pz;
  const int tid = threadIdx.x, d = q.rows;
  auto total = [&](double v) {  // block sum, known to every thread
    const double s = block_sum(v, red);
    if (tid == 0) bc = s;
    __syncthreads();
    const double t = bc;
    __syncthreads();
    return t;
  };
  double s = 0.0;
  for (int i = tid; i < d; i += kSmallThreads) s += q.M[i * q.ld + i];
  const double trace = total(s), lam = ridge * trace / d;
  s = 0.0;
  for (int e = tid; e < d * d; e += kSmallThreads) {
    const int i = e / d, j = e - i * d;
    const double v = q.M[i * q.ld + j] + (i == j ? lam : 0.0);
    s += v * v;
  }
  const double c = sqrt(total(s)), inv = 1.0 / c;
  s = 0.0;
  for (int e = tid; e < d * d; e += kSmallThreads) {
    const int i = e / d, j = e - i * d;
    const double v = (q.M[i * q.ld + j] + (i == j ? lam : 0.0)) * inv;
    Y[0][e] = v;
    const double o = v - (i == j ? 1.0 : 0.0);
    s += o * o;
  }
  double res = sqrt(total(s));
  if (tid == 0) {
    *q.lam = lam;
    *q.norm = c;
    st = ns_initial(1.0);
    st.low = ns_root_bound(d, trace + ridge * trace, c, lam);
    ns_update(&st, res);
  }
  __syncthreads();
  for (int e = tid; e < d * d; e += kSmallThreads) {
    const int i = e / d, j = e - i * d;
    Z[1][e] = st.alpha * Y[0][e] + (i == j ? st.beta : 0.0);
  }
  {
    SmallProduct g[1] = {small_product(d, d, d, Y[0], d, false, Y[0], d, true, Y[1], d)};
    g[0].alpha = st.alpha;
    g[0].beta = st.beta;
    g[0].C = Y[0];
    g[0].ldc = d;
    small_products(g);
  }
  for (int it = 1; it < most; ++it) {
    const int a = it & 1, b = a ^ 1;
    {
      const SmallProduct g[1] = {small_product(d, d, d, Z[a], d, false, Y[a], d, true, P, d)};
      res = sqrt(total(small_products(g)));
    }
    if (tid == 0) ns_update(&st, res);
    __syncthreads();
    if (st.done) break;
    SmallProduct g[2] = {small_product(d, d, d, Y[a], d, false, P, d, true, Y[b], d),
                         small_product(d, d, d, P, d, false, Z[a], d, true, Z[b], d)};
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      g[z].alpha = st.alpha;
      g[z].beta = st.beta;
      g[z].C = z ? Z[a] : Y[a];
      g[z].ldc = d;
    }
    small_products(g);
  }
  if (tid == 0) *q.st = st;
}

// Everything after the roots: the whitened cross-covariance, its polar factor
// (as ns_polar), A and b, and the record of the three iterations.
struct SmallRest {
  int p, q, most;
  const double* mu;
  const double* cov;
  const double* Yy[2];
  const double* Zz[2];
  const double* Zy[2];
  const double* cz;
  const double* cy;
  double* X[2];
  double* P;
  double* T1;
  double* T2;
  double* A;
  double* b;
  NsState* st;
  hf_recolor_info* info;
};
__global__ __launch_bounds__(kSmallThreads) void small_rest_kernel(const SmallRest w) {
  __shared__ double red[kSmallThreads / 64];
  __shared__ NsState st;
  __shared__ double bc;
  const int tid = threadIdx.x, p = w.p, q = w.q, pq = p + q;
  auto total = [&](double v) {
    const double s = block_sum(v, red);
    if (tid == 0) bc = s;
    __syncthreads();
    const double t = bc;
    __syncthreads();
    return t;
  };
  const double* Zz = w.Zz[w.st[0].iters & 1];
  const double* Zy = w.Zy[w.st[1].iters & 1];
  const double* Yy = w.Yy[w.st[1].iters & 1];
  {
    const SmallProduct g[1] = {small_product(p, q, p, Zz, p, false, w.cov + p, pq, true, w.T1, q)};
    small_products(g);
  }
  {
    const SmallProduct g[1] = {small_product(p, q, q, w.T1, q, false, Zy, q, true, w.X[0], q)};
    small_products(g);
  }
  double s = 0.0;
  for (int e = tid; e < p * q; e += kSmallThreads) s += w.X[0][e] * w.X[0][e];
  const double inv = 1.0 / sqrt(total(s));
  for (int e = tid; e < p * q; e += kSmallThreads) w.X[0][e] *= inv;
  if (tid == 0) {
    st = ns_initial(kNsFloorPolar);
    st.low = kNsFloorPolar;
  }
  __syncthreads();
  const bool tall = p >= q;
  const int e = tall ? q : p;
  for (int it = 0; it < w.most; ++it) {
    const int a = it & 1, b = a ^ 1;
    double res;
    {
      SmallProduct g[1] = {small_product(e, e, tall ? p : q, w.X[a], q, tall, w.X[a], q, tall, w.P, e)};
      g[0].sym = true;
      res = sqrt(total(small_products(g)));
    }
    if (tid == 0) ns_update(&st, res);
    __syncthreads();
    if (st.done) break;
    SmallProduct g[1] = {tall ? small_product(p, q, q, w.X[a], q, false, w.P, q, true, w.X[b], q)
                              : small_product(p, q, p, w.P, p, true, w.X[a], q, true, w.X[b], q)};
    g[0].alpha = st.alpha;
    g[0].beta = st.beta;
    g[0].C = w.X[a];
    g[0].ldc = q;
    small_products(g);
  }
  const double* X = w.X[st.iters & 1];
  {
    const SmallProduct g[1] = {small_product(q, p, p, X, q, true, Zz, p, true, w.T2, p)};
    small_products(g);
  }
  {
    SmallProduct g[1] = {small_product(q, p, q, Yy, q, false, w.T2, p, true, w.A, p)};
    g[0].alpha = sqrt(*w.cy / *w.cz);
    small_products(g);
  }
  for (int i = tid >> 6; i < q; i += kSmallThreads / 64) {  // b = mu_Y - A mu_Z, a wave per row
    double v = 0.0;
    for (int k = tid & 63; k < p; k += 64) v += w.A[(long long)i * p + k] * w.mu[k];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((tid & 63) == 0) w.b[i] = w.mu[p + i] - v;
  }
  if (w.info && tid < 3) {
    const NsState z = tid < 2 ? w.st[tid] : st;
    w.info->iterations[tid] = z.iters;
    w.info->converged[tid] = z.done;
    w.info->residual[tid] = z.res;
  }
}

// ---------------------------------------------------------------------------
// Column statistics of the samples: weighted sums per column and the weighted
// sum of squares of the X columns, per chunk of rows.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void colstats_kernel(long long n, int p, int q, const T* X,
                                                        long long ldx, const T* Y, long long ldy,
                                                        const float* w, long long rows_per_chunk,
                                                        double* part_sum, double* part_sq,
                                                        double* part_w) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int chunk = blockIdx.y;
  const long long r0 = (long long)chunk * rows_per_chunk;
  const long long r1 = r0 + rows_per_chunk < n ? r0 + rows_per_chunk : n;
  const int pq = p + q;
  if (c < pq) {
    double s = 0.0, ss = 0.0;
#pragma unroll 8
    for (long long r = r0; r < r1; ++r) {
      const double wv = w ? (double)w[r] : 1.0;
      const double v = c < p ? load_elem(X, r * ldx + c) : load_elem(Y, r * ldy + (c - p));
      s += wv * v;
      ss += wv * v * v;
    }
    part_sum[(long long)chunk * pq + c] = s;
    if (c < p) part_sq[(long long)chunk * p + c] = ss;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double sw = 0.0;
    for (long long r = r0; r < r1; ++r) sw += w ? (double)w[r] : 1.0;
    part_w[chunk] = sw;
  }
}

// Per column: total weighted sum and (X columns) sum of squares over the chunks.
// 64 columns x 16 groups of chunks per workgroup, the groups added in order
// (one thread per column, down all 512 chunks of 4096 columns: 217 us).
constexpr int kCsGroups = 16;
__global__ __launch_bounds__(64 * kCsGroups) void colstats_reduce_kernel(
    int p, int q, int n_chunks, const double* part_sum, const double* part_sq, double* col_sum,
    double* col_sq) {
  __shared__ double ts[kCsGroups][64], tss[kCsGroups][64];
  const int x = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + x;
  const int pq = p + q;
  double s = 0.0, ss = 0.0;
  if (c < pq) {
#pragma unroll 4
    for (int k = g; k < n_chunks; k += kCsGroups) s += part_sum[(long long)k * pq + c];
    if (c < p) {
#pragma unroll 4
      for (int k = g; k < n_chunks; k += kCsGroups) ss += part_sq[(long long)k * p + c];
    }
  }
  ts[g][x] = s;
  tss[g][x] = ss;
  __syncthreads();
  if (g != 0 || c >= pq) return;
  for (int k = 1; k < kCsGroups; ++k) {
    s += ts[k][x];
    ss += tss[k][x];
  }
  col_sum[c] = s;
  if (c < p) col_sq[c] = ss;
}

// W, r (Eq. 3), raw means (centring shifts), column scales (1/r for X, 1 for
// Y), the means of [x/r | y], and 1/W.
__global__ __launch_bounds__(kRedThreads) void moments_scalars_kernel(
    int p, int q, int n_chunks, const double* part_w, const double* col_sum, const double* col_sq,
    double* shift, double* scale, double* mu, double* r_out, double* inv_w) {
  __shared__ double red[kRedThreads / 64];
  __shared__ double sh_w, sh_r;
  const double W = sum_partials(part_w, n_chunks, red);
  double s = 0.0;
  for (int c = threadIdx.x; c < p; c += blockDim.x) s += col_sq[c];
  s = block_sum(s, red);
  if (threadIdx.x == 0) {
    sh_w = W;
    sh_r = sqrt(s / ((double)p * W));
    *r_out = sh_r;
    *inv_w = 1.0 / W;
  }
  __syncthreads();
  const double Wv = sh_w, rv = sh_r;
  for (int c = threadIdx.x; c < p + q; c += blockDim.x) {
    const double m = col_sum[c] / Wv;
    shift[c] = m;
    scale[c] = c < p ? 1.0 / rv : 1.0;
    mu[c] = c < p ? m / rv : m;
  }
}

int grid_for(long long total, int threads = 256, int cap = 4096) {
  long long b = (total + threads - 1) / threads;
  if (b < 1) b = 1;
  return (int)(b < cap ? b : cap);
}

// Tiles of height bm of a product; of a symmetric one, those that reach its
// upper triangle.
long long tiles_of(const GemmJob& j, int bm) {
  const long long tm = (j.m + bm - 1) / bm, tn = (j.n + kBN - 1) / kBN;
  const bool sym = j.kind == kGramSym;
  return sym ? tm * tn - (bm / kBN) * (tm * (tm - 1) / 2) : tm * tn;
}

// Products that run in one launch.
struct Batch {
  GemmBatch g{};
  GemmJob& add(int m, int n, long long k, const double* A, long long lda, bool ak, const double* B,
               long long ldb, bool bk, double* D, long long ldd, int kind = kPlain) {
    GemmJob& j = g.job[g.n_jobs];
    j = GemmJob{};
    j.m = m;
    j.n = n;
    j.k = k;
    j.A = j.A1 = A;
    j.lda = lda;
    j.B = j.B1 = B;
    j.ldb = ldb;
    j.D = D;
    j.ldd = ldd;
    j.alpha = 1.0;
    j.kind = kind;
    j.a_kmajor = ak;
    j.b_kmajor = bk;
    // 16-byte loads need aligned bases and even leading dimensions; edge tiles
    // read one element at a time
    j.fast = (uintptr_t)A % 16 == 0 && lda % 2 == 0 && (uintptr_t)B % 16 == 0 && ldb % 2 == 0 &&
             k % kBK == 0;
    ++g.n_jobs;
    return j;
  }
  // Numbers the tiles of height bm.
  long long number(int bm) {
    g.bm = bm;
    for (int i = 0; i < g.n_jobs; ++i) g.first[i + 1] = g.first[i] + tiles_of(g.job[i], bm);
    return g.first[g.n_jobs];
  }
  // Chooses the tile and numbers the tiles.
  long long cut() {
    const long long tall = number(128);
    return tall >= kGemmSmallTiles ? tall : number(64);
  }
  // A short product's tiles are mostly staging and stores: small tiles with one slice
  // in flight, of which four instead of three workgroups fit a CU, also where three
  // a CU would leave a nearly empty last wave.  us that way and otherwise, k = 16, 64,
  // 256: 50000 x 64 12/15, 19/22, 43/45; 2600 x 2600 18/22, 29/35, 72/84; 4096 x 4096
  // 32/33, 55/58.  With fewer tiles, or many waves, k = 256 is better off with the
  // others: 640 x 640 18.2/17.4, 4096 x 4096 157/152.  A workgroup per tile, so that
  // one's stores run beside the next one's loads: 8192 x 4096, k = 64 106, resident
  // workgroups 111.
  hipError_t launch(hipStream_t s) {
    const long long k = g.n_jobs == 1 ? g.job[0].k : INT64_MAX;
    const long long small = number(64);
    if (k <= 64 || (k <= 256 && small > kGemmResident && small < 2048)) {
      if (small <= 0) return hipSuccess;
      const dim3 grid((unsigned)std::min<long long>(small, 1 << 20));
      hipLaunchKernelGGL((gemm_f64_kernel<64, 1>), grid, dim3(kGemmThreads), 0, s, g);
      return hipGetLastError();
    }
    const long long tiles = cut();
    if (tiles <= 0) return hipSuccess;
    const dim3 grid((unsigned)std::min<long long>(tiles, kGemmResident));
    if (g.bm == 128) hipLaunchKernelGGL((gemm_f64_kernel<128, 1>), grid, dim3(kGemmThreads), 0, s, g);
    else hipLaunchKernelGGL((gemm_f64_kernel<64, 2>), grid, dim3(kGemmThreads), 0, s, g);
    return hipGetLastError();
  }
};

// The plan of an iteration: products described in the workspace.
struct Plan {
  GemmBatch* dev;
  int n = 0;
  PlanPart part;
  long long tiles[8];
  int bm[8];
  hipError_t store(int count, hipStream_t s) const {
    hipLaunchKernelGGL(store_plan_kernel, dim3(1), dim3(256), 0, s, part, dev + n - count, count);
    return hipGetLastError();
  }
  // Adds a description; the last of kPlanPart of them, or `flush`, stores them.
  hipError_t add(Batch& b, bool flush, hipStream_t s) {
    const int at = n % kPlanPart;
    tiles[n] = b.cut();
    bm[n++] = b.g.bm;
    part.g[at] = b.g;
    return at + 1 == kPlanPart || flush ? store(at + 1, s) : hipSuccess;
  }
  hipError_t launch(int i, hipStream_t s) const {
    const dim3 grid((unsigned)(tiles[i] < kGemmResident ? tiles[i] : kGemmResident));
    const GemmBatch* d = dev + i;
    if (bm[i] == 128)
      hipLaunchKernelGGL(gemm_f64_planned_kernel<128>, grid, dim3(kGemmThreads), 0, s, d);
    else
      hipLaunchKernelGGL(gemm_f64_planned_kernel<64>, grid, dim3(kGemmThreads), 0, s, d);
    return hipGetLastError();
  }
};
constexpr int kPlanMax = 5;  // descriptions of an iteration

// Plain fp64 product D = alpha * op(A) op(B) + beta * C + gamma * I with
// op(A) m x k (ak: stored k-major, A[kk * lda + i]) and op(B) k x n (bk: stored
// k-major, B[kk * ldb + j]).
hipError_t gemm(int m, int n, long long k, const double* A, long long lda, bool ak,
                const double* B, long long ldb, bool bk, double* D, long long ldd,
                hipStream_t s, double alpha = 1.0, double beta = 0.0, const double* C = nullptr,
                long long ldc = 0, double gamma = 0.0) {
  Batch b;
  GemmJob& j = b.add(m, n, k, A, lda, ak, B, ldb, bk, D, ldd);
  j.alpha = alpha;
  j.beta = beta;
  j.C = C;
  j.ldc = ldc;
  j.gamma = gamma;
  return b.launch(s);
}

hipError_t matvec(int rows, int k, const double* M, long long si, long long sk, const double* x,
                  double alpha, double beta, const double* c, double* out, hipStream_t s) {
  hipLaunchKernelGGL(matvec_kernel, dim3((unsigned)rows), dim3(64), 0, s, rows, k, M, si, sk, x,
                     alpha, beta, c, out);
  return hipGetLastError();
}

#define HF_CHECK(x)                   \
  do {                                \
    hipError_t e_ = (x);              \
    if (e_ != hipSuccess) return e_;  \
  } while (0)

// Scratch carving from the workspace (256-byte aligned pieces).
struct Carve {
  char* p;
  template <typename U>
  U* take(size_t count) {
    U* r = reinterpret_cast<U*>(p);
    p += (count * sizeof(U) + 255) / 256 * 256;
    return r;
  }
};

// Steps after which an iteration is given up.  With the scaling, whatever 64 and
// 128 plain steps bring to convergence (singular values down to 1e-10 and 7e-22
// of the norm, in exact arithmetic) takes at most 60 and 80.  In fp64 the roots
// converge up to condition numbers of about 1e14, as with plain steps: past that
// rounding keeps |I - Z Y|_F from falling.
constexpr int kSqrtMaxIter = 60;
constexpr int kPolarMaxIter = 88;

// Shares of a residual: one per tile of a d x d product, or one per workgroup of
// an elementwise kernel.
size_t ns_partials(int d) {
  const size_t nt = ((size_t)d + kBN - 1) / kBN, tiles = nt * nt;
  return tiles > (size_t)kMaxRedBlocks ? tiles : (size_t)kMaxRedBlocks;
}

// A root iteration's buffers: Y and Z ping-pong, P the product Z Y.
struct RootBuffers {
  double* Y[2];
  double* Z[2];
  double* P;
};

// The two coupled Newton-Schulz iterations (S = M + lam I, d x d, SPD), side by
// side in the same launches:
//   Y0 = S / c, Z0 = I, P = Z Y, Y <- beta Y + alpha Y P, Z <- beta Z + alpha P Z,
// Y -> (S/c)^{1/2}, Z -> (S/c)^{-1/2}, with c = |S|_F.  Results in buffer
// st->iters & 1.  Y, Z and P are symmetric in exact arithmetic, and none is taken to
// be so: every product is whole, and reads its factors in this order and not
// transposed.  Errors of Y and Z then go over into errors that do not grow; the
// rounding of P, dZ Y + Z dY, is not symmetric, and a mirrored triangle of Y or Z, or
// one read as its transpose, feeds that back.  |A S_Z A^T - S_Y| / |S_Y| at condition
// numbers 1e4, 1e8, 1e12 of S_Y (150 x 140): 5e-15, 2e-13, 2e-11 as it is; 2e-14, 5e-11,
// 5e-7 with Y and Z mirrored.  In fp64 on the host, Z read transposed doubles the error,
// Y read transposed diverges at 1e12, and with Y alone mirrored the error is that of
// whole products but one eigenvalue of 1e-14 no longer converges.
hipError_t ns_roots(const NsPair& pr, const RootBuffers (&rb)[2], double ridge, NsState* polar,
                    GemmBatch* plan_ws, hipStream_t s) {
  Plan plan{plan_ws};
  const long long most = (long long)std::max(pr.q[0].rows, pr.q[1].rows);
  const dim3 red((unsigned)grid_for(most * most, kRedThreads, kMaxRedBlocks), 2);
  hipLaunchKernelGGL(ns_start_kernel, dim3(2), dim3(kRedThreads), 0, s, pr, ridge, polar);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(ns_norm_kernel, red, dim3(kRedThreads), 0, s, pr);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(ns_root_init_kernel, red, dim3(kRedThreads), 0, s, pr);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(ns_root_first_kernel, red, dim3(kRedThreads), 0, s, pr);
  HF_CHECK(hipGetLastError());
  // plan 0: step 0; 1, 2: P of odd and even steps; 3, 4: odd and even steps
  for (int i = 0; i < 5; ++i) {
    const bool first = i == 0, gram = i == 1 || i == 2;
    const int a = first ? 0 : (i & 1), b = a ^ 1;
    Batch t;
    for (int z = 0; z < 2; ++z) {
      const int d = pr.q[z].rows;
      if (gram) {
        GemmJob& j = t.add(d, d, d, rb[z].Z[a], d, false, rb[z].Y[a], d, true, rb[z].P, d, kGram);
        j.st = pr.q[z].st;
        j.partial = pr.q[z].partial;
        continue;
      }
      const double* P = first ? rb[z].Y[0] : rb[z].P;
      GemmJob& y = t.add(d, d, d, rb[z].Y[a], d, false, P, d, true, rb[z].Y[b], d, kStep);
      y.C = rb[z].Y[a];
      y.ldc = d;
      y.st = pr.q[z].st;
      if (first) continue;  // Z1 is there
      GemmJob& w = t.add(d, d, d, P, d, false, rb[z].Z[a], d, true, rb[z].Z[b], d, kStep);
      w.C = rb[z].Z[a];
      w.ldc = d;
      w.st = pr.q[z].st;
    }
    HF_CHECK(plan.add(t, i == 4, s));
  }
  HF_CHECK(plan.launch(0, s));
  for (int it = 1; it < kSqrtMaxIter; ++it) {
    HF_CHECK(plan.launch(2 - (it & 1), s));
    HF_CHECK(plan.launch(4 - (it & 1), s));
  }
  return hipSuccess;
}

// Newton-Schulz iteration for the polar factor of the p x q matrix in X[0]:
// X0 = M / |M|_F, then X <- beta X + alpha X (X^T X) (p >= q) or
// X <- beta X + alpha (X X^T) X (p < q).  Result in X[st->iters & 1].
hipError_t ns_polar(int p, int q, double* X[2], double* P, double* partial, double* nrm,
                    NsState* st, GemmBatch* plan_ws, hipStream_t s) {
  Plan plan{plan_ws};
  const long long pq = (long long)p * q;
  NsPair pr{};
  pr.q[0].M = X[0];
  pr.q[0].ld = q;
  pr.q[0].rows = p;
  pr.q[0].cols = q;
  pr.q[0].norm = nrm;
  pr.q[0].st = st;
  pr.q[0].partial = partial;
  hipLaunchKernelGGL(ns_norm_kernel, dim3((unsigned)grid_for(pq, kRedThreads, kMaxRedBlocks), 1),
                     dim3(kRedThreads), 0, s, pr);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(scale_kernel, dim3(grid_for(pq)), dim3(256), 0, s, X[0], pq,
                     (const double*)nrm);
  HF_CHECK(hipGetLastError());
  // plan 0, 1: P of even and odd steps; 2, 3: even and odd steps
  const bool tall = p >= q;
  const int e = tall ? q : p;
  for (int i = 0; i < 4; ++i) {
    const int a = i & 1, b = a ^ 1;
    Batch t;
    if (i < 2) {
      GemmJob& g = t.add(e, e, tall ? p : q, X[a], q, tall, X[a], q, tall, P, e, kGramSym);
      g.st = st;
      g.partial = partial;
    } else {
      GemmJob& j = tall ? t.add(p, q, q, X[a], q, false, P, q, true, X[b], q, kStep)
                        : t.add(p, q, p, P, p, true, X[a], q, true, X[b], q, kStep);
      j.C = X[a];
      j.ldc = q;
      j.st = st;
    }
    HF_CHECK(plan.add(t, i == 3, s));
  }
  for (int it = 0; it < kPolarMaxIter; ++it) {
    HF_CHECK(plan.launch(it & 1, s));
    HF_CHECK(plan.launch(2 + (it & 1), s));
  }
  return hipSuccess;
}

// Scalar slots of the solve's workspace.
enum { kScLamZ = 0, kScLamY = 1, kScCZ = 2, kScCY = 3, kScNormM = 4, kScTrZ = 5, kScTrY = 6, kScCount = 16 };

}  // namespace

// Row chunks of the column statistics: 32 rows each, so that 3,000 samples make
// 94 of them (with 256 rows, 12 chains of loads took 57 us), at most 512 chunks.
int moments_chunks(long long n) {
  long long c = (n + 31) / 32;
  if (c > 512) c = 512;
  if (c < 1) c = 1;
  return (int)c;
}

namespace {

struct CovPlan {
  int nt, n_tiles, splits;
  long long rows_per_split;
};

// Rows are split so that the (split, tile) items fill the resident workgroups
// with the least idle tail, each split keeping at least 32 steps of rows -- or
// 4 where even so fewer items than resident workgroups would come out (3,000 x
// 137 samples: 47 splits of 4 steps instead of 5 of 38).
CovPlan cov_plan(long long n, int m) {
  CovPlan c;
  c.nt = (m + kCT - 1) / kCT;
  c.n_tiles = c.nt * (c.nt + 1) / 2;
  const long long steps = (n + kCK - 1) / kCK;
  long long max_splits = std::min<long long>(std::max<long long>(steps / 32, 1), 64);
  if (max_splits * c.n_tiles < kCovResident) {
    const long long fill = (kCovResident + c.n_tiles - 1) / c.n_tiles;
    max_splits = std::max(max_splits, std::min(std::max<long long>(steps / 4, 1), fill));
  }
  int best = 1;
  double best_waste = 1e30;
  for (int s = 1; s <= max_splits; ++s) {
    const long long items = (long long)s * c.n_tiles;
    if (items < kCovResident && s < max_splits) continue;
    const long long rounds = (items + kCovResident - 1) / kCovResident;
    const double waste = (double)(rounds * kCovResident) / (double)items - 1.0;
    if (waste < best_waste - 0.01) {
      best_waste = waste;
      best = s;
    }
  }
  c.splits = best;
  c.rows_per_split = (steps + best - 1) / best * kCK;
  return c;
}

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

size_t recolor_moments_workspace_bytes(long long n, int p, int q) {
  const size_t n_chunks = (size_t)moments_chunks(n);
  const size_t pq = (size_t)p + q;
  const CovPlan c = cov_plan(n, p + q);
  return align256(n_chunks * pq * 8) + align256(n_chunks * (size_t)p * 8) +
         align256(n_chunks * 8) + align256(pq * 8) + align256((size_t)p * 8) +
         2 * align256(pq * 8) + align256(8) +
         align256((size_t)c.splits * c.n_tiles * kCT * kCT * 8);
}

hipError_t launch_recolor_stats(int dtype, long long n, int p, int q, const void* X,
                                long long ldx, const void* Y, long long ldy, const float* w,
                                double* r, double* mu, void* workspace, hipStream_t s) {
  const int n_chunks = moments_chunks(n);
  const long long rows_per_chunk = (n + n_chunks - 1) / n_chunks;
  const int pq = p + q;
  Carve cv{static_cast<char*>(workspace)};
  double* part_sum = cv.take<double>((size_t)n_chunks * pq);
  double* part_sq = cv.take<double>((size_t)n_chunks * p);
  double* part_w = cv.take<double>(n_chunks);
  double* col_sum = cv.take<double>(pq);
  double* col_sq = cv.take<double>(p);
  double* shift = cv.take<double>(pq);
  double* scale = cv.take<double>(pq);
  double* inv_w = cv.take<double>(1);

  dim3 g1((pq + 255) / 256, n_chunks);
  if (dtype == HF_BF16)
    hipLaunchKernelGGL(colstats_kernel<uint16_t>, g1, dim3(256), 0, s, n, p, q,
                       static_cast<const uint16_t*>(X), ldx, static_cast<const uint16_t*>(Y), ldy,
                       w, rows_per_chunk, part_sum, part_sq, part_w);
  else
    hipLaunchKernelGGL(colstats_kernel<float>, g1, dim3(256), 0, s, n, p, q,
                       static_cast<const float*>(X), ldx, static_cast<const float*>(Y), ldy, w,
                       rows_per_chunk, part_sum, part_sq, part_w);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(colstats_reduce_kernel, dim3((pq + 63) / 64), dim3(64 * kCsGroups), 0, s, p, q,
                     n_chunks, (const double*)part_sum, (const double*)part_sq, col_sum, col_sq);
  HF_CHECK(hipGetLastError());
  hipLaunchKernelGGL(moments_scalars_kernel, dim3(1), dim3(kRedThreads), 0, s, p, q, n_chunks,
                     (const double*)part_w, (const double*)col_sum, (const double*)col_sq, shift,
                     scale, mu, r, inv_w);
  HF_CHECK(hipGetLastError());
  return hipSuccess;
}

hipError_t launch_recolor_cov(int dtype, long long n, int p, int q, const void* X, long long ldx,
                              const void* Y, long long ldy, const float* w, void* workspace,
                              hipStream_t s) {
  const int n_chunks = moments_chunks(n);
  const int pq = p + q;
  Carve cv{static_cast<char*>(workspace)};
  (void)cv.take<double>((size_t)n_chunks * pq);
  (void)cv.take<double>((size_t)n_chunks * p);
  (void)cv.take<double>(n_chunks);
  (void)cv.take<double>(pq);
  (void)cv.take<double>(p);
  double* shift = cv.take<double>(pq);
  (void)cv.take<double>(pq);  // column scales (applied by the reduction)
  (void)cv.take<double>(1);   // 1 / W
  const CovPlan plan = cov_plan(n, pq);
  double* partial = cv.take<double>((size_t)plan.splits * plan.n_tiles * kCT * kCT);
  CovArgs g{};
  g.n = n;
  g.p = p;
  g.m = pq;
  g.X = X;
  g.ldx = ldx;
  g.Y = Y;
  g.ldy = ldy;
  g.w = w;
  g.shift = shift;
  g.nt = plan.nt;
  g.n_tiles = plan.n_tiles;
  g.rows_per_split = plan.rows_per_split;
  g.partial = partial;
  // groups of 4 columns: whole in X or Y, each 4 elements aligned
  const uintptr_t al = dtype == HF_BF16 ? 8 : 16;
  const bool vec = p % 4 == 0 && q % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 &&
                   (uintptr_t)X % al == 0 && (uintptr_t)Y % al == 0;
  const dim3 grid((unsigned)((long long)plan.splits * plan.n_tiles));
  if (dtype == HF_BF16) {
    if (vec) hipLaunchKernelGGL((cov_kernel<uint16_t, true>), grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL((cov_kernel<uint16_t, false>), grid, dim3(256), 0, s, g);
  } else {
    if (vec) hipLaunchKernelGGL((cov_kernel<float, true>), grid, dim3(256), 0, s, g);
    else hipLaunchKernelGGL((cov_kernel<float, false>), grid, dim3(256), 0, s, g);
  }
  return hipGetLastError();
}

hipError_t launch_recolor_cov_reduce(long long n, int p, int q, double* cov, void* workspace,
                                     hipStream_t s) {
  const int n_chunks = moments_chunks(n);
  const int pq = p + q;
  Carve cv{static_cast<char*>(workspace)};
  (void)cv.take<double>((size_t)n_chunks * pq);
  (void)cv.take<double>((size_t)n_chunks * p);
  (void)cv.take<double>(n_chunks);
  (void)cv.take<double>(pq);
  (void)cv.take<double>(p);
  (void)cv.take<double>(pq);
  double* scale = cv.take<double>(pq);
  double* inv_w = cv.take<double>(1);
  const CovPlan plan = cov_plan(n, pq);
  double* partial = cv.take<double>((size_t)plan.splits * plan.n_tiles * kCT * kCT);
  hipLaunchKernelGGL(cov_reduce_kernel,
                     dim3((unsigned)(plan.n_tiles * (kCT / kRB) * (kCT / kRB))), dim3(256), 0, s, (const double*)partial, plan.splits, plan.n_tiles, plan.nt, pq,
                     (const double*)scale, (const double*)inv_w, cov);
  return hipGetLastError();
}

size_t recolor_solve_workspace_bytes(int p, int q) {
  auto a = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t pp = (size_t)p * p, qq = (size_t)q * q, pq = (size_t)p * q;
  const size_t e = p < q ? p : q;
  return a(kScCount * 8) + a(3 * sizeof(NsState)) + 2 * a(kPlanMax * sizeof(GemmBatch)) +
         a(ns_partials(p) * 8) + a(ns_partials(q) * 8) +
         5 * a(pp * 8) + 5 * a(qq * 8) + 2 * a(pq * 8) + a(e * e * 8) + a(pq * 8) + a(pq * 8);
}

hipError_t launch_recolor_solve(int p, int q, const double* mu, const double* cov, double lam,
                                double* A, double* b, hf_recolor_info* info, void* workspace,
                                hipStream_t s) {
  const int pq = p + q;
  Carve cv{static_cast<char*>(workspace)};
  double* sc = cv.take<double>(kScCount);
  NsState* st = cv.take<NsState>(3);
  GemmBatch* plan_roots = cv.take<GemmBatch>(kPlanMax);
  GemmBatch* plan_polar = cv.take<GemmBatch>(kPlanMax);
  NsPair pr{};
  RootBuffers rb[2];
  for (int i = 0; i < 2; ++i) pr.q[i].partial = cv.take<double>(ns_partials(i ? q : p));
  for (int i = 0; i < 2; ++i) {
    const int d = i ? q : p;
    const size_t dd = (size_t)d * d;
    rb[i].Y[0] = cv.take<double>(dd);
    rb[i].Y[1] = cv.take<double>(dd);
    rb[i].Z[0] = cv.take<double>(dd);
    rb[i].Z[1] = cv.take<double>(dd);
    rb[i].P = cv.take<double>(dd);
    NsProblem& n = pr.q[i];
    n.M = i ? cov + (long long)p * pq + p : cov;
    n.ld = pq;
    n.rows = n.cols = d;
    n.lam = sc + (i ? kScLamY : kScLamZ);
    n.norm = sc + (i ? kScCY : kScCZ);
    n.Y = rb[i].Y[0];
    n.Z1 = rb[i].Z[1];
    n.st = st + i;
    n.trace = sc + (i ? kScTrY : kScTrZ);
  }
  double* Xp[2] = {cv.take<double>((size_t)p * q), cv.take<double>((size_t)p * q)};
  const size_t e = p < q ? p : q;
  double* Pp = cv.take<double>(e * e);
  double* Tmp1 = cv.take<double>((size_t)p * q);  // Z_z C (p x q)
  double* Tmp2 = cv.take<double>((size_t)p * q);  // R^T Z_z (q x p)

  if (p <= kSmallDim && q <= kSmallDim) {
    hipLaunchKernelGGL(small_roots_kernel, dim3(2), dim3(kSmallThreads), 0, s, pr, lam, rb[0].Y[1],
                       rb[0].Z[0], rb[0].P, rb[1].Y[1], rb[1].Z[0], rb[1].P, kSqrtMaxIter);
    HF_CHECK(hipGetLastError());
    const SmallRest w{p, q, kPolarMaxIter, mu, cov, {rb[1].Y[0], rb[1].Y[1]},
                      {rb[0].Z[0], rb[0].Z[1]}, {rb[1].Z[0], rb[1].Z[1]}, sc + kScCZ, sc + kScCY,
                      {Xp[0], Xp[1]}, Pp, Tmp1, Tmp2, A, b, st, info};
    hipLaunchKernelGGL(small_rest_kernel, dim3(1), dim3(kSmallThreads), 0, s, w);
    return hipGetLastError();
  }
  HF_CHECK(ns_roots(pr, rb, lam, st + 2, plan_roots, s));
  // M ~ Sigma_Z^{-1/2} Sigma_ZY Sigma_Y^{-1/2} (positive scale: the polar factor ignores it)
  {
    Batch t;
    GemmJob& j = t.add(p, q, p, rb[0].Z[0], p, false, cov + p, pq, true, Tmp1, q);
    j.a_sel = st;
    j.A1 = rb[0].Z[1];
    HF_CHECK(t.launch(s));
  }
  {
    Batch t;
    GemmJob& j = t.add(p, q, q, Tmp1, q, false, rb[1].Z[0], q, true, Xp[0], q);
    j.b_sel = st + 1;
    j.B1 = rb[1].Z[1];
    HF_CHECK(t.launch(s));
  }
  HF_CHECK(ns_polar(p, q, Xp, Pp, pr.q[0].partial, sc + kScNormM, st + 2, plan_polar, s));
  // A (stored q x p) = Sigma_Y^{1/2} R^T Sigma_Z^{-1/2} = sqrt(c_Y / c_Z) Y_y R^T Z_z
  {
    Batch t;
    GemmJob& j = t.add(q, p, p, Xp[0], q, true, rb[0].Z[0], p, true, Tmp2, p);
    j.a_sel = st + 2;
    j.A1 = Xp[1];
    j.b_sel = st;
    j.B1 = rb[0].Z[1];
    HF_CHECK(t.launch(s));
  }
  {
    Batch t;
    GemmJob& j = t.add(q, p, q, rb[1].Y[0], q, false, Tmp2, p, true, A, p);
    j.a_sel = st + 1;
    j.A1 = rb[1].Y[1];
    j.ratio_num = sc + kScCY;
    j.ratio_den = sc + kScCZ;
    HF_CHECK(t.launch(s));
  }
  HF_CHECK(matvec(q, p, A, p, 1, mu, -1.0, 1.0, mu + p, b, s));  // b = mu_Y - A mu_Z
  if (info) {
    hipLaunchKernelGGL(info_kernel, dim3(1), dim3(64), 0, s, (const NsState*)st, info);
    HF_CHECK(hipGetLastError());
  }
  return hipSuccess;
}

size_t fold_workspace_bytes(int p, int rank) {
  return ((size_t)rank * p * 8 + 255) / 256 * 256 + ((size_t)rank * 8 + 255) / 256 * 256;
}

hipError_t launch_fold(int p, int q, int rank, const double* A, const double* b, const double* B,
                       const double* G, double* A_out, double* b_out, void* workspace,
                       hipStream_t s) {
  Carve cv{static_cast<char*>(workspace)};
  double* T = cv.take<double>((size_t)rank * p);
  double* t = cv.take<double>(rank);
  // stored maps: A_out = (I + B G)^T A = A + G^T (B^T A); same for the bias column
  HF_CHECK(gemm(rank, p, q, B, rank, true, A, p, true, T, p, s));
  HF_CHECK(matvec(rank, q, B, 1, rank, b, 1.0, 0.0, nullptr, t, s));
  HF_CHECK(gemm(q, p, rank, G, q, true, T, p, true, A_out, p, s, 1.0, 1.0, A, p));
  HF_CHECK(matvec(q, rank, G, 1, q, t, 1.0, 1.0, b, b_out, s));
  return hipSuccess;
}

hipError_t launch_gemm_f64(int m, int n, long long k, const double* A, long long lda, int ak,
                           const double* B, long long ldb, int bk, double* D, long long ldd,
                           double alpha, double beta, const double* C, long long ldc,
                           double gamma, hipStream_t s) {
  return gemm(m, n, k, A, lda, ak != 0, B, ldb, bk != 0, D, ldd, s, alpha, beta, C, ldc, gamma);
}

}  // namespace hf
