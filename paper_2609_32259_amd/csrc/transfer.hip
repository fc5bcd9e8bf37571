// KV transfer kernels: RoPE cos/sin tables, map packing, and the transfer
// itself (layer interpolation + RoPE un-rotation + overlap-weighted segment
// mean, then the folded affine map of Eq. 9 with bias and receiver RoPE in
// the epilogue, written straight into the receiver cache layout).
#include <hip/hip_runtime.h>

#include <limits.h>

#include <mutex>
#include <type_traits>

#include "hf_device.h"
#include "hf_internal.h"

namespace hf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

// ---------------------------------------------------------------------------
// bf16 helpers.  bf16 -> f32 is exact (the bf16 bits are the top half of the
// f32); f32 -> bf16 rounds to nearest even (v_cvt_pk_bf16_f32).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint4 pack8(const float* f) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

// One 16-byte-per-lane global -> LDS copy: lane l writes 16 bytes at
// lds_wave_base + 16 l (lds_wave_base must be the same for the whole wave).
__device__ __forceinline__ void copy16_to_lds(const void* gsrc, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds(gsrc, (lds_void_t*)lds_wave_base, 16, 0, 0);
}

// ---------------------------------------------------------------------------
// RoPE tables: row pos holds cos(pos w_k) for k < d/2, then sin(pos w_k), with
// w_k = theta^(-2k/d); the angle is formed in fp64.  Only the rows a call reads
// are written: [0, head) and [lo, P).
// A workgroup of 512 threads owns 64 angles (k) and 8 ppt rows; each thread forms
// its w_k once, for ppt rows.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void rope_rows(const RopeTab& t, int blk, int half, int d) {
  const int n_k = (half + 63) / 64;
  const int k = (blk % n_k) * 64 + (threadIdx.x & 63);
  if (k >= half) return;
  const double w = pow(t.theta, -2.0 * k / d);
  const int rows = t.head + (t.P - t.lo);
  const int v0 = ((blk / n_k) * 8 + (int)(threadIdx.x >> 6)) * t.ppt;
  for (int v = v0; v < min(v0 + t.ppt, rows); ++v) {
    const int pos = v < t.head ? v : t.lo + (v - t.head);
    double s, c;
    sincos((double)pos * w, &s, &c);
    t.tab[(long long)pos * d + k] = (float)c;
    t.tab[(long long)pos * d + half + k] = (float)s;
  }
}

// ---------------------------------------------------------------------------
// Map packing for the bf16 matrix-core kernels.  One 1 KB fragment holds the
// 32 x 16 block (rows n, columns k) one v_mfma_f32_32x32x16_bf16 consumes as
// its A operand: lane l holds row n = 32 nb + l%32, columns
// k = 16 ks + 8 (l/32) + 0..7.  Fragments are ordered [lc][ks][nb], so a wave
// reads one fragment with a single fully coalesced 16-byte-per-lane load.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint16_t* A, uint4* Wp,
                                                        long long n_frag_lanes, int d_r, int d_in) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n_frag_lanes) return;
  const int NB = d_r / 32, KS = d_in / 16;
  const int lane = (int)(idx & 63);
  long long t = idx >> 6;
  const int nb = (int)(t % NB);
  t /= NB;
  const int ks = (int)(t % KS);
  const long long lc = t / KS;
  const int n = nb * 32 + (lane & 31);
  const int k = ks * 16 + 8 * (lane >> 5);
  Wp[idx] = *reinterpret_cast<const uint4*>(A + ((lc * d_r + n) * (long long)d_in + k));
}

// Header of a packed map buffer: what hf_pack_maps packed, ahead of the data.
__global__ __launch_bounds__(64) void pack_header_kernel(uint32_t* hdr, int dtype, int L_r,
                                                         int d_r, int d_in) {
  const int i = threadIdx.x;
  uint32_t v = 0;
  if (i == 0) v = kPackedMagic;
  if (i == 1) v = 1;  // layout version
  if (i == 2) v = (uint32_t)dtype;
  if (i == 3) v = (uint32_t)L_r;
  if (i == 4) v = (uint32_t)d_r;
  if (i == 5) v = (uint32_t)d_in;
  hdr[i] = v;  // 64 words = HF_PACKED_HEADER_BYTES
}

__global__ __launch_bounds__(256) void copy_f32_kernel(const float4* A, float4* Wp, long long n4) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx < n4) Wp[idx] = A[idx];
}

constexpr int kDH = 128;
constexpr int kXS = kDH + 8;  // LDS row stride of X / staging, bf16 elements (16-byte pad)

// Per-(layer, role, sequence) constants of the bf16 kernels.
struct Ctx {
  const uint16_t* S_lo;   // sender cache at (b, lo, c), head 0, token 0
  const uint16_t* S_hi;
  const float* cs_s;      // sender RoPE table row of position pos0_s (nullptr: no un-rotation)
  float wlo, whi;
  bool two_tap;
  int Ts;
};

// Tap t of the layer map: with concatenated taps, sender layer taps[l][t]
// with weight 1; otherwise (t = 0) the interpolation of lo and hi.
__device__ __forceinline__ Ctx make_ctx(const TransferArgs& p, const Item& it, int t = 0) {
  Ctx x;
  const uint16_t* Sb = static_cast<const uint16_t*>(p.S) + it.b * p.s_sb + it.c * p.s_sc;
  const int lo = p.concat ? arg_byte(&p.taps[0][0], 3 * it.l + t) : arg_byte(p.lo, it.l);
  x.S_lo = Sb + (long long)lo * p.s_sl;
  x.S_hi = Sb + (long long)(p.concat ? lo : arg_byte(p.hi, it.l)) * p.s_sl;
  x.cs_s = (it.c == 0 && p.unrot) ? p.cs_s + (long long)p.pos0_s[it.b] * kDH : nullptr;
  x.wlo = p.concat ? 1.0f : p.wlo[it.l];
  x.whi = p.concat ? 0.0f : p.whi[it.l];
  x.two_tap = x.whi != 0.0f;
  if (p.inv_r) {  // the map sees x / r: scale the layer weights
    const float s = p.inv_r[it.l * 2 + it.c];
    x.wlo *= s;
    x.whi *= s;
  }
  x.Ts = p.Ts[it.b];
  return x;
}

// One entry added to a row's sums: x[u] and x[u + 8] from the taps' features
// (lo: l0, l1; hi: h0, h1), with the layer weights a, bq times the entry's own, and
// for keys the rotation U(p_i) of the pair.  Every operation rounds as written: the
// callers have branches in different places, and what the compiler would fuse (a
// product into a later sum) would depend on them.
__device__ __forceinline__ void add_entry(float* x, const uint4& L0, const uint4& L1,
                                          const uint4& H0, const uint4& H1, float a, float bq,
                                          bool two_tap, bool unrot, const float* cc,
                                          const float* ss) {
#pragma clang fp contract(off)
  const uint32_t l0[4] = {L0.x, L0.y, L0.z, L0.w}, l1[4] = {L1.x, L1.y, L1.z, L1.w};
  const uint32_t h0[4] = {H0.x, H0.y, H0.z, H0.w}, h1[4] = {H1.x, H1.y, H1.z, H1.w};
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    float ma = a * ((u & 1) ? bf_hi(l0[u >> 1]) : bf_lo(l0[u >> 1]));
    float mb = a * ((u & 1) ? bf_hi(l1[u >> 1]) : bf_lo(l1[u >> 1]));
    if (two_tap) {
      ma = fmaf(bq, (u & 1) ? bf_hi(h0[u >> 1]) : bf_lo(h0[u >> 1]), ma);
      mb = fmaf(bq, (u & 1) ? bf_hi(h1[u >> 1]) : bf_lo(h1[u >> 1]), mb);
    }
    if (unrot) {  // U(p) = R(-p) on the pair (e0 + u, e0 + 64 + u)
      x[u] = fmaf(ma, cc[u], fmaf(mb, ss[u], x[u]));
      x[u + 8] = fmaf(mb, cc[u], fmaf(-ma, ss[u], x[u + 8]));
    } else {
      x[u] += ma;
      x[u + 8] += mb;
    }
  }
}

// Accumulate the aligned features of one receiver row straight from global
// memory: x[0..7] = features e0..e0+7 and x[8..15] = e0+64..e0+71 of sender
// head h (a RoPE pair per index).  Used where the staged path does not apply.
__device__ __forceinline__ void build_row_global(const TransferArgs& p, const Ctx& cx, int g,
                                                 int h, int e0, float* x) {
  const int e_beg = p.row_ptr[g], e_end = p.row_ptr[g + 1];
  const float dinv = (float)p.den[g];
  for (int e = e_beg; e < e_end; ++e) {
    const int i = min(max(p.col[e], 0), cx.Ts - 1);
    const float w = (float)p.num[e] / dinv;
    const long long off = h * p.s_sh + (long long)i * p.s_st + e0;
    const uint4 L0 = *reinterpret_cast<const uint4*>(cx.S_lo + off);
    const uint4 L1 = *reinterpret_cast<const uint4*>(cx.S_lo + off + 64);
    uint4 H0 = make_uint4(0, 0, 0, 0), H1 = H0;
    if (cx.two_tap) {
      H0 = *reinterpret_cast<const uint4*>(cx.S_hi + off);
      H1 = *reinterpret_cast<const uint4*>(cx.S_hi + off + 64);
    }
    const float a = w * cx.wlo, bq = w * cx.whi;
    float cc[8], ss[8];
    if (cx.cs_s) {
      const float* row = cx.cs_s + (long long)i * kDH;
      const float4 c0 = *reinterpret_cast<const float4*>(row + e0);
      const float4 c1 = *reinterpret_cast<const float4*>(row + e0 + 4);
      const float4 s0 = *reinterpret_cast<const float4*>(row + 64 + e0);
      const float4 s1 = *reinterpret_cast<const float4*>(row + 64 + e0 + 4);
      cc[0] = c0.x; cc[1] = c0.y; cc[2] = c0.z; cc[3] = c0.w;
      cc[4] = c1.x; cc[5] = c1.y; cc[6] = c1.z; cc[7] = c1.w;
      ss[0] = s0.x; ss[1] = s0.y; ss[2] = s0.z; ss[3] = s0.w;
      ss[4] = s1.x; ss[5] = s1.y; ss[6] = s1.z; ss[7] = s1.w;
    }
    // straight code for each case: 700 rows of 20 entries, 8 -> 8 heads 394 us without
    // rotation and 461 with it, 437 and 482 with the conditions inside
    if (cx.cs_s) {
      if (cx.two_tap) add_entry(x, L0, L1, H0, H1, a, bq, true, true, cc, ss);
      else add_entry(x, L0, L1, H0, H1, a, bq, false, true, cc, ss);
    } else {
      if (cx.two_tap) add_entry(x, L0, L1, H0, H1, a, bq, true, false, cc, ss);
      else add_entry(x, L0, L1, H0, H1, a, bq, false, false, cc, ss);
    }
  }
}

// y[q][4 g + u] *= inv * weight of its feature feat[q] + 8 g + hi4 + u.
template <int NTW>
__device__ __forceinline__ void scale_by_weights(float (*y)[16], const int* feat, int hi4,
                                                 const float* wrow, float inv) {
#pragma unroll
  for (int q = 0; q < NTW; ++q)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 w = *reinterpret_cast<const float4*>(wrow + feat[q] + 8 * g + hi4);
      y[q][4 * g + 0] *= inv * w.x;
      y[q][4 * g + 1] *= inv * w.y;
      y[q][4 * g + 2] *= inv * w.z;
      y[q][4 * g + 3] *= inv * w.w;
    }
}

// ---------------------------------------------------------------------------
// bf16 transfer kernel, tiled (d_h = 128; 2, 4 or 8 receiver heads; X holds up to 8
// sender heads, more take a pass per group of 8).
//
// One workgroup = 8 waves computes 64 receiver rows x all d_r receiver
// features of one (layer, role), in three phases after copying the tile's
// staging record (written by prologue_kernel) into LDS, or staging it there
// itself (OWN):
//   build: all 512 threads form the whole aligned feature block X[64][d_in]
//          in fp32 -- gather the tile's CSR entries (from the record), mix the
//          two sender-layer taps, un-rotate keys, weight and sum -- and store
//          it once as bf16 in LDS.  Sender rows come straight from global
//          memory through a register ring of trips; no matrix-core work is in
//          flight, so nothing waits behind these loads.  Each lane group walks
//          a run of rows holding an equal share of the tile's entries.
//   mma:   each wave multiplies its output tiles by X over all d_in/16 k-steps
//          (v_mfma_f32_32x32x16_bf16: packed map fragment from global memory as
//          A, X from LDS as B) with a four-deep register prefetch of the map
//          fragments and no barrier inside the loop.  In plain work order
//          workgroups start the loop at different sender heads so that
//          concurrent workgroups stream different parts of the map.
//   store: the tile's receiver RoPE rows and the bias are copied into LDS
//          once; bias, rotation and bf16 rounding, then staged row writes.
// Wave w owns 32-feature tiles of one receiver head: with 8 heads all four tiles
// of head w, with 4 heads tiles {w%2, w%2 + 2} of head w/2, with 2 heads tiles
// {w/2%2, w/2%2 + 2} of head w/4 for the 32 rows from 32 (w%2) on.  So RoPE pairs
// (f, f + 64) stay inside a lane; the accumulator of lane l, row block mt,
// tile q, register i holds receiver row 32 mt + l%32 (of the wave's rows) and
// feature feat[q] + 8 (i/4) + 4 (l/32) + i%4.
//
// Where the tile's record is prepared (4 or 8 receiver heads, up to 8 sender
// heads), the un-rotation of sender row i at position p_i is split as
// U(p_i) = U(q_g) U(p_i - q_g) with q_g the position of the smallest sender
// token of the lane group's run: the small-offset rotations U(0..15) sit in
// LDS and U(q_g) is applied once to each row's sum.  Tiles whose entry count or
// run sender span exceed what is staged build X entry by entry from the CSR
// and the full RoPE table in global memory.
// ---------------------------------------------------------------------------
constexpr int kEMax = 512;             // CSR entries staged per tile
constexpr int kDMax = kRopeDeltaRows;  // in-row sender offsets handled with the LDS table
constexpr int kHMax = 8;               // sender heads held in LDS
constexpr int kXF = kHMax * kDH + 8;   // LDS row stride of X, bf16 elements (16-byte pad)
constexpr int kXBytes = 64 * kXF * 2;
constexpr int kDtBytes = kDMax * kDH * 4;            // U(delta) rows: cos | sin, fp32
constexpr int kOffDt = kXBytes;
constexpr int kOffEnt = kOffDt + kDtBytes;
// Staged tile record: estart, gbase, ecol, ew, einfo, flags, gstart, row min /
// max sender index; written once per row tile by the prologue and copied whole
// into LDS by every (layer, role) of the tile.
constexpr int kEntInts = 65 + 64 + kEMax * 3 + 4 + 65 + 2 * 64;
constexpr int kRecBytes = 8192;  // 8 waves x 64 lanes x 16 bytes
static_assert(kEntInts * 4 <= kRecBytes, "tile record size");
constexpr int kOffNext = kOffEnt + kRecBytes;  // the workgroup's next work item
constexpr int kSmemBytes = kOffNext + 16;
// Store phase, inside the (then free) X region: receiver RoPE rows, bias, staging.
constexpr int kOffRcs = 0;                           // [64][cos 64 | sin 64] fp32
constexpr int kOffBias = kOffRcs + 64 * kDH * 4;     // [d_r <= 1024] fp32
constexpr int kOffStage = kOffBias + 1024 * 4;       // 8 waves x [32][kXS] bf16
constexpr int kOffRsum = kOffStage + 8 * 32 * kXS * 2;  // 8 waves x 32 fp32
static_assert(kOffRsum + 8 * 32 * 4 <= kXBytes, "store phase must fit the X region");
static_assert(kSmemBytes <= 160 * 1024, "LDS budget");

// Group-walk build.  WPH waves share a sender head, 8 WPH lane groups (8
// lanes, 16 features each) over the tile's 64 rows: group g walks the CSR
// entries of a run of consecutive rows in order, one entry per trip, so a
// sender token shared by neighbouring rows is read twice in a row (the second
// read hits the cache).  The runs hold equal shares of the tile's entries, as
// a wave takes as many trips as its longest run.  Trips past a group's last entry
// use an out-of-range buffer offset, which returns zeros without touching
// memory, so every trip issues the same loads and a ring of R trips keeps
// R - 1 trips of loads in flight.
// ABS (the kernels that stage their tiles themselves): each entry is rotated by its
// own U(p_i) from the table, and added by add_entry, so that the results are those of
// build_row_global bit for bit.  The split rotation differs in the last bits of fp32,
// which moves 0.2% of the bf16 results; it is 1 to 4% faster (8 -> 2 heads, 1,821 rows:
// 198 against 202 us; 14,250 rows: 1,300 against 1,361).
constexpr int kOOB = (int)0x80000000;  // buffer offset past any slab extent (extents < 2^31)

struct GroupLds {
  const int* estart;  // [65] CSR offsets of the tile rows
  const int* ecol;    // staged sender indices
  const float* ew;    // staged weights num / den
  const int* einfo;   // staged row | last-entry-of-row << 8 | first-entry-of-row << 9
  const float* dt;    // U(0..15), swizzled
  int e_base;
};

template <bool TWO_TAP, bool ABS>
struct Trip {
  uint4 a0, a1, b0, b1;  // tap lo / hi: features e0..e0+7 and e0+64..e0+71
  uint4 c0, c1, s0, s1;  // ABS: U(p_i) of features e0..e0+7 (cos, sin)
  int code;              // -1: no entry; else row | last << 6 | (i - base) << 8
  float w;
};

// Rotation rows of the swizzled U(0..15) table: row t holds cos chunks 0..15
// then sin chunks 16..31 (4 floats each), chunk c stored at slot c ^ (t & 1).
__device__ __forceinline__ void table_row(const float* tab, int t, int e0, float* c, float* s) {
  const float4* row = reinterpret_cast<const float4*>(tab) + t * 32;
  const int cw = t & 1;
  const float4 c0 = row[(e0 >> 2) ^ cw], c1 = row[((e0 >> 2) + 1) ^ cw];
  const float4 s0 = row[(16 + (e0 >> 2)) ^ cw], s1 = row[(17 + (e0 >> 2)) ^ cw];
  c[0] = c0.x; c[1] = c0.y; c[2] = c0.z; c[3] = c0.w;
  c[4] = c1.x; c[5] = c1.y; c[6] = c1.z; c[7] = c1.w;
  s[0] = s0.x; s[1] = s0.y; s[2] = s0.z; s[3] = s0.w;
  s[4] = s1.x; s[5] = s1.y; s[6] = s1.z; s[7] = s1.w;
}

__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, int off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Where a built X row goes: sink(r, f, v) stores features f..f+7 of tile row r.
struct LdsSink {  // the X tile in LDS (row stride kXF)
  uint16_t* Xs;
  __device__ __forceinline__ void operator()(int r, int f, uint4 v) const {
    *reinterpret_cast<uint4*>(Xs + r * kXF + f) = v;
  }
};

template <bool TWO_TAP, bool UNROT, bool ABS, int R, class Sink>
__device__ __forceinline__ void build_groups(const Ctx& cx, const TransferArgs& p, const GroupLds& L,
                                             int base, int src_head, int head, int r_first, int rpg,
                                             int lane, const Sink& sink) {
  const int e0 = (lane & 7) * 8;
  const int kb = L.estart[r_first] - L.e_base;
  const int E = L.estart[r_first + rpg] - L.e_base - kb;
  int T = 0;  // trips of the wave: the longest group
#pragma unroll
  for (int g = 0; g < 8; ++g) T = max(T, __builtin_amdgcn_readlane(E, 8 * g));
  for (int q = 0; q < rpg; ++q) {  // rows without entries stay zero
    const int r = r_first + q;
    if (L.estart[r + 1] == L.estart[r]) {
      sink(r, head * kDH + e0, make_uint4(0, 0, 0, 0));
      sink(r, head * kDH + 64 + e0, make_uint4(0, 0, 0, 0));
    }
  }
  float rc[8], rs[8];  // U(p_base): closes every row of the group
  if (UNROT && !ABS) {
    const float* row = cx.cs_s + (long long)base * kDH;
    const float4 c0 = *reinterpret_cast<const float4*>(row + e0);
    const float4 c1 = *reinterpret_cast<const float4*>(row + e0 + 4);
    const float4 s0 = *reinterpret_cast<const float4*>(row + 64 + e0);
    const float4 s1 = *reinterpret_cast<const float4*>(row + 64 + e0 + 4);
    rc[0] = c0.x; rc[1] = c0.y; rc[2] = c0.z; rc[3] = c0.w;
    rc[4] = c1.x; rc[5] = c1.y; rc[6] = c1.z; rc[7] = c1.w;
    rs[0] = s0.x; rs[1] = s0.y; rs[2] = s0.z; rs[3] = s0.w;
    rs[4] = s1.x; rs[5] = s1.y; rs[6] = s1.z; rs[7] = s1.w;
  }
  const __amdgpu_buffer_rsrc_t rlo =
      __builtin_amdgcn_make_buffer_rsrc((void*)cx.S_lo, 0, p.s_extent, 0x00020000);
  const __amdgpu_buffer_rsrc_t rhi =
      __builtin_amdgcn_make_buffer_rsrc((void*)cx.S_hi, 0, p.s_extent, 0x00020000);
  const __amdgpu_buffer_rsrc_t rcs =
      __builtin_amdgcn_make_buffer_rsrc((void*)cx.cs_s, 0, cx.Ts * kDH * 4, 0x00020000);
  const int hoff = (int)(src_head * p.s_sh + e0) * 2;  // bytes
  const int tstride = (int)p.s_st * 2;

  Trip<TWO_TAP, UNROT && ABS> ring[R];
  float x[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) x[u] = 0.0f;

  auto issue = [&](Trip<TWO_TAP, UNROT && ABS>& t, int k) {
    const bool valid = k < E;
    int i = 0, info = 0;
    float w = 0.0f;
    if (valid) {
      i = L.ecol[kb + k];
      w = L.ew[kb + k];
      info = L.einfo[kb + k];
    }
    const int off = valid ? hoff + i * tstride : kOOB;
    t.a0 = buf_load16(rlo, off);
    t.a1 = buf_load16(rlo, off + 128);
    if (TWO_TAP) {
      t.b0 = buf_load16(rhi, off);
      t.b1 = buf_load16(rhi, off + 128);
    }
    if (UNROT && ABS) {
      const int co = valid ? i * (kDH * 4) + e0 * 4 : kOOB;  // fewer than 2^22 sender rows
      t.c0 = buf_load16(rcs, co);
      t.c1 = buf_load16(rcs, co + 16);
      t.s0 = buf_load16(rcs, co + 256);
      t.s1 = buf_load16(rcs, co + 272);
    }
    t.code = valid ? ((info & 63) | ((info >> 8) << 6) | ((UNROT && !ABS ? i - base : 0) << 8)) : -1;
    t.w = w;
  };
  auto consume = [&](const Trip<TWO_TAP, UNROT && ABS>& t) {
    if (t.code < 0) return;
    const uint32_t l0[4] = {t.a0.x, t.a0.y, t.a0.z, t.a0.w};
    const uint32_t l1[4] = {t.a1.x, t.a1.y, t.a1.z, t.a1.w};
    uint32_t h0[4] = {0, 0, 0, 0}, h1[4] = {0, 0, 0, 0};
    if (TWO_TAP) {
      h0[0] = t.b0.x; h0[1] = t.b0.y; h0[2] = t.b0.z; h0[3] = t.b0.w;
      h1[0] = t.b1.x; h1[1] = t.b1.y; h1[2] = t.b1.z; h1[3] = t.b1.w;
    }
    const float a = t.w * cx.wlo, bq = t.w * cx.whi;  // weight folded into the layer mix
    float cc[8], ss[8];
    if (UNROT && !ABS) table_row(L.dt, t.code >> 8, e0, cc, ss);  // U(p_i - p_base)
    if (ABS && UNROT) {
      const uint4 v[4] = {t.c0, t.c1, t.s0, t.s1};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float* d = (g < 2 ? cc : ss) + 4 * (g & 1);
        d[0] = __uint_as_float(v[g].x);
        d[1] = __uint_as_float(v[g].y);
        d[2] = __uint_as_float(v[g].z);
        d[3] = __uint_as_float(v[g].w);
      }
    }
    if (ABS) {
      const uint4 z = make_uint4(0, 0, 0, 0);
      add_entry(x, t.a0, t.a1, TWO_TAP ? t.b0 : z, TWO_TAP ? t.b1 : z, a, bq, TWO_TAP, UNROT, cc, ss);
    } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      float ma = a * ((u & 1) ? bf_hi(l0[u >> 1]) : bf_lo(l0[u >> 1]));
      float mb = a * ((u & 1) ? bf_hi(l1[u >> 1]) : bf_lo(l1[u >> 1]));
      if (TWO_TAP) {
        ma = fmaf(bq, (u & 1) ? bf_hi(h0[u >> 1]) : bf_lo(h0[u >> 1]), ma);
        mb = fmaf(bq, (u & 1) ? bf_hi(h1[u >> 1]) : bf_lo(h1[u >> 1]), mb);
      }
      if (UNROT) {
        x[u] = fmaf(ma, cc[u], fmaf(mb, ss[u], x[u]));
        x[u + 8] = fmaf(mb, cc[u], fmaf(-ma, ss[u], x[u + 8]));
      } else {
        x[u] += ma;
        x[u + 8] += mb;
      }
    }
    }
    if ((t.code >> 6) & 1) {  // last entry of the row: close the rotation, round, store
      if (UNROT && !ABS) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float a = x[u], b = x[u + 8];
          x[u] = fmaf(a, rc[u], b * rs[u]);
          x[u + 8] = fmaf(b, rc[u], -a * rs[u]);
        }
      }
      sink(t.code & 63, head * kDH + e0, pack8(x));
      sink(t.code & 63, head * kDH + 64 + e0, pack8(x + 8));
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = 0.0f;
    }
  };

#pragma unroll
  for (int s = 0; s < R - 1; ++s) issue(ring[s], s);
  for (int t0 = 0; t0 < T; t0 += R) {
#pragma unroll
    for (int s = 0; s < R; ++s) {
      issue(ring[(s + R - 1) % R], t0 + s + R - 1);
      if (t0 + s < T) consume(ring[s]);
    }
  }
}

// ---------------------------------------------------------------------------
// Per-tile staging for the tiled kernel, one workgroup per 64-row tile of the
// batch.  The record holds the tile's CSR entries with their row, weight
// num/den and first / last-of-row flags; the cut of the rows into runs of
// consecutive rows with equal shares of the entries (a wave takes as many
// trips as its longest run); each run's smallest sender index; and two flags:
// [0] some run spans kDMax sender tokens or more (too wide for the LDS
// rotation table), [1] the tile has more than kEMax entries.  Every (layer,
// role) of the tile reads the same record.
// ---------------------------------------------------------------------------
// Tile t's record into ent (LDS), by 512 threads.
__device__ __forceinline__ void stage_tile(const TransferArgs& p, int t, int* ent) {
  int* estart = ent;
  int* gbase = estart + 65;
  int* ecol = gbase + 64;
  float* ew = reinterpret_cast<float*>(ecol + kEMax);
  int* einfo = reinterpret_cast<int*>(ew + kEMax);
  int* flag = einfo + kEMax;
  int* gstart = flag + 4;     // lane group g walks tile rows [gstart[g], gstart[g + 1])
  int* rmin = gstart + 65;    // smallest / largest sender index of each tile row
  int* rmax = rmin + 64;

  int b = 0;
  while (b + 1 < p.B && p.tile_start[b + 1] <= t) ++b;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = (t - p.tile_start[b]) * 64;
  const int nrows = min(64, p.Tr[b] - j0);
  const int g0 = p.row0[b] + j0;
  const int Ts = p.Ts[b];
  const int H = p.H_s;
  const int WPH = H == 1 ? 8 : H == 2 ? 4 : H <= 4 ? 2 : 1;  // waves per sender head

  if (tid <= 64) estart[tid] = p.row_ptr[g0 + min(tid, nrows)];
  if (tid < 4) flag[tid] = 0;
  __syncthreads();
  const int e_base = estart[0];
  const int nnz = estart[nrows] - e_base;
  const bool fits = nnz <= kEMax;
  if (fits) {
    for (int k = tid; k < nnz; k += 512) {
      int lo = 0, hi = nrows;  // row r with estart[r] <= e_base + k < estart[r + 1]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (estart[mid] <= e_base + k) lo = mid; else hi = mid;
      }
      const int e = e_base + k;
      ecol[k] = min(max(p.col[e], 0), Ts - 1);
      ew[k] = (float)p.num[e] / (float)p.den[g0 + lo];
      einfo[k] = lo | ((int)(e + 1 == estart[lo + 1]) << 8) | ((int)(e == estart[lo]) << 9);
    }
  }
  __syncthreads();
  const int NG = 8 * WPH;  // lane groups over the tile's rows
  if (wave == 0) {
    // Boundaries gstart[0..NG]; with one sender head NG = 64, one more than the
    // wave has lanes, so lane 0 also writes the closing boundary gstart[NG].
    if (lane == 0) gstart[NG] = 64;
    if (lane < NG) {
      int bnd = 0;
      if (lane > 0) {
        const int target = (lane * nnz + NG / 2) / NG;
        int lo = 0, hi = nrows;  // smallest r with estart[r] - e_base >= target
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (estart[mid] - e_base >= target) hi = mid; else lo = mid + 1;
        }
        bnd = lo;
      }
      gstart[lane] = bnd;
    }
    int lmin = INT_MAX, lmax = -1;  // lane = tile row
    if (fits && lane < nrows)
      for (int k = estart[lane] - e_base; k < estart[lane + 1] - e_base; ++k) {
        lmin = min(lmin, ecol[k]);
        lmax = max(lmax, ecol[k]);
      }
    rmin[lane] = lmin;
    rmax[lane] = lmax;
    if (lane < NG) {  // sender span of each run
      int gmin = INT_MAX, gmax = -1;
      for (int r = gstart[lane]; r < gstart[lane + 1]; ++r) {
        gmin = min(gmin, rmin[r]);
        gmax = max(gmax, rmax[r]);
      }
      gbase[lane] = gmax < 0 ? 0 : gmin;
      if (gmax >= 0 && gmax - gmin >= kDMax) flag[0] = 1;
    }
    if (lane == 0 && !fits) flag[1] = 1;
  }
  __syncthreads();
}

// Work items in plain order, or dealt in kQueues queues (transfer_order says when):
// queue q then holds the tiles of every eighth (layer, role) from q on.  Workgroup i
// takes from queue i % 8 and runs on XCD i % 8, so the workgroups of an XCD share one
// map in its L2.
constexpr int kQueues = 8;
constexpr int kCtrStride = 8;  // ints between the queues' counters (256 bytes in all)
constexpr int kCtrTotal = 4;   // the count of all items taken, between the first two

__device__ __forceinline__ int queue_items(const TransferArgs& p, int q) {
  return p.tiles_per_lc * ((2 * p.L_r - q + kQueues - 1) / kQueues);
}
// Item v of queue q, in plain order.
__device__ __forceinline__ int queue_item(const TransferArgs& p, int q, int v) {
  const int i = v / p.tiles_per_lc;
  return (kQueues * i + q) * p.tiles_per_lc + (v - i * p.tiles_per_lc);
}
// An item of the queues after `own` (which is empty), or n_items if they are too.
__device__ __forceinline__ int other_queue_item(const TransferArgs& p, int own, int n_items) {
#pragma unroll 1
  for (int i = 1; i < kQueues; ++i) {
    const int q = (own + i) % kQueues, n = queue_items(p, q);
    if (n <= 0) continue;
    const int v = atomicAdd(p.work_ctr + q * kCtrStride, 1);
    if (v < n) return queue_item(p, q, v);
  }
  return n_items;
}
// The next item for a workgroup of queue `own`, n_items if none is left.  A count of
// all items taken goes along, so that the end is found with one look and not eight.
__device__ __forceinline__ int next_item_of(const TransferArgs& p, int own, int n_items) {
  const int v = atomicAdd(p.work_ctr + own * kCtrStride, 1);
  const int t = atomicAdd(p.work_ctr + kCtrTotal, 1);
  if (v < queue_items(p, own)) return queue_item(p, own, v);
  return t < n_items ? other_queue_item(p, own, n_items) : n_items;
}

// What a transfer needs before its kernels, in one launch (each costs 5 to 6 us on
// the GPU whatever it does: a call on 200 tokens took 18 us for two tables and the
// records, 5.7 now): first the staging of the tiles (n_stage workgroups),
// then the RoPE tables.
__global__ __launch_bounds__(512) void prologue_kernel(const TransferArgs p, int* rec, int n_stage,
                                                       const RopeTabs r) {
  __shared__ __attribute__((aligned(16))) int ent[kRecBytes / 4];
  int blk = blockIdx.x;
  if (blk < n_stage) {
    if (blk == 0 && threadIdx.x < kQueues) {  // the first items are taken statically
      const int q = threadIdx.x, wgs = (p.n_wg - q + kQueues - 1) / kQueues;
      if (p.queued) p.work_ctr[q * kCtrStride] = min(wgs, queue_items(p, q));
      else if (q == 0) p.work_ctr[0] = p.n_wg;
      if (q == 0) p.work_ctr[kCtrTotal] = p.n_wg;
    }
    stage_tile(p, blk, ent);
    int4* dst = reinterpret_cast<int4*>(rec + (long long)blk * (kRecBytes / 4));
    dst[threadIdx.x] = reinterpret_cast<const int4*>(ent)[threadIdx.x];
    return;
  }
  blk -= n_stage;
  for (int i = 0; i < r.n; ++i) {
    if (blk < r.t[i].blocks) {
      rope_rows(r.t[i], blk, p.d_h / 2, p.d_h);
      return;
    }
    blk -= r.t[i].blocks;
  }
}

// HR: receiver heads.  MULTI: several passes over the X tile (concatenated taps,
// or more than kHMax sender heads).  OWN: the call's workspace has no records
// and no work counter (two receiver heads, or more than kHMax sender heads), so
// every workgroup does one item and stages its tile itself.  QUEUED: a persistent
// workgroup takes its items from the queues (the others map their one item with
// p.queued).  A kernel of its own for the plain order: with the queues' search in it
// the 8 -> 4-head kernel has 68 bytes of scratch a lane instead of none, and calls of
// 32K tokens take 0.5 to 0.8% longer.
template <int HR, bool MULTI, bool OWN, bool QUEUED>
__global__ __launch_bounds__(512, 1) void transfer_bf16_tiled_kernel(const TransferArgs p) {
  constexpr int NTW = HR == 8 ? 4 : 2;  // 32-feature tiles per wave
  constexpr int MT = HR == 2 ? 1 : 2;   // 32-row blocks per wave
  __shared__ __attribute__((aligned(16))) unsigned char smem[kSmemBytes];
  uint16_t* Xs = reinterpret_cast<uint16_t*>(smem);
  float* dt = reinterpret_cast<float*>(smem + kOffDt);
  int* estart = reinterpret_cast<int*>(smem + kOffEnt);
  int* gbase = estart + 65;
  int* ecol = gbase + 64;
  float* ew = reinterpret_cast<float*>(ecol + kEMax);
  int* einfo = reinterpret_cast<int*>(ew + kEMax);
  const int* flag = einfo + kEMax;  // [0] a run too wide for U(0..15), [1] too many entries
  const int* gstart = flag + 4;     // lane group g walks tile rows [gstart[g], gstart[g + 1])
  int* next_item = reinterpret_cast<int*>(smem + kOffNext);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int H = p.H_s;
  // WPH waves share a sender head; each lane group walks a run of rows
  const int WPH = H == 1 ? 8 : H == 2 ? 4 : H <= 4 ? 2 : 1;
  const int n_items = p.tiles_per_lc * p.L_r * 2;
  // The tile's staging record into LDS, one 16-byte-per-lane copy per wave.
  auto copy_record = [&](int item) {
    const Item ni = decode_item(p, item);
    const int* rec = p.tile_rec + (long long)(p.tile_start[ni.b] + ni.tile) * (kRecBytes / 4);
    copy16_to_lds(rec + wave * 256 + 4 * lane, estart + wave * 256);
  };

  // Persistent (interpolating map): the workgroup starts on item blockIdx.x, or item
  // blockIdx.x / 8 of its queue, and takes the next one from the counter (set to the
  // items started this way by the prologue) while it builds, so the items in flight
  // stay a contiguous run of the order or of each queue, and the next record is copied
  // in during the store.  With several passes (which leave no registers for the loop)
  // a workgroup does one item, and the queues are equally long.
  constexpr bool kPersist = !MULTI && !OWN;
  const int queue = blockIdx.x % kQueues, first = blockIdx.x / kQueues;
  int item = blockIdx.x;
  if (!kPersist) {
    if (p.queued) item = queue_item(p, queue, first);
  } else if (QUEUED) {
    if (first < queue_items(p, queue)) {
      item = queue_item(p, queue, first);
    } else {  // more workgroups than items in this queue
      if (tid == 0) *next_item = other_queue_item(p, queue, n_items);
      __syncthreads();
      item = *next_item;
      if (item >= n_items) return;
    }
  }
  if (OWN) stage_tile(p, item % p.tiles_per_lc, estart);
  else copy_record(item);
  if (!OWN && p.unrot) {  // U(0..15): rows 0..15 of the sender table, 2 per wave
    const int ri = wave * 2 + (lane >> 5);
    const int c = (lane & 31) ^ (ri & 1);
    copy16_to_lds(p.cs_s + (long long)ri * kDH + 4 * c, dt + wave * 2 * kDH);
  }
  __builtin_amdgcn_s_waitcnt(0);  // both copies have landed
  __syncthreads();

  for (;;) {
  const Item it = decode_item(p, item);
  const Ctx cx = make_ctx(p, it);
  const int Tr = p.Tr[it.b];
  const int j0 = it.tile * 64;
  const int nrows = min(64, Tr - j0);
  const int g0 = p.row0[it.b] + j0;
  const bool unrot = cx.cs_s != nullptr;
  const int e_base = estart[0];
  const bool staged = p.s_extent > 0 && flag[1] == 0 &&
                      !(unrot && (OWN ? cx.Ts >= (1 << 22) : flag[0] != 0));
  int grabbed = n_items;
  if (kPersist && tid == 0)
    grabbed = QUEUED ? next_item_of(p, queue, n_items) : atomicAdd(p.work_ctr, 1);

  f32x16 acc[MT][NTW];  // zeroed after the first pass's build
  // This wave's accumulators: receiver head `head`, n-tiles feat[q].
  const int head = HR == 8 ? wave : HR == 4 ? (wave >> 1) : (wave >> 2);
  const int nt0 = HR == 8 ? 0 : HR == 4 ? (wave & 1) : ((wave >> 1) & 1);
  const int row0 = HR == 2 ? 32 * (wave & 1) : 0;  // the wave's first tile row
  constexpr int NTS = 4 / NTW;  // n-tile stride inside the head
  int feat[NTW];
#pragma unroll
  for (int q = 0; q < NTW; ++q) feat[q] = 32 * (nt0 + q * NTS);
  const int NB = p.H_r * (kDH / 32);
  const int lc_store = it.l * 2 + it.c;

  // One pass per tap of the layer map (concatenated taps, each one sender layer)
  // and group of kHMax sender heads: build its X, multiply it by the matching k
  // block of the map into the same accumulators.  From the second pass on the
  // accumulators are live during the build, which then keeps fewer loads in
  // flight.
  const int n_grp = OWN ? (H + kHMax - 1) / kHMax : 1;
  const int n_pass = MULTI ? p.n_taps * n_grp : 1;
  for (int pass = 0; pass < n_pass; ++pass) {
    if (pass > 0) __syncthreads();  // every wave is done reading the previous pass's X
    const int tap = pass / n_grp, h_first = OWN ? kHMax * (pass - tap * n_grp) : 0;
    const int Hp = OWN ? min(kHMax, H - h_first) : H;  // sender heads of this pass
    const int KS = Hp * (kDH / 16);                    // and its k-steps
    // The first one.  In plain order, where all workgroups share a map, they start at
    // different sender heads; an XCD's few start at the same one and meet in its L2.
    // OWN: all at the first, so that a result does not depend on the work order.
    const int ks0 =
        OWN ? 0
            : (int)((unsigned)((kPersist ? QUEUED : p.queued != 0) ? lc_store : item) %
                    (unsigned)Hp) * (kDH / 16);
    const Ctx ct = make_ctx(p, it, tap);
    // ---- build X[64][Hp d_h] of this pass ----
    if (staged) {
      const LdsSink xsink{Xs};
      const int sh = wave / WPH;  // sender head this wave builds
      if (sh < Hp) {
        const GroupLds L{estart, ecol, ew, einfo, dt, e_base};
        const int grp = (wave % WPH) * 8 + (lane >> 3);
        const int r_first = gstart[grp];
        const int rpg = gstart[grp + 1] - r_first;
        const int base = gbase[grp];
        const int src = h_first + sh;
        auto build = [&](auto two, auto rotate, auto ring) {
          build_groups<decltype(two)::value, decltype(rotate)::value, OWN, decltype(ring)::value>(
              ct, p, L, base, src, sh, r_first, rpg, lane, xsink);
        };
        using T = std::true_type;
        using F = std::false_type;
        using R3 = std::integral_constant<int, 3>;
        using R2 = std::integral_constant<int, 2>;
        // Trips in flight in the first pass and the later ones.  Two receiver heads
        // leave registers for the deeper ring in every pass; eight with the entries'
        // own rotations in none (16 -> 8 heads, 1,821 rows: 685 us with 53 registers
        // spilled, 647 with 3).
        using R0 = std::conditional_t<OWN && HR == 8, R2, R3>;
        using Rn = std::conditional_t<HR == 2, R3, R2>;
        if ((!MULTI || OWN) && ct.two_tap) {  // concatenated taps are one sender layer each
          if (!MULTI || pass == 0) {
            if (unrot) build(T(), T(), R0());
            else build(T(), F(), R0());
          } else {
            if (unrot) build(T(), T(), Rn());
            else build(T(), F(), Rn());
          }
        } else if (!MULTI || pass == 0) {
          if (unrot) build(F(), T(), R0());
          else build(F(), F(), R0());
        } else {
          if (unrot) build(F(), T(), Rn());
          else build(F(), F(), Rn());
        }
      }
    } else {
      const int r = tid >> 3;         // 8 threads per row
      const int e0 = (tid & 7) * 8;   // features e0..e0+7 and e0+64..e0+71 of every head
      for (int h = 0; h < Hp; ++h) {
        float x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = 0.0f;
        if (r < nrows) build_row_global(p, ct, g0 + r, h_first + h, e0, x);
        uint16_t* xr = Xs + r * kXF + h * kDH;
        *reinterpret_cast<uint4*>(xr + e0) = pack8(x);
        *reinterpret_cast<uint4*>(xr + 64 + e0) = pack8(x + 8);
      }
    }
    __syncthreads();
    if (pass == 0) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < NTW; ++q)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[mt][q][i] = 0.0f;
    }

    // ---- multiply ----
    // The map block of this (layer, role, pass) through a buffer resource: a
    // 32-bit per-lane offset plus the k-step's scalar offset, so a refill costs
    // no 64-bit address arithmetic.
    const bf16x8* Wblk =
        static_cast<const bf16x8*>(p.Wp) +
        (((long long)lc_store * p.n_taps + tap) * H + h_first) * (kDH / 16) * NB * 64;
    const __amdgpu_buffer_rsrc_t rW =
        __builtin_amdgcn_make_buffer_rsrc((void*)Wblk, 0, KS * NB * 64 * 16, 0x00020000);
    const int w_lane = ((4 * head + nt0) * 64 + lane) * 16;  // bytes within a k-step
    // Map fragments of four consecutive k-steps, kept as integers: as bf16 vectors
    // the compiler copied the first slot through registers and waited for
    // every load in flight once per four k-steps (2.5% of a 4-head transfer).
    u32x4 wr[4][NTW];
    auto kstep = [&](int ks) { int k = ks + ks0; return k >= KS ? k - KS : k; };
    auto load_w = [&](u32x4* dst, int ks) {
      const int k_off = kstep(ks) * NB * 64 * 16;
#pragma unroll
      for (int q = 0; q < NTW; ++q)
        dst[q] = __builtin_amdgcn_raw_buffer_load_b128(rW, w_lane + q * NTS * 64 * 16, k_off, 0);
    };
    auto read_x = [&](bf16x8* xa, int ks) {
      const int k = kstep(ks);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        xa[mt] = *reinterpret_cast<const bf16x8*>(Xs + (row0 + 32 * mt + (lane & 31)) * kXF + 16 * k +
                                                8 * (lane >> 5));
    };
    bf16x8 xc[MT], xn[MT];  // X fragments of this k-step and the next
    // One k-step: read next X from LDS, multiply, then refill this map slot with
    // k-step ks + 4.  LOAD is a constant so that the loop body has no branches
    // and every wait on a map fragment keeps the three younger k-steps in flight.
    auto step = [&](u32x4* wf, int ks, auto load) {
      read_x(xn, ks + 1);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < NTW; ++q)
          acc[mt][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[q]), xc[mt],
                                                               acc[mt][q], 0, 0, 0);
      if (decltype(load)::value) load_w(wf, ks + 4);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xc[mt] = xn[mt];
      __builtin_amdgcn_sched_barrier(0);  // keep the refill in this k-step
    };
    using Load = std::true_type;
    using NoLoad = std::false_type;
#pragma unroll
    for (int u = 0; u < 4; ++u) load_w(wr[u], u);  // KS is a multiple of 8
    read_x(xc, 0);
    for (int ks = 0; ks < KS - 4; ks += 4) {
      step(wr[0], ks, Load());
      step(wr[1], ks + 1, Load());
      step(wr[2], ks + 2, Load());
      step(wr[3], ks + 3, Load());
    }
    step(wr[0], KS - 4, NoLoad());
    step(wr[1], KS - 3, NoLoad());
    step(wr[2], KS - 2, NoLoad());
    step(wr[3], KS - 1, NoLoad());
  }
  if (tid == 0) *next_item = grabbed;
  __syncthreads();  // every wave is done reading X; the X region is free
  const int next = *next_item;

  // ---- store ----
  const bool rot = it.c == 0 && p.rot;
  float* rcs = reinterpret_cast<float*>(smem + kOffRcs);
  float* bias_s = reinterpret_cast<float*>(smem + kOffBias);
  const int d_r = NB * 32;
  if (rot) {  // receiver RoPE rows j0..j0+63: 2 per wave instruction; slot c holds chunk
              // (c & 16) | ((c ^ r) & 15) so that lanes of different rows hit different banks
    for (int q = wave; q < 32; q += 8) {
      const int rr = 2 * q + (lane >> 5);
      const int c = lane & 31;
      const int cs = (c & 16) | ((c ^ rr) & 15);
      const int jr = p.pos0_r[it.b] + j0 + min(rr, nrows - 1);
      copy16_to_lds(p.cs_r + (long long)jr * kDH + 4 * cs, rcs + q * 2 * kDH);
    }
  }
  if (p.bias && wave < d_r / 256)  // 256 floats per wave instruction
    copy16_to_lds(p.bias + (long long)lc_store * d_r + wave * 256 + 4 * lane, bias_s + wave * 256);
  if (next < n_items) copy_record(next);  // this item's record is no longer read
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  uint16_t* stage = reinterpret_cast<uint16_t*>(smem + kOffStage) + wave * 32 * kXS;
  uint16_t* dst_head = static_cast<uint16_t*>(p.R) + it.b * p.r_sb + (long long)it.l * p.r_sl +
                       it.c * p.r_sc + head * p.r_sh;
  float* rsum = reinterpret_cast<float*>(smem + kOffRsum);  // [8 waves][32] row sums of squares
  const float* knorm = (it.c == 0 && p.k_norm) ? p.k_norm + (long long)it.l * kDH : nullptr;
  const int hi4 = 4 * (lane >> 5);
  const int mcol = lane & 31;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int rl = row0 + 32 * mt + mcol;  // tile row held by this lane
    float y[NTW][16];
#pragma unroll
    for (int q = 0; q < NTW; ++q)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p.bias) bv = *reinterpret_cast<const float4*>(bias_s + head * kDH + feat[q] + 8 * g + hi4);
        y[q][4 * g + 0] = acc[mt][q][4 * g + 0] + bv.x;
        y[q][4 * g + 1] = acc[mt][q][4 * g + 1] + bv.y;
        y[q][4 * g + 2] = acc[mt][q][4 * g + 2] + bv.z;
        y[q][4 * g + 3] = acc[mt][q][4 * g + 3] + bv.w;
      }
    if (knorm) {  // receiver key RMSNorm over each head's 128 features
      float ss = 0.0f;
#pragma unroll
      for (int q = 0; q < NTW; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) ss = fmaf(y[q][i], y[q][i], ss);
      ss += __shfl_xor(ss, 32);  // lane ^ 32 holds the same row's other features
      if (NTW == 2) {            // another wave holds the other half of the head
        rsum[wave * 32 + mcol] = ss;
        __syncthreads();
        ss += rsum[(wave ^ (HR == 2 ? 2 : 1)) * 32 + mcol];
        __syncthreads();
      }
      const float inv = 1.0f / sqrtf(ss * (1.0f / kDH) + p.k_norm_eps);
      scale_by_weights<NTW>(y, feat, hi4, knorm, inv);
    }
    if (rot) {
      const float4* crow = reinterpret_cast<const float4*>(rcs) + rl * 32;
#pragma unroll
      for (int q = 0; q < NTW / 2; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = (feat[q] + 8 * g + hi4) >> 2;  // cos chunk, < 16
          const float4 cv = crow[(c ^ rl) & 15];
          const float4 sv = crow[16 | ((c ^ rl) & 15)];
          const float cc[4] = {cv.x, cv.y, cv.z, cv.w};
          const float ss[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float a = y[q][4 * g + u], b = y[q + NTW / 2][4 * g + u];
            y[q][4 * g + u] = fmaf(a, cc[u], -b * ss[u]);
            y[q + NTW / 2][4 * g + u] = fmaf(b, cc[u], a * ss[u]);
          }
        }
    }
#pragma unroll
    for (int q = 0; q < NTW; ++q)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 v = make_uint2(pack2(y[q][4 * g], y[q][4 * g + 1]), pack2(y[q][4 * g + 2], y[q][4 * g + 3]));
        *reinterpret_cast<uint2*>(stage + mcol * kXS + 32 * q + 8 * g + hi4) = v;
      }
    constexpr int LPR = NTW * 4;  // lanes per row, 16 bytes each
    constexpr int RPP = 64 / LPR;
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int rr = pass * RPP + lane / LPR;
      const int ci = lane % LPR;
      const uint4 v = *reinterpret_cast<const uint4*>(stage + rr * kXS + 8 * ci);
      const int jj = j0 + row0 + 32 * mt + rr;
      if (jj < Tr)  // streaming store: the receiver rows are not read again here, so
                    // they should not push the shared map out of L2
        __builtin_nontemporal_store(
            u32x4{v.x, v.y, v.z, v.w},
            reinterpret_cast<u32x4*>(dst_head + (long long)jj * p.r_st + feat[ci / 4] + 8 * (ci % 4)));
    }
  }
  if (!kPersist || next >= n_items) break;
  __syncthreads();  // every wave is done with the staging rows; the next build writes X
  item = next;
  }
}

// ---------------------------------------------------------------------------
// Staged path, build: the aligned features of one (slab, 64-row tile) written
// to global memory in the layout the staged GEMM reads.  The tile is built in
// LDS and then written out: in the slab's [256-row tile][k-tile][256][32]
// layout its rows are one 4 KB run per k-tile, so every wave store is 1 KB of
// whole lines (rows past the sequence end carry zeros the GEMM never stores).
// Each wave writes its own sender head as soon as its walk ends.  A slab is (role,
// receiver layer) for the interpolating map -- x_j of Sec. 3.1 with the layer
// weights of its two taps -- or (role, sender layer) for concatenated taps --
// one block x_j^t of Eq. 2, shared by every receiver layer that reads that
// sender layer.  The arithmetic is the fused kernel's build (same staging
// record, same group walk, one bf16 rounding per feature).
// ---------------------------------------------------------------------------
// 16 bytes from LDS to global memory as a streaming (non-temporal) store: the
// slab is read back only after the whole build, so it need not stay in L2.
__device__ __forceinline__ void nt_store16(uint16_t* g, const uint16_t* l) {
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(*reinterpret_cast<const v4u*>(l), reinterpret_cast<v4u*>(g));
}

__global__ __launch_bounds__(512) void staged_build_kernel(const TransferArgs p) {
  __shared__ __attribute__((aligned(16))) uint16_t xl[64 * kXF];  // the built tile, fused-kernel layout
  __shared__ __attribute__((aligned(16))) int ent[kRecBytes / 4];
  __shared__ __attribute__((aligned(16))) float dt[kDMax * kDH];
  int* estart = ent;
  int* gbase = estart + 65;
  int* ecol = gbase + 64;
  float* ew = reinterpret_cast<float*>(ecol + kEMax);
  int* einfo = reinterpret_cast<int*>(ew + kEMax);
  const int* flag = einfo + kEMax;
  const int* gstart = flag + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  const int slab = blockIdx.x / p.tiles_per_lc;  // (role, layer), role-major
  const int t = blockIdx.x - slab * p.tiles_per_lc;
  Item it;
  it.c = slab / p.n_slab_layers;
  it.l = slab - it.c * p.n_slab_layers;
  int b = 0;
  while (b + 1 < p.B && p.tile_start[b + 1] <= t) ++b;
  it.b = b;
  it.tile = t - p.tile_start[b];
  Ctx cx;
  if (p.concat) {  // one sender layer, weight 1
    const uint16_t* Sb = static_cast<const uint16_t*>(p.S) + it.b * p.s_sb + it.c * p.s_sc;
    cx.S_lo = cx.S_hi = Sb + (long long)it.l * p.s_sl;
    cx.cs_s = (it.c == 0 && p.unrot) ? p.cs_s + (long long)p.pos0_s[it.b] * kDH : nullptr;
    cx.wlo = 1.0f;
    cx.whi = 0.0f;
    cx.two_tap = false;
    cx.Ts = p.Ts[it.b];
  } else {
    cx = make_ctx(p, it);
  }
  // Keys un-rotate at the sender positions when the call asks for it; values
  // never do (their context carries no sender table).
  const bool unrot = cx.cs_s != nullptr;
  copy16_to_lds(p.tile_rec + (long long)t * (kRecBytes / 4) + wave * 256 + 4 * lane, estart + wave * 256);
  if (unrot) {  // U(0..15): rows 0..15 of the sender table, 2 per wave
    const int ri = wave * 2 + (lane >> 5);
    const int c = (lane & 31) ^ (ri & 1);
    copy16_to_lds(p.cs_s + (long long)ri * kDH + 4 * c, dt + wave * 2 * kDH);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const int Tr = p.Tr[it.b];
  const int j0 = it.tile * 64;
  const int nrows = min(64, Tr - j0);
  const int g0 = p.row0[it.b] + j0;
  const LdsSink sink{xl};
  const int rt = p.rt_start[it.b] + (it.tile >> 2);
  uint16_t* dst = p.xs + slab * p.xs_slab + (long long)rt * (kStagedRows * kHMax * kDH) +
                  (it.tile & 3) * 64 * 32;
  const bool staged = p.s_extent > 0 && flag[1] == 0 && !(unrot && flag[0] != 0);
  if (staged) {  // eight sender heads: wave w builds head w
    const GroupLds L{estart, ecol, ew, einfo, dt, estart[0]};
    const int grp = lane >> 3;
    const int r_first = gstart[grp], rpg = gstart[grp + 1] - r_first, base = gbase[grp];
    if (cx.two_tap && unrot) build_groups<true, true, false, 3>(cx, p, L, base, wave, wave, r_first, rpg, lane, sink);
    else if (cx.two_tap) build_groups<true, false, false, 3>(cx, p, L, base, wave, wave, r_first, rpg, lane, sink);
    else if (unrot) build_groups<false, true, false, 3>(cx, p, L, base, wave, wave, r_first, rpg, lane, sink);
    else build_groups<false, false, false, 3>(cx, p, L, base, wave, wave, r_first, rpg, lane, sink);
    // The wave's own head (k-tiles 4 wave .. 4 wave + 3 of the 64 rows) goes
    // out as soon as its walk ends: LDS operations of one wave run in order.
    const int c8 = (lane & 3) * 8;
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
      const int kt = 4 * wave + (i >> 2), r = 16 * (i & 3) + (lane >> 2);
      nt_store16(dst + kt * (kStagedRows * 32) + r * 32 + c8, xl + r * kXF + kt * 32 + c8);
    }
  } else {
    const int r = tid >> 3;        // 8 threads per row
    const int e0 = (tid & 7) * 8;  // features e0..e0+7 and e0+64..e0+71 of every head
    for (int h = 0; h < kHMax; ++h) {
      float x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = 0.0f;
      if (r < nrows) build_row_global(p, cx, g0 + r, h, e0, x);
      sink(r, h * kDH + e0, pack8(x));
      sink(r, h * kDH + 64 + e0, pack8(x + 8));
    }
    __syncthreads();
    const int r2 = (tid & 255) >> 2, c8 = (tid & 3) * 8;
#pragma unroll 4
    for (int kt = tid >> 8; kt < kHMax * kDH / 32; kt += 2)
      nt_store16(dst + kt * (kStagedRows * 32) + r2 * 32 + c8, xl + r2 * kXF + kt * 32 + c8);
  }
}

}  // namespace

int transfer_rows_per_tile(int dtype, int H_r, int H_s, int n_taps, int d_h) {
  if (dtype == HF_BF16) return 64;
  return transfer_f32_rows_per_tile(H_s, n_taps, d_h);
}

// Shapes whose workspace holds the tile records and the work counter.
static bool uses_records(int dtype, int H_r, int H_s, int d_h) {
  return dtype == HF_BF16 && d_h == kDH && (H_r == 4 || H_r == 8) && H_s <= kHMax;
}

size_t transfer_tile_record_bytes(int dtype, int H_r, int H_s, int d_h) {
  return uses_records(dtype, H_r, H_s, d_h) ? kRecBytes : 0;
}

// In queues up to kQueueTiles row tiles, in plain order past that.  In plain order the
// tiles of a (layer, role) lie on all XCDs and each fetches the map (2 MB for 8 -> 8
// heads, half that for 8 -> 4 and 4 -> 8): 577, 1130 and 1905 MB fetched at 3, 7 and 14
// tiles for 168 MB of maps, and 249, 403 and 627 MB in queues.  Queued over plain
// kernel time at 3, 7, 14, 28, 56, 78, 100, 125, 167 and 223 tiles (200 to 16K tokens):
//   8 -> 8         .59 .69 .76 .81 .93 .97 .99 .98 1.00 1.00  (93 -> 55 us at 3 tiles)
//   8 -> 4         .74 .71 .90 .96 1.00 .98 1.00 .98 1.00 .99
//   4 -> 8         .70 .71 .86 .94 1.00 1.00 1.03 .99 1.01 1.01
//   2 -> 4         .83 .94 .98 .98 .98 .98 1.02 1.02 1.03 1.01
//   8 -> 4, 3 taps .74 .60 .81 .99 .99 1.00 1.03 1.00 1.00 .98
//   8 -> 2         .96 .89 .97 1.02 1.01 1.00 1.01 1.00 1.02 1.01
//   16 -> 8        .76 .63 .78 .90 .95 .97
// Runs differ by 1 to 2%.  On a second card whole calls of 8 -> 8 heads at 89, 100, 114
// and 125 tiles .97 .99 1.00 .98, of 4 -> 8 1.00 1.02 1.02 1.00, of 8 -> 4 .98 1.00 1.01
// .99; on a third 8 -> 8 at 115 tiles 1.03.  So the line lies where no shape loses.
// A kernel of one item per workgroup needs queues of one length.
constexpr int kQueueTiles = 96;

void transfer_order(TransferArgs& a) {
  const bool one_each = a.concat || a.H_s > kHMax || !uses_records(HF_BF16, a.H_r, a.H_s, a.d_h);
  const bool even = 2 * a.L_r % kQueues == 0;
  a.queued = a.tiles_per_lc <= kQueueTiles && (even || !one_each);
}

int transfer_persistent_grid(const TransferArgs& a, int n_cu) {
  const long long items = (long long)a.tiles_per_lc * a.L_r * 2;
  return (int)(items < n_cu ? items : n_cu);
}

hipError_t launch_prologue(int dtype, const TransferArgs& a, bool stage, const RopeTabs& tabs,
                           hipStream_t s) {
  int n_stage = 0;
  if (stage && uses_records(dtype, a.H_r, a.H_s, a.d_h)) {
    n_stage = a.tile_start[a.B];
    if (n_stage > 0 && (!a.tile_rec || !a.work_ctr || a.n_wg < 1)) return hipErrorInvalidValue;
  }
  RopeTabs r = tabs;
  const int half = a.d_h / 2, n_k = (half + 63) / 64;
  long long blocks = n_stage;
  for (int i = 0; i < r.n; ++i) {
    RopeTab& t = r.t[i];
    t.head = t.head < t.lo ? t.head : 0;  // rows [0, head) below the range
    if (t.head == 0 && tabs.t[i].head > 0) t.lo = 0;
    const int rows = t.head + (t.P - t.lo);
    // 16 rows share a w_k, fewer where that would leave the chip idle
    t.ppt = rows >= 16384 ? 16 : rows >= 4096 ? 4 : 1;
    t.blocks = n_k * ((rows + 8 * t.ppt - 1) / (8 * t.ppt));
    blocks += t.blocks;
  }
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(prologue_kernel, dim3((unsigned)blocks), dim3(512), 0, s, a,
                     const_cast<int*>(a.tile_rec), n_stage, r);
  return hipGetLastError();
}

hipError_t launch_pack_maps(int dtype, int n_lc, int d_r, int d_in, const void* A, void* A_packed,
                            hipStream_t s) {
  static_assert(HF_PACKED_HEADER_BYTES == 64 * 4, "header kernel writes 64 words");
  hipLaunchKernelGGL(pack_header_kernel, dim3(1), dim3(64), 0, s, static_cast<uint32_t*>(A_packed),
                     dtype, n_lc / 2, d_r, d_in);
  void* Wp = static_cast<char*>(A_packed) + HF_PACKED_HEADER_BYTES;
  if (dtype == HF_BF16) {
    const long long n = (long long)n_lc * (d_r / 32) * (d_in / 16) * 64;
    if (n > 0)
      hipLaunchKernelGGL(pack_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                         static_cast<const uint16_t*>(A), static_cast<uint4*>(Wp), n, d_r, d_in);
  } else {
    const long long n4 = (long long)n_lc * d_r * d_in / 4;
    if (n4 > 0)
      hipLaunchKernelGGL(copy_f32_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                         static_cast<const float4*>(A), static_cast<float4*>(Wp), n4);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of hf_transfer_kv_noalloc: the workspace of a transfer (RoPE
// tables, staged tile records, work counter) in a file-scope device array, so
// that the call allocates nothing.  Each device holds its own copy from module
// load until the process ends.  Host code never passes the array's name to a
// kernel: it resolves the device address once per device and uses that.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[HF_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* per_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(mu);
  if (!per_device[dev]) {  // first call on this device, with it current
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

bool staged_supported(int dtype, int H_s, int H_r, int d_h) {
  return dtype == HF_BF16 && d_h == kDH && H_s == kHMax && H_r == kHMax;
}

hipError_t launch_staged_build(const TransferArgs& a, hipStream_t s) {
  const long long items = (long long)a.tiles_per_lc * a.n_slab_layers * 2;
  if (items <= 0) return hipSuccess;
  if (!a.xs || !a.tile_rec || items > INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)items);
  hipLaunchKernelGGL(staged_build_kernel, grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_transfer(int dtype, const TransferArgs& a, hipStream_t s) {
  const long long items = (long long)a.tiles_per_lc * a.L_r * 2;
  if (items <= 0) return hipSuccess;
  const dim3 grid((unsigned)items);
  const bool rec = uses_records(dtype, a.H_r, a.H_s, a.d_h);
  if (rec && (!a.tile_rec || !a.work_ctr || a.n_wg < 1)) return hipErrorInvalidValue;
  const dim3 pgrid((unsigned)a.n_wg);  // persistent (interpolating map): one workgroup per CU
  const dim3 block(512);
  if (dtype == HF_BF16) {
    const bool multi = a.concat || a.H_s > kHMax;  // several passes over the X tile
#define HF_TILED(GRID, ...) \
  hipLaunchKernelGGL((transfer_bf16_tiled_kernel<__VA_ARGS__>), GRID, block, 0, s, a)
    if (rec && a.H_r == 8) {
      if (multi) HF_TILED(grid, 8, true, false, false);
      else if (a.queued) HF_TILED(pgrid, 8, false, false, true);
      else HF_TILED(pgrid, 8, false, false, false);
    } else if (rec) {
      if (multi) HF_TILED(grid, 4, true, false, false);
      else if (a.queued) HF_TILED(pgrid, 4, false, false, true);
      else HF_TILED(pgrid, 4, false, false, false);
    } else if (a.H_r == 8) {
      HF_TILED(grid, 8, true, true, false);
    } else if (a.H_r == 4) {
      HF_TILED(grid, 4, true, true, false);
    } else if (a.H_r == 2) {
      if (multi) HF_TILED(grid, 2, true, true, false);
      else HF_TILED(grid, 2, false, true, false);
#undef HF_TILED
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    return launch_transfer_f32(a, s);
  }
  return hipGetLastError();
}

}  // namespace hf
