// fp32 transfer kernels: the definitions of the bf16 kernels (transfer.hip)
// with fp32 operands, fp32 sums throughout, and head sizes that are multiples of 4.
#include <hip/hip_runtime.h>

#include "hf_device.h"
#include "hf_internal.h"

namespace hf {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kF32Threads = 256;

// ---------------------------------------------------------------------------
// fp32 transfer kernel on the matrix cores (heads of up to 256 channels).
//
// One workgroup = 4 waves computes 32 receiver rows x one group of receiver
// heads (at most kF32Cols features) of one (layer, role).  The map row is
// walked in chunks of whole (tap, sender head) blocks, at most kF32Cols
// features: all threads build the chunk's aligned features X[32][chunk] in LDS
// from the tile's staged CSR entries, then each wave multiplies its 32-feature
// tiles by X with v_mfma_f32_32x32x2_f32 (the map as operand A straight from
// global memory, 8 consecutive inputs per lane; X as operand B, so a lane
// holds one receiver row).  The result goes through LDS once, where bias, key
// norm and RoPE see whole heads.
//
// What bounds it: at 24 -> 28 layers, 4 -> 2 heads of 64, 1,778 receiver rows,
// the products take 42 us at the 157 TFLOP/s of the fp32 matrix cores and the
// caches 33 us of memory traffic; the kernel takes 127 us there, 72 without the
// products and their map loads, 41 without the sender rows too.  One
// scalar FMA per two loads, with the map read down its columns and every
// feature behind a chain of three dependent loads (the kernel for larger heads
// below), takes 965 us.  On 340 -> 301 tokens, 4 -> 6 layers, 2 heads of 64:
// 13.5 against 111 us.
// 32 rows fill the instruction's 32 columns; kF32Cols keeps X and the result
// (which take turns in the same LDS) under 58 KB, so that two or three
// workgroups of a CU hide each other's loads.  Loading the first map values
// ahead of the build costs registers and with them one of three workgroups
// per CU (146 us).
// ---------------------------------------------------------------------------
constexpr int kF32Rows = 32;
constexpr int kF32Cols = 448;  // features of a chunk and of a head group
constexpr int kF32Ent = 256;   // CSR entries of a tile staged in LDS
constexpr int kF32MaxHead = 256;

struct F32Plan {
  int hg;      // receiver heads per workgroup
  int nb;      // (tap, sender head) blocks per chunk
  int stride;  // LDS row stride of X, floats
  int ystride; // LDS row stride of the result, floats
};

template <int VW>
struct VecF;
template <>
struct VecF<4> {
  typedef float4 T;
};
template <>
struct VecF<2> {
  typedef float2 T;
};

template <int VW>
__device__ __forceinline__ void ldv(const float* p, float (&v)[VW]) {
  const auto t = *reinterpret_cast<const typename VecF<VW>::T*>(p);
  const float* f = reinterpret_cast<const float*>(&t);
#pragma unroll
  for (int u = 0; u < VW; ++u) v[u] = f[u];
}
template <int VW>
__device__ __forceinline__ void stv(float* p, const float (&v)[VW]) {
  typename VecF<VW>::T t;
  float* f = reinterpret_cast<float*>(&t);
#pragma unroll
  for (int u = 0; u < VW; ++u) f[u] = v[u];
  *reinterpret_cast<typename VecF<VW>::T*>(p) = t;
}

// TPW: 32-feature tiles per wave.  VW: channels per lane of the build and the
// epilogue (4, or 2 where half a head is not a multiple of 4 channels).
template <int TPW, int VW>
__global__ __launch_bounds__(kF32Threads) void transfer_f32_kernel(const TransferArgs p,
                                                                   const F32Plan q) {
  extern __shared__ __attribute__((aligned(16))) float xs[];
  __shared__ int estart[kF32Rows + 1];
  __shared__ int ecol[kF32Ent];
  __shared__ float ew[kF32Ent];

  const Item it = decode_item(p, blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = p.d_h, half = d / 2, Q = half / VW;
  const int NV = p.n_taps * p.H_s;
  const int d_all = NV * d;
  const int j0 = it.tile * kF32Rows;
  const int Tr = p.Tr[it.b], Ts = p.Ts[it.b];
  const int nrows = min(kF32Rows, Tr - j0);
  const int g0 = p.row0[it.b] + j0;
  const int h0 = blockIdx.y * q.hg;           // first receiver head of the group
  const int nh = min(q.hg, p.H_r - h0);
  const int GF = nh * d;                      // features of the group
  const bool keys = it.c == 0;
  const bool unrot = keys && p.unrot, rot = keys && p.rot;
  const int lc = it.l * 2 + it.c;
  const float sr = p.inv_r ? p.inv_r[lc] : 1.0f;  // the map sees x / r
  const float wlo = p.wlo[it.l] * sr, whi = p.whi[it.l] * sr;
  const bool two_tap = p.whi[it.l] != 0.0f;

  // ---- the tile's CSR entries ----
  if (tid <= kF32Rows) estart[tid] = p.row_ptr[g0 + min(tid, nrows)];
  __syncthreads();
  const int e_base = estart[0];
  const int nnz = estart[nrows] - e_base;
  const bool staged = nnz <= kF32Ent;
  if (staged) {
    for (int k = tid; k < nnz; k += kF32Threads) {
      int lo = 0, hi = nrows;  // row r with estart[r] <= e_base + k < estart[r + 1]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (estart[mid] <= e_base + k) lo = mid; else hi = mid;
      }
      ecol[k] = min(max(p.col[e_base + k], 0), Ts - 1);
      ew[k] = (float)p.num[e_base + k] / (float)p.den[g0 + lo];
    }
    __syncthreads();
  }

  f32x16 acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int u = 0; u < 16; ++u) acc[i][u] = 0.0f;

  const float* Sb = static_cast<const float*>(p.S) + it.b * p.s_sb + it.c * p.s_sc;
  const float* csb = unrot ? p.cs_s + (long long)p.pos0_s[it.b] * d : nullptr;
  const float* W = static_cast<const float*>(p.Wp) + ((long long)lc * p.H_r + h0) * d * d_all;
  const float* wrow[TPW];  // this lane's map rows (rows past the group repeat its last one)
#pragma unroll
  for (int i = 0; i < TPW; ++i)
    wrow[i] = W + (long long)min(32 * (wave + 4 * i) + (lane & 31), GF - 1) * d_all;
  const int kh = 8 * (lane >> 5);  // the lane's 8 inputs of each 16

  for (int v0 = 0; v0 < NV; v0 += q.nb) {
    const int nb = min(q.nb, NV - v0);
    const int K = nb * d, Kp = (K + 15) & ~15;
    if (v0 > 0) __syncthreads();  // the previous chunk is read
    // ---- build: two heads of a tap at a time, the next entry's rows loading
    // while this entry's are summed ----
    for (int bi = 0; bi < nb;) {
      const int v = v0 + bi, t = v / p.H_s, h = v - t * p.H_s;
      const bool pair = bi + 1 < nb && h + 1 < p.H_s;
      const int lo = p.concat ? arg_byte(&p.taps[0][0], 3 * it.l + t) : arg_byte(p.lo, it.l);
      const int hi = p.concat ? lo : arg_byte(p.hi, it.l);
      const float* S_lo = Sb + (long long)lo * p.s_sl + h * p.s_sh;
      const float* S_hi = Sb + (long long)hi * p.s_sl + h * p.s_sh;
      const long long hstep = pair ? p.s_sh : 0;  // a lone head is read twice and stored once
      for (int u0 = tid; u0 < kF32Rows * Q; u0 += kF32Threads) {
        const int r = u0 / Q, f = (u0 - r * Q) * VW;
        struct Rows {  // one entry: sender rows of the two heads and their rotation
          float m[2][2][VW], n[2][2][VW], c[VW], s[VW], w;
        };
        float x[2][2][VW];
#pragma unroll
        for (int u = 0; u < VW; ++u) x[0][0][u] = x[0][1][u] = x[1][0][u] = x[1][1][u] = 0.0f;
        auto load = [&](Rows& z, int e) {
          int i;
          if (staged) {
            i = ecol[e - e_base];
            z.w = ew[e - e_base];
          } else {
            i = min(max(p.col[e], 0), Ts - 1);
            z.w = (float)p.num[e] / (float)p.den[g0 + r];
          }
          const long long off = (long long)i * p.s_st + f;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            ldv<VW>(S_lo + off + g * hstep, z.m[g][0]);
            ldv<VW>(S_lo + off + g * hstep + half, z.m[g][1]);
            if (two_tap) {
              ldv<VW>(S_hi + off + g * hstep, z.n[g][0]);
              ldv<VW>(S_hi + off + g * hstep + half, z.n[g][1]);
            }
          }
          if (unrot) {
            const float* cs = csb + (long long)i * d + f;
            ldv<VW>(cs, z.c);
            ldv<VW>(cs + half, z.s);
          }
        };
        auto add = [&](const Rows& z) {
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int u = 0; u < VW; ++u) {
              float m1 = wlo * z.m[g][0][u], m2 = wlo * z.m[g][1][u];
              if (two_tap) {
                m1 = fmaf(whi, z.n[g][0][u], m1);
                m2 = fmaf(whi, z.n[g][1][u], m2);
              }
              if (unrot) {
                const float u1 = fmaf(m1, z.c[u], m2 * z.s[u]);
                const float u2 = fmaf(m2, z.c[u], -m1 * z.s[u]);
                m1 = u1;
                m2 = u2;
              }
              x[g][0][u] = fmaf(z.w, m1, x[g][0][u]);
              x[g][1][u] = fmaf(z.w, m2, x[g][1][u]);
            }
        };
        const int e_end = r < nrows ? estart[r + 1] : 0;
        int e = r < nrows ? estart[r] : 0;
        if (e < e_end) {
          Rows z[2];
          load(z[0], e);
          for (; e < e_end; e += 2) {
            if (e + 1 < e_end) load(z[1], e + 1);
            add(z[0]);
            if (e + 1 < e_end) {
              if (e + 2 < e_end) load(z[0], e + 2);
              add(z[1]);
            }
          }
        }
        float* xr = xs + r * q.stride + bi * d + f;
        stv<VW>(xr, x[0][0]);
        stv<VW>(xr + half, x[0][1]);
        if (pair) {
          stv<VW>(xr + d, x[1][0]);
          stv<VW>(xr + d + half, x[1][1]);
        }
      }
      bi += pair ? 2 : 1;
    }
    if (Kp > K)  // the last 16 inputs of the chunk are completed with zeros
      for (int u = tid; u < kF32Rows * (Kp - K); u += kF32Threads) {
        const int r = u / (Kp - K);
        xs[r * q.stride + K + (u - r * (Kp - K))] = 0.0f;
      }
    __syncthreads();

    // ---- multiply: 16 inputs per step, lane half h holds inputs 8 h .. 8 h + 7 ----
    const int steps = Kp / 16;
    const float* xrow = xs + (lane & 31) * q.stride + kh;
    constexpr int R = TPW == 1 ? 4 : 2;  // steps of map values in flight
    float4 wr[R][TPW][2];
    auto load_w = [&](float4 (&dst)[TPW][2], int step) {
#pragma unroll
      for (int i = 0; i < TPW; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int k = 16 * step + kh + 4 * j;  // K is a multiple of 4
          dst[i][j] = k < K ? *reinterpret_cast<const float4*>(wrow[i] + v0 * d + k)
                            : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
#pragma unroll
    for (int s = 0; s < R; ++s) load_w(wr[s], s);
    for (int s0 = 0; s0 < steps; s0 += R) {
#pragma unroll
      for (int s = 0; s < R; ++s) {
        if (s0 + s < steps) {
          const float4 xa = *reinterpret_cast<const float4*>(xrow + 16 * (s0 + s));
          const float4 xb = *reinterpret_cast<const float4*>(xrow + 16 * (s0 + s) + 4);
          const float xv[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
              const float4 w4 = wr[s][i][u >> 2];
              const float wv = (u & 3) == 0 ? w4.x : (u & 3) == 1 ? w4.y : (u & 3) == 2 ? w4.z : w4.w;
              acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, xv[u], acc[i], 0, 0, 0);
            }
        }
        load_w(wr[s], s0 + s + R);
      }
    }
  }

  // ---- result through LDS: row j = lane & 31, features 8 (u / 4) + 4 (lane / 32) + u % 4 ----
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = 32 * (wave + 4 * i) + 8 * g + 4 * (lane >> 5);
      if (n < GF)  // GF is a multiple of 4
        *reinterpret_cast<float4*>(xs + (lane & 31) * q.ystride + n) =
            make_float4(acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]);
    }
  __syncthreads();

  float* Rb = static_cast<float*>(p.R) + it.b * p.r_sb + (long long)it.l * p.r_sl + it.c * p.r_sc;
  const float* bias = p.bias ? p.bias + ((long long)lc * p.H_r + h0) * d : nullptr;
  const float* knorm = (keys && p.k_norm) ? p.k_norm + (long long)it.l * d : nullptr;
  // Rows are whole-wave work: 32 nh Q units are a multiple of 64 wherever the
  // key norm is served (d_h 64 and 128: a head's Q units are Q consecutive lanes).
  const int per_row = nh * Q;
  for (int u0 = tid; u0 < kF32Rows * per_row; u0 += kF32Threads) {
    const int r = u0 / per_row, c0 = u0 - r * per_row;
    const int h = c0 / Q, f = (c0 - h * Q) * VW;
    float y1[VW], y2[VW];
    ldv<VW>(xs + r * q.ystride + h * d + f, y1);
    ldv<VW>(xs + r * q.ystride + h * d + f + half, y2);
    if (bias) {
      float b1[VW], b2[VW];
      ldv<VW>(bias + h * d + f, b1);
      ldv<VW>(bias + h * d + f + half, b2);
#pragma unroll
      for (int u = 0; u < VW; ++u) {
        y1[u] += b1[u];
        y2[u] += b2[u];
      }
    }
    if (knorm) {  // RMSNorm over the head's d features, held by Q consecutive lanes
      float ss = 0.0f;
#pragma unroll
      for (int u = 0; u < VW; ++u) ss = fmaf(y1[u], y1[u], fmaf(y2[u], y2[u], ss));
      for (int o = 1; o < Q; o <<= 1) ss += __shfl_xor(ss, o);
      const float inv = 1.0f / sqrtf(ss / (float)d + p.k_norm_eps);
#pragma unroll
      for (int u = 0; u < VW; ++u) {
        y1[u] *= inv * knorm[f + u];
        y2[u] *= inv * knorm[f + half + u];
      }
    }
    const int j = j0 + r;
    if (j >= Tr) continue;
    if (rot) {
      const float* cs = p.cs_r + (long long)(p.pos0_r[it.b] + j) * d + f;
      float c[VW], s[VW];
      ldv<VW>(cs, c);
      ldv<VW>(cs + half, s);
#pragma unroll
      for (int u = 0; u < VW; ++u) {
        const float u1 = fmaf(y1[u], c[u], -y2[u] * s[u]);
        const float u2 = fmaf(y2[u], c[u], y1[u] * s[u]);
        y1[u] = u1;
        y2[u] = u2;
      }
    }
    float* dst = Rb + (long long)(h0 + h) * p.r_sh + (long long)j * p.r_st + f;
    stv<VW>(dst, y1);
    stv<VW>(dst + half, y2);
  }
}

// ---------------------------------------------------------------------------
// fp32 transfer kernel for heads of more than 256 channels, whose features
// outgrow the tile above: plain FMA, one workgroup = RT receiver rows of one
// (layer, role).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kF32Threads) void transfer_f32_plain_kernel(const TransferArgs p) {
  extern __shared__ float xs[];  // [RT][d_in]
  const Item it = decode_item(p, blockIdx.x);
  const int RT = p.rows_per_tile;
  const int d = p.d_h, half = d / 2;
  const int NV = p.n_taps * p.H_s;  // (tap, sender head) blocks of the map row
  const int d_in = NV * d, d_r = p.H_r * d;
  const int j0 = it.tile * RT;
  const int Tr = p.Tr[it.b], Ts = p.Ts[it.b];
  const bool keys = it.c == 0;
  const bool unrot = keys && p.unrot, rot = keys && p.rot;
  const float sr = p.inv_r ? p.inv_r[it.l * 2 + it.c] : 1.0f;  // the map sees x / r
  const float wlo = p.wlo[it.l] * sr, whi = p.whi[it.l] * sr;
  const bool two_tap = p.whi[it.l] != 0.0f;
  const float* Sb = static_cast<const float*>(p.S) + it.b * p.s_sb + it.c * p.s_sc;
  const int lc_store = it.l * 2 + it.c;

  for (int idx = threadIdx.x; idx < RT * NV * half; idx += kF32Threads) {
    const int r = idx / (NV * half);
    const int rem = idx - r * (NV * half);
    const int vh = rem / half, f = rem - vh * half;
    const int h = vh % p.H_s, t = vh / p.H_s;
    const int lo = p.concat ? p.taps[it.l][t] : p.lo[it.l];
    const float* S_lo = Sb + (long long)lo * p.s_sl;
    const float* S_hi = Sb + (long long)(p.concat ? lo : p.hi[it.l]) * p.s_sl;
    const int j = j0 + r;
    float x1 = 0.f, x2 = 0.f;
    if (j < Tr) {
      const int g = p.row0[it.b] + j;
      const float dinv = (float)p.den[g];
      for (int e = p.row_ptr[g]; e < p.row_ptr[g + 1]; ++e) {
        int i = min(max(p.col[e], 0), Ts - 1);
        const float w = (float)p.num[e] / dinv;
        const long long off = h * p.s_sh + (long long)i * p.s_st + f;
        float m1 = wlo * S_lo[off], m2 = wlo * S_lo[off + half];
        if (two_tap) {
          m1 = fmaf(whi, S_hi[off], m1);
          m2 = fmaf(whi, S_hi[off + half], m2);
        }
        if (unrot) {
          const float* cs = p.cs_s + (long long)(p.pos0_s[it.b] + i) * d;
          const float c = cs[f], s = cs[half + f];
          const float u1 = fmaf(m1, c, m2 * s);
          const float u2 = fmaf(m2, c, -m1 * s);
          m1 = u1;
          m2 = u2;
        }
        x1 = fmaf(w, m1, x1);
        x2 = fmaf(w, m2, x2);
      }
    }
    xs[r * d_in + vh * d + f] = x1;
    xs[r * d_in + vh * d + f + half] = x2;
  }
  __syncthreads();

  const float* W = static_cast<const float*>(p.Wp) + (long long)lc_store * d_r * d_in;
  float* Rb = static_cast<float*>(p.R) + it.b * p.r_sb + (long long)it.l * p.r_sl + it.c * p.r_sc;
  constexpr int kMaxRT = 16;
  const float* knorm = (keys && p.k_norm) ? p.k_norm + (long long)it.l * d : nullptr;
  // Every thread takes the same number of trips (pc past the end computes
  // nothing and stores nothing), so the key norm's shuffles see whole waves;
  // the half = d/2 threads of one receiver head are consecutive lanes.
  for (int pc0 = 0; pc0 < p.H_r * half; pc0 += kF32Threads) {
    const int pc = pc0 + threadIdx.x;
    const bool live = pc < p.H_r * half;
    const int hr = live ? pc / half : 0, f = live ? pc - hr * half : 0;
    const int n1 = hr * d + f, n2 = n1 + half;
    float y1[kMaxRT], y2[kMaxRT];
#pragma unroll
    for (int r = 0; r < kMaxRT; ++r) y1[r] = y2[r] = 0.f;
    const float* W1 = W + (long long)n1 * d_in;
    const float* W2 = W + (long long)n2 * d_in;
    for (int k = 0; k < (live ? d_in : 0); ++k) {
      const float a1 = W1[k], a2 = W2[k];
#pragma unroll
      for (int r = 0; r < kMaxRT; ++r) {
        if (r < RT) {
          const float xv = xs[r * d_in + k];
          y1[r] = fmaf(a1, xv, y1[r]);
          y2[r] = fmaf(a2, xv, y2[r]);
        }
      }
    }
    const float b1 = (p.bias && live) ? p.bias[(long long)lc_store * d_r + n1] : 0.f;
    const float b2 = (p.bias && live) ? p.bias[(long long)lc_store * d_r + n2] : 0.f;
    const float g1 = knorm ? knorm[f] : 1.f, g2 = knorm ? knorm[f + half] : 1.f;
#pragma unroll
    for (int r = 0; r < kMaxRT; ++r) {
      const int j = j0 + r;
      if (r >= RT) continue;  // uniform: the shuffles below stay whole-wave
      float v1 = y1[r] + b1, v2 = y2[r] + b2;
      if (knorm) {  // RMSNorm over the head's d features, held by half lanes
        float ss = fmaf(v1, v1, v2 * v2);
        for (int o = 1; o < half; o <<= 1) ss += __shfl_xor(ss, o);
        const float inv = 1.0f / sqrtf(ss / (float)d + p.k_norm_eps);
        v1 *= inv * g1;
        v2 *= inv * g2;
      }
      if (!live || j >= Tr) continue;
      if (rot) {
        const float* cs = p.cs_r + (long long)(p.pos0_r[it.b] + j) * d;
        const float c = cs[f], s = cs[half + f];
        const float u1 = fmaf(v1, c, -v2 * s);
        const float u2 = fmaf(v2, c, v1 * s);
        v1 = u1;
        v2 = u2;
      }
      float* dst = Rb + hr * p.r_sh + (long long)j * p.r_st;
      dst[f] = v1;
      dst[f + half] = v2;
    }
  }
}

bool f32_on_matrix_cores(int d_h) { return d_h <= kF32MaxHead; }

template <int VW>
void launch_f32(int tpw, dim3 grid, size_t lds, hipStream_t s, const TransferArgs& a,
                const F32Plan& q) {
  if (tpw <= 1)
    hipLaunchKernelGGL((transfer_f32_kernel<1, VW>), grid, dim3(kF32Threads), lds, s, a, q);
  else if (tpw <= 2)
    hipLaunchKernelGGL((transfer_f32_kernel<2, VW>), grid, dim3(kF32Threads), lds, s, a, q);
  else
    hipLaunchKernelGGL((transfer_f32_kernel<4, VW>), grid, dim3(kF32Threads), lds, s, a, q);
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

}  // namespace

int transfer_f32_rows_per_tile(int H_s, int n_taps, int d_h) {
  if (f32_on_matrix_cores(d_h)) return kF32Rows;
  const int d_in = n_taps * H_s * d_h;
  int rt = 8192 / (d_in > 0 ? d_in : 1);  // fp32 X tile <= 32 KB of LDS
  return rt < 1 ? 1 : (rt > 16 ? 16 : rt);
}

hipError_t launch_transfer_f32(const TransferArgs& a, hipStream_t s) {
  const long long items = (long long)a.tiles_per_lc * a.L_r * 2;
  if (items <= 0) return hipSuccess;
  const int NV = a.n_taps * a.H_s;
  if (!f32_on_matrix_cores(a.d_h)) {
    const size_t shmem = (size_t)a.rows_per_tile * NV * a.d_h * sizeof(float);
    hipLaunchKernelGGL(transfer_f32_plain_kernel, dim3((unsigned)items), dim3(kF32Threads), shmem,
                       s, a);
    return hipGetLastError();
  }
  F32Plan q;
  // whole heads per group and per chunk, in equal shares
  const int most = kF32Cols / a.d_h;  // >= 1
  const int groups = ceil_div(a.H_r, most);
  q.hg = ceil_div(a.H_r, groups);
  q.nb = ceil_div(NV, ceil_div(NV, most));
  // a row stride of 4 mod 16 floats spreads 16 rows over all LDS banks
  q.stride = (q.nb * a.d_h + 15) / 16 * 16 + 4;
  q.ystride = (q.hg * a.d_h + 15) / 16 * 16 + 4;
  const size_t lds = (size_t)kF32Rows * (q.stride > q.ystride ? q.stride : q.ystride) * 4;
  const dim3 grid((unsigned)items, (unsigned)ceil_div(a.H_r, q.hg));
  const int tpw = ceil_div(ceil_div(q.hg * a.d_h, 32), 4);
  if ((a.d_h / 2) % 4 == 0) launch_f32<4>(tpw, grid, lds, s, a, q);
  else launch_f32<2>(tpw, grid, lds, s, a, q);
  return hipGetLastError();
}

}  // namespace hf
