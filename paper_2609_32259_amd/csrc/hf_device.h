// Device helpers shared by the transfer kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "hf_internal.h"

namespace hf {

// ---------------------------------------------------------------------------
// Work decoding shared by the transfer kernels.  Work items run role-major,
// then layer, then sequence, then row tile, so the workgroups in flight at
// any time share one map A[l, c] (kept in L2) and the two sender layers it
// reads, and consecutive receiver layers reuse a sender layer.
// ---------------------------------------------------------------------------
struct Item {
  int c, l, b, tile;
};

__device__ __forceinline__ Item decode_item(const TransferArgs& p, int item) {
  Item it;
  const int lc = item / p.tiles_per_lc;
  int t = item - lc * p.tiles_per_lc;
  it.c = lc / p.L_r;
  it.l = lc - it.c * p.L_r;
  int b = 0;
  while (b + 1 < p.B && p.tile_start[b + 1] <= t) ++b;
  it.b = b;
  it.tile = t - p.tile_start[b];
  return it;
}

// Byte i of a kernel-argument byte array (lo, hi, taps), read as the aligned
// dword that holds it with a uniform index: gfx950 has no scalar byte loads,
// and a vector load here would wait (in order) for every load and store the
// workgroup still has in flight, such as the previous tile's receiver rows.
static_assert(offsetof(TransferArgs, lo) % 4 == 0 && offsetof(TransferArgs, hi) % 4 == 0 &&
                  offsetof(TransferArgs, taps) % 4 == 0,
              "layer-map byte arrays must be dword aligned");
__device__ __forceinline__ int arg_byte(const uint8_t* base, int i) {
  i = __builtin_amdgcn_readfirstlane(i);
  const uint32_t w = reinterpret_cast<const uint32_t*>(base)[i >> 2];
  return (int)((w >> (8 * (i & 3))) & 0xffu);
}

}  // namespace hf
