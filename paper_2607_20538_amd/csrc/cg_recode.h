// Token rows with a non-finite channel, coded again after a three-plane encoder's range (one copy per
// translation unit).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cg_device.h"

namespace cg {
namespace {

// Set in a lane's flags where an encoder met a row to be coded again (not a flag of the interface)
constexpr int kFlagRecode = 1 << 16;

// Codes the bf16 token rows that have a non-finite (or huge, at least 2^100) channel by the binary32 FMA
// chain over the channel's own gauge group, with block ranges that leave NaN out.  The matrix cores take G
// in three planes: 0 times an infinity and infinities times planes of two signs are NaN where the chain
// gives the infinity, and products that span several groups carry them into the others.
// Encoders only note that there is such a row, and the workgroup runs this after its range: the same work
// inside the pipelined loop of the paged encoder, though hardly ever run, cost it 1.4 to 2.2 %.
//   x: the first row (bytes; pitch tstride), nrow <= 64 rows; Gh: the head's blocks [d / g][g][g];
//   codes, side: the cache's first row (per-token blocks of n channels); flagged (64) and z (d): LDS.
// All of the workgroup's threads, at least d of them; returns flags.
__device__ inline int recode_rows(const char* x, int64_t tstride, int nrow, int d, int n, int bits, const float* Gh,
                                  int g, uint8_t* codes, uint32_t* side, int* flagged, float* z) {
  const int tid = int(threadIdx.x), nb = d / n;
  int flags = 0;
  __syncthreads();  // what the LDS held is read
  if (tid < nrow) flagged[tid] = 0;
  __syncthreads();
  for (int idx = tid; idx < nrow * (d / 8); idx += int(blockDim.x)) {
    const int t = idx / (d / 8), c8 = idx - t * (d / 8);
    const uint4 v = *reinterpret_cast<const uint4*>(x + t * tstride + 16 * c8);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = (w[e] >> 7) & 0xffu, hi = (w[e] >> 23) & 0xffu;  // exponents
      if (lo >= 227u || hi >= 227u) flagged[t] = 1;
      if (lo == 255u || hi == 255u) flags |= CG_FLAG_NONFINITE;
    }
  }
  __syncthreads();
  for (int t = 0; t < nrow; ++t) {
    if (!flagged[t]) continue;
    if (tid < d) {
      const int r = tid / g;
      const float* row = Gh + size_t(r) * g * g + size_t(tid - r * g) * g;
      const uint16_t* xr = reinterpret_cast<const uint16_t*>(x + t * tstride) + r * g;
      float acc = 0.0f;
      for (int k = 0; k < g; ++k) acc = fmaf(row[k], bf16_to_f32(xr[k]), acc);
      z[tid] = acc;
    }
    __syncthreads();
    if (tid < nb) {
      const float* zb = z + tid * n;
      float mn = zb[0], mx = zb[0];
      for (int e = 1; e < n; ++e) {
        mn = fminf(mn, zb[e]);
        mx = fmaxf(mx, zb[e]);
      }
      const Side sd = make_side(mn, mx, bits);
      uint32_t* dst = reinterpret_cast<uint32_t*>(codes + size_t(t) * (d * bits / 8) + tid * (n * bits / 8));
      const float qmax = float((1 << bits) - 1);
      uint64_t acc = 0;
      int nbit = 0;
      for (int e = 0; e < n; ++e) {
        acc |= uint64_t(quantize(zb[e], sd.mn, sd.inv, qmax)) << nbit;
        nbit += bits;
        if (nbit >= 32) {
          *dst++ = uint32_t(acc);
          acc >>= 32;
          nbit -= 32;
        }
      }
      side[size_t(t) * nb + tid] = sd.word;
      flags |= sd.flags;
    }
    __syncthreads();
  }
  return flags;
}

}  // namespace
}  // namespace cg
