// Device parts shared by the general kernels (encode, decode, rolling append): the binary32 gauge
// of a tile of tokens and the block quantiser (one copy per translation unit).
#pragma once

#include <type_traits>

#include "cg_internal.h"
#include "cg_device.h"

namespace cg {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ size_t gauge_block(int l, int s, int h, int r, int H, int R) {
  return ((size_t(l) * 2 + s) * H + h) * R + r;
}

// Channels off .. off + 7 of a view row as loaded (16-byte aligned: rows and channel offsets are), and
// their binary32 values
struct Raw8 {
  uint4 v[2];
};
template <bool BF16>
__device__ __forceinline__ Raw8 load_raw8(const void* ptr, size_t off) {
  Raw8 r;
  if constexpr (BF16) {
    r.v[0] = *reinterpret_cast<const uint4*>((const uint16_t*)ptr + off);
    r.v[1] = make_uint4(0u, 0u, 0u, 0u);
  } else {
    r.v[0] = *reinterpret_cast<const uint4*>((const float*)ptr + off);
    r.v[1] = *reinterpret_cast<const uint4*>((const float*)ptr + off + 4);
  }
  return r;
}
__device__ __forceinline__ void raw8_values(const Raw8& r, bool bf16, float (&x)[8]) {
  const uint32_t w[8] = {r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w, r.v[1].x, r.v[1].y, r.v[1].z, r.v[1].w};
#pragma unroll
  for (int e = 0; e < 8; ++e)
    x[e] = __uint_as_float(bf16 ? ((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16)) : w[e]);
}

// LDS row pitch of the token tiles (floats): rows stay 16-byte aligned for vector accesses, and
// d + 4 is an odd multiple of 4 (d is a multiple of 8), so the 16 rows x 4 words of a matrix-core
// operand read fall into 64 distinct banks
constexpr int kPad = 4;

// ------------------------------------------------------------------------------------------
// gauge on the vector ALU: groups the matrix-core variant does not take
// ------------------------------------------------------------------------------------------
// zs[t][i] = sum_j G_{l,s,h,r}[i%g][j] xs[t][r*g + j] for t < ntok: one binary32 FMA chain per
// element in increasing j.  With g a multiple of 4 each thread computes a 4-token x 4-channel
// block, reading 4 consecutive j of 4 rows of G and of 4 token rows per step (16-byte loads).
__device__ void gauge_tile(const float* xs, float* zs, int ntok, int d, int dp, const GaugeDev& G, int l, int s,
                           int h) {
  const int g = G.g;
  if (g % 4) {
    for (int idx = threadIdx.x; idx < ntok * d; idx += blockDim.x) {
      const int t = idx / d, i = idx - t * d;
      const int r = i / g, ii = i - r * g;
      const float* Gr = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + size_t(ii) * g;
      const float* xr = xs + t * dp + r * g;
      float acc = 0.0f;
      for (int j = 0; j < g; ++j) acc = fmaf(Gr[j], xr[j], acc);
      zs[t * dp + i] = acc;
    }
    return;
  }
  const int ntb = (ntok + 3) / 4, ncb = d / 4;
  for (int idx = threadIdx.x; idx < ntb * ncb; idx += blockDim.x) {
    const int tb = idx / ncb, cb = idx - tb * ncb;
    const int t0 = 4 * tb, i0 = 4 * cb, r = i0 / g;
    const float* Gb = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + size_t(i0 - r * g) * g;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float acc[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[t][a] = 0.0f;
    for (int j = 0; j < g; j += 4) {
      float4 gv[4], xv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) gv[a] = *reinterpret_cast<const float4*>(Gb + size_t(a) * g + j);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        xv[t] = t0 + t < ntok ? *reinterpret_cast<const float4*>(xs + (t0 + t) * dp + r * g + j) : zero;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          acc[t][a] = fmaf(gv[a].x, xv[t].x, acc[t][a]);
          acc[t][a] = fmaf(gv[a].y, xv[t].y, acc[t][a]);
          acc[t][a] = fmaf(gv[a].z, xv[t].z, acc[t][a]);
          acc[t][a] = fmaf(gv[a].w, xv[t].w, acc[t][a]);
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t0 + t < ntok) *reinterpret_cast<float4*>(zs + (t0 + t) * dp + i0) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
  }
}

// ------------------------------------------------------------------------------------------
// gauge on the binary32 matrix cores
// ------------------------------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one fused multiply-add after
// the other in increasing k, so a chain of them over a group gives, bit for bit, the binary32 FMA
// chain of gauge_tile.  Lane (m = lane % 16, q = lane / 16) holds A = row m at k = q, B = column
// m at k = q and four results: column m, rows 4q .. 4q + 3.  Rows are 16 output channels of one
// group, columns 16 tokens.  A wave owns up to NBW consecutive channel blocks and keeps their
// rows of G in registers (A[j][k]: step k of block j, g = 4 KR) for all of its tokens.
typedef float f32x4_mat __attribute__((ext_vector_type(4)));

// Which blocks of 16 channels and of 16 tokens a wave takes: NBW consecutive channel blocks; heads
// of at most 32 channels leave waves over, which split the tokens.
struct WaveTile {
  int cb0, ncb;      // first channel block, channel blocks (none: the wave is idle)
  int tb0, tstep;    // token blocks tb0, tb0 + tstep, ...
  int last;          // last channel block of the head: a wave with fewer than NBW repeats it
};
template <int NBW>
__device__ __forceinline__ WaveTile wave_tile(int d) {
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), nc = d / 16;
  WaveTile t;
  t.last = nc - 1;
  if (NBW == 1 && nc <= 2) {
    t.cb0 = w & (nc - 1);
    t.ncb = 1;
    t.tb0 = nc == 2 ? w >> 1 : w;
    t.tstep = 4 / nc;
  } else {
    t.cb0 = w * NBW;
    t.ncb = max(0, min(NBW, nc - t.cb0));
    t.tb0 = 0;
    t.tstep = 1;
  }
  return t;
}

// 4 x 4 transpose between the four 16-lane rows of a wave and four registers: v[e] of lane row i
// becomes v[i] of lane row e
__device__ __forceinline__ void row_transpose4(uint32_t (&v)[4]) {
  const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto e = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  v[0] = c[0]; v[1] = c[1]; v[2] = e[0]; v[3] = e[1];
}

// A[j][k] = G[row m of block j][4k + q].  The 16-byte loads along the rows come first, with no branch
// between them, so that all are in flight together (and beside the caller's loads); the transpose
// between the lane rows follows where the operands are needed.
template <int KR, int NBW>
struct GaugeRaw {
  uint4 v[NBW][KR / 4];
};
template <int KR, int NBW>
__device__ __forceinline__ void load_gauge_rows(GaugeRaw<KR, NBW>& raw, const GaugeDev& G, int l, int s, int h,
                                                const WaveTile& wt) {
  constexpr int g = 4 * KR;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    const int i0 = 16 * min(wt.cb0 + j, wt.last), r = i0 / g;
    const float* row = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + size_t(i0 - r * g + m) * g + 4 * q;
#pragma unroll
    for (int kk = 0; kk < KR / 4; ++kk) raw.v[j][kk] = *reinterpret_cast<const uint4*>(row + 16 * kk);
  }
}
template <int KR, int NBW>
__device__ __forceinline__ void gauge_operand(const GaugeRaw<KR, NBW>& raw, float (&A)[NBW][KR]) {
#pragma unroll
  for (int j = 0; j < NBW; ++j)
#pragma unroll
    for (int kk = 0; kk < KR / 4; ++kk) {
      uint32_t v[4] = {raw.v[j][kk].x, raw.v[j][kk].y, raw.v[j][kk].z, raw.v[j][kk].w};
      row_transpose4(v);
#pragma unroll
      for (int u = 0; u < 4; ++u) A[j][4 * kk + u] = __uint_as_float(v[u]);
    }
}

// The same operand of G^T (the inverse gauge): A[j][k] = G[4k + q][column m of block j], 16 neighbouring
// columns of a row per 16 lanes
template <int KR, int NBW>
struct GaugeCols {
  float v[NBW][KR];
};
template <int KR, int NBW>
__device__ __forceinline__ void load_gauge_cols(float (&A)[NBW][KR], const GaugeDev& G, int l, int s, int h,
                                                const WaveTile& wt) {
  constexpr int g = 4 * KR;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    const int i0 = 16 * min(wt.cb0 + j, wt.last), r = i0 / g;
    const float* col = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + size_t(q) * g + (i0 - r * g + m);
#pragma unroll
    for (int kk = 0; kk < KR; ++kk) A[j][kk] = col[size_t(4 * kk) * g];
  }
}

// out[t][i] = sum_k A_i[k] in[t][r g + k] for the wave's channel blocks and token blocks
// tb < ntb (rows 16 ntb of both tiles are addressed)
template <int KR, int NBW>
__device__ __forceinline__ void gauge_mfma(const float (&A)[NBW][KR], const float* in, float* out, int ntb, int dp,
                                           const WaveTile& wt) {
  constexpr int g = 4 * KR;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  if (wt.ncb == 0) return;
  int off[NBW];  // first channel of each block's group
#pragma unroll
  for (int j = 0; j < NBW; ++j) off[j] = 16 * min(wt.cb0 + j, wt.last) / g * g;
  // blocks of one wave share their group when a group holds all of them (operands read once)
  const bool same = g >= 16 * NBW && off[0] == off[NBW - 1];
  for (int tb = wt.tb0; tb < ntb; tb += wt.tstep) {
    const float* row = in + (16 * tb + m) * dp + q;
    f32x4_mat acc[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j) acc[j] = f32x4_mat{0.0f, 0.0f, 0.0f, 0.0f};
    if (NBW == 1 || same) {
      const float* rj = row + off[0];
#pragma unroll
      for (int k0 = 0; k0 < KR; k0 += 16) {  // up to 16 operand reads in flight
        float b[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (k0 + k < KR) b[k] = rj[4 * (k0 + k)];
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (k0 + k < KR) {
#pragma unroll
            for (int j = 0; j < NBW; ++j)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[j][k0 + k], b[k], acc[j], 0, 0, 0);
          }
      }
    } else {
#pragma unroll
      for (int k = 0; k < KR; ++k)
#pragma unroll
        for (int j = 0; j < NBW; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[j][k], row[off[j] + 4 * k], acc[j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < NBW; ++j)
      if (j < wt.ncb)
        *reinterpret_cast<float4*>(out + (16 * tb + m) * dp + 16 * (wt.cb0 + j) + 4 * q) =
            make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
  }
}

// ------------------------------------------------------------------------------------------
// gauge on the bf16 matrix cores: bf16 tokens, groups that are a multiple of 32 channels
// ------------------------------------------------------------------------------------------
// x is exact in bf16 and G = G0 + G1 + G2 to 24 significant bits, so three products of
// v_mfma_f32_16x16x32_bf16 per 32 channels give z closer to the binary64 product than the binary32
// chain (relative error 1.2e-7 against 2.0e-7 at g = 128, 0.7e-7 against 1.0e-7 at g = 32) in 3/16 of the
// matrix-core time.  Lane (m, q) holds A = row m and B = column m at k = 8q .. 8q + 7, and the same
// results as the binary32 step.
typedef __bf16 bf16x8_gen __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_gen __attribute__((ext_vector_type(4)));

template <int KK, int NBW>  // g = 32 KK
struct GaugePlanes {
  u32x4_gen v[NBW][KK][3];
};
template <int KK, int NBW>
__device__ __forceinline__ void load_gauge_planes(GaugePlanes<KK, NBW>& A, const GaugeDev& G, int l, int s, int h,
                                                  const WaveTile& wt) {
  constexpr int g = 32 * KK;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
#pragma unroll
  for (int j = 0; j < NBW; ++j) {
    const int i0 = 16 * min(wt.cb0 + j, wt.last), r = i0 / g;
    const size_t off = gauge_block(l, s, h, r, G.H, G.R) * g * g + size_t(i0 - r * g + m) * g + 8 * q;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int p = 0; p < 3; ++p) A.v[j][kk][p] = *reinterpret_cast<const u32x4_gen*>(G.hi[p] + off + 32 * kk);
  }
}
// bytes between token rows of the staged bf16 tile: rows stay 16-byte aligned and start 4 banks apart
__device__ __host__ __forceinline__ int bf16_pitch(int d) { return 2 * d + 16; }

// out[t][i] = sum_k G_i[k] in[t][r g + k], in: the bf16 tile (pitch bf16_pitch), out: binary32 (pitch dp)
template <int KK, int NBW>
__device__ __forceinline__ void gauge_planes_mfma(const GaugePlanes<KK, NBW>& A, const uint8_t* in, float* out, int ntb,
                                                  int d, int dp, const WaveTile& wt) {
  constexpr int g = 32 * KK;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  if (wt.ncb == 0) return;
  int off[NBW];  // first byte of each block's group
#pragma unroll
  for (int j = 0; j < NBW; ++j) off[j] = 2 * (16 * min(wt.cb0 + j, wt.last) / g * g) + 16 * q;
  for (int tb = wt.tb0; tb < ntb; tb += wt.tstep) {
    const uint8_t* row = in + (16 * tb + m) * bf16_pitch(d);
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
      f32x4_mat acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8_gen b = __builtin_bit_cast(bf16x8_gen, *reinterpret_cast<const u32x4_gen*>(row + off[j] + 64 * kk));
#pragma unroll
        for (int p = 0; p < 3; ++p)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_gen, A.v[j][kk][p]), b, acc, 0, 0, 0);
      }
      if (j < wt.ncb)
        *reinterpret_cast<float4*>(out + (16 * tb + m) * dp + 16 * (wt.cb0 + j) + 4 * q) =
            make_float4(acc[0], acc[1], acc[2], acc[3]);
    }
  }
}

// idx / c for 0 <= idx < 2^14, 1 <= c <= 32, inv = 1.0f / c: (idx + 1/2) / c lies at least 1/64 from
// an integer and the product is off by less than 2^-8
__device__ __forceinline__ int small_div(int idx, float inv) { return int((float(idx) + 0.5f) * inv); }

// ------------------------------------------------------------------------------------------
// block quantiser
// ------------------------------------------------------------------------------------------
// Quantise n values (stride `stride` in LDS) as one block and write its packed stream and
// side word.  n * bits is a multiple of 32.
__device__ int quantize_block_to(const float* z, int stride, int n, int bits, uint32_t* dst, uint32_t* side_dst) {
  float mn = z[0], mx = z[0];
  for (int e = 1; e < n; ++e) {
    mn = fminf(mn, z[e * stride]);
    mx = fmaxf(mx, z[e * stride]);
  }
  Side sd = make_side(mn, mx, bits);
  const float qmax = (float)((1 << bits) - 1);
  uint64_t acc = 0;
  int nbit = 0, wi = 0;
  for (int e = 0; e < n; ++e) {
    acc |= (uint64_t)quantize(z[e * stride], sd.mn, sd.inv, qmax) << nbit;
    nbit += bits;
    if (nbit >= 32) {
      dst[wi++] = (uint32_t)acc;
      acc >>= 32;
      nbit -= 32;
    }
  }
  *side_dst = sd.word;
  return sd.flags;
}

// Blocks of 8, 16, ... 256 channels (a power of two) are quantised by n / 8 neighbouring lanes, 8
// channels each (quantise_rows below); others by one thread per block.
__device__ __host__ __forceinline__ bool lane_blocks(int n) { return n >= 8 && n <= 256 && (n & (n - 1)) == 0; }

// (min, max) of a lane and the lane a DPP control brings (a lane of the same 16-lane row)
template <int CTRL>
__device__ __forceinline__ void lane_range(float& mn, float& mx) {
  mn = fminf(mn, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(mn), CTRL, 0xF, 0xF, true)));
  mx = fmaxf(mx, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(mx), CTRL, 0xF, 0xF, true)));
}

// quantize() in four instructions: the clamp to [0, qmax] (whole numbers) commutes with the rounding to
// nearest even that v_cvt_pk_u8_f32 does
__device__ __forceinline__ uint32_t quantize_u8(float z, float mn, float inv, float qmax) {
  return code_u8(fminf(fmaxf(quantize_t(z, mn, inv), 0.0f), qmax));
}

// Rows [0, ntok) of a tile, bt = 1: one range per row and block of n channels (lane_blocks(n));
// bt > 1: one range per bt rows and block (ntok a multiple of bt).  A lane takes 8 channels, the
// lanes of a block exchange their ranges, and the 8 codes leave as `bits` bytes of the packed row
// in LDS (cst, row pitch d bits / 8).  live(t): whether row t is stored; side(t, kb): where the
// side word of row t's block kb goes (bt > 1: asked for the first row of a tile).  red: LDS,
// ntok d / n pairs (bt > 1 only).  Ranges are the same minimum and maximum as
// quantize_block_to's (fminf / fmaxf skip a NaN in any order), so the results are.
template <class Live, class SideAt>
__device__ int quantise_rows(const float* zs, int ntok, int d, int dp, int n, int bits, int bt, float2* red,
                             uint8_t* cst, Live live, SideAt side) {
  int flags = 0;
  const int c8n = d / 8, lg = n / 8, nb = d / n, lsh = 31 - __builtin_clz(lg);
  const float inv8 = 1.0f / float(c8n);
  const float qmax = (float)((1 << bits) - 1);
  auto finish = [&](int t, int c8, const float (&z)[8], float mn, float mx) {
    const Side sd = make_side<true>(mn, mx, bits);
    uint32_t half[2];  // four codes each (at most 32 bits)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t q[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = quantize_u8(z[4 * u + e], sd.mn, sd.inv, qmax);
      half[u] = q[0] | (q[1] << bits) | ((q[2] | (q[3] << bits)) << (2 * bits));
    }
    const uint64_t acc = half[0] | (uint64_t(half[1]) << (4 * bits));
    uint8_t* dst = cst + (t * c8n + c8) * bits;
    switch (bits) {
      case 2: *reinterpret_cast<uint16_t*>(dst) = (uint16_t)acc; break;
      case 3:
        dst[0] = (uint8_t)acc;
        dst[1] = (uint8_t)(acc >> 8);
        dst[2] = (uint8_t)(acc >> 16);
        break;
      case 4: *reinterpret_cast<uint32_t*>(dst) = (uint32_t)acc; break;
      case 6:
        reinterpret_cast<uint16_t*>(dst)[0] = (uint16_t)acc;
        reinterpret_cast<uint16_t*>(dst)[1] = (uint16_t)(acc >> 16);
        reinterpret_cast<uint16_t*>(dst)[2] = (uint16_t)(acc >> 32);
        break;
      default: *reinterpret_cast<uint64_t*>(dst) = acc; break;
    }
    if ((c8 & (lg - 1)) == 0 && (t & (bt - 1)) == 0) *side(t, c8 >> lsh) = sd.word;
    flags |= sd.flags;
  };
  auto read8 = [&](int t, int c8, float (&z)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(zs + t * dp + 8 * c8);
    const float4 b = *reinterpret_cast<const float4*>(zs + t * dp + 8 * c8 + 4);
    z[0] = a.x; z[1] = a.y; z[2] = a.z; z[3] = a.w;
    z[4] = b.x; z[5] = b.y; z[6] = b.z; z[7] = b.w;
  };
  for (int idx = threadIdx.x; idx < ntok * c8n; idx += blockDim.x) {
    const int t = small_div(idx, inv8), c8 = idx - t * c8n;
    float z[8];
    read8(t, c8, z);
    float mn = z[0], mx = z[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) {
      mn = fminf(mn, z[e]);
      mx = fmaxf(mx, z[e]);
    }
    // the lanes of a block are neighbours of one wave (idx is aligned to lg) and active together;
    // once the lanes of a quad agree, a mirror of 8 (16) lanes brings the other quad's (half's) value
    if (lg >= 2) lane_range<0xB1>(mn, mx);    // quad_perm [1,0,3,2]
    if (lg >= 4) lane_range<0x4E>(mn, mx);    // quad_perm [2,3,0,1]
    if (lg >= 8) lane_range<0x141>(mn, mx);   // row_half_mirror
    if (lg >= 16) lane_range<0x140>(mn, mx);  // row_mirror
    if (lg >= 32) {
      mn = fminf(mn, __shfl_xor(mn, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
    }
    if (bt > 1) {
      if ((c8 & (lg - 1)) == 0) red[t * nb + (c8 >> lsh)] = make_float2(mn, mx);
    } else if (live(t)) {
      finish(t, c8, z, mn, mx);
    }
  }
  if (bt > 1) {
    __syncthreads();
    for (int idx = threadIdx.x; idx < ntok * c8n; idx += blockDim.x) {
      const int t = small_div(idx, inv8), c8 = idx - t * c8n;
      const float2* rr = red + (t & -bt) * nb + (c8 >> lsh);
      float mn = rr[0].x, mx = rr[0].y;
      for (int v = 1; v < bt; ++v) {
        mn = fminf(mn, rr[v * nb].x);
        mx = fmaxf(mx, rr[v * nb].y);
      }
      float z[8];
      read8(t, c8, z);
      if (live(t)) finish(t, c8, z, mn, mx);
    }
  }
  return flags;
}

// Block-uniform (or KIVI value) rows: tile rows t < ntok go to cache positions pos0 + t.
__device__ int store_rows_blocks(const float* zs, int ntok, int d, int dp, int n, int bits, const CacheDev& k,
                                 size_t slc, int pos0) {
  int flags = 0;
  const int nb = d / n, row_bytes = d * bits / 8, blk_bytes = n * bits / 8;
  for (int w = threadIdx.x; w < ntok * nb; w += blockDim.x) {
    const int t = w / nb, kb = w - t * nb;
    const size_t row = slc * k.T_cap + pos0 + t;
    uint32_t* dst = (uint32_t*)(k.codes + row * row_bytes + size_t(kb) * blk_bytes);
    flags |= quantize_block_to(zs + t * dp + kb * n, 1, n, bits, dst, k.side + row * nb + kb);
  }
  return flags;
}

// Block-uniform token-channel tiles: tile rows [u*bt, u*bt + bt) form tile (pos0 / bt) + u; one
// (tile, channel block) per thread takes the range of its bt x n values and packs every token's
// n codes into that token's row.
__device__ int store_tiles(const float* zs, int ntile, int bt, int d, int dp, int n, int bits, const CacheDev& k,
                           size_t slc, int pos0) {
  int flags = 0;
  const int nb = d / n, row_bytes = d * bits / 8, blk_bytes = n * bits / 8;
  for (int w = threadIdx.x; w < ntile * nb; w += blockDim.x) {
    const int u = w / nb, kb = w - u * nb;
    const float* zt = zs + (u * bt) * dp + kb * n;
    float mn = zt[0], mx = zt[0];
    for (int v = 0; v < bt; ++v)
      for (int e = 0; e < n; ++e) {
        mn = fminf(mn, zt[v * dp + e]);
        mx = fmaxf(mx, zt[v * dp + e]);
      }
    const Side sd = make_side(mn, mx, bits);
    const float qmax = (float)((1 << bits) - 1);
    for (int v = 0; v < bt; ++v) {
      const size_t row = slc * k.T_cap + pos0 + u * bt + v;
      uint32_t* dst = (uint32_t*)(k.codes + row * row_bytes + size_t(kb) * blk_bytes);
      uint64_t acc = 0;
      int nbit = 0, wi = 0;
      for (int e = 0; e < n; ++e) {
        acc |= (uint64_t)quantize(zt[v * dp + e], sd.mn, sd.inv, qmax) << nbit;
        nbit += bits;
        if (nbit >= 32) {
          dst[wi++] = (uint32_t)acc;
          acc >>= 32;
          nbit -= 32;
        }
      }
    }
    k.side[(slc * (k.T_cap / bt) + (pos0 / bt + u)) * nb + kb] = sd.word;
    flags |= sd.flags;
  }
  return flags;
}

// KIVI key groups: tile rows [u*kg, u*kg + kg) form token group grp0 + u; one channel per
// thread.
__device__ int store_key_groups(const float* zs, int ngrp, int kg, int d, int dp, int bits, const CacheDev& k,
                                size_t slc, int grp0) {
  int flags = 0;
  const int cb = kg * bits / 8;
  for (int w = threadIdx.x; w < ngrp * d; w += blockDim.x) {
    const int u = w / d, ch = w - u * d;
    const size_t gi = slc * (k.T_cap / kg) + grp0 + u;
    uint32_t* dst = (uint32_t*)(k.codes + (gi * d + ch) * cb);
    flags |= quantize_block_to(zs + (u * kg) * dp + ch, dp, kg, bits, dst, k.side + gi * d + ch);
  }
  return flags;
}

// ------------------------------------------------------------------------------------------
// choice of the kernel variant
// ------------------------------------------------------------------------------------------
// (KR, NBW) of the matrix-core gauge for groups of 4 KR channels: NBW channel blocks per wave (four
// waves cover the d / 16 blocks of a head); (0, 1): the vector ALU, for the other groups (8 channels are
// 8 FMAs per value, and the 16-channel operand rows would mix two groups).
template <class Fn>
auto by_gauge(int g, int d, Fn&& fn) {
  auto nbw = [&](auto kr) {
    constexpr int KR = decltype(kr)::value;
    if constexpr (4 * KR <= 64) {
      if (d <= 64) return fn(kr, std::integral_constant<int, 1>());
    }
    if constexpr (4 * KR <= 128) {
      if (d <= 128) return fn(kr, std::integral_constant<int, 2>());
    }
    return fn(kr, std::integral_constant<int, 4>());
  };
  switch (g) {
    case 16: return nbw(std::integral_constant<int, 4>());
    case 32: return nbw(std::integral_constant<int, 8>());
    case 64: return nbw(std::integral_constant<int, 16>());
    case 80: return nbw(std::integral_constant<int, 20>());
    case 96: return nbw(std::integral_constant<int, 24>());
    case 128: return nbw(std::integral_constant<int, 32>());
    case 192: return nbw(std::integral_constant<int, 48>());
    case 256: return nbw(std::integral_constant<int, 64>());
    default: return fn(std::integral_constant<int, 0>(), std::integral_constant<int, 1>());
  }
}

inline hipError_t set_smem(const void* fn, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace
}  // namespace cg
