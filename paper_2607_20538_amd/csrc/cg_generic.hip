// General-purpose codec kernels (any supported g, n, b, backend, bf16 or binary32 input).
//
// One workgroup owns a tile of tokens of one (layer, batch, head) slice.  The tile is staged
// in LDS in binary32, the gauge z = G x of every channel group is applied on the VALU with a
// binary32 accumulator (section 3: Z[b,h,t,r] = G_{l,s,h,r} X[b,h,t,r]), and the backend of
// section 4.3 quantises the gauge-space tile from LDS: block-uniform / KIVI values one block
// per thread, KIVI keys one channel of a token group per thread.  Decode mirrors it: codes
// are unpacked and dequantised into an LDS tile, then Xhat = G^T Zhat is applied per
// channel.  These kernels carry every configuration; the MFMA kernels take over the
// large-group bf16 block-uniform case.
#include "cg_internal.h"
#include "cg_device.h"
#include "cg_general.h"
#include "cg_zfp.h"

namespace cg {

namespace {

// xs[t][i] = sum_j G_{l,s,h,r}[j][i%g] zs[t][r*g + j] (inverse gauge, G^T), the same chains and
// blocking (4 consecutive columns of G are one 16-byte read of row j).
__device__ void inverse_tile(const float* zs, float* xs, int ntok, int d, int dp, const GaugeDev& G, int l, int s,
                             int h) {
  const int g = G.g;
  if (g % 4) {
    for (int idx = threadIdx.x; idx < ntok * d; idx += blockDim.x) {
      const int t = idx / d, i = idx - t * d;
      const int r = i / g, ii = i - r * g;
      const float* Gr = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + ii;
      const float* zr = zs + t * dp + r * g;
      float acc = 0.0f;
      for (int j = 0; j < g; ++j) acc = fmaf(Gr[size_t(j) * g], zr[j], acc);
      xs[t * dp + i] = acc;
    }
    return;
  }
  const int ntb = (ntok + 3) / 4, ncb = d / 4;
  for (int idx = threadIdx.x; idx < ntb * ncb; idx += blockDim.x) {
    const int tb = idx / ncb, cb = idx - tb * ncb;
    const int t0 = 4 * tb, i0 = 4 * cb, r = i0 / g;
    const float* Gb = G.f32 + gauge_block(l, s, h, r, G.H, G.R) * g * g + (i0 - r * g);
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float acc[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[t][a] = 0.0f;
    for (int j = 0; j < g; j += 4) {
      float4 gv[4], zv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) gv[q] = *reinterpret_cast<const float4*>(Gb + size_t(j + q) * g);  // G[j+q][i0..i0+3]
#pragma unroll
      for (int t = 0; t < 4; ++t)
        zv[t] = t0 + t < ntok ? *reinterpret_cast<const float4*>(zs + (t0 + t) * dp + r * g + j) : zero;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float zz[4] = {zv[t].x, zv[t].y, zv[t].z, zv[t].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[t][0] = fmaf(gv[q].x, zz[q], acc[t][0]);
          acc[t][1] = fmaf(gv[q].y, zz[q], acc[t][1]);
          acc[t][2] = fmaf(gv[q].z, zz[q], acc[t][2]);
          acc[t][3] = fmaf(gv[q].w, zz[q], acc[t][3]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t0 + t < ntok) *reinterpret_cast<float4*>(xs + (t0 + t) * dp + i0) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
  }
}

// zfp-style rows: tile rows [4u, 4u + 4) x channels [4cb, 4cb + 4) form block (pos0 / 4 + u, cb)
__device__ int store_zfp(const float* zs, int ntok, int d, int dp, int rate, const CacheDev& k, size_t slc,
                         int pos0, const ZfpTables& tab) {
  return zfp_by_rate(rate, [&](auto R) {
    constexpr int RATE = decltype(R)::value;
    int flags = 0;
    const int nbc = d / 4;
    for (int idx = threadIdx.x; idx < (ntok / 4) * nbc; idx += blockDim.x) {
      const int u = idx / nbc, cb = idx - u * nbc;
      float v[16];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * j + i] = zs[(4 * u + j) * dp + 4 * cb + i];
      uint32_t w[4];
      flags |= zfp_encode_block<RATE>(v, tab, w);
      zfp_store<RATE>(k.codes + ((slc * (k.T_cap / 4) + pos0 / 4 + u) * nbc + cb) * size_t(2 * RATE), w);
    }
    return flags;
  });
}

__device__ void load_zfp(float* zs, int ntok, int d, int dp, int rate, const CacheDev& k, size_t slc, int pos0,
                         const ZfpTables& tab) {
  zfp_by_rate(rate, [&](auto R) {
    constexpr int RATE = decltype(R)::value;
    const int nbc = d / 4;
    for (int idx = threadIdx.x; idx < (ntok / 4) * nbc; idx += blockDim.x) {
      const int u = idx / nbc, cb = idx - u * nbc;
      uint32_t w[4];
      zfp_load<RATE>(k.codes + ((slc * (k.T_cap / 4) + pos0 / 4 + u) * nbc + cb) * size_t(2 * RATE), w);
      float v[16];
      zfp_decode_block<RATE>(w, tab, v);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) zs[(4 * u + j) * dp + 4 * cb + i] = v[4 * j + i];
    }
    return 0;
  });
}

// ------------------------------------------------------------------------------------------
// encode
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void enc_generic(int s, ViewDev X, int l0, GaugeDev G, CodecDev c, CacheDev k,
                                                        int t0, int tq, int TT, int* err, PageDev pt) {
  extern __shared__ float sm[];
  const int d = X.d, dp = d + kPad;
  float* xs = sm;
  float* zs = sm + TT * dp;
  const int sv = blockIdx.y;
  const int h = sv % X.H, b = (sv / X.H) % X.B, lv = sv / (X.H * X.B);
  const int l = lv + l0;
  const int tile0 = blockIdx.x * TT;
  const int ntok = min(TT, X.T - tile0);
  int crow = b;  // cache batch row: the page of a paged cache (a tile never crosses a page)
  if (pt.pages) {
    const int lp = (t0 + tile0) / pt.page_size;
    crow = lp < pt.max_pages ? pt.pages[size_t(b) * pt.max_pages + lp] : -1;
    if (crow < 0 || crow >= k.B) {
      if (threadIdx.x == 0 && err) atomicOr(err, CG_FLAG_POS_RANGE);
      return;
    }
    t0 -= lp * pt.page_size;  // positions inside the page
  }
  const size_t slc = (size_t(l) * k.B + crow) * k.H + h;
  const size_t xbase = size_t(lv) * X.sl + size_t(b) * X.sb + size_t(h) * X.sh;

  if (c.backend == CG_BACKEND_KIVI && tile0 >= tq) {
    // full-precision window: raw bf16 rows into the ring
    const int ringsz = c.win + c.kg;
    for (int idx = threadIdx.x; idx < ntok * d; idx += blockDim.x) {
      const int t = idx / d, ch = idx - t * d;
      const int tok = tile0 + t;
      k.ring[(slc * ringsz + tok % ringsz) * d + ch] = ((const uint16_t*)X.ptr)[xbase + size_t(tok) * X.st + ch];
    }
    return;
  }
  // block-uniform tiles: rows of the unfinished tile (view rows >= tq) wait raw in the
  // staging window (slot = cache position mod bt; t0 is a multiple of bt)
  const bool tiles = c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1;
  const int nq = tiles ? max(0, min(ntok, tq - tile0)) : ntok;
  if (tiles) {
    for (int idx = nq * d + threadIdx.x; idx < ntok * d; idx += blockDim.x) {
      const int t = idx / d, ch = idx - t * d;
      const int tok = tile0 + t;
      k.ring[(slc * c.bt + (t0 + tok) % c.bt) * d + ch] = ((const uint16_t*)X.ptr)[xbase + size_t(tok) * X.st + ch];
    }
    if (nq == 0) return;
  }

  __shared__ ZfpTables ztab;
  if (c.backend == CG_BACKEND_ZFP) zfp_tables_init(ztab);  // read after the barriers below
  int flags = 0;
  for (int idx = threadIdx.x; idx < TT * d; idx += blockDim.x) {
    const int t = idx / d, ch = idx - t * d;
    float v = 0.0f;
    if (t < ntok) {
      v = load_x(X, xbase + size_t(tile0 + t) * X.st + ch);
      if (t < nq && !isfinite(v)) flags |= CG_FLAG_NONFINITE;  // staged rows: checked when quantised
    }
    xs[t * dp + ch] = v;
  }
  __syncthreads();
  gauge_tile(xs, zs, ntok, d, dp, G, l, s, h);
  __syncthreads();

  if (c.backend == CG_BACKEND_PASSTHROUGH) {
    store_rows_pass(zs, ntok, d, dp, k, slc, t0 + tile0);
  } else if (c.backend == CG_BACKEND_ZFP) {
    flags |= store_zfp(zs, ntok, d, dp, c.bits, k, slc, t0 + tile0, ztab);
  } else if (tiles) {
    flags |= store_tiles(zs, nq / c.bt, c.bt, d, dp, c.n, c.bits, k, slc, t0 + tile0);
  } else if (c.backend == CG_BACKEND_BLOCK_UNIFORM) {
    flags |= store_rows_blocks(zs, ntok, d, dp, c.n, c.bits, k, slc, t0 + tile0);
  } else if (s == 1) {
    flags |= store_rows_blocks(zs, ntok, d, dp, c.kvc, c.bits, k, slc, tile0);
  } else {
    flags |= store_key_groups(zs, ntok / c.kg, c.kg, d, dp, c.bits, k, slc, tile0 / c.kg);
  }
  if (flags && err) atomicOr(err, flags);
}

// ------------------------------------------------------------------------------------------
// decode
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void dec_generic(int s, CacheDev k, int l0, GaugeDev G, CodecDev c, int t0,
                                                        int len, const int* pos, int pos_add, ViewDev Y, int TT,
                                                        int* err) {
  extern __shared__ float sm[];
  const int d = Y.d, dp = d + kPad;
  float* zs = sm;
  float* xs = sm + TT * dp;
  const int sv = blockIdx.y;
  const int h = sv % Y.H, b = (sv / Y.H) % Y.B, lv = sv / (Y.H * Y.B);
  const int l = lv + l0;
  const int tile0 = blockIdx.x * TT;
  int ntok = min(TT, Y.T - tile0);
  const size_t slc = (size_t(l) * k.B + b) * k.H + h;
  const size_t ybase = size_t(lv) * Y.sl + size_t(b) * Y.sb + size_t(h) * Y.sh;

  // Positions the cache holds bound the rows written: pos[b] + pos_add per row (a rolling step's
  // newest position + 1, or kv_decode's per-row lengths; outside [0, T_cap] the row is flagged
  // and skipped), else `len` for a KIVI or tile cache, otherwise every requested position (the
  // host checked the capacity).
  const bool kivi = c.backend == CG_BACKEND_KIVI;
  const bool tiles = c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1;
  int held = INT_MAX;
  if (pos) {
    const int hb = pos[b] + pos_add;
    if (hb < 0 || hb > k.T_cap) {
      if (err && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err, CG_FLAG_POS_RANGE);
      return;
    }
    held = hb;
  } else if (kivi || tiles) {
    held = len;
  }
  const int p0 = t0 + tile0;  // cache position of tile row 0
  if (held != INT_MAX) ntok = min(ntok, held - p0);
  if (ntok <= 0) return;
  // KIVI quantises the first T_q positions and keeps the rest in the window, tiles the whole
  // tiles and keep the unfinished one staged; the other backends quantise every position.
  const int tq = kivi ? (held < c.win ? 0 : ((held - c.win) / c.kg) * c.kg)
                      : (tiles ? (held / c.bt) * c.bt : INT_MAX);
  const int nq = max(0, min(ntok, tq - p0));  // quantised rows of this tile

  // 1. dequantise the quantised rows into zs
  const int bits = c.bits;
  if (c.backend == CG_BACKEND_ZFP) {  // the backend is the same for the whole workgroup
    __shared__ ZfpTables ztab;
    zfp_tables_init(ztab);
    __syncthreads();
    load_zfp(zs, nq, d, dp, bits, k, slc, p0, ztab);
  }
  for (int idx = threadIdx.x; c.backend != CG_BACKEND_ZFP && idx < nq * d; idx += blockDim.x) {
    const int t = idx / d, ch = idx - t * d;
    const int p = p0 + t;
    float zv;
    if (c.backend == CG_BACKEND_PASSTHROUGH) {
      zv = ((const float*)k.codes)[(slc * k.T_cap + p) * d + ch];
    } else if (c.backend == CG_BACKEND_BLOCK_UNIFORM || s == 1) {
      const int n = c.backend == CG_BACKEND_BLOCK_UNIFORM ? c.n : c.kvc;
      const int nb = d / n, kb = ch / n;
      const size_t row = slc * k.T_cap + p;
      const uint32_t* stream = (const uint32_t*)(k.codes + row * (d * bits / 8) + size_t(kb) * (n * bits / 8));
      const uint32_t q = extract_code(stream, ch - kb * n, bits);
      const uint32_t sw = k.side[(tiles ? slc * (k.T_cap / c.bt) + p / c.bt : row) * nb + kb];
      zv = dequantize(q, f16_bits_to_f32(sw & 0xffffu), f16_bits_to_f32(sw >> 16));
    } else {
      const int kg = c.kg;
      const size_t gi = slc * (k.T_cap / kg) + p / kg;
      const uint32_t* stream = (const uint32_t*)(k.codes + (gi * d + ch) * (kg * bits / 8));
      const uint32_t q = extract_code(stream, p % kg, bits);
      const uint32_t sw = k.side[gi * d + ch];
      zv = dequantize(q, f16_bits_to_f32(sw & 0xffffu), f16_bits_to_f32(sw >> 16));
    }
    zs[t * dp + ch] = zv;
  }
  __syncthreads();
  // 2. inverse gauge
  inverse_tile(zs, xs, nq, d, dp, G, l, s, h);
  __syncthreads();
  // 3. write rows: inverse-gauged rows, then window / staged rows copied raw
  const int ringsz = tiles ? c.bt : c.win + c.kg;
  for (int idx = threadIdx.x; idx < ntok * d; idx += blockDim.x) {
    const int t = idx / d, ch = idx - t * d;
    const size_t off = ybase + size_t(tile0 + t) * Y.st + ch;
    if (t < nq) {
      const float v = xs[t * dp + ch];
      if (Y.bf16) ((uint16_t*)Y.ptr)[off] = (uint16_t)f32_to_bf16_rne(v);
      else ((float*)Y.ptr)[off] = v;
    } else if (kivi || tiles) {
      const uint16_t raw = k.ring[(slc * ringsz + (p0 + t) % ringsz) * d + ch];
      if (Y.bf16) ((uint16_t*)Y.ptr)[off] = raw;
      else ((float*)Y.ptr)[off] = bf16_to_f32(raw);
    }
  }
}

// KIVI tiles are exactly one key token group, so the quantised / window split (a multiple of
// the group) never cuts a tile.
int tile_tokens(const CodecDev& c) { return c.backend == CG_BACKEND_KIVI ? c.kg : 32; }

}  // namespace

hipError_t launch_encode_generic(int s, const ViewDev& X, int l0, const GaugeDev& G, const CodecDev& c,
                                 const CacheDev& k, int t0, int tq, int* err, hipStream_t st, const PageDev& pt) {
  if (X.T == 0) return hipSuccess;
  const int TT = tile_tokens(c);
  const size_t smem = size_t(2) * TT * (X.d + kPad) * sizeof(float);
  hipError_t e = set_smem((const void*)enc_generic, smem);
  if (e != hipSuccess) return e;
  dim3 grid((X.T + TT - 1) / TT, X.L * X.B * X.H);
  hipLaunchKernelGGL(enc_generic, grid, dim3(kThreads), smem, st, s, X, l0, G, c, k, t0, tq, TT, err, pt);
  return hipGetLastError();
}

hipError_t launch_decode_generic(int s, const CacheDev& k, int l0, const GaugeDev& G, const CodecDev& c, int t0,
                                 int len, const int* pos, int pos_add, const ViewDev& Y, int* err, hipStream_t st) {
  if (Y.T == 0) return hipSuccess;
  const int TT = tile_tokens(c);
  const size_t smem = size_t(2) * TT * (Y.d + kPad) * sizeof(float);
  hipError_t e = set_smem((const void*)dec_generic, smem);
  if (e != hipSuccess) return e;
  dim3 grid((Y.T + TT - 1) / TT, Y.L * Y.B * Y.H);
  hipLaunchKernelGGL(dec_generic, grid, dim3(kThreads), smem, st, s, k, l0, G, c, t0, len, pos, pos_add, Y, TT, err);
  return hipGetLastError();
}

}  // namespace cg
