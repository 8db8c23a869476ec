// General-purpose codec kernels (any supported g, n, b, backend, bf16 or binary32 input).
//
// A workgroup owns a range of token tiles of one (layer, batch, head) slice.  A tile is staged in LDS in
// binary32, the gauge z = G x of every channel group (section 3: Z[b,h,t,r] = G_{l,s,h,r} X[b,h,t,r])
// runs on the binary32 matrix cores with the wave's rows of G in registers for the whole range
// (v_mfma_f32_16x16x4_f32 gives the binary32 FMA chain bit for bit; other group sizes than those of
// by_gauge stay on the vector ALU), and the backend of section 4.3 quantises the gauge-space tile
// from LDS, 8 channels per lane, the packed rows leaving as one contiguous run.  Decode mirrors it:
// codes are unpacked and dequantised into an LDS tile, Xhat = G^T Zhat is applied the same way, and
// the rows leave as 16-byte stores.  The next tile's loads are in flight beside a tile's work.  These
// kernels carry every configuration; the bf16 matrix-core kernels take over head dimension 128.
//
// What bounds them: the binary32 matrix cores (256 flops per CU and cycle), then the tile's four
// dependent phases.  16 layers x 2 x 8 heads x 2048 tokens of 64 channels, g = 64, 4 bits, block 32,
// bf16: encode 256 -> 74 us, decode 210 -> 66 us per tensor (vector-ALU gauge re-reading G per tile, one
// thread per block; the matrix-core floor is 27 us, the bytes' 18 us); with the three bf16 planes of G
// (general_planes) encode 44 us.
#include <algorithm>

#include "cg_internal.h"
#include "cg_device.h"
#include "cg_general.h"
#include "cg_recode.h"
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
struct EncArgs {
  int s;
  ViewDev X;
  int l0;
  GaugeDev G;
  CodecDev c;
  CacheDev k;
  int t0, tq;
  int TT, tiles_per_wg;  // tokens per tile, tiles per workgroup
  int* err;
  PageDev pt;
};

// granules of 8 channels of a tile that a thread fetches ahead (tiles of more go unfetched)
constexpr int kAhead = 2;

// Rows of packed codes staged in LDS (cst) to the cache rows [row0, row0 + nrow), one contiguous run.
__device__ __forceinline__ void store_code_rows(const uint8_t* cst, uint8_t* codes, size_t row0, int nrow,
                                                int row_bytes) {
  uint8_t* dst = codes + row0 * row_bytes;
  const int nbytes = nrow * row_bytes;  // a multiple of 4 (n bits is a multiple of 32)
  if (((reinterpret_cast<uintptr_t>(dst) | uintptr_t(nbytes)) & 15) == 0) {
    for (int i = threadIdx.x; i < nbytes / 16; i += kThreads)
      reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(cst)[i];
  } else {
    for (int i = threadIdx.x; i < nbytes / 4; i += kThreads)
      reinterpret_cast<uint32_t*>(dst)[i] = reinterpret_cast<const uint32_t*>(cst)[i];
  }
}

// How the tile is stored.  Token rows quantised over the lanes are the common case and have a variant
// of their own: the zfp-style coder alone would take every variant to 200 VGPRs (two waves per SIMD).
constexpr int kStoreRows = 0;   // per-token blocks (or KIVI values), 8 channels per lane
constexpr int kStoreOther = 1;  // passthrough, zfp-style, KIVI keys, tiles, odd block sizes

// Waves per SIMD the kernels are compiled for: four where the gauge takes at most 16 registers (heads of
// 64 channels), three up to 64.
constexpr int general_waves(int kr, int nbw, int store) {
  return store == kStoreRows ? (kr * nbw <= 16 ? 4 : (kr * nbw <= 64 ? 3 : 1)) : 1;
}

// Whether token rows of bf16 tensors take the three bf16 planes of G (by groups of 4 KR channels): where
// g is a multiple of 32 and the planes fit a wave's registers.  The other stores keep the binary32 chain
// (the error-free backend returns z itself, the zfp-style coder follows its last bits).
constexpr bool general_planes(int kr, int nbw, int store) {
  return store == kStoreRows && kr > 0 && kr % 8 == 0 && kr * nbw <= 64;
}

// The workgroup's rows with a non-finite channel once more (recode_rows).  Everything is derived from the
// kernel's argument segment (EncArgs is its only argument, at offset 0) and block indexes behind an asm
// barrier, so that the compiler keeps no scalar register for this call through the tile loop: with the
// kernel's own values a paged encode of K and V (5 layers, 4 x 16 rows of 1676 tokens, 64 channels, g = 32,
// 3 bits) takes 104.9 us, this way 101.3, without the call 100.0.
// flagged (64) and z (d floats): LDS; the smallest launch has 16 rows of d floats and more.
__device__ __forceinline__ int recode_range(int* flagged, float* z) {
  int bx = blockIdx.x, sv = blockIdx.y;
  auto args = (const __attribute__((address_space(4))) EncArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(bx), "+s"(sv), "+s"(args));
  const EncArgs& a = *(const EncArgs*)args;
  const ViewDev& X = a.X;
  const CacheDev& k = a.k;
  const bool kivi = a.c.backend == CG_BACKEND_KIVI;
  const int TT = a.TT, d = X.d, n = kivi ? a.c.kvc : a.c.n;
  const int h = sv % X.H, b = (sv / X.H) % X.B, lv = sv / (X.H * X.B), l = lv + a.l0;
  const int T = kivi ? min(X.T, a.tq) : X.T, row_bytes = d * a.c.bits / 8;
  const int tb = bx * a.tiles_per_wg, te = min((T + TT - 1) / TT, tb + a.tiles_per_wg);
  const char* x = static_cast<const char*>(X.ptr) + 2 * (size_t(lv) * X.sl + size_t(b) * X.sb + size_t(h) * X.sh);
  const float* Gh = a.G.f32 + gauge_block(l, a.s, h, 0, a.G.H, a.G.R) * a.G.g * a.G.g;
  int flags = 0;
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores, before those over them
  for (int tile = tb; tile < te; ++tile) {
    int crow = b, pos0 = a.t0 + tile * TT;
    if (a.pt.pages) {
      const int lp = pos0 / a.pt.page_size;
      crow = lp < a.pt.max_pages ? a.pt.pages[size_t(b) * a.pt.max_pages + lp] : -1;
      if (crow < 0 || crow >= k.B) continue;
      pos0 -= lp * a.pt.page_size;
    }
    const size_t row0 = ((size_t(l) * k.B + crow) * k.H + h) * k.T_cap + pos0;
    flags |= recode_rows(x + 2 * size_t(tile) * TT * X.st, 2 * X.st, min(TT, T - tile * TT), d, n, a.c.bits, Gh, a.G.g,
                         k.codes + row0 * row_bytes, k.side + row0 * (d / n), flagged, z);
  }
  return flags;
}

// PL: bf16 tokens stay bf16 in LDS and the gauge runs as three bf16 planes; rows with a non-finite channel
// are coded again after the range (recode_rows)
template <int KR, int NBW, int STORE, bool PL>
__global__ __launch_bounds__(kThreads, general_waves(KR, NBW, STORE)) void enc_general(EncArgs a) {
  static_assert(!PL || general_planes(KR, NBW, STORE), "groups of 32 KK channels");
  // the alignment matters: the dynamic part starts behind the static one, and at an offset of 4 every 16-byte
  // access to the tiles is misaligned (16 layers x 2 x 8 heads x 2048 tokens of 64 channels: 41 -> 77 us)
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ std::conditional_t<STORE == kStoreOther, ZfpTables, char> ztab;
  __shared__ int recode;  // PL: the workgroup met such a row
  const ViewDev& X = a.X;
  const CodecDev& c = a.c;
  const CacheDev& k = a.k;
  const int s = a.s, TT = a.TT, d = X.d, dp = d + kPad, d8 = d / 8, tid = threadIdx.x;
  const float inv8 = 1.0f / float(d8);
  const bool kivi = c.backend == CG_BACKEND_KIVI;
  const bool tiles = c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1;
  const int rows16 = (TT + 15) & ~15;
  const int n = kivi ? c.kvc : c.n, row_bytes = d * c.bits / 8;
  float* xs = sm;
  uint8_t* xb = reinterpret_cast<uint8_t*>(sm);
  const int xpitch = bf16_pitch(d);
  float* zs = PL ? reinterpret_cast<float*>(xb + rows16 * xpitch) : xs + rows16 * dp;
  float2* red = reinterpret_cast<float2*>(zs + rows16 * dp);
  uint8_t* cst = reinterpret_cast<uint8_t*>(red + (tiles ? TT * (d / n) : 0));
  const int sv = blockIdx.y;
  const int h = sv % X.H, b = (sv / X.H) % X.B, lv = sv / (X.H * X.B);
  const int l = lv + a.l0;
  const int ntiles = (X.T + TT - 1) / TT;
  const int tb = blockIdx.x * a.tiles_per_wg, te = min(ntiles, tb + a.tiles_per_wg);
  const size_t xbase = size_t(lv) * X.sl + size_t(b) * X.sb + size_t(h) * X.sh;

  GaugeRaw<(KR > 0 ? KR : 4), NBW> graw;
  GaugePlanes<(PL ? KR / 8 : 1), NBW> gp;
  const WaveTile wt = wave_tile<NBW>(d);
  if constexpr (PL) load_gauge_planes<KR / 8, NBW>(gp, a.G, l, s, h, wt);
  else if constexpr (KR > 0) load_gauge_rows<KR, NBW>(graw, a.G, l, s, h, wt);
  if constexpr (STORE == kStoreOther) {
    if (c.backend == CG_BACKEND_ZFP) zfp_tables_init(ztab);  // read after the barriers below
  }

  // this thread's granules of a tile: row gt[i], channels 8 gc[i] .. + 7 (rows past the view repeat its
  // last token; they are not stored)
  const bool ahead = TT * d8 <= kAhead * kThreads;
  int gt[kAhead], gc[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    gt[i] = small_div(tid + i * kThreads, inv8);
    gc[i] = tid + i * kThreads - gt[i] * d8;
  }
  Raw8 xr[kAhead];
  auto fetch = [&](int tile) {
    size_t off[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) off[i] = xbase + size_t(min(tile * TT + gt[i], X.T - 1)) * X.st + 8 * gc[i];
    if (PL || X.bf16) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
        if (i * kThreads < TT * d8) xr[i] = load_raw8<true>(X.ptr, off[i]);
    } else {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
        if (i * kThreads < TT * d8) xr[i] = load_raw8<false>(X.ptr, off[i]);
    }
  };
  auto raw_tile = [&](int tile) { return kivi && tile * TT >= a.tq; };  // KIVI window rows: no gauge
  if (ahead && !raw_tile(tb)) fetch(tb);
  float A[NBW][KR > 0 ? KR : 1];
  if constexpr (KR > 0 && !PL) gauge_operand<KR, NBW>(graw, A);
  int flags = 0;
  if (PL && tid == 0) recode = 0;  // set after the range, behind its barriers
  for (int tile = tb; tile < te; ++tile) {
    const int tile0 = tile * TT, ntok = min(TT, X.T - tile0);
    int crow = b, pos0 = a.t0 + tile0;  // cache batch row and its position of tile row 0
    bool skip = false;
    if (a.pt.pages) {  // a tile never crosses a page
      const int lp = pos0 / a.pt.page_size;
      crow = lp < a.pt.max_pages ? a.pt.pages[size_t(b) * a.pt.max_pages + lp] : -1;
      skip = crow < 0 || crow >= k.B;
      if (skip && tid == 0 && a.err) atomicOr(a.err, CG_FLAG_POS_RANGE);
      pos0 -= lp * a.pt.page_size;
    }
    const size_t slc = (size_t(l) * k.B + crow) * k.H + h;
    // KIVI window, or rows of an unfinished tile (view rows >= tq; t0 is a multiple of bt): raw bf16
    // rows into the ring (slot = cache position mod its slots)
    const int nq = kivi || tiles ? max(0, min(ntok, a.tq - tile0)) : ntok;
    if (nq < ntok) {
      const int slots = kivi ? c.win + c.kg : c.bt;
      for (int idx = tid; idx < (ntok - nq) * d8; idx += kThreads) {
        const int t = small_div(idx, inv8), c8 = idx - t * d8, tok = tile0 + nq + t;
        *reinterpret_cast<uint4*>(k.ring + (slc * slots + (a.t0 + tok) % slots) * d + 8 * c8) =
            *reinterpret_cast<const uint4*>((const uint16_t*)X.ptr + xbase + size_t(tok) * X.st + 8 * c8);
      }
    }
    if (nq == 0) continue;
    auto stage = [&](int t, int c8, const Raw8& r) {
      if constexpr (PL) {
        const uint32_t w[4] = {r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w};
        if (t < nq && !skip) {
#pragma unroll
          for (int e = 0; e < 4; ++e)  // an exponent of at least 2^100
            if ((w[e] & 0x7f80u) >= 0x7180u || (w[e] & 0x7f800000u) >= 0x71800000u) flags |= kFlagRecode;
        }
        *reinterpret_cast<uint4*>(xb + t * xpitch + 16 * c8) = r.v[0];
        return;
      }
      float x[8];
      raw8_values(r, X.bf16, x);
      if (t < nq && !skip) {  // staged rows: checked when quantised
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (!isfinite(x[e])) flags |= CG_FLAG_NONFINITE;
      }
      *reinterpret_cast<float4*>(xs + t * dp + 8 * c8) = make_float4(x[0], x[1], x[2], x[3]);
      *reinterpret_cast<float4*>(xs + t * dp + 8 * c8 + 4) = make_float4(x[4], x[5], x[6], x[7]);
    };
    if (ahead) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
        if (gt[i] < TT) stage(gt[i], gc[i], xr[i]);
    } else {
      for (int idx = tid; idx < TT * d8; idx += kThreads) {
        const int t = small_div(idx, inv8), c8 = idx - t * d8;
        const size_t off = xbase + size_t(min(tile0 + t, X.T - 1)) * X.st + 8 * c8;
        stage(t, c8, PL || X.bf16 ? load_raw8<true>(X.ptr, off) : load_raw8<false>(X.ptr, off));
      }
    }
    __syncthreads();
    if (ahead && tile + 1 < te && !raw_tile(tile + 1)) fetch(tile + 1);
    if constexpr (PL) gauge_planes_mfma<KR / 8, NBW>(gp, xb, zs, (ntok + 15) / 16, d, dp, wt);
    else if constexpr (KR > 0) gauge_mfma<KR, NBW>(A, xs, zs, (ntok + 15) / 16, dp, wt);
    else gauge_tile(xs, zs, ntok, d, dp, a.G, l, s, h);
    __syncthreads();
    if (skip) continue;

    if constexpr (STORE == kStoreRows) {
      const size_t row0 = slc * k.T_cap + pos0;
      const int nb = d / n;
      flags |= quantise_rows(
          zs, nq, d, dp, n, c.bits, 1, nullptr, cst, [](int) { return true; },
          [&](int t, int kb) { return k.side + (row0 + t) * nb + kb; });
      __syncthreads();
      store_code_rows(cst, k.codes, row0, nq, row_bytes);
    } else if (c.backend == CG_BACKEND_PASSTHROUGH) {
      float* out = reinterpret_cast<float*>(k.codes) + (slc * k.T_cap + pos0) * d;
      for (int idx = tid; idx < ntok * d8; idx += kThreads) {
        const int t = small_div(idx, inv8), c8 = idx - t * d8;
        float4* dst = reinterpret_cast<float4*>(out + size_t(t) * d + 8 * c8);
        const float4* src = reinterpret_cast<const float4*>(zs + t * dp + 8 * c8);
        dst[0] = src[0];
        dst[1] = src[1];
      }
    } else if (c.backend == CG_BACKEND_ZFP) {
      flags |= store_zfp(zs, ntok, d, dp, c.bits, k, slc, pos0, ztab);
    } else if (kivi && s == 0) {
      flags |= store_key_groups(zs, ntok / c.kg, c.kg, d, dp, c.bits, k, slc, pos0 / c.kg);
    } else if (tiles && lane_blocks(n)) {
      const size_t row0 = slc * k.T_cap + pos0;
      const int nb = d / n;
      flags |= quantise_rows(
          zs, nq, d, dp, n, c.bits, c.bt, red, cst, [](int) { return true; },
          [&](int t, int kb) { return k.side + ((row0 + t) / c.bt) * nb + kb; });
      __syncthreads();
      store_code_rows(cst, k.codes, row0, nq, row_bytes);
    } else if (tiles) {
      flags |= store_tiles(zs, nq / c.bt, c.bt, d, dp, n, c.bits, k, slc, pos0);
    } else {
      flags |= store_rows_blocks(zs, ntok, d, dp, n, c.bits, k, slc, pos0);
    }
  }
  if constexpr (PL) {
    if (flags & kFlagRecode) recode = 1;
    __syncthreads();
    if (recode) {
      flags &= ~kFlagRecode;
      flags |= recode_range(reinterpret_cast<int*>(sm), sm + 64);
    }
  }
  if (flags && a.err) atomicOr(a.err, flags);
}

// ------------------------------------------------------------------------------------------
// decode
// ------------------------------------------------------------------------------------------
struct DecArgs {
  int s;
  CacheDev k;
  int l0;
  GaugeDev G;
  CodecDev c;
  int t0, len;
  const int* pos;
  int pos_add;
  ViewDev Y;
  int TT, tiles_per_wg;
  int* err;
};

// A lane's 8 channels of a token row of block-uniform codes (or KIVI values) as loaded: the two dwords
// holding its 8 codes and the side words of its first and last four channels (blocks hold at least 4)
struct Code8 {
  uint32_t w0, w1, s0, s1;
};
__device__ __forceinline__ Code8 load_code8(const CacheDev& k, int d, int bits, int n, int bt, size_t slc, int p,
                                            int ch0) {
  const size_t row = slc * k.T_cap + p;
  const int rw = d * bits / 32, byte = ch0 * bits / 8, d0 = byte >> 2;
  const uint32_t* w = reinterpret_cast<const uint32_t*>(k.codes) + row * rw;
  const uint32_t* side = k.side + (bt > 1 ? slc * (k.T_cap / bt) + p / bt : row) * (d / n);
  Code8 c;
  c.w0 = w[d0];
  c.w1 = w[min(d0 + 1, rw - 1)];
  c.s0 = side[ch0 / n];
  c.s1 = side[(ch0 + 4) / n];
  return c;
}
__device__ __forceinline__ void code8_values(const Code8& c, int bits, int ch0, float (&z)[8]) {
  const uint32_t mask = (1u << bits) - 1u;
  const uint64_t v = ((uint64_t(c.w1) << 32) | c.w0) >> (((ch0 * bits / 8) & 3) * 8);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t sw = e < 4 ? c.s0 : c.s1;
    z[e] = dequantize(uint32_t(v >> (bits * e)) & mask, f16_bits_to_f32(sw & 0xffffu), f16_bits_to_f32(sw >> 16));
  }
}

// STORE as in the encoder: kStoreRows for codes by token rows (block-uniform, KIVI values)
template <int KR, int NBW, int STORE>
__global__ __launch_bounds__(kThreads, general_waves(KR, NBW, STORE)) void dec_general(DecArgs a) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ std::conditional_t<STORE == kStoreOther, ZfpTables, char> ztab;
  const ViewDev& Y = a.Y;
  const CodecDev& c = a.c;
  const CacheDev& k = a.k;
  const int s = a.s, TT = a.TT, d = Y.d, dp = d + kPad, d8 = d / 8, tid = threadIdx.x;
  const float inv8 = 1.0f / float(d8);
  const int rows16 = (TT + 15) & ~15;
  float* zs = sm;
  float* xs = zs + rows16 * dp;
  const int sv = blockIdx.y;
  const int h = sv % Y.H, b = (sv / Y.H) % Y.B, lv = sv / (Y.H * Y.B);
  const int l = lv + a.l0;
  const size_t slc = (size_t(l) * k.B + b) * k.H + h;
  const size_t ybase = size_t(lv) * Y.sl + size_t(b) * Y.sb + size_t(h) * Y.sh;

  GaugeCols<(KR > 0 ? KR : 4), NBW> A;
  const WaveTile wt = wave_tile<NBW>(d);
  if constexpr (KR > 0) load_gauge_cols<KR, NBW>(A.v, a.G, l, s, h, wt);

  // Positions the cache holds bound the rows written: pos[b] + pos_add per row (a rolling step's
  // newest position + 1, or kv_decode's per-row lengths; outside [0, T_cap] the row is flagged
  // and skipped), else `len` for a KIVI or tile cache, otherwise every requested position (the
  // host checked the capacity).
  const bool kivi = c.backend == CG_BACKEND_KIVI;
  const bool tiles = c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1;
  int held = INT_MAX;
  if (a.pos) {
    const int hb = a.pos[b] + a.pos_add;
    if (hb < 0 || hb > k.T_cap) {
      if (a.err && blockIdx.x == 0 && tid == 0) atomicOr(a.err, CG_FLAG_POS_RANGE);
      return;
    }
    held = hb;
  } else if (kivi || tiles) {
    held = a.len;
  }
  const int Tv = held == INT_MAX ? Y.T : min(Y.T, held - a.t0);  // view rows to write
  const int ntiles = (Tv + TT - 1) / TT;
  const int tb = blockIdx.x * a.tiles_per_wg, te = min(ntiles, tb + a.tiles_per_wg);
  if (tb >= te) return;
  // KIVI quantises the first T_q positions and keeps the rest in the window, tiles the whole
  // tiles and keep the unfinished one staged; the other backends quantise every position.
  const int tq = kivi ? (held < c.win ? 0 : ((held - c.win) / c.kg) * c.kg)
                      : (tiles ? (held / c.bt) * c.bt : INT_MAX);
  const int bits = c.bits, n = kivi ? c.kvc : c.n;
  auto quantised = [&](int tile) {  // quantised rows of a tile
    return max(0, min(min(TT, Tv - tile * TT), tq - (a.t0 + tile * TT)));
  };
  if constexpr (STORE == kStoreOther) {
    if (c.backend == CG_BACKEND_ZFP) {  // the backend is the same for the whole workgroup
      zfp_tables_init(ztab);
      __syncthreads();
    }
  }

  const bool ahead = STORE == kStoreRows && TT * d8 <= kAhead * kThreads;
  int gt[kAhead], gc[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    gt[i] = small_div(tid + i * kThreads, inv8);
    gc[i] = tid + i * kThreads - gt[i] * d8;
  }
  Code8 cr[kAhead];
  auto fetch = [&](int tile) {  // rows past the quantised ones repeat the last one
    const int nq = quantised(tile);
    if (nq == 0) return;
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (i * kThreads < TT * d8)
        cr[i] = load_code8(k, d, bits, n, c.bt, slc, a.t0 + tile * TT + min(gt[i], nq - 1), 8 * gc[i]);
  };
  auto put8 = [&](int t, int c8, const float (&z)[8]) {
    *reinterpret_cast<float4*>(zs + t * dp + 8 * c8) = make_float4(z[0], z[1], z[2], z[3]);
    *reinterpret_cast<float4*>(zs + t * dp + 8 * c8 + 4) = make_float4(z[4], z[5], z[6], z[7]);
  };
  if (ahead) fetch(tb);
  for (int tile = tb; tile < te; ++tile) {
    const int tile0 = tile * TT, p0 = a.t0 + tile0, ntok = min(TT, Tv - tile0), nq = quantised(tile);
    // 1. dequantise the quantised rows into zs
    if (ahead) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
        if (gt[i] < nq) {
          float z[8];
          code8_values(cr[i], bits, 8 * gc[i], z);
          put8(gt[i], gc[i], z);
        }
    } else if constexpr (STORE == kStoreRows) {
      for (int idx = tid; idx < nq * d8; idx += kThreads) {
        const int t = small_div(idx, inv8), c8 = idx - t * d8;
        float z[8];
        code8_values(load_code8(k, d, bits, n, c.bt, slc, p0 + t, 8 * c8), bits, 8 * c8, z);
        put8(t, c8, z);
      }
    } else if (c.backend == CG_BACKEND_PASSTHROUGH) {
      const float* src = reinterpret_cast<const float*>(k.codes) + (slc * k.T_cap + p0) * d;
      for (int idx = tid; idx < nq * d8; idx += kThreads) {
        const int t = small_div(idx, inv8), c8 = idx - t * d8;
        const float4* v = reinterpret_cast<const float4*>(src + size_t(t) * d + 8 * c8);
        float4* dst = reinterpret_cast<float4*>(zs + t * dp + 8 * c8);
        const float4 v0 = v[0], v1 = v[1];
        dst[0] = v0;
        dst[1] = v1;
      }
    } else if (c.backend == CG_BACKEND_ZFP) {
      load_zfp(zs, nq, d, dp, bits, k, slc, p0, ztab);
    } else {  // KIVI keys: per-channel streams of a token group
      const int kg = c.kg;
      for (int idx = tid; idx < nq * d; idx += kThreads) {
        const int t = idx / d, ch = idx - t * d, p = p0 + t;
        const size_t gi = slc * (k.T_cap / kg) + p / kg;
        const uint32_t* stream = (const uint32_t*)(k.codes + (gi * d + ch) * (kg * bits / 8));
        const uint32_t q = extract_code(stream, p % kg, bits);
        const uint32_t sw = k.side[gi * d + ch];
        zs[t * dp + ch] = dequantize(q, f16_bits_to_f32(sw & 0xffffu), f16_bits_to_f32(sw >> 16));
      }
    }
    __syncthreads();
    if (ahead && tile + 1 < te) fetch(tile + 1);
    // 2. inverse gauge
    if (nq > 0) {
      if constexpr (KR > 0) gauge_mfma<KR, NBW>(A.v, zs, xs, (nq + 15) / 16, dp, wt);
      else inverse_tile(zs, xs, nq, d, dp, a.G, l, s, h);
    }
    __syncthreads();
    // 3. write rows: inverse-gauged rows, then window / staged rows copied raw
    const int slots = tiles ? c.bt : c.win + c.kg;
    for (int idx = tid; idx < ntok * d8; idx += kThreads) {
      const int t = small_div(idx, inv8), c8 = idx - t * d8;
      const size_t off = ybase + size_t(tile0 + t) * Y.st + 8 * c8;
      if (t < nq) {
        const float4 v0 = *reinterpret_cast<const float4*>(xs + t * dp + 8 * c8);
        const float4 v1 = *reinterpret_cast<const float4*>(xs + t * dp + 8 * c8 + 4);
        if (Y.bf16) {
          *reinterpret_cast<uint4*>((uint16_t*)Y.ptr + off) =
              make_uint4(f32_to_bf16_rne(v0.x) | (f32_to_bf16_rne(v0.y) << 16), f32_to_bf16_rne(v0.z) | (f32_to_bf16_rne(v0.w) << 16),
                         f32_to_bf16_rne(v1.x) | (f32_to_bf16_rne(v1.y) << 16), f32_to_bf16_rne(v1.z) | (f32_to_bf16_rne(v1.w) << 16));
        } else {
          float4* dst = reinterpret_cast<float4*>((float*)Y.ptr + off);
          dst[0] = v0;
          dst[1] = v1;
        }
      } else if (kivi || tiles) {
        const uint4 r = *reinterpret_cast<const uint4*>(k.ring + (slc * slots + (p0 + t) % slots) * d + 8 * c8);
        if (Y.bf16) {
          *reinterpret_cast<uint4*>((uint16_t*)Y.ptr + off) = r;
        } else {
          Raw8 raw;
          raw.v[0] = r;
          raw.v[1] = make_uint4(0u, 0u, 0u, 0u);
          float x[8];
          raw8_values(raw, true, x);
          float4* dst = reinterpret_cast<float4*>((float*)Y.ptr + off);
          dst[0] = make_float4(x[0], x[1], x[2], x[3]);
          dst[1] = make_float4(x[4], x[5], x[6], x[7]);
        }
      }
    }
  }
}

// KIVI tiles are exactly one key token group, so the quantised / window split (a multiple of
// the group) never cuts a tile.  Otherwise a tile holds about 4096 values, two granules of 8 channels per
// thread: 64 tokens for heads of at most 64 channels where that leaves every CU a workgroup of at least
// two tiles, 32 up to 128 channels, 16 above.  (32 against 64 tokens, encode / decode of a bf16 tensor,
// d = 64: 2^15 tokens 7.4 / 8.9 against 6.3 / 8.3 us, 2^19 46 / 62 against 41 / 60; d = 32: 2^15 7.3 / 7.2 against
// 7.1 / 7.3, 2^19 37 / 35 against 26 / 28; below 2^15 the two are within 1 us either way.)  Paged caches take at
// most 32: positions start at multiples of 32, so only such a tile always lies inside one page;
// block-uniform tiles take whole ones.
int tile_tokens(const CodecDev& c, int d, bool paged, int T, int nslices) {
  if (c.backend == CG_BACKEND_KIVI) return c.kg;
  if (d > 128) return c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 16 ? 32 : 16;
  return !paged && d <= 64 && int64_t(T) * nslices >= 64 * 2 * cu_count() ? 64 : 32;
}

// Tiles per workgroup: each slice in as many chunks as bring the workgroups to about four per CU, all
// resident, so that a gauge is loaded once per several tiles and the next tile's loads run
// beside this one's work; one tile while there are fewer than that.
int tiles_per_wg(int ntiles, int nslices) {
  const int chunks = std::max(1, std::min(ntiles, (4 * cu_count() + nslices / 2) / nslices));
  return (ntiles + chunks - 1) / chunks;
}

}  // namespace

hipError_t launch_encode_generic(int s, const ViewDev& X, int l0, const GaugeDev& G, const CodecDev& c,
                                 const CacheDev& k, int t0, int tq, int* err, hipStream_t st, const PageDev& pt) {
  if (X.T == 0) return hipSuccess;
  EncArgs a;
  a.s = s;
  a.X = X;
  a.l0 = l0;
  a.G = G;
  a.c = c;
  a.k = k;
  a.t0 = t0;
  a.tq = tq;
  a.err = err;
  a.pt = pt;
  const int d = X.d, nslices = X.L * X.B * X.H;
  a.TT = tile_tokens(c, d, pt.pages != nullptr, X.T, nslices);
  a.tiles_per_wg = tiles_per_wg((X.T + a.TT - 1) / a.TT, nslices);
  const int rows16 = (a.TT + 15) & ~15;
  const size_t tile_f32 = size_t(rows16) * (d + kPad) * sizeof(float);
  size_t smem = tile_f32;  // zs, codes and ranges
  if (c.backend == CG_BACKEND_BLOCK_UNIFORM || (c.backend == CG_BACKEND_KIVI && s == 1)) {
    smem += size_t(a.TT) * (d * c.bits / 8);
    if (c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1) smem += size_t(a.TT) * (d / c.n) * sizeof(float2);
  }
  const bool kivi = c.backend == CG_BACKEND_KIVI;
  const bool by_rows = kivi ? s == 1 && lane_blocks(c.kvc)
                            : c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt == 1 && lane_blocks(c.n);
  const dim3 grid(((X.T + a.TT - 1) / a.TT + a.tiles_per_wg - 1) / a.tiles_per_wg, nslices);
  return by_gauge(G.g, d, [&](auto kr, auto nbw) {
    constexpr int KR = decltype(kr)::value, NBW = decltype(nbw)::value;
    const void* fn = by_rows ? (const void*)enc_general<KR, NBW, kStoreRows, false>
                             : (const void*)enc_general<KR, NBW, kStoreOther, false>;
    size_t bytes = smem + tile_f32;  // and the binary32 tokens
    if constexpr (general_planes(KR, NBW, kStoreRows)) {
      if (by_rows && X.bf16) {
        fn = (const void*)enc_general<KR, NBW, kStoreRows, true>;
        bytes = smem + size_t(rows16) * bf16_pitch(d);
      }
    }
    hipError_t e = set_smem(fn, bytes + sizeof(ZfpTables));
    if (e != hipSuccess) return e;
    void* args[] = {&a};
    return hipLaunchKernel(fn, grid, dim3(kThreads), args, bytes, st);
  });
}

hipError_t launch_decode_generic(int s, const CacheDev& k, int l0, const GaugeDev& G, const CodecDev& c, int t0,
                                 int len, const int* pos, int pos_add, const ViewDev& Y, int* err, hipStream_t st) {
  if (Y.T == 0) return hipSuccess;
  DecArgs a;
  a.s = s;
  a.k = k;
  a.l0 = l0;
  a.G = G;
  a.c = c;
  a.t0 = t0;
  a.len = len;
  a.pos = pos;
  a.pos_add = pos_add;
  a.Y = Y;
  a.err = err;
  const int nslices = Y.L * Y.B * Y.H;
  a.TT = tile_tokens(c, Y.d, false, Y.T, nslices);
  a.tiles_per_wg = tiles_per_wg((Y.T + a.TT - 1) / a.TT, nslices);
  const bool by_rows = c.backend == CG_BACKEND_BLOCK_UNIFORM || (c.backend == CG_BACKEND_KIVI && s == 1);
  const size_t smem = size_t(2) * ((a.TT + 15) & ~15) * (Y.d + kPad) * sizeof(float);
  const dim3 grid(((Y.T + a.TT - 1) / a.TT + a.tiles_per_wg - 1) / a.tiles_per_wg, nslices);
  return by_gauge(G.g, Y.d, [&](auto kr, auto nbw) {
    constexpr int KR = decltype(kr)::value, NBW = decltype(nbw)::value;
    const void* fn = by_rows ? (const void*)dec_general<KR, NBW, kStoreRows> : (const void*)dec_general<KR, NBW, kStoreOther>;
    hipError_t e = set_smem(fn, smem + sizeof(ZfpTables));
    if (e != hipSuccess) return e;
    void* args[] = {&a};
    return hipLaunchKernel(fn, grid, dim3(kThreads), args, smem, st);
  });
}

}  // namespace cg
