// Rolling append (section 4.4 step 1): the new key and value token of every (layer, batch row, head)
// gauged and quantised at its position, K and V in one launch.
//
// A step moves little (the gauges of the layers, once, and a few hundred bytes per token), so it is
// bound by the chain of dependent loads from the launch to the stores; the kernels keep that chain
// short.  append_rows takes the batch rows of one (layer, head), which share a gauge, as the 16
// columns of the binary32 matrix cores (the same FMA chains as the general encoder, gauge rows straight
// from global memory into the operand registers), so a gauge is read once per 16 rows and all of
// its loads are in flight together.  Measured on MI355X, K and V of one layer of 8 heads, d = g = 128,
// batch 1: 41 us in two launches (a 128-step chain of dependent 4-byte-per-lane loads and a block
// quantised by one thread) -> 7 us in one.
#include "cg_internal.h"
#include "cg_device.h"
#include "cg_general.h"

namespace cg {

namespace {

struct AppendArgs {
  ViewDev x[2];    // new tokens, keys and values
  CacheDev k[2];
  int l0;
  const int* pos;
  GaugeDev G;
  CodecDev c;
  int* err;
  PageDev pt;
};

// Cache batch row and position inside it of batch row b's new token at position p of the row; false
// (and flagged) when the position or its page is outside the cache.
__device__ __forceinline__ bool token_slot(const AppendArgs& a, const CacheDev& k, int b, int& row, int& p) {
  row = b;
  if (a.pt.pages) {
    const int lp = p >= 0 ? p / a.pt.page_size : -1;
    row = lp >= 0 && lp < a.pt.max_pages ? a.pt.pages[size_t(b) * a.pt.max_pages + lp] : -1;
    p -= lp * a.pt.page_size;
  }
  if (row < 0 || row >= k.B || p < 0 || p >= k.T_cap) {
    if (a.err) atomicOr(a.err, CG_FLAG_POS_RANGE);
    return false;
  }
  return true;
}

// Per-token blocks and the error-free backend: workgroup (layer and head, 16 batch rows, K or V).
constexpr int kRows = 16;

template <int KR, int NBW>
__global__ __launch_bounds__(kThreads) void append_rows(AppendArgs a) {
  extern __shared__ float sm[];
  __shared__ int64_t rowi[kRows];  // cache token row of each batch row, or -1
  const int s = blockIdx.z;
  const ViewDev& X = a.x[s];
  const CacheDev& k = a.k[s];
  const int d = X.d, dp = d + kPad, d8 = d / 8;
  float* xs = sm;
  float* zs = sm + kRows * dp;
  uint8_t* cst = reinterpret_cast<uint8_t*>(zs + kRows * dp);
  const float inv8 = 1.0f / float(d8);
  const int h = blockIdx.x % X.H, lv = blockIdx.x / X.H, l = lv + a.l0;
  const int b0 = kRows * blockIdx.y, nr = min(kRows, X.B - b0);
  const int tid = threadIdx.x;

  GaugeRaw<(KR > 0 ? KR : 4), NBW> raw;
  const WaveTile wt = wave_tile<NBW>(d);
  const int pv = a.pos[min(b0 + (tid & (kRows - 1)), X.B - 1)];
  if constexpr (KR > 0) load_gauge_rows<KR, NBW>(raw, a.G, l, s, h, wt);
  // the tokens' channels, 8 per lane (at most 2 x 8: 16 rows of 256 channels); rows past the batch
  // repeat its last one and are not stored
  Raw8 xr[2];
  size_t xo[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = tid + i * kThreads, t = min(small_div(idx, inv8), nr - 1), c8 = idx - small_div(idx, inv8) * d8;
    xo[i] = size_t(lv) * X.sl + size_t(b0 + t) * X.sb + size_t(h) * X.sh + 8 * c8;
  }
  if (X.bf16) {
#pragma unroll
    for (int i = 0; i < 2; ++i) xr[i] = load_raw8<true>(X.ptr, xo[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) xr[i] = load_raw8<false>(X.ptr, xo[i]);
  }
  if (tid < kRows) {
    int row, p = pv;
    rowi[tid] = tid < nr && token_slot(a, k, b0 + tid, row, p)
                    ? int64_t((size_t(l) * k.B + row) * k.H + h) * k.T_cap + p
                    : int64_t(-1);
  }
  float x[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = tid + i * kThreads, t = small_div(idx, inv8), c8 = idx - t * d8;
    raw8_values(xr[i], X.bf16, x[i]);
    if (t < kRows) {
      *reinterpret_cast<float4*>(xs + t * dp + 8 * c8) = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
      *reinterpret_cast<float4*>(xs + t * dp + 8 * c8 + 4) = make_float4(x[i][4], x[i][5], x[i][6], x[i][7]);
    }
  }
  __syncthreads();
  int flags = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = small_div(tid + i * kThreads, inv8);
    if (t < nr && rowi[t] >= 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (!isfinite(x[i][e])) flags |= CG_FLAG_NONFINITE;
    }
  }
  if constexpr (KR > 0) {
    float A[NBW][KR];
    gauge_operand<KR, NBW>(raw, A);
    gauge_mfma<KR, NBW>(A, xs, zs, 1, dp, wt);
  } else gauge_tile(xs, zs, nr, d, dp, a.G, l, s, h);
  __syncthreads();

  const int bits = a.c.bits, n = a.c.n;
  if (a.c.backend == CG_BACKEND_PASSTHROUGH) {
    float* out = reinterpret_cast<float*>(k.codes);
    for (int idx = tid; idx < nr * (d / 4); idx += kThreads) {
      const int t = idx / (d / 4), c4 = idx - t * (d / 4);
      if (rowi[t] >= 0)
        *reinterpret_cast<float4*>(out + size_t(rowi[t]) * d + 4 * c4) = *reinterpret_cast<const float4*>(zs + t * dp + 4 * c4);
    }
  } else {
    const int nb = d / n, rw = d * bits / 32;  // side words and dwords per row
    if (lane_blocks(n)) {
      flags |= quantise_rows(
          zs, nr, d, dp, n, bits, 1, nullptr, cst, [&](int t) { return rowi[t] >= 0; },
          [&](int t, int kb) { return k.side + size_t(rowi[t]) * nb + kb; });
      __syncthreads();
      for (int idx = tid; idx < nr * rw; idx += kThreads) {
        const int t = idx / rw, wd = idx - t * rw;
        if (rowi[t] >= 0)
          reinterpret_cast<uint32_t*>(k.codes)[size_t(rowi[t]) * rw + wd] = reinterpret_cast<const uint32_t*>(cst)[idx];
      }
    } else {
      for (int w = tid; w < nr * nb; w += kThreads) {
        const int t = w / nb, kb = w - t * nb;
        if (rowi[t] < 0) continue;
        uint32_t* dst = reinterpret_cast<uint32_t*>(k.codes) + size_t(rowi[t]) * rw + kb * (n * bits / 32);
        flags |= quantize_block_to(zs + t * dp + kb * n, 1, n, bits, dst, k.side + size_t(rowi[t]) * nb + kb);
      }
    }
  }
  if (flags && a.err) atomicOr(a.err, flags);
}

// KIVI caches and token-channel tiles: the token goes raw into the window or the staging tile; when
// it completes a group (KIVI: the cache holds T tokens with T - W a positive multiple of kg; tiles:
// the tile's last token) the workgroup, one per (layer, batch row, head) and K or V, gauges and
// quantises the kg oldest window tokens or the tile.
template <int KR, int NBW>
__global__ __launch_bounds__(kThreads) void append_staged(AppendArgs a) {
  extern __shared__ float sm[];
  const int s = blockIdx.z;
  const ViewDev& X = a.x[s];
  const CacheDev& k = a.k[s];
  const CodecDev& c = a.c;
  const int d = X.d, dp = d + kPad, d8 = d / 8;
  const float inv8 = 1.0f / float(d8);
  const int sv = blockIdx.x;
  const int h = sv % X.H, b = (sv / X.H) % X.B, lv = sv / (X.H * X.B);
  const int l = lv + a.l0;
  const int p = a.pos[b];
  if (p < 0 || p >= k.T_cap) {
    if (threadIdx.x == 0 && a.err) atomicOr(a.err, CG_FLAG_POS_RANGE);
    return;
  }
  const size_t slc = (size_t(l) * k.B + b) * k.H + h;
  const bool kivi = c.backend == CG_BACKEND_KIVI;
  const int unit = kivi ? c.kg : c.bt, slots = kivi ? c.win + c.kg : c.bt;
  const uint16_t* src = (const uint16_t*)X.ptr + size_t(lv) * X.sl + size_t(b) * X.sb + size_t(h) * X.sh;
  for (int i = threadIdx.x; i < d8; i += kThreads)
    *reinterpret_cast<uint4*>(k.ring + (slc * slots + p % slots) * d + 8 * i) = *reinterpret_cast<const uint4*>(src + 8 * i);
  const int T = p + 1;
  if (kivi ? !(T - c.win >= c.kg && (T - c.win) % c.kg == 0) : T % c.bt != 0) return;
  const int tb = T - (kivi ? c.win : 0) - unit;  // first token of the group
  const int ntb = (unit + 15) / 16;
  float* xs = sm;
  float* zs = sm + 16 * ntb * dp;
  float2* red = reinterpret_cast<float2*>(zs + 16 * ntb * dp);
  uint8_t* cst = reinterpret_cast<uint8_t*>(red + (kivi ? 0 : unit * (d / c.n)));
  GaugeRaw<(KR > 0 ? KR : 4), NBW> raw;
  const WaveTile wt = wave_tile<NBW>(d);
  if constexpr (KR > 0) load_gauge_rows<KR, NBW>(raw, a.G, l, s, h, wt);
  __syncthreads();  // the new token's row is written
  int flags = 0;
  for (int idx = threadIdx.x; idx < 16 * ntb * d8; idx += kThreads) {
    const int t = small_div(idx, inv8), c8 = idx - t * d8;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (t < unit) v = *reinterpret_cast<const uint4*>(k.ring + (slc * slots + (tb + t) % slots) * d + 8 * c8);
    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
    float x[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = __uint_as_float(wv[e] << 16);
      x[2 * e + 1] = __uint_as_float(wv[e] & 0xffff0000u);
    }
    if (!kivi) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (!isfinite(x[e])) flags |= CG_FLAG_NONFINITE;
    }
    *reinterpret_cast<float4*>(xs + t * dp + 8 * c8) = make_float4(x[0], x[1], x[2], x[3]);
    *reinterpret_cast<float4*>(xs + t * dp + 8 * c8 + 4) = make_float4(x[4], x[5], x[6], x[7]);
  }
  __syncthreads();
  if constexpr (KR > 0) {
    float A[NBW][KR];
    gauge_operand<KR, NBW>(raw, A);
    gauge_mfma<KR, NBW>(A, xs, zs, ntb, dp, wt);
  } else gauge_tile(xs, zs, unit, d, dp, a.G, l, s, h);
  __syncthreads();

  const int n = kivi ? c.kvc : c.n, bits = c.bits, nb = d / n;
  if (kivi && s == 0) {
    flags |= store_key_groups(zs, 1, c.kg, d, dp, bits, k, slc, tb / c.kg);
  } else if (lane_blocks(n)) {
    const size_t row0 = slc * k.T_cap + tb;
    flags |= quantise_rows(
        zs, unit, d, dp, n, bits, c.bt, red, cst, [](int) { return true; },
        [&](int t, int kb) { return k.side + ((row0 + t) / c.bt) * nb + kb; });
    __syncthreads();
    const int rw = d * bits / 32;
    for (int idx = threadIdx.x; idx < unit * rw; idx += kThreads)
      reinterpret_cast<uint32_t*>(k.codes)[row0 * rw + idx] = reinterpret_cast<const uint32_t*>(cst)[idx];
  } else if (kivi) {
    flags |= store_rows_blocks(zs, c.kg, d, dp, c.kvc, bits, k, slc, tb);
  } else {
    flags |= store_tiles(zs, 1, c.bt, d, dp, c.n, bits, k, slc, tb);
  }
  if (flags && a.err) atomicOr(a.err, flags);
}

}  // namespace

hipError_t launch_append(const ViewDev& Kn, const ViewDev& Vn, int l0, const int* pos, const GaugeDev& G,
                         const CodecDev& c, const CacheDev& kc, const CacheDev& vc, int* err, hipStream_t st,
                         const PageDev& pt) {
  AppendArgs a;
  a.x[0] = Kn; a.x[1] = Vn;
  a.k[0] = kc; a.k[1] = vc;
  a.l0 = l0;
  a.pos = pos;
  a.G = G;
  a.c = c;
  a.err = err;
  a.pt = pt;
  const int d = Kn.d, dp = d + kPad;
  const bool kivi = c.backend == CG_BACKEND_KIVI, staged = kivi || c.bt > 1;
  // codes of a staged tile: the widest row a codec can have (passthrough writes from the tile)
  const int unit = staged ? (kivi ? c.kg : c.bt) : kRows, rows = (unit + 15) / 16 * 16;
  size_t smem = size_t(2) * rows * dp * sizeof(float) + size_t(unit) * d;
  if (staged && !kivi) smem += size_t(unit) * (d / c.n) * sizeof(float2);
  const dim3 grid = staged ? dim3(Kn.L * Kn.B * Kn.H, 1, 2) : dim3(Kn.L * Kn.H, (Kn.B + kRows - 1) / kRows, 2);
  return by_gauge(G.g, d, [&](auto kr, auto nbw) {
    constexpr int KR = decltype(kr)::value, NBW = decltype(nbw)::value;
    const void* fn = staged ? (const void*)append_staged<KR, NBW> : (const void*)append_rows<KR, NBW>;
    hipError_t e = set_smem(fn, smem);
    if (e != hipSuccess) return e;
    void* args[] = {&a};
    return hipLaunchKernel(fn, grid, dim3(kThreads), args, smem, st);
  });
}

}  // namespace cg
