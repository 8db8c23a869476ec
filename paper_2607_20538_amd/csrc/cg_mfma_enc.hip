// Matrix-core codec kernels for bf16 caches with head dimension 128 and the block-uniform
// backend (the configuration the paper's Llama-class KV caches take).
//
// The gauge (section 3: z = G_{l,s,h,r} x per channel group) is a dense contraction over the
// channel axis, so it runs on the gfx950 matrix cores with v_mfma_f32_32x32x16_bf16.  The
// input x is exact in bf16; the binary32 gauge enters as kNP bf16 planes G0 + G1 (+ G2) of
// its split (the gauge buffer holds three), each multiplied on the matrix core with a
// binary32 accumulator.  Two planes carry 16 significant bits of every entry (entry error at
// most 2^-16 relative), which keeps z within a few 1e-6 of the binary32 gauge per group,
// inside the 1e-5 gauge tolerance, at two thirds of the matrix-core work of three planes.
//
// Work split: a workgroup of four wave64s owns a range of 32-token tiles of one
// (layer, batch, head) slice; wave w computes output channels [32w, 32w+32) (one 32-row MFMA
// tile) for the tile's 32 tokens.  The wave keeps its 32 rows of every split plane in VGPRs
// for the whole range, so the matrix core never re-reads G.  Output rows are permuted so
// that lane (token n, half hc) ends up with the 16 consecutive channels 32w + 16hc + [0, 16):
// its codes form one contiguous stretch of the packed row.  Tokens are staged through LDS
// with an XOR swizzle of the 16-byte granules of each 256-byte row, so the B-operand reads
// (lane n reads granule j of row n) hit distinct banks.
//
// Encode epilogue (section 4.3 block-uniform): block minimum / maximum in-lane, across the
// two lane halves (n = 32) and across the wave pair through LDS (n = 64); binary16 side
// information; binary32 quantisation without contraction; LSB-first packing; stores.
//
#include <cstdlib>
#include <type_traits>

#include "cg_internal.h"
#include "cg_device.h"
#include "cg_mfma_util.h"
#include "cg_mfma_common.h"
#include "cg_recode.h"
#include "cg_zfp.h"

namespace cg {

namespace {

constexpr int kStages = 5;       // encoder LDS ring: tiles in flight + the one being read

// Packs 16 codes of BITS bits into 16*BITS/32 words (BITS even) LSB-first.
template <int BITS>
__device__ __forceinline__ void pack16(const uint32_t (&q)[16], uint32_t* out) {
  constexpr int NW = (16 * BITS + 31) / 32;
#pragma unroll
  for (int w = 0; w < NW; ++w) out[w] = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int bit = e * BITS, w = bit >> 5, off = bit & 31;
    out[w] |= q[e] << off;
    if (off + BITS > 32) out[w + 1] |= q[e] >> (32 - off);
  }
}

template <int NW>
__device__ __forceinline__ void store_words(uint32_t* dst, const uint32_t* v) {
  // dst is 4-byte aligned; use the widest aligned vector stores available
  if constexpr (NW == 4) {
    *(u32x4_t*)dst = u32x4_t{v[0], v[1], v[2], v[3]};
  } else if constexpr (NW == 2) {
    *(uint2*)dst = make_uint2(v[0], v[1]);
  } else {
#pragma unroll
    for (int i = 0; i < NW; ++i) dst[i] = v[i];
  }
}

// ------------------------------------------------------------------------------------------
// encode
// ------------------------------------------------------------------------------------------

// z (32 rows x 32 tokens) of one tile: the NP split planes times the tile, one chain.
// TR: the tile as the A operand and the gauge rows as the B operand, so the accumulator holds
// z transposed (lane (n, hc): tokens 8i + 4hc + j of channel row n).
template <int NP, int KS, bool TR = false>
__device__ __forceinline__ f32x16_t mfma_chain(const bf16x8_t (&A)[NP][KS], const bf16x8_t (&Bf)[KS]) {
  f32x16_t acc = {};
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
#pragma unroll
    for (int p = 0; p < NP; ++p) acc = TR ? mfma(Bf[kk], A[p][kk], acc) : mfma(A[p][kk], Bf[kk], acc);
  return acc;
}


// min / max over the 16 lanes of a DPP row (quad swaps, then rotations by 4 and 8 lanes)
__device__ __forceinline__ float row16_min(float v) {
  v = min_nan(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
  v = min_nan(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
  v = min_nan(v, dpp_mov<0x124>(v));  // row_ror:4
  return min_nan(v, dpp_mov<0x128>(v));  // row_ror:8
}
__device__ __forceinline__ float row16_max(float v) {
  v = max_nan(v, dpp_mov<0xB1>(v));
  v = max_nan(v, dpp_mov<0x4E>(v));
  v = max_nan(v, dpp_mov<0x124>(v));
  return max_nan(v, dpp_mov<0x128>(v));
}


// encoder modes
constexpr int kModeBU = 0;     // block-uniform (or KIVI values: n = value channel group)
constexpr int kModePass = 1;   // error-free backend: binary32 z
constexpr int kModeKeys = 2;   // KIVI keys: one block per channel over a 32-token group
constexpr int kModeZfp = 3;    // zfp-style fixed-rate blocks of 4 tokens x 4 channels (BITS = rate)

// Software pipeline over 32-token tiles, one barrier per tile.  Iteration t:
//   1. block-range partials of tile t from its accumulator (64-channel blocks: wave-pair
//      exchange through red[t & 1]);
//   2. wait for tile t+1's LDS-direct loads, barrier, issue the loads of tile t+kStages-1
//      into the buffer tile t-1 used, read the B fragments of tile t+1, write tile t-1's
//      staged codes and side words to the cache as contiguous runs;
//   3. matrix-core chain of tile t+1 interleaved with side info, quantisation and packing of
//      tile t into the staging buffers.
// kStages - 1 tiles are in flight between global memory and LDS.  The codes of a tile are one
// contiguous run of 32 RB bytes in the cache and its side words one run of 32 NBK words, so
// the staged copy leaves with whole-line stores instead of 32 scattered row pieces.
// PAGED: the cache is a page pool; the rows of a tile (always inside one page) go to the page its
// positions map to, looked up one tile ahead of the tile's first use.  Blocks with a non-finite value are
// coded again after the range (recode_rows).
template <int NP, int KS, int BITS, int NB, int MODE, int TB = 1, bool PAGED = false>
__global__ __launch_bounds__(kThreads, NP == 2 ? 3 : 2) void enc_mfma(MfmaArgs a) {
  constexpr bool PASS = MODE == kModePass, KEYS = MODE == kModeKeys, ZFP = MODE == kModeZfp;
  constexpr bool QUANT = !PASS && !ZFP;  // block ranges, staged codes and side words
  // token-channel tiles: one range per TB tokens x NB channels (NB spans whole waves)
  constexpr bool TILE = TB > 1;
  static_assert(!TILE || (TB == 16 && MODE == kModeBU && (NB == 64 || NB == 128)), "tile shape");
  constexpr int RB = kD * BITS / 8;   // packed code bytes per token row
  constexpr int NBK = kD / NB;        // side words per token row (per tile row of tiles)
  // ring depth: the zfp-style coder is bound by its VALU work, so it keeps one tile fewer in
  // flight and gives the LDS to the block transpose below (three workgroups per CU either way)
  constexpr int ST = ZFP ? kStages - 1 : kStages;
  __shared__ __attribute__((aligned(16))) uint8_t xtile[ST][kTok * kRowBytes];
  __shared__ float2 red[2][4][kTok];  // per-wave (min, max) of each token, for 64-channel blocks
  // a tile's packed rows and side words, staged so that they leave as contiguous stores
  __shared__ __attribute__((aligned(16))) uint8_t cstage[2][QUANT ? kTok * RB : 16];
  __shared__ uint32_t sstage[2][QUANT ? kTok * NBK : 1];  // KIVI keys: NB = 32, one word per channel
  __shared__ std::conditional_t<ZFP, ZfpTables, char> ztab;
  // zfp-style: each wave's 32 tokens x 32 channels of z, written by token rows and read back as
  // 4 x 4 blocks by the same wave (LDS operations of a wave complete in order, so no barrier)
  constexpr int QP = 36;  // row pitch in floats (16-byte rows, rows 4 banks apart)
  __shared__ __attribute__((aligned(16))) float zq[ZFP ? 4 : 1][ZFP ? kTok * QP : 4];

  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = lane & 31, hc = lane >> 5;
  const int logical = xcd_remap(blockIdx.x, gridDim.x);
  const int slice = logical / a.chunks, chunk = logical - slice * a.chunks;
  if (slice >= a.nslices) return;
  const int h = slice % a.H, b = (slice / a.H) % a.B, lv = slice / (a.H * a.B);
  const int l = lv + a.l0;
  const int ntiles = (a.T + kTok - 1) / kTok;
  const int tb = chunk * a.tiles_per_wg;
  const int te_all = min(ntiles, tb + a.tiles_per_wg);
  if (tb >= te_all) return;
  // tiles below tq / 32 are quantised (tq is a multiple of 32 for KIVI, T otherwise)
  const int te = min(te_all, (a.tq + kTok - 1) / kTok);

  const char* xs = a.x + 2 * (size_t(lv) * a.sl + size_t(b) * a.sb + size_t(h) * a.sh);
  const size_t cslice = (size_t(l) * a.cB + b) * a.cH + h;
  const int64_t tstride = 2 * a.st;  // bytes between tokens

  // KIVI full-precision window / staged tokens of an unfinished tile: this workgroup's rows
  // at or past tq copied raw into the ring (slot = cache position mod ring_slots)
  auto ring_copy = [&]() {
    constexpr int GR = kRowBytes / 16;  // granules per row
    const int r0 = max(a.tq, tb * kTok), r1 = min(a.T, te_all * kTok);
    for (int gi = r0 * GR + int(threadIdx.x); gi < r1 * GR; gi += kThreads) {
      const int row = gi / GR, j = gi % GR;
      uint16_t* dst = a.ring + (cslice * a.ring_slots + (a.t0 + row) % a.ring_slots) * kD;
      *(u32x4_t*)((char*)dst + 16 * j) = *(const u32x4_t*)(xs + int64_t(row) * tstride + 16 * j);
    }
  };
  if (tb >= te) {
    ring_copy();
    return;
  }
  if constexpr (ZFP) zfp_tables_init(ztab);  // read after the prologue's barrier

  // K range of this wave's rows: the group of channels 32w.. (whole head for g = 128)
  const int kbase = a.g >= 32 ? (32 * w / a.g) * a.g : 32 * w;
  // A row m of this wave computes output channel 32w + 16*((m/4)%2) + 4*(m/8) + m%4
  const int chA = 32 * w + 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  bf16x8_t A[NP][KS];
  load_a<NP, KS>(A, a, l, h, chA, kbase, hc);

  // Tiles stream global -> LDS without VGPRs (LDS-direct loads): wave w moves rows
  // 8w .. 8w+7 of a tile with two 1 KB instructions whose lanes write consecutive 16-byte
  // LDS granules; lane l of instruction q fetches the logical granule that the XOR swizzle
  // puts at physical granule l % 16 of row 8w + 4q + l / 16.
  const int wu = __builtin_amdgcn_readfirstlane(w);  // the wave index as a scalar
  int drow[2];
  const char* dsrc[2];  // this lane's source granule in tile 0
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    drow[q] = 8 * w + 4 * q + (lane >> 4);
    dsrc[q] = xs + drow[q] * tstride + 16 * swz(drow[q], lane & 15);
  }
  auto issue = [&](int tile) {
    uint8_t* dst = xtile[(tile - tb) % ST] + 8 * wu * kRowBytes;
    if ((tile + 1) * kTok <= a.T) {
      const int64_t off = int64_t(tile) * kTok * tstride;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        __builtin_amdgcn_global_load_lds(dsrc[q] + off, (__attribute__((address_space(3))) void*)(dst + 4 * q * kRowBytes),
                                         16, 0, kLoadStreamPolicy);
    } else {
      // ragged last tile: rows past the view repeat its last token
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int tok = min(tile * kTok + drow[q], a.T - 1);
        __builtin_amdgcn_global_load_lds(dsrc[q] + (int64_t(tok) - drow[q]) * tstride,
                                         (__attribute__((address_space(3))) void*)(dst + 4 * q * kRowBytes), 16, 0,
                                         kLoadStreamPolicy);
      }
    }
  };
  // Before a barrier: wait until this wave's loads of tile X have landed while the loads of
  // tiles X+1 .. I (the last one issued) may stay in flight, and until its LDS writes are
  // done.  VMEM operations complete in issue order; stores issued after those loads only make
  // the count stricter.
  auto wait_tile = [&](int X, int I) {
    switch (I - X) {
      case 0: __builtin_amdgcn_s_waitcnt(waitcnt_imm(0)); break;
      case 1: __builtin_amdgcn_s_waitcnt(waitcnt_imm(2)); break;
      case 2: __builtin_amdgcn_s_waitcnt(waitcnt_imm(4)); break;
      case 3: __builtin_amdgcn_s_waitcnt(waitcnt_imm(6)); break;
      default: __builtin_amdgcn_s_waitcnt(waitcnt_imm(8)); break;
    }
  };
  int boff[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) boff[kk] = n * kRowBytes + 16 * swz(n, (kbase >> 3) + 2 * kk + hc);
  bf16x8_t Bf[KS];
  auto bfrags = [&](int tile) {
    const uint8_t* src = xtile[(tile - tb) % ST];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) Bf[kk] = as_bf16x8(*(const u32x4_t*)(src + boff[kk]));
  };

  // prologue: tiles tb .. tb+ST-2 in flight, tile tb on the matrix core
  for (int t = tb; t < min(te, tb + ST - 1); ++t) issue(t);
  wait_tile(tb, min(te - 1, tb + ST - 2));
  __builtin_amdgcn_s_barrier();
  bfrags(tb);
  f32x16_t acc[2];
  acc[0] = mfma_chain<NP, KS, KEYS>(A, Bf);
  int flags = 0;
  // cache row of tile t's first token: positions t0 + 32 t of the row, or of its page (-1: outside
  // the table or the pool); paged caches keep the rows of the tile being flushed and of this one
  auto page_of = [&](int tile) {
    const int lp = (a.t0 + tile * kTok) / a.T_cap;
    return lp < a.max_pages ? a.pages[size_t(b) * a.max_pages + lp] : -1;
  };
  auto page_row = [&](int tile, int pg) {
    if (pg < 0 || pg >= a.cB) return int64_t(-1);
    return int64_t((size_t(l) * a.cB + pg) * a.cH + h) * a.T_cap + (a.t0 + tile * kTok) % a.T_cap;
  };
  int64_t prow[2] = {-1, -1};
  __shared__ int recode;  // PAGED: the workgroup met a non-finite z
  if constexpr (PAGED) {
    if (threadIdx.x == 0) recode = 0;  // a barrier follows in every step
  }
  if constexpr (PAGED) prow[0] = page_row(tb, page_of(tb));
  // staged tile -> cache: thread i stores 16-byte granule i of the codes (row i / BITS) and,
  // counting from the last thread, side word i (row i / NBK); rows past the view are skipped
  auto flush = [&](int tile, auto parity) {
    constexpr int P = decltype(parity)::value;
    const int tid = int(threadIdx.x);
    const int nlive = min(a.T, a.tq) - tile * kTok;  // quantised rows of the tile
    if (PAGED && prow[P] < 0) return;
    const size_t crow0 = PAGED ? size_t(prow[P]) : cslice * a.T_cap + size_t(a.t0 + tile * kTok);
    if (tid < kTok * BITS && tid / BITS < nlive)
      *(u32x4_t*)(a.codes + crow0 * RB + 16 * tid) = *(const u32x4_t*)(cstage[P] + 16 * tid);
    // side words: one per (row, block), or per (tile of TB rows, block); t0 % TB == 0
    const int si = kThreads - 1 - tid;
    if (si < (kTok / TB) * NBK && (si / NBK) * TB < nlive) a.side[crow0 / TB * NBK + si] = sstage[P][si];
  };
  // one pipeline step; P = parity of (tile - tb) selects the accumulator, LDS buffer, register
  // stage and exchange slot at compile time
  auto step = [&](int tile, auto parity) {
    constexpr int P = decltype(parity)::value;
    float z[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = acc[P][e];
    const int tok = tile * kTok + n;
    bool live = tok < (TILE ? a.tq : a.T);
    int pg_next = -1;
    if constexpr (PAGED) {
      live = live && prow[P] >= 0;
      if (prow[P] < 0) flags |= CG_FLAG_POS_RANGE;
    }
    const size_t crow = cslice * a.T_cap + size_t(a.t0 + tok);

    // 1. block-range partials (NaN-propagating: a NaN anywhere in the block reaches the range)
    float mn = z[0], mx = z[0];
    if constexpr (QUANT) {
#pragma unroll
      for (int e = 1; e < 16; ++e) {
        mn = min_nan(mn, z[e]);
        mx = max_nan(mx, z[e]);
      }
      if constexpr (TILE) {  // the 16 tokens of the lane's tile: one DPP row
        mn = row16_min(mn);
        mx = row16_max(mx);
      }
      if constexpr (NB >= 32) halves_minmax(mn, mx);
      if constexpr (TILE) {
        if (hc == 0 && (n & 15) == 0) red[P][w][n >> 4] = make_float2(mn, mx);
      } else if constexpr (NB == 64) {
        if (hc == 0) red[P][w][n] = make_float2(mn, mx);
      }
    }
    // 2. tile+1 landed in every wave (and every wave is done with tile-1's buffer), refill
    //    that buffer with tile+ST-1, read tile+1's B fragments
    if (tile + 1 < te) wait_tile(tile + 1, min(te - 1, tile + ST - 2));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(63));  // LDS writes only
    __builtin_amdgcn_s_barrier();
    if (tile + ST - 1 < te) issue(tile + ST - 1);
    if constexpr (PAGED) {
      if (tile + 1 < te) pg_next = page_of(tile + 1);  // used once this tile is staged
    }
    bfrags(tile + 1);
    if constexpr (QUANT) {
      if (tile > tb) flush(tile - 1, std::integral_constant<int, P ^ 1>());
    }
    // 5. next tile on the matrix core (past the range it reads a stale buffer and is unused),
    //    this tile's epilogue on the VALU; no branch until the stores
    acc[P ^ 1] = mfma_chain<NP, KS, KEYS>(A, Bf);

    if constexpr (ZFP) {
      // the lane's 4 x 4 block of this tile, through the wave's LDS region: tokens
      // 4(n/4) .. +3 x channels 32w + 16hc + 4(n%4) .. +3; range, transform and top planes
      // alongside the chain, then the planes (blocks past the view, at token counts that are
      // multiples of 4, are skipped)
      (void)live;
      float* zw = zq[w];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(float4*)(zw + n * QP + 16 * hc + 4 * q) = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
      __builtin_amdgcn_wave_barrier();  // keep the reads after the writes
      float v[16];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 t = *(const float4*)(zw + (4 * (n >> 2) + j) * QP + 16 * hc + 4 * (n & 3));
        v[4 * j] = t.x; v[4 * j + 1] = t.y; v[4 * j + 2] = t.z; v[4 * j + 3] = t.w;
      }
      ZfpPrep zp;
      zfp_prepare(v, zp);
#pragma unroll
      for (int i = 0; i < KS * NP; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 20, 0);
      }
      if (tile * kTok + 4 * (n >> 2) < a.T) {
        uint32_t wd[4];
        flags |= zfp_encode_planes<BITS>(zp, ztab, wd);
        const size_t blk = (cslice * size_t(a.T_cap / 4) + (a.t0 + tile * kTok) / 4 + (n >> 2)) * (kD / 4) +
                           8 * w + 4 * hc + (n & 3);
        zfp_store<BITS>(a.codes + blk * (2 * BITS), wd);
      }
    } else if constexpr (PASS) {
#pragma unroll
      for (int i = 0; i < KS * NP; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
      }
      if (live) {
        float* dst = (float*)a.codes + crow * kD + 32 * w + 16 * hc;
#pragma unroll
        for (int q = 0; q < 4; ++q) *(float4*)(dst + 4 * q) = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
      }
    } else if constexpr (KEYS) {
      // z^T: lane (n, hc) holds tokens 8i + 4hc + j (e = 4i + j) of channel chA; the block is
      // the channel over the tile's 32 tokens (in-lane 16 + the other half-wave's 16)
      const bool bad = !(mn >= -3.0e38f && mx <= 3.0e38f);  // NaN or +-inf in the block
      const Side sd = make_side<true>(mn, mx, BITS);
      // the channel's LSB-first stream of 32 codes in token order (BITS words): this lane's
      // codes placed as if hc = 0 (token 8i + j at bit (8i + j) BITS), shifted by 4 BITS bits
      // for hc = 1, then the two half-wave patterns OR-ed together
      uint32_t words[BITS];
#pragma unroll
      for (int i = 0; i < BITS; ++i) words[i] = 0;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t q = code_u8(quantize_t(z[e], sd.mn, sd.inv));
        const int bit = (8 * (e >> 2) + (e & 3)) * BITS, wd = bit >> 5, off = bit & 31;
        words[wd] |= q << off;
        if (off + BITS > 32) words[wd + 1] |= q >> (32 - off);
      }
      if (hc) {
        constexpr int SH = 4 * BITS;  // <= 32
#pragma unroll
        for (int i = BITS - 1; i >= 0; --i) {
          const uint32_t lo = i > 0 ? words[i - 1] : 0u;
          words[i] = SH == 32 ? lo : ((words[i] << (SH & 31)) | (lo >> ((32 - SH) & 31)));
        }
      }
#pragma unroll
      for (int i = 0; i < BITS; ++i) {  // both half-waves' patterns (v_permlane32_swap: own and partner's)
        const auto u = __builtin_amdgcn_permlane32_swap(words[i], words[i], false, false);
        words[i] = u[0] | u[1];
      }
#pragma unroll
      for (int i = 0; i < BITS; ++i) asm volatile("" ::"v"(words[i]));
      asm volatile("" ::"v"(sd.word));
#pragma unroll
      for (int i = 0; i < KS * NP; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
      }
      if (hc == 0) {
        store_words<BITS>((uint32_t*)(cstage[P] + chA * 4 * BITS), words);
        sstage[P][chA] = sd.word;
      }
      flags |= sd.flags | (bad ? CG_FLAG_NONFINITE : 0);
    } else {
      if constexpr (TILE) {  // the other waves of the tile's channel block
#pragma unroll
        for (int o = 1; o < NB / 32; ++o) {
          const float2 v = red[P][w ^ o][n >> 4];
          mn = min_nan(mn, v.x);
          mx = max_nan(mx, v.y);
        }
      } else if constexpr (NB == 64) {
        const float2 o = red[P][w ^ 1][n];
        mn = min_nan(mn, o.x);
        mx = max_nan(mx, o.y);
      }
      const bool bad = !(mn >= -3.0e38f && mx <= 3.0e38f);  // NaN or +-inf in the block
      const Side sd = make_side<true>(mn, mx, BITS);
      float r[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        // v_cvt_pk_u8_f32 below rounds to nearest even (packing bytes, or code_u8)
        r[e] = quantize_t(z[e], sd.mn, sd.inv);
      }
      constexpr int NW = (BITS & 1) ? BITS : BITS / 2;  // words this lane stores
      uint32_t words[NW];
      // v_cvt_pk_u8_f32 rounds to nearest even (the quantiser's rint) and saturates to
      // [0, 255] (codes are in [0, 2^b - 1] by construction of the side information); bytes
      // then go to b-bit fields of the LSB-first stream
      auto pk4 = [](float c0, float c1, float c2, float c3) {
        uint32_t v = __builtin_amdgcn_cvt_pk_u8_f32(c0, 0, 0u);
        v = __builtin_amdgcn_cvt_pk_u8_f32(c1, 1, v);
        v = __builtin_amdgcn_cvt_pk_u8_f32(c2, 2, v);
        return __builtin_amdgcn_cvt_pk_u8_f32(c3, 3, v);
      };
      if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) words[i] = pk4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]);
      } else if constexpr (BITS == 4) {
        // byte j of the word holds codes 2j (low nibble) and 2j+1 (high nibble)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float* c = r + 8 * i;
          words[i] = pk4(c[0], c[2], c[4], c[6]) | (pk4(c[1], c[3], c[5], c[7]) << 4);
        }
      } else if constexpr (BITS == 2) {
        // byte j holds codes 4j .. 4j+3 in 2-bit fields
        words[0] = pk4(r[0], r[4], r[8], r[12]) | (pk4(r[1], r[5], r[9], r[13]) << 2) |
                   (pk4(r[2], r[6], r[10], r[14]) << 4) | (pk4(r[3], r[7], r[11], r[15]) << 6);
      } else {
        uint32_t q[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) q[e] = code_u8(r[e]);
        if constexpr (BITS == 6) {
          pack16<BITS>(q, words);
        } else {
          // 16 odd-width codes span 1.5 words: the lane packs its own 16, the upper half-wave's words
          // cross over (v_permlane32_swap), and the lower half joins and stores the 32 codes' BITS words
          static_assert(BITS == 3, "odd widths");
          uint32_t own[2];
          pack16<BITS>(q, own);
          const auto u0 = __builtin_amdgcn_permlane32_swap(own[0], own[0], false, false);
          const auto u1 = __builtin_amdgcn_permlane32_swap(own[1], own[1], false, false);
          words[0] = own[0];
          words[1] = own[1] | (u0[1] << 16);
          words[2] = (u0[1] >> 16) | (u1[1] << 16);
        }
      }
      // keep the epilogue in this block (not sunk into the store branch) so the scheduler can
      // interleave it with the matrix-core chain
#pragma unroll
      for (int i = 0; i < NW; ++i) asm volatile("" ::"v"(words[i]));
      asm volatile("" ::"v"(sd.word));
#pragma unroll
      for (int i = 0; i < KS * NP; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
      }
      uint8_t* crowp = cstage[P] + n * RB;
      if constexpr ((BITS & 1) == 0) {
        store_words<NW>((uint32_t*)(crowp + (4 * w + 2 * hc) * BITS), words);
      } else if (hc == 0) {
        uint32_t* dst = (uint32_t*)(crowp + (4 * w) * BITS);
#pragma unroll
        for (int i = 0; i < BITS; ++i) dst[i] = words[i];
      }
      if (live) flags |= PAGED ? (bad ? kFlagRecode : sd.flags) : (sd.flags | (bad ? CG_FLAG_NONFINITE : 0));
      if constexpr (TILE) {
        if (hc == 0 && (n & 15) == 0 && w % (NB / 32) == 0) sstage[P][(n >> 4) * NBK + w / (NB / 32)] = sd.word;
      } else if constexpr (NB == 16) {
        sstage[P][n * NBK + 2 * w + hc] = sd.word;
      } else if constexpr (NB == 32) {
        if (hc == 0) sstage[P][n * NBK + w] = sd.word;
      } else {
        if (hc == 0 && (w & 1) == 0) sstage[P][n * NBK + (w >> 1)] = sd.word;
      }
    }
    if constexpr (PAGED) prow[P ^ 1] = page_row(tile + 1, pg_next);
  };
  for (int tile = tb; tile < te; tile += 2) {
    step(tile, std::integral_constant<int, 0>());
    if (tile + 1 < te) step(tile + 1, std::integral_constant<int, 1>());
  }
  if constexpr (QUANT) {
    // the last tile's staging: every wave's LDS writes done, then the final contiguous stores
    if (PAGED && (flags & kFlagRecode)) recode = 1;
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(63));
    __builtin_amdgcn_s_barrier();
    if ((te - tb) & 1) flush(te - 1, std::integral_constant<int, 0>());
    else flush(te - 1, std::integral_constant<int, 1>());
  }
  if constexpr (PAGED) {
    if (recode) {
      flags &= ~kFlagRecode;
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(0));  // this wave's stores, before those over them
      for (int tile = tb; tile < te; ++tile) {
        const int64_t row = page_row(tile, page_of(tile));
        if (row < 0) continue;
        flags |= recode_rows(xs + int64_t(tile) * kTok * tstride, tstride, min(kTok, a.T - tile * kTok), kD, NB, BITS,
                             a.g32 + ((size_t(l) * 2 + a.s) * a.Hg + h) * a.R * a.g * a.g, a.g,
                             a.codes + size_t(row) * RB, a.side + size_t(row) * NBK, (int*)xtile[0], (float*)xtile[1]);
      }
    }
  } else {
    ring_copy();
  }
  if (flags && a.err) atomicOr(a.err, flags);
}

// Split planes of the gauge on the matrix core.  Decoding takes two (16 significant bits per
// entry: a few 1e-6 of the group norm).  Encoding takes two up to 4-bit codes and three
// above: a finer grid turns the same z error into more codes moved across a rounding
// boundary (with two planes about 3e-5 of 4-bit codes but 1.4e-4 of 6-bit codes move, against
// the 1e-4 budget).
constexpr int enc_planes(int bits) { return bits >= 6 ? 3 : 2; }

template <int KS, int BITS, int NB>
void* enc_kernel(int mode, int bt) {
  if (mode == kModePass) return (void*)enc_mfma<kNP, KS, 8, 64, kModePass>;
  if (mode == kModeZfp) return NB == 64 ? (void*)enc_mfma<kNP, KS, BITS, 64, kModeZfp> : nullptr;
  if (mode == kModeKeys) return (void*)enc_mfma<enc_planes(BITS), KS, BITS, 32, kModeKeys>;
  if constexpr (NB >= 64) {
    if (bt == 16) return (void*)enc_mfma<enc_planes(BITS), KS, BITS, NB, kModeBU, 16>;
  }
  if constexpr (NB <= 64) {
    if (bt == 1) return (void*)enc_mfma<enc_planes(BITS), KS, BITS, NB, kModeBU>;
  }
  return nullptr;
}

// Paged caches take three planes at every width: their encoder was the binary32 FMA chain, and three
// planes (24 significant bits of every entry) keep z closer to the binary64 product than that chain does
// (relative error 1.2e-7 against 2.0e-7 at g = 128, 0.7e-7 against 1.0e-7 at g = 32).  8 layers x 4 rows x
// 8 heads x 2000 tokens in 256-position pages, g = 128, 4 bits: 1058 us per tensor on the vector ALU, 236
// on the binary32 matrix cores (the general kernel, which other shapes keep), 70 here.
constexpr int kModePaged = 4;

template <int KS, int BITS>
void* enc_by_nb(int nb, int mode, int bt) {
  if (mode == kModePaged) {
    switch (nb) {
      case 16: return (void*)enc_mfma<3, KS, BITS, 16, kModeBU, 1, true>;
      case 32: return (void*)enc_mfma<3, KS, BITS, 32, kModeBU, 1, true>;
      case 64: return (void*)enc_mfma<3, KS, BITS, 64, kModeBU, 1, true>;
    }
    return nullptr;
  }
  switch (nb) {
    case 16: return enc_kernel<KS, BITS, 16>(mode, bt);
    case 32: return enc_kernel<KS, BITS, 32>(mode, bt);
    case 64: return enc_kernel<KS, BITS, 64>(mode, bt);
    case 128: return enc_kernel<KS, BITS, 128>(mode, bt);
  }
  return nullptr;
}

template <int KS>
void* enc_by_bits(int bits, int nb, int mode, int bt) {
  switch (bits) {
    case 2: return enc_by_nb<KS, 2>(nb, mode, bt);
    case 3: return enc_by_nb<KS, 3>(nb, mode, bt);
    case 4: return enc_by_nb<KS, 4>(nb, mode, bt);
    case 6: return enc_by_nb<KS, 6>(nb, mode, bt);
    case 8: return enc_by_nb<KS, 8>(nb, mode, bt);
  }
  return nullptr;
}

}  // namespace

bool mfma_encode_supported(const ViewDev& X, const GaugeDev& G, const CodecDev& c, bool paged) {
  if (!X.bf16 || X.d != kD || !group_ok(G.g)) return false;
  if (paged && c.backend != CG_BACKEND_BLOCK_UNIFORM) return false;  // the error-free backend: general kernels
  if (c.backend == CG_BACKEND_PASSTHROUGH) return true;
  if (c.backend == CG_BACKEND_ZFP) return bits_ok(c.bits);
  if (c.backend == CG_BACKEND_KIVI)
    return bits_ok(c.bits) && c.kg == kTok && (c.kvc == 16 || c.kvc == 32 || c.kvc == 64) && c.win % kTok == 0;
  if (c.backend != CG_BACKEND_BLOCK_UNIFORM || !bits_ok(c.bits)) return false;
  if (c.bt == 16) return c.n == 64 || c.n == 128;  // token-channel tiles
  return c.bt == 1 && (c.n == 16 || c.n == 32 || c.n == 64);
}

hipError_t launch_encode_mfma(int s, const ViewDev& X, int l0, const GaugeDev& G, const CodecDev& c,
                              const CacheDev& k, int t0, int tq, int* err, hipStream_t st, const PageDev& pt) {
  if (X.T == 0) return hipSuccess;
  MfmaArgs m{};
  m.x = (char*)X.ptr;
  m.sl = X.sl; m.sb = X.sb; m.sh = X.sh; m.st = X.st;
  m.L = X.L; m.B = X.B; m.H = X.H; m.T = X.T;
  m.l0 = l0; m.s = s; m.t0 = t0;
  for (int p = 0; p < 3; ++p) m.gp[p] = G.hi[p];
  m.g32 = G.f32; m.g = G.g; m.R = G.R; m.Hg = G.H;
  m.codes = k.codes; m.side = k.side; m.T_cap = k.T_cap; m.cB = k.B; m.cH = k.H;
  m.err = err;
  const bool pass = c.backend == CG_BACKEND_PASSTHROUGH, kivi = c.backend == CG_BACKEND_KIVI;
  const bool zfp = c.backend == CG_BACKEND_ZFP;
  const bool tiles = c.backend == CG_BACKEND_BLOCK_UNIFORM && c.bt > 1;
  m.tq = kivi || tiles ? tq : X.T;
  m.ring = k.ring;
  m.ring_slots = kivi ? c.win + c.kg : (tiles ? c.bt : 0);
  m.pages = pt.pages;
  m.max_pages = pt.max_pages;
  const int mode = pt.pages ? kModePaged : pass ? kModePass : (zfp ? kModeZfp : (kivi && s == 0 ? kModeKeys : kModeBU));
  const int nb = pass || zfp ? 64 : (kivi ? c.kvc : c.n), bits = pass ? 8 : c.bits, bt = tiles ? c.bt : 1;
  void* fn = nullptr;
  switch (ksteps(G.g)) {
    case 2: fn = enc_by_bits<2>(bits, nb, mode, bt); break;
    case 4: fn = enc_by_bits<4>(bits, nb, mode, bt); break;
    case 8: fn = enc_by_bits<8>(bits, nb, mode, bt); break;
  }
  if (!fn) return hipErrorInvalidValue;
  plan(m, X.L * X.B * X.H, X.T, fn);
  const int nwg = ((m.nslices * m.chunks + 7) / 8) * 8;
  void* args[] = {&m};
  return hipLaunchKernel(fn, dim3(nwg), dim3(kThreads), args, 0, st);
}

}  // namespace cg
