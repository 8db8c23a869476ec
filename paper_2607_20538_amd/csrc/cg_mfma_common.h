// What the bf16 matrix-core encoder and decoders share (one copy per translation unit): kernel
// arguments, the gauge operand, split of the work into workgroups.
#pragma once

#include <cstdlib>
#include <type_traits>

#include "cg_internal.h"
#include "cg_device.h"
#include "cg_mfma_util.h"

namespace cg {

namespace {

constexpr int kNP = kDecPlanes;  // split planes of the gauge a decoder multiplies

struct MfmaArgs {
  // view (input for encode, output for decode)
  char* x;
  int64_t sl, sb, sh, st;        // element strides
  int L, B, H, T;                // view dims (L = layers of the view)
  int l0;                        // cache layer of view layer 0
  int s;                         // 0 keys, 1 values
  int t0;                        // cache position of view token 0
  // gauge planes ([nblk][g][g] bf16) and binary32 blocks
  const uint16_t* gp[3];
  const float* g32;
  const float* cs8;              // decoder column sums per 8-channel segment [head][d/8][d]
  int g, R;                      // group size, groups per head
  int Hg;                        // heads of the gauge shape
  // cache
  uint8_t* codes;
  uint32_t* side;
  int T_cap, cB, cH;             // cache capacity and dims
  // KIVI: tokens [0, tq) are quantised, [tq, T) go raw into the ring of ring_slots rows;
  // the decoders derive tq from the positions the cache holds (len, or pos[b] + 1)
  int tq, ring_slots;
  uint16_t* ring;
  int kivi, win, kg, len;
  // paged encode: the page of batch row b's positions [i P, (i + 1) P) is pages[b max_pages + i], and
  // T_cap = P = page_size, cB = pages of the pool
  const int* pages;
  int max_pages;
  // work split
  int nslices, chunks, tiles_per_wg;
  // decode only: batch row b holds positions [0, pos[b] + pos_add) (rolling step: pos_add = 1,
  // the row's newest position; per-row lengths: pos_add = 0); NULL: every row holds `len`
  const int* pos;
  int pos_add;
  int* err;
};


// Load the wave's A fragments: plane p, K-step kk: 8 bf16 of row `ch` (an output channel of
// this wave) at input channels j0..j0+7 of the full block-diagonal matrix (zero outside the
// row's group).  `tr` selects G^T planes (decode).
template <int NP, int KS>
__device__ void load_a(bf16x8_t (&A)[NP][KS], const MfmaArgs& a, int l, int h, int ch, int kbase, int kh) {
  const int g = a.g;
  const int r = ch / g;
  const size_t blk = ((size_t(l) * 2 + a.s) * a.Hg + h) * a.R + r;
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const int j0 = kbase + 16 * kk + 8 * kh;
    const bool in_group = (j0 / g) == r;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (in_group) v = *(const u32x4_t*)(a.gp[p] + blk * g * g + size_t(ch % g) * g + (j0 % g));
      A[p][kk] = as_bf16x8(v);
    }
  }
}

// Split the (slice, tile) space into workgroups: as many as can be resident at once (the
// kernel's occupancy per CU times the CUs), each a contiguous tile range of one slice; the
// count is padded to a multiple of 8 (XCD remap).
//
// CG_TILES_PER_WG=k (read at every launch) fixes the tiles per workgroup instead, so that small
// inputs run the multi-tile pipeline (ring wrap, prefetch, overlapped flush, exact waits) that
// the resident grid only reaches on large ones; the tests compare both geometries.
inline int forced_tiles_per_wg() {
  const char* e = getenv("CG_TILES_PER_WG");
  if (!e || !*e) return 0;
  const long v = strtol(e, nullptr, 10);
  return v > 0 && v < (1 << 20) ? int(v) : 0;
}

inline void plan(MfmaArgs& m, int nslices, int T, const void* fn) {
  const int ntiles = (T + kTok - 1) / kTok;
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, kThreads, 0) != hipSuccess || occ < 1) occ = 2;
  const int target = occ * cu_count();
  int chunks = (target + nslices - 1) / nslices;
  chunks = chunks < 1 ? 1 : (chunks > ntiles ? ntiles : chunks);
  m.tiles_per_wg = (ntiles + chunks - 1) / chunks;
  if (const int f = forced_tiles_per_wg()) m.tiles_per_wg = f < ntiles ? f : (ntiles > 0 ? ntiles : 1);
  m.chunks = (ntiles + m.tiles_per_wg - 1) / m.tiles_per_wg;
  m.nslices = nslices;
}

inline int ksteps(int g) { return g >= 128 ? 8 : (g == 64 ? 4 : 2); }

inline bool group_ok(int g) { return g == 8 || g == 16 || g == 32 || g == 64 || g == 128; }

inline bool bits_ok(int b) { return b == 2 || b == 3 || b == 4 || b == 6 || b == 8; }

}  // namespace
}  // namespace cg
