// The selection of one pass of a stretch beside the first launch of the next.
//
// A selection is one workgroup per slice, bound by its barriers: most of the
// chip idles through it. What the next pass needs first does not depend on its
// outcome: the value norms of the frames that come next, and the recent-key
// table, if the window lies in those frames. So these run in the selection's
// launch, on the CUs it leaves. 16x16 video (7 passes, 112 slices of 12288
// rows): selection 26.6 us and the next table + VaN launch 41 us apart, 54 us
// together (58 with one tile in flight, the same with four); 1114 -> 1056 us a call.
//
// The norms cannot go to `van`, which the selection reads: they wait in the rows
// of patch_idx that the next pass's new rows will have. The metadata of a
// stretch's new rows is arithmetic, so nothing else is there; the next pass's
// TaR launch moves each norm to `van` and stores the row's patch id in its place.
#pragma once

#include "ipv_select.hpp"
#include "ipv_stretch.hpp"

namespace ipv {

// The next pass's first launch.
struct Ahead {
  const char *K, *V;  // the cache (its rows are not read: every row is in the frames)
  int32_t kind;       // element type and head size: kind_of
  Stretch st;         // the next pass's
  int32_t n, r, p;
  float* norm;        // patch_idx as floats
  FastDiv slices;
  uint32_t n_work, tile_blocks;
  float* table;       // null: no table (the consecutive-frame mode)
  FastDiv table_blocks;
  uint32_t table_real, table_padded;
  int32_t* first_recent;
  uint32_t* zero;
  int32_t zero_per_slice;
  uint32_t sel_padded, sel_real;
};

constexpr int kAheadThreads = 1024;
// The selection's registers leave room for one of these blocks on a CU, half the
// waves a launch of its own would have, so each has twice the loads in flight.
constexpr int kAheadTiles = 2;

// One kernel serves every element type and head size (a uniform branch), so that
// the selection's own variants are not multiplied by them.
constexpr int kind_of(bool bf16, int64_t D) { return (bf16 ? 0 : 4) + (D == 32 ? 0 : D == 64 ? 1 : D == 128 ? 2 : 3); }

// Block `i` of the next pass's first launch: as k_stretch_table_van, four times
// kAheadTiles VaN tiles to a block.
template <typename T, int D>
__device__ __forceinline__ void ahead_block(const Ahead& a, const int32_t* frame_idx, const int32_t* patch_idx,
                                            int64_t S, uint32_t* err, uint32_t i) {
  using C = SweepCfg<T, D>;
  if (i < a.table_padded) {
    if (i >= a.table_real) return;
    constexpr int GROUPS = kAheadThreads / C::LPR;
    const uint32_t slice = fast_div(i, a.table_blocks);
    const int32_t q0 = (int32_t)(i - slice * a.table_blocks.d) * GROUPS;
    if (a.zero && q0 == 0)
      for (int j = threadIdx.x; j < a.zero_per_slice; j += kAheadThreads) a.zero[(int64_t)slice * a.zero_per_slice + j] = 0u;
    // the window lies in the frames (the host has checked): no scan, no slots
    stretch_table_block<T, D, kAheadThreads, true>(a.K, a.st, frame_idx, patch_idx, S, a.n, a.r, a.p, slice, q0, a.table,
                                                   a.first_recent, err, nullptr);
    return;
  }
  const uint32_t logical = xcd_logical_id(i - a.table_padded, a.tile_blocks) * 4u + threadIdx.x / 256u;
  if (logical >= a.n_work) return;
  const uint32_t t = fast_div(logical, a.slices), slice = logical - t * a.slices.d;
  stretch_van_tile<T, D, kAheadTiles>(a.V, a.st, S, (uint32_t)a.n, a.norm, slice,
                                      a.st.n0 + t * (C::GROUPS * C::U * kAheadTiles), threadIdx.x % 256u);
}

// Selection blocks first (those at or past sel_real return at once); sel_padded
// is a multiple of 8, so the rest map to XCDs as in a launch of their own.
template <int RPT, bool VEC>
__global__ __launch_bounds__(kAheadThreads) void k_select_ahead(const float* __restrict__ tar,
                                                                const float* van, const int32_t* frame_idx,
                                                                const int32_t* patch_idx, int64_t S,
                                                                int32_t n, int32_t budget, int32_t tar_total, int32_t r,
                                                                uint32_t* err, int32_t heads, uint32_t tflip,
                                                                uint32_t vflip, Stretch st, Emit em, Ahead a) {
  __shared__ SelShared<kAheadThreads> sh;
  if (blockIdx.x < a.sel_padded) {
    if (blockIdx.x < a.sel_real)
      select_slice<kAheadThreads, RPT, VEC>(tar, van, frame_idx, S, n, budget, tar_total, r, nullptr, err,
                                            (int64_t)blockIdx.x * heads, heads, tflip, vflip, sh, st, em);
    return;
  }
  const uint32_t i = blockIdx.x - a.sel_padded;
  switch (a.kind) {
    case kind_of(true, 32): return ahead_block<uint16_t, 32>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(true, 64): return ahead_block<uint16_t, 64>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(true, 128): return ahead_block<uint16_t, 128>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(true, 256): return ahead_block<uint16_t, 256>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(false, 32): return ahead_block<float, 32>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(false, 64): return ahead_block<float, 64>(a, frame_idx, patch_idx, S, err, i);
    case kind_of(false, 128): return ahead_block<float, 128>(a, frame_idx, patch_idx, S, err, i);
    default: return ahead_block<float, 256>(a, frame_idx, patch_idx, S, err, i);
  }
}

}  // namespace ipv
