// Passes over rows that are not in the cache yet: the continual-compression
// loop over a stretch of resident frames (Algorithm 1).
//
// Appending every frame and compacting at every pass moves a row that is kept
// for P passes P + 1 times and a dropped row once, and reads each value once
// per pass although its norm never changes. Here the rows of a stretch stay
// where they are while its passes run: a pass reads new rows from the frame
// buffers, old rows through an index (`src`), and its selection compacts the
// metadata, the index and the value norms only. After a stream's last pass of
// the call one gather writes the surviving rows into the cache.
// 7B-class cache, 16 new frames a pass: about 1.08 GB of traffic a pass before
// (append 360 MB, sweeps 360, compaction 360), 270 MB for a pass without the
// gather now, 360 MB more for the pass that ends with it. Measured: a 16x16
// video of 192 frames (7 passes, 112 slices of 12288 rows) 2915 -> 1114 us a
// call, a 64-frame 7B-class clip in calls of 16 frames 720 -> 557 us, a 172-frame
// 72B-class clip (one pass) 8.41 -> 4.49 ms; with the later changes to the
// selection, the tile order and the launches 1046 us, 560 us and 4.12 ms.
//
// Row x of a slice is "old" (x < n0: it was a row of the slice before the
// stretch's pending frames) or "new" (row x - n0 of the pending frames). An old
// row's place is src[x]: s >= 0 is cache row s, s < 0 is row ~s of the call's
// frames (frame ~s / rows); without an index (the first pass of a call) it is
// cache row x. The metadata of new rows is arithmetic and is never stored
// before the selection keeps them.
#pragma once

#include "ipv_adjacent.hpp"
#include "ipv_compact.hpp"
#include "ipv_scores.hpp"

namespace ipv {

// The address of row `s` (a src value) of `slice`: cache / frames are K's or
// V's base pointers (slice 0 of the launch).
template <uint32_t RB>
__device__ __forceinline__ const char* row_place(const char* cache, const char* frames, const Stretch& st, int64_t S,
                                                 uint32_t slice, int32_t s) {
  const uint32_t e = (uint32_t)~s;
  const uint32_t f = fast_div(e, st.rows);
  const char* in_frame = frames + (int64_t)f * st.stride + ((int64_t)slice * st.rows.d + (e - f * st.rows.d)) * RB;
  const char* in_cache = cache + ((int64_t)slice * S + s) * RB;
  return s < 0 ? in_frame : in_cache;
}

// One address per lane quad member, handed to the quad by DPP: lane l of a
// quad computes the place of the lane group's row l % 4.
template <int CTRL>
__device__ __forceinline__ const char* dpp_ptr(uint64_t p) {
  const uint32_t lo = dpp_u32<CTRL>((uint32_t)p), hi = dpp_u32<CTRL>((uint32_t)(p >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ Raw16 load16_stream(const char* p) {
  const U32x4 v = __builtin_nontemporal_load(reinterpret_cast<const U32x4*>(p));
  return Raw16{{v[0], v[1], v[2], v[3]}};
}

// ---------------------------------------------------------------- recent-key table
// When the window lies wholly in the new frames (more new frames than r: every
// old row is then older than the window unless frame ids decrease, which the
// selection reports), the key of recent frame j at position q is known without
// a scan. Otherwise the window's metadata is scanned as in table_block.
// CLOSED: known on the host (slot may then be null).
template <typename T, int D, int NT, bool CLOSED = false>
__device__ __forceinline__ void stretch_table_block(const char* __restrict__ K, const Stretch& st,
                                                    const int32_t* __restrict__ frame_idx,
                                                    const int32_t* __restrict__ patch_idx, int64_t S, int32_t n,
                                                    int32_t r, int32_t p, uint32_t slice, int32_t q0,
                                                    float* __restrict__ table, int32_t* __restrict__ first_recent,
                                                    uint32_t* err, int32_t* slot) {
  constexpr int EPL = Lane<T>::EPL, LPR = D / EPL, GROUPS = NT / LPR;
  constexpr uint32_t RB = D * (uint32_t)sizeof(T);
  const int tid = threadIdx.x, g = tid / LPR, lane = tid % LPR;
  const int32_t q1 = min(p, q0 + GROUPS), q = q0 + g;
  const int64_t base = (int64_t)slice * S;
  const int32_t rows = (int32_t)st.rows.d, n0 = (int32_t)st.n0;
  const int32_t new_frames = (int32_t)fast_div((uint32_t)(n - n0), st.rows);
  const bool closed = CLOSED || new_frames > r;
  if (closed) {
    if (q0 == 0 && tid == 0) first_recent[slice] = n - r * rows;
  } else {
    const int32_t thr_frame = st.frame_of(n - 1);
    const int64_t thr = (int64_t)thr_frame - r + 1;
    const int32_t t0 = (int32_t)max((int64_t)0, (int64_t)n - (int64_t)r * p);
    for (int i = tid; i < GROUPS * r; i += NT) slot[i] = -1;
    __syncthreads();
    uint32_t ebits = 0;
    for (int32_t t = t0 + tid; t < n; t += NT) {
      const bool nw = t >= n0;
      const int32_t f = nw ? st.frame_of(t) : frame_idx[base + t];
      const int32_t pq = nw ? st.patch_of(t) : patch_idx[base + t];
      const int32_t before = t - 1;
      const int32_t fprev = before < t0 ? INT32_MIN : before >= n0 ? st.frame_of(before) : frame_idx[base + before];
      if (f < thr) continue;
      if (q0 == 0 && (t == t0 || fprev < thr)) first_recent[slice] = t;
      const int64_t fo = (int64_t)f - thr;
      if (pq < 0 || pq >= p) {
        ebits |= 1u;
      } else if (fo >= r) {
        ebits |= 2u;
      } else if (pq >= q0 && pq < q1) {
        if (atomicExch(&slot[(pq - q0) * r + fo], t) != -1) ebits |= 2u;
      }
    }
    if (ebits) raise_error(err, ebits);
    __syncthreads();
  }
  if (q >= q1) return;
  float acc[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) acc[i] = 0.f;
  int cnt = 0;
  // batches of 4 independent key loads, summed in frame order
  for (int j0 = 0; j0 < r; j0 += 4) {
    Raw16 raw[4];
    bool have[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int j = j0 + b;
      int32_t s;
      if (closed) {
        have[b] = j < r && q >= st.patch0 && q < st.patch0 + rows;
        s = ~(int32_t)(st.eoff + (uint32_t)(n - (r - j) * rows + q - st.patch0));
      } else {
        const int32_t y = j < r ? slot[g * r + j] : -1;
        have[b] = y >= 0;
        s = y >= n0 ? ~(int32_t)(st.eoff + (uint32_t)y) : st.src ? st.src[(int64_t)slice * st.src_stride + max(y, 0)] : y;
      }
      if (have[b]) raw[b] = load16(row_place<RB>(K, st.K, st, S, slice, s) + lane * 16);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (!have[b]) continue;  // uniform within the lane group
      ++cnt;
      float f[EPL];
      Lane<T>::decode(raw[b], f);
      const float ss = group_sum<LPR>(Lane<T>::sumsq(raw[b]));
      const float inv = ss > 0.f ? fast_rsqrt(ss) : 0.f;
#pragma unroll
      for (int i = 0; i < EPL; ++i) acc[i] = __builtin_fmaf(f[i], inv, acc[i]);
    }
  }
  const float scale = cnt ? 1.f / (float)cnt : 0.f;
  float* out = table + ((int64_t)slice * p + q) * D + lane * EPL;
#pragma unroll
  for (int i = 0; i < EPL; i += 4)
    *reinterpret_cast<float4*>(out + i) = make_float4(acc[i] * scale, acc[i + 1] * scale, acc[i + 2] * scale,
                                                      acc[i + 3] * scale);
}

// ---------------------------------------------------------------- value norms
// A slice's norms to compute: rows [v0, n) (v0 = n0: the old rows' norms are in
// van already; v0 = 0: all rows), 4 * GROUPS consecutive rows a tile. TILES
// tiles from x0 on are in flight together.
template <typename T, int D, int TILES = 1>
__device__ __forceinline__ void stretch_van_tile(const char* __restrict__ V, const Stretch& st, int64_t S, uint32_t n,
                                                 float* __restrict__ van, uint32_t slice, uint32_t x0, int tid) {
  using C = SweepCfg<T, D>;
  constexpr int LPR = C::LPR, GROUPS = C::GROUPS, U = C::U;
  constexpr uint32_t RB = D * (uint32_t)sizeof(T), ROWS = GROUPS * U;
  const uint32_t g = (uint32_t)(tid / LPR);
  const int lane = tid % LPR;
  const uint32_t lo = (uint32_t)lane * 16u;
  Raw16 v[TILES][U];
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    // lane l's own row is row l % 4 of its group; rows past n read row n - 1
    const uint32_t xm = min(x0 + t * ROWS + (uint32_t)(lane & 3) * GROUPS + g, n - 1);
    const int32_t old = st.src && xm < st.n0 ? st.src[(int64_t)slice * st.src_stride + xm] : (int32_t)xm;
    const int32_t s = xm < st.n0 ? old : ~(int32_t)(st.eoff + xm);
    const uint64_t mine = reinterpret_cast<uint64_t>(row_place<RB>(V, st.V, st, S, slice, s));
    v[t][0] = load16_stream(dpp_ptr<0x00>(mine) + lo);
    v[t][1] = load16_stream(dpp_ptr<0x55>(mine) + lo);
    v[t][2] = load16_stream(dpp_ptr<0xAA>(mine) + lo);
    v[t][3] = load16_stream(dpp_ptr<0xFF>(mine) + lo);
  }
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    float part[U][1], tot[1];
#pragma unroll
    for (int u = 0; u < U; ++u) part[u][0] = Lane<T>::sumsq(v[t][u]);
    reduce_scatter4<LPR, 1>(part, tot, lane);
    constexpr int Q = (LPR > 16 ? 16 : LPR) / 4;
    const uint32_t x = x0 + t * ROWS + (uint32_t)scatter_row<LPR>(lane) * GROUPS + g;
    if (lane < 16 && lane % Q == 0 && x < n) van[(int64_t)slice * S + x] = fast_sqrt(tot[0]);
  }
}

// Recent-key table blocks first, then the VaN tiles (as in k_table_van).
// tiles: VaN tiles per slice; v0: first row they cover.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_stretch_table_van(const char* __restrict__ K, const char* __restrict__ V,
                                                           Stretch st, const int32_t* __restrict__ frame_idx,
                                                           const int32_t* __restrict__ patch_idx, int64_t S, int32_t n,
                                                           int32_t r, int32_t p, FastDiv blocks_per_slice,
                                                           uint32_t table_padded, uint32_t table_real,
                                                           float* __restrict__ table,
                                                           int32_t* __restrict__ first_recent, uint32_t* err,
                                                           uint32_t* __restrict__ zero, int32_t zero_per_slice,
                                                           float* __restrict__ van, uint32_t v0, FastDiv tiles,
                                                           FastDiv vslices, uint32_t n_work, uint32_t tile_blocks) {
  extern __shared__ int32_t slot[];
  constexpr int GROUPS = 256 / (D / Lane<T>::EPL);
  if (blockIdx.x < table_padded) {
    if (blockIdx.x >= table_real) return;
    const uint32_t slice = fast_div(blockIdx.x, blocks_per_slice);
    const int32_t q0 = (int32_t)(blockIdx.x - slice * blocks_per_slice.d) * GROUPS;
    if (zero && q0 == 0)
      for (int i = threadIdx.x; i < zero_per_slice; i += 256) zero[(int64_t)slice * zero_per_slice + i] = 0u;
    stretch_table_block<T, D, 256>(K, st, frame_idx, patch_idx, S, n, r, p, slice, q0, table, first_recent, err, slot);
    return;
  }
  const uint32_t logical = xcd_logical_id(blockIdx.x - table_padded, tile_blocks);
  if (logical >= n_work) return;
  uint32_t slice, t;
  if (v0 >= st.n0) {  // frames only: neighbouring slices in turn (640 slices of 12288 rows 1514 -> 1481 us a call)
    t = fast_div(logical, vslices);
    slice = logical - t * vslices.d;
  } else {
    slice = fast_div(logical, tiles);
    t = logical - slice * tiles.d;
  }
  stretch_van_tile<T, D>(V, st, S, (uint32_t)n, van, slice, v0 + t * (GROUPS * 4), threadIdx.x);
}

// ---------------------------------------------------------------- TaR rows
template <int EPL>
__device__ __forceinline__ void load_m(const __amdgpu_buffer_rsrc_t& mrs, uint32_t off, float4 (&m)[EPL / 4]) {
#pragma unroll
  for (int i = 0; i < EPL / 4; ++i) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(mrs, off + 16u * i, 0, 0);
    m[i] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
  }
}

// Old rows [x0, x0 + 4 * GROUPS) of a slice, in row order. After a compaction
// neighbouring rows rarely share a patch position, so each row takes its own m
// vector; patch ids and places are read first, then the four keys and m
// vectors of a lane group are in flight together.
template <typename T, int D>
__device__ __forceinline__ void stretch_tar_old(const char* __restrict__ K, const Stretch& st,
                                                const int32_t* __restrict__ patch_idx, int64_t S, uint32_t p,
                                                const float* __restrict__ table, uint32_t rec, float* __restrict__ tar,
                                                uint32_t* err, uint32_t slice, uint32_t x0, int tid) {
  using C = SweepCfg<T, D>;
  constexpr int EPL = C::EPL, LPR = C::LPR, GROUPS = C::GROUPS, U = C::U;
  constexpr uint32_t RB = D * (uint32_t)sizeof(T);
  constexpr uint32_t kSkip = 0xfffffff0u;
  const uint32_t g = (uint32_t)(tid / LPR);
  const int lane = tid % LPR;
  const int64_t base = (int64_t)slice * S;
  const uint32_t past_end = min(st.n0, rec);
  const uint32_t xm = x0 + (uint32_t)(lane & 3) * GROUPS + g;
  const bool past_m = xm < past_end;
  const uint32_t xc = past_m ? xm : 0u;
  const int32_t q_m = patch_idx[base + xc];
  const int32_t s_m = st.src ? st.src[(int64_t)slice * st.src_stride + xc] : (int32_t)xc;
  const bool ok_m = past_m && q_m >= 0 && q_m < (int32_t)p;
  if (past_m && !ok_m && lane < 4) raise_error(err, 1u);
  const uint64_t mine = reinterpret_cast<uint64_t>(row_place<RB>(K, st.K, st, S, slice, s_m));
  const uint32_t lo = (uint32_t)lane * 16u;
  // rows without a score read row 0's key and a zero m vector
  const uint32_t moff_m = ok_m ? (uint32_t)q_m * (D * 4u) : kSkip;
  const __amdgpu_buffer_rsrc_t mrs = buffer_rsrc(table + (int64_t)slice * p * D, p * D * 4u);
  const char* kp[U] = {dpp_ptr<0x00>(mine), dpp_ptr<0x55>(mine), dpp_ptr<0xAA>(mine), dpp_ptr<0xFF>(mine)};
  const uint32_t mo[U] = {dpp_u32<0x00>(moff_m), dpp_u32<0x55>(moff_m), dpp_u32<0xAA>(moff_m), dpp_u32<0xFF>(moff_m)};
  Raw16 k[U];
  float4 m[U][EPL / 4];
#pragma unroll
  for (int u = 0; u < U; ++u) k[u] = load16_stream(kp[u] + lo);
#pragma unroll
  for (int u = 0; u < U; ++u) load_m<EPL>(mrs, mo[u] == kSkip ? kSkip - 64u : mo[u] + (uint32_t)lane * (EPL * 4u), m[u]);
  float part[U][2], tot[2];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    tar_parts<T>(k[u], m[u], part[u]);
    if (mo[u] == kSkip) part[u][0] = part[u][1] = 0.f;
  }
  reduce_scatter4<LPR, 2>(part, tot, lane);
  constexpr int Q = (LPR > 16 ? 16 : LPR) / 4;
  const uint32_t x = x0 + (uint32_t)scatter_row<LPR>(lane) * GROUPS + g;
  if (lane < 16 && lane % Q == 0 && x < st.n0) tar[base + x] = x < past_end ? tar_score(tot) : 0.f;
}

// New rows: GROUPS columns of 4 pending frames from `f`. A column's patch
// position is the same in every frame, so its m vector is read once.
// ahead (may be null): patch_idx, where the row's norm waits (ipv_ahead.hpp); it
// goes to van, and the row's patch id takes its place.
__device__ __forceinline__ void take_norm(int32_t* __restrict__ ahead, float* __restrict__ van, const Stretch& st,
                                          int64_t at, uint32_t x) {
  van[at] = __int_as_float(ahead[at]);
  ahead[at] = st.patch_of(x);
}

template <typename T, int D>
__device__ __forceinline__ void stretch_tar_new(const Stretch& st, int64_t S, uint32_t n, uint32_t p,
                                                const float* __restrict__ table, uint32_t rec, float* __restrict__ tar,
                                                int32_t* __restrict__ ahead, float* __restrict__ van, uint32_t slice,
                                                uint32_t f, uint32_t colblock, int tid) {
  using C = SweepCfg<T, D>;
  constexpr int EPL = C::EPL, LPR = C::LPR, GROUPS = C::GROUPS, U = C::U;
  constexpr uint32_t RB = D * (uint32_t)sizeof(T);
  constexpr uint32_t kSkip = 0xfffffff0u;
  const uint32_t col = colblock * GROUPS + (uint32_t)(tid / LPR), rows = st.rows.d;
  const int lane = tid % LPR;
  if (col >= rows) return;  // the whole lane group idles: it is in no cross-lane sum
  const uint32_t x0 = st.n0 + f * rows + col, past_end = min(n, rec);
  Raw16 k[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    // one frame of one slice is contiguous; frames past the last and recent ones read nothing
    const __amdgpu_buffer_rsrc_t krs =
        buffer_rsrc(st.K + (int64_t)(st.f0 + f + u) * st.stride + (int64_t)slice * rows * RB, rows * RB);
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(
        krs, x0 + u * rows < past_end ? col * RB + (uint32_t)lane * 16u : kSkip, 0, kNontemporal);
    k[u] = Raw16{{v[0], v[1], v[2], v[3]}};
  }
  float4 m[EPL / 4];
  const __amdgpu_buffer_rsrc_t mrs = buffer_rsrc(table + (int64_t)slice * p * D, p * D * 4u);
  const uint32_t q = (uint32_t)st.patch0 + col;
  load_m<EPL>(mrs, x0 < past_end ? (q * D + (uint32_t)lane * EPL) * 4u : kSkip - 64u, m);
  float part[U][2], tot[2];
#pragma unroll
  for (int u = 0; u < U; ++u) tar_parts<T>(k[u], m, part[u]);
  reduce_scatter4<LPR, 2>(part, tot, lane);
  constexpr int Q = (LPR > 16 ? 16 : LPR) / 4;
  const uint32_t x = x0 + (uint32_t)scatter_row<LPR>(lane) * rows;
  if (lane < 16 && lane % Q == 0 && x < n) {
    const int64_t at = (int64_t)slice * S + x;
    tar[at] = x < past_end ? tar_score(tot) : 0.f;
    if (ahead) take_norm(ahead, van, st, at, x);
  }
}

// Frames of all slices lie one after another, so tiles that run together read
// nearby memory when neighbouring slices take the same tile in turn. The TaR
// tiles of a pass without old rows go 1, 2, 4 or 8 slices at a time (log2 here): as
// many as have m tables of 1.2 MB together (an XCD's L2 holds 4 MB and the keys
// stream through it), and 7 groups to an XCD at least (an XCD takes a run of slices,
// and the groups that two of them share have their tables in both). A call with one
// pass and its gather, us, 1 / 2 / 4 / 8 / 16 slices at a time:
//   112 slices, tables of 100 KB   171 / 168 / 169 / 173 / 172
//   640 slices                    4081 / 4062 / 4039 / 4029 / 4079
//   112 slices, 131 KB             291 / 287 / 292 / 300 / 296
//   640 slices                    1518 / 1500 / 1490 / 1479 / 1506
//   640 slices, 295 KB            2363 / 2357 / 2356 / 2376 / 2406
//   112 slices, 590 KB             415 / 416 / 421 / 431 / 435
//   320 slices                    2290 / 2291 / 2307 / 2371 / 2376
//   224 slices, 25 KB              583 / 586 / 568 / 563 / 568
// Old rows are strewn over their slice's table, and only that one stays in L2 with
// them: one slice at a time (75 us a pass of the 16x16 video, 78 us with 8 in turn).
inline uint32_t slice_group(uint32_t slices, uint32_t table_bytes) {
  uint32_t g = 0;
  while (g < 3 && slices / 56u >= 2u << g && (2u << g) * (uint64_t)table_bytes <= 1200000u) ++g;
  return g;
}

// The TaR launch of a pass, with the pooling CV blocks first (cv_padded = 0:
// none). tiles: tiles per slice, the first old_tiles of them over the old rows.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_stretch_tar(const char* __restrict__ K, Stretch st,
                                                     const int32_t* patch_idx, int32_t* ahead, int64_t S, int32_t n,
                                                     int32_t p, const float* __restrict__ table,
                                                     const int32_t* __restrict__ first_recent, float* __restrict__ tar,
                                                     uint32_t* err, FastDiv tiles, uint32_t old_tiles, FastDiv col_blocks,
                                                     uint32_t n_work, uint32_t tile_blocks, uint32_t slices,
                                                     uint32_t group, int32_t sure_past, float* van, int32_t H,
                                                     double tau1, double tau2, double tau3,
                                                     int32_t* __restrict__ pool_ws, uint32_t cv_padded,
                                                     uint32_t cv_real) {
  __shared__ double red[256 / kWave];
  if (blockIdx.x < cv_padded) {
    if (blockIdx.x < cv_real)
      pool_cv_block<256>(van, S, n, H, tau1, tau2, tau3, pool_ws, nullptr, blockIdx.x, threadIdx.x, red);
    return;
  }
  using C = SweepCfg<T, D>;
  const uint32_t logical = xcd_logical_id(blockIdx.x - cv_padded, tile_blocks);
  if (logical >= n_work) return;
  // 1 << group slices take their tiles in turn
  const uint32_t turn = logical >> group, grp = fast_div(turn, tiles), t = turn - grp * tiles.d;
  const uint32_t slice = (grp << group) + (logical & ((1u << group) - 1u));
  if (slice >= slices) return;
  if (t < old_tiles) {
    const uint32_t x0 = t * (C::GROUPS * C::U);
    const bool tail = (int64_t)x0 + C::GROUPS * C::U > sure_past;
    const uint32_t rec = tail ? (uint32_t)first_recent[slice] : (uint32_t)n;
    stretch_tar_old<T, D>(K, st, patch_idx, S, (uint32_t)p, table, rec, tar, err, slice, x0, threadIdx.x);
  } else {
    const uint32_t fb = fast_div(t - old_tiles, col_blocks), cb = t - old_tiles - fb * col_blocks.d;
    const bool tail = (int64_t)st.n0 + (int64_t)(fb + 1) * C::U * st.rows.d > sure_past;
    const uint32_t rec = tail ? (uint32_t)first_recent[slice] : (uint32_t)n;
    stretch_tar_new<T, D>(st, S, (uint32_t)n, (uint32_t)p, table, rec, tar, ahead, van, slice, fb * C::U, cb,
                          threadIdx.x);
  }
}

// ---------------------------------------------------------------- consecutive-frame TaR
// Prev-row walks first, then four VaN tiles to a block (as in k_prev_van).
template <typename T, int D>
__global__ __launch_bounds__(kPrevThreads) void k_stretch_prev_van(const char* __restrict__ V, Stretch st,
    const int32_t* __restrict__ frame_idx, const int32_t* __restrict__ patch_idx, int64_t S, int32_t n, int32_t r,
    int32_t p, int32_t* __restrict__ prev, int32_t* __restrict__ first_recent, uint32_t* err,
    uint32_t* __restrict__ zero, int32_t zero_per_slice, uint32_t prev_padded, uint32_t slices, float* __restrict__ van,
    uint32_t v0, FastDiv tiles, uint32_t n_work, uint32_t tile_blocks) {
  if (blockIdx.x < prev_padded) {
    if (blockIdx.x < slices)
      prev_rows_block(blockIdx.x, frame_idx, patch_idx, S, n, r, p, prev, first_recent, err, zero, zero_per_slice, st);
    return;
  }
  constexpr int GROUPS = SweepCfg<T, D>::GROUPS;
  const uint32_t logical = xcd_logical_id(blockIdx.x - prev_padded, tile_blocks) * 4u + threadIdx.x / 256u;
  if (logical >= n_work) return;
  const uint32_t slice = fast_div(logical, tiles);
  stretch_van_tile<T, D>(V, st, S, (uint32_t)n, van, slice, v0 + (logical - slice * tiles.d) * (GROUPS * 4),
                         threadIdx.x % 256u);
}

// As k_adjacent_sweep, with both keys found through the index.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_stretch_adjacent(const char* __restrict__ K, Stretch st,
                                                          const int32_t* __restrict__ prev, int64_t S, int32_t n,
                                                          const int32_t* __restrict__ first_recent,
                                                          float* __restrict__ tar, int32_t* ahead, float* van,
                                                          FastDiv tiles, uint32_t n_work, uint32_t tile_blocks) {
  using C = SweepCfg<T, D>;
  constexpr int LPR = C::LPR, GROUPS = C::GROUPS, U = C::U;
  constexpr uint32_t RB = D * (uint32_t)sizeof(T);
  const uint32_t logical = xcd_logical_id(blockIdx.x, tile_blocks);
  if (logical >= n_work) return;
  const uint32_t slice = fast_div(logical, tiles), x0 = (logical - slice * tiles.d) * (GROUPS * U);
  const uint32_t g = threadIdx.x / LPR;
  const int lane = threadIdx.x % LPR;
  const int64_t base = (int64_t)slice * S;
  const uint32_t past_end = min((uint32_t)n, (uint32_t)first_recent[slice]);
  const int32_t* src = st.src ? st.src + (int64_t)slice * st.src_stride : nullptr;
  auto place = [&](uint32_t x) {
    const int32_t old = src && x < st.n0 ? src[x] : (int32_t)x;
    const int32_t s = x < st.n0 ? old : ~(int32_t)(st.eoff + x);
    return reinterpret_cast<uint64_t>(row_place<RB>(K, st.K, st, S, slice, s));
  };
  const uint32_t xm = x0 + (uint32_t)(lane & 3) * GROUPS + g;
  const bool past_m = xm < past_end;
  const uint32_t xc = past_m ? xm : 0u;
  const int32_t yl = prev[base + xc];
  const int32_t y_m = past_m ? yl : -1;
  const uint64_t px = place(xc), py = place(y_m >= 0 ? (uint32_t)y_m : 0u);
  const uint32_t lo = (uint32_t)lane * 16u;
  const bool has[U] = {(int32_t)dpp_u32<0x00>((uint32_t)y_m) >= 0, (int32_t)dpp_u32<0x55>((uint32_t)y_m) >= 0,
                       (int32_t)dpp_u32<0xAA>((uint32_t)y_m) >= 0, (int32_t)dpp_u32<0xFF>((uint32_t)y_m) >= 0};
  const Raw16 kx[U] = {load16(dpp_ptr<0x00>(px) + lo), load16(dpp_ptr<0x55>(px) + lo), load16(dpp_ptr<0xAA>(px) + lo),
                       load16(dpp_ptr<0xFF>(px) + lo)};
  const Raw16 ky[U] = {load16(dpp_ptr<0x00>(py) + lo), load16(dpp_ptr<0x55>(py) + lo), load16(dpp_ptr<0xAA>(py) + lo),
                       load16(dpp_ptr<0xFF>(py) + lo)};
  float tsc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const float dot = group_sum<LPR>(Lane<T>::dot(kx[u], ky[u]));
    const float aa = group_sum<LPR>(Lane<T>::sumsq(kx[u]));
    const float cc = group_sum<LPR>(Lane<T>::sumsq(ky[u]));
    float sc = (has[u] && aa != 0.f && cc != 0.f) ? -(dot * fast_rsqrt(aa) * fast_rsqrt(cc)) : 0.f;  // NaN stays NaN
    if (sc == 0.f) sc = 0.f;  // -0.0 -> +0.0
    tsc[u] = sc;
  }
  if (lane < U) {
    const uint32_t x = x0 + lane * GROUPS + g;
    if (x < (uint32_t)n) {
      tar[base + x] = lane == 0 ? tsc[0] : lane == 1 ? tsc[1] : lane == 2 ? tsc[2] : tsc[3];
      if (ahead && x >= st.n0) take_norm(ahead, van, st, base + x, x);
    }
  }
}

// ---------------------------------------------------------------- gather
// After a stream's last pass: cache row j <- row src[j] for j < C, K and V
// (the metadata is in place already). The walks, chunks, ticket and flags are
// those of k_compact: only cache rows are sources that a store can overwrite,
// they come before the frame rows in row order and their src values ascend, so
// src[j] >= j for them. HAZARD false: no row was in the cache before the call,
// nothing to wait for and no ticket. n_entry: cache rows there were.
template <int RB, int NT, int CHR, int CBMAX, bool HAZARD>
__global__ __launch_bounds__(NT) void k_stretch_gather(char* __restrict__ K, char* __restrict__ V, Stretch st,
                                                       const int32_t* __restrict__ src, int64_t S, int32_t n_entry,
                                                       int32_t budget, uint32_t* err, uint32_t* flags,
                                                       uint32_t n_chunks, FastDiv walks) {
  using C = CompactCfg<RB, NT, CHR, CBMAX>;
  constexpr int LPP = C::LPP, RPS = C::RPS, U = C::U, CH = C::CH, PARTS = 2 * C::NCB;
  __shared__ uint32_t ticket, ok_all;
  const uint32_t kexp = fast_div(blockIdx.x, walks), w = blockIdx.x - kexp * walks.d;
  const uint32_t slice = w / PARTS, part = w % PARTS;
  const int tid = threadIdx.x, sub = tid / LPP, lane = tid % LPP;
  uint32_t* wflags = flags + (int64_t)w * walk_words(n_chunks);
  uint32_t drawn = 0;
  if (HAZARD && tid == 0) drawn = atomicAdd(&wflags[n_chunks], 1u);
  char* cache = part < C::NCB ? K : V;
  const char* frames = part < C::NCB ? st.K : st.V;
  const uint32_t col = (part % C::NCB) * C::CB + lane * 16;
  char* base = cache + (int64_t)slice * S * RB;
  const int32_t* from = src + (int64_t)slice * S;
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(from, (uint32_t)budget * 4u);
  Raw16 buf[U];
  bool move[U];
  auto load_chunk = [&](uint32_t k) {
    const uint32_t c0 = k * CH, c1 = min((uint32_t)budget, c0 + CH);
    int32_t s[U];
#pragma unroll
    for (int u = 0; u < U; ++u)  // past the chunk's end: its first row, not stored
      s[u] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(
          srs, (c0 + u * RPS + sub < c1 ? c0 + u * RPS + sub : c0) * 4u, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = c0 + u * RPS + sub;
      move[u] = j < c1 && s[u] != (int32_t)j;
      buf[u] = load16_stream(row_place<RB>(cache, frames, st, S, slice, s[u]) + col);
    }
    // wait here for every loaded register (the barrier that follows then
    // covers the loads of every wave)
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" ::"v"(buf[u].w[0]));
  };
  load_chunk(kexp);
  uint32_t k = kexp;
  if (HAZARD) {
    if (tid == 0) ticket = drawn;
    __syncthreads();
    k = ticket;
    if (k >= n_chunks) {  // the counter was not zero: a workspace shared by overlapping calls
      if (tid == 0) raise_error(err, 32u);
      return;
    }
    if (k != kexp) {
      load_chunk(k);
      __syncthreads();
    }
    const int32_t c0 = (int32_t)(k * CH), c1 = min(budget, c0 + CH);
    if (tid == 0) store_flag(&wflags[k], 1u);
    if (tid < kWave) {
      bool ok = true;
      for (uint32_t j0 = 0; j0 < k && ok; j0 += kWave) {
        const uint32_t jc = j0 + tid;
        bool need = false;
        if (jc < k) {
          const int32_t lo = from[(int64_t)jc * CH];
          const int32_t last = from[min((int64_t)budget, (int64_t)(jc + 1) * CH) - 1];
          need = lo >= 0 && (last < 0 ? n_entry - 1 : last) >= c0 && lo < c1;
        }
        for (uint32_t spins = 0;; ++spins) {
          const bool pending = need && load_flag(&wflags[jc]) == 0u;
          if (__ballot(pending) == 0) break;
          if (spins >= kSpinLimit) {
            ok = false;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      if (tid == 0) ok_all = ok;
    }
    __syncthreads();
    if (!ok_all) {
      if (tid == 0) raise_error(err, 32u);
      return;
    }
  }
  const uint32_t c0 = k * CH;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (move[u]) store16(base + (int64_t)(c0 + u * RPS + sub) * RB + col, buf[u]);
}

}  // namespace ipv
