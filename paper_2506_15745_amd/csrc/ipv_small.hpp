// A whole pass over small slices in one launch, one workgroup per slice.
//
// A pass over a few hundred rows is bound by its launches: every kernel works
// for 2-4 us and the chain of them waits for the one before (host: about 3 us
// a launch). A slice's steps depend on that slice only, so one workgroup takes
// them in turn with barriers between: the recent-key table, the VaN and TaR
// tiles, the selection, and the move of the kept rows, each by the code of the
// large launches and so with the same bits. What one workgroup loses against
// many is bandwidth, so the slice has to be small: see small_pass().
//
// Scores and the table go through global memory (the workgroup's own L1);
// no kernel argument is `__restrict__`, so that the compiler does not take them for
// constants and read them through the scalar cache. (The steps' functions hold the
// qualifier over their own extent, where it is true.)
#pragma once

#include "ipv_select.hpp"
#include "ipv_stretch.hpp"

namespace ipv {

constexpr int kSmallThreads = 1024;
constexpr int kSmallRows = 256;  // most rows of a slice (a thread holds one in the selection and the metadata's move)

// A word that a wave of this workgroup stored before the last barrier (a vector load).
__device__ __forceinline__ int32_t published(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// K and V rows: row j <- row from(j) for j < budget, in place. Sources lie at or
// after their row and ascend among the rows that are in place (see k_compact),
// so ascending batches, each loaded before any of it is stored, overwrite
// nothing that is still to be read.
template <int RB, typename From>
__device__ __forceinline__ void small_move(char* K, char* V, int32_t budget, From from) {
  constexpr int NT = kSmallThreads, LPP = RB / 16, RPS = NT / LPP, U = 2;
  const int sub = threadIdx.x / LPP, lane = threadIdx.x % LPP;
  for (int32_t j0 = 0; j0 < budget; j0 += RPS * U) {
    Raw16 k[U], v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t j = min(j0 + u * RPS + sub, budget - 1);
      k[u] = load16(from(j, false) + lane * 16);
      v[u] = load16(from(j, true) + lane * 16);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      asm volatile("" ::"v"(k[u].w[0]), "v"(k[u].w[1]), "v"(k[u].w[2]), "v"(k[u].w[3]), "v"(v[u].w[0]), "v"(v[u].w[1]),
                   "v"(v[u].w[2]), "v"(v[u].w[3]));
    __syncthreads();  // every wave's loads of this batch have landed
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t j = j0 + u * RPS + sub;
      if (j >= budget) continue;
      store16(K + (int64_t)j * RB + lane * 16, k[u]);
      store16(V + (int64_t)j * RB + lane * 16, v[u]);
    }
  }
}

// Rows in the cache (Whole, Ragged): scores, keep set and compaction.
template <typename T, int D, class ST>
__global__ __launch_bounds__(kSmallThreads) void k_small_pass(char* K, char* V, int32_t* frame_idx, int32_t* patch_idx,
                                                              int64_t S, int32_t n, int32_t r, int32_t p, int32_t budget,
                                                              int32_t tar_total, float* table, int32_t* first_recent,
                                                              float* tar, float* van, int32_t* keep_idx, uint32_t* err,
                                                              uint32_t tflip, uint32_t vflip, ST st) {
  using C = SweepCfg<T, D>;
  constexpr int TG = kSmallThreads / C::LPR, RB = D * (int)sizeof(T);
  extern __shared__ int32_t slot[];
  __shared__ SelShared<kSmallThreads> sh;
  const uint32_t slice = blockIdx.x;
  const int tid = threadIdx.x;
  n = slice_rows(st, n, slice);
  if (ST::kRagged && n == 0) return;
  const T* k = reinterpret_cast<const T*>(K);
  const T* v = reinterpret_cast<const T*>(V);
  for (int32_t q0 = 0; q0 < p; q0 += TG) {
    if (q0) __syncthreads();  // the slots are free
    table_block<T, D, kSmallThreads>(k, frame_idx, patch_idx, S, n, r, p, slice, q0, table, first_recent, err, slot);
  }
  const uint32_t cols = (uint32_t)(p + C::GROUPS - 1) / C::GROUPS;
  const uint32_t tiles = ((uint32_t)(n + p - 1) / p + C::U - 1) / C::U * cols;
  for (uint32_t t = tid / 256; t < tiles; t += kSmallThreads / 256)
    sweep_tile<T, D, false, true>(k, v, patch_idx, S, (uint32_t)n, (uint32_t)p, table, (uint32_t)n, nullptr, van, err,
                                  slice, t / cols * C::U, t % cols, tid % 256);
  __syncthreads();
  const uint32_t rec = (uint32_t)published(first_recent + slice);
  for (uint32_t t = tid / 256; t < tiles; t += kSmallThreads / 256)
    sweep_tile<T, D, true, false>(k, v, patch_idx, S, (uint32_t)n, (uint32_t)p, table, rec, tar, nullptr, err, slice,
                                  t / cols * C::U, t % cols, tid % 256);
  __syncthreads();
  select_slice<kSmallThreads, 1, false>(tar, van, frame_idx, S, n, budget, tar_total, r, keep_idx, err, slice, 1, tflip,
                                        vflip, sh, st, NoEmit{});
  __syncthreads();
  // the keep set still stands in the stage; the metadata first (one row a thread)
  auto row = [&](int32_t j) { return min((uint32_t)sh.stage[j], (uint32_t)n - 1u); };
  int32_t* fr = frame_idx + slice * S;
  int32_t* pa = patch_idx + slice * S;
  const uint32_t x = row(min(tid, budget - 1));
  const int32_t f = fr[x], q = pa[x];
  asm volatile("" ::"v"(f), "v"(q));
  __syncthreads();
  if (tid < budget) {
    fr[tid] = f;
    pa[tid] = q;
  }
  char* kd = K + (int64_t)slice * S * RB;
  char* vd = V + (int64_t)slice * S * RB;
  small_move<RB>(kd, vd, budget, [&](int32_t j, bool val) { return (val ? vd : kd) + (int64_t)row(j) * RB; });
}

// A pass of a stretch of resident frames. gather: the stream's last pass of the
// call, whose rows also go into the cache. The places are then kept in LDS:
// the workspace's place for them is the table region, which other workgroups
// still read.
template <typename T, int D>
__global__ __launch_bounds__(kSmallThreads) void k_small_stretch(char* K, char* V, Stretch st, int32_t* frame_idx,
                                                                 int32_t* patch_idx, int64_t S, int32_t n, int32_t r,
                                                                 int32_t p, int32_t budget, int32_t tar_total,
                                                                 float* table, int32_t* first_recent, float* tar,
                                                                 float* van, uint32_t v0, uint32_t* err, uint32_t tflip,
                                                                 uint32_t vflip, Emit em, bool gather) {
  using C = SweepCfg<T, D>;
  constexpr int TG = kSmallThreads / C::LPR, RB = D * (int)sizeof(T);
  constexpr uint32_t TILE = C::GROUPS * C::U;
  extern __shared__ int32_t slot[];
  __shared__ SelShared<kSmallThreads> sh;
  __shared__ int32_t places[kSmallRows];
  const uint32_t slice = blockIdx.x;
  const int tid = threadIdx.x;
  for (int32_t q0 = 0; q0 < p; q0 += TG) {
    if (q0) __syncthreads();  // the slots are free
    stretch_table_block<T, D, kSmallThreads>(K, st, frame_idx, patch_idx, S, n, r, p, slice, q0, table, first_recent, err,
                                             slot);
  }
  for (uint32_t x0 = v0 + tid / 256 * TILE; x0 < (uint32_t)n; x0 += kSmallThreads / 256 * TILE)
    stretch_van_tile<T, D>(V, st, S, (uint32_t)n, van, slice, x0, tid % 256);
  __syncthreads();
  const uint32_t rec = (uint32_t)published(first_recent + slice), rows = st.rows.d;
  for (uint32_t x0 = tid / 256 * TILE; x0 < st.n0; x0 += kSmallThreads / 256 * TILE)
    stretch_tar_old<T, D>(K, st, patch_idx, S, (uint32_t)p, table, rec, tar, err, slice, x0, tid % 256);
  const uint32_t cols = (rows + C::GROUPS - 1) / C::GROUPS;
  const uint32_t tiles = (((uint32_t)n - st.n0) / rows + C::U - 1) / C::U * cols;
  for (uint32_t t = tid / 256; t < tiles; t += kSmallThreads / 256)
    stretch_tar_new<T, D>(st, S, (uint32_t)n, (uint32_t)p, table, rec, tar, nullptr, nullptr, slice, t / cols * C::U, t % cols,
                          tid % 256);
  __syncthreads();
  if (gather) {
    em.src = places;
    em.src_stride = 0;
  }
  select_slice<kSmallThreads, 1, false>(tar, van, frame_idx, S, n, budget, tar_total, r, nullptr, err, slice, 1, tflip,
                                        vflip, sh, st, em);
  if (!gather) return;
  __syncthreads();
  char* kd = K + (int64_t)slice * S * RB;
  char* vd = V + (int64_t)slice * S * RB;
  small_move<RB>(kd, vd, budget, [&](int32_t j, bool val) {
    return row_place<RB>(val ? V : K, val ? st.V : st.K, st, S, slice, places[j]);
  });
}

}  // namespace ipv
