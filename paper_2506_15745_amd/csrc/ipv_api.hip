// C ABI of the compression pass: argument validation, workspace layout and
// kernel launches. Every check that the host can make happens before the
// first launch, so a rejected call enqueues nothing and touches no buffer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <vector>

#include "../../include/ipv.h"
#include "ipv_adjacent.hpp"
#include "ipv_ahead.hpp"
#include "ipv_compact.hpp"
#include "ipv_scores.hpp"
#include "ipv_select.hpp"
#include "ipv_small.hpp"
#include "ipv_stretch.hpp"

using namespace ipv;

#define IPV_TRY(x)               \
  do {                           \
    const ipv_status _s = (x);   \
    if (_s != IPV_OK) return _s; \
  } while (0)

namespace {

constexpr int32_t kMaxRows = 65536;  // select: 1024 threads x 64 row flags
constexpr int64_t kMaxWindowRows = 65536;        // r * p: recent rows scanned per table block
constexpr int32_t kMaxRecentFrames = 256;
static_assert(kPrevMaxPositions >= kPoolCells, "the prev-row walk holds one entry per patch position");
constexpr int kCompactThreads = 1024;
constexpr int kCompactRows = 512;      // rows per compaction chunk
constexpr int kCompactColBytes = 256;  // largest column block a compaction walk copies

struct Dims {
  int64_t B, L, H, S, D, p, slices;
  int32_t gh, gw, dtype;
  int64_t elem;  // bytes per element
};

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

ipv_status check_shape(const ipv_shape* s, Dims* d) {
  if (!s) return IPV_ERR_NULL;
  if (s->dtype != IPV_BF16 && s->dtype != IPV_F32) return IPV_ERR_DTYPE;
  if (s->streams < 1 || s->layers < 1 || s->kv_heads < 1 || s->capacity < 1 || s->grid_h < 1 || s->grid_w < 1)
    return IPV_ERR_SHAPE;
  if (s->head_dim != 32 && s->head_dim != 64 && s->head_dim != 128 && s->head_dim != 256) return IPV_ERR_SHAPE;
  const int64_t p = (int64_t)s->grid_h * s->grid_w;
  if (p > kPoolCells) return IPV_ERR_SHAPE;
  d->B = s->streams;
  d->L = s->layers;
  d->H = s->kv_heads;
  d->S = s->capacity;
  d->D = s->head_dim;
  d->p = p;
  d->slices = d->B * d->L * d->H;
  d->gh = s->grid_h;
  d->gw = s->grid_w;
  d->dtype = s->dtype;
  d->elem = s->dtype == IPV_BF16 ? 2 : 4;
  if (d->slices > (int64_t)INT32_MAX / 8) return IPV_ERR_SHAPE;
  // buffer loads address one slice's rows with 32-bit byte offsets
  if (d->S * d->D * d->elem > (int64_t)UINT32_MAX - 16) return IPV_ERR_SHAPE;
  return IPV_OK;
}

ipv_status check_mode(uint32_t mode) { return (mode & ~(uint32_t)IPV_MODE_ALL) ? IPV_ERR_ARG : IPV_OK; }

// Uniform Select decides from frame ids: no score buffers are read or written
bool scores_needed(uint32_t mode) { return (mode & IPV_UNIFORM_SELECT) == 0; }

ipv_status check_rows(const Dims& d, int32_t n) {
  if (n < 1 || n > d.S || n > kMaxRows) return IPV_ERR_SHAPE;
  return IPV_OK;
}

ipv_status check_recent(const Dims& d, int32_t r) {
  if (r < 1 || r > kMaxRecentFrames) return IPV_ERR_ARG;
  if ((int64_t)r * d.p > kMaxWindowRows) return IPV_ERR_ARG;
  return IPV_OK;
}

// A pass keeps budget rows of n: 1 <= budget <= n. Whether the budget also
// holds the recent window |R| depends on the frame ids, which only the device
// reads: the selection reports a larger window (IPV_DEV_RECENT_OVER).
ipv_status check_budget(int32_t n, int32_t budget) {
  return (budget < 1 || budget > n) ? IPV_ERR_BUDGET : IPV_OK;
}

// The continual-compression loop runs many passes without reading the device
// between them, so it asks for a budget that holds any window the cache can
// have: |R| <= min(n, r * p) (a frame holds each patch position at most once).
ipv_status check_loop_budget(const Dims& d, int32_t n, int32_t budget, int32_t r) {
  IPV_TRY(check_budget(n, budget));
  return budget < std::min<int64_t>(n, (int64_t)r * d.p) ? IPV_ERR_BUDGET : IPV_OK;
}

// ------------------------------------------------------------ workspace layout
// [0, 256)                 device error word (uint32) + padding
// table  slices * p * D    fp32 m_q vectors of the recent window; in the
//                          consecutive-frame TaR mode the same region holds
//                          prev(x) per row instead (slices * S int32)
// first  slices            int32 first recent row of each slice
// pool   B * L             int32 pooling window per (stream, layer)
// flags  walks * (chunks+1) per compaction walk: a uint32 per chunk (1 once its
//                          rows are loaded), then the walk's ticket counter
size_t up256(size_t x) { return (x + 255) / 256 * 256; }
int64_t compact_parts(const Dims& d) { return 2 * std::max<int64_t>(1, d.D * d.elem / kCompactColBytes) + 1; }
int64_t max_chunks(const Dims& d) { return (d.S + kCompactRows - 1) / kCompactRows; }
size_t table_offset() { return kWsHeader; }
size_t table_bytes(const Dims& d) {
  return std::max((size_t)(d.slices * d.p * d.D) * sizeof(float), (size_t)(d.slices * d.S) * sizeof(int32_t));
}
size_t first_offset(const Dims& d) { return up256(table_offset() + table_bytes(d)); }
size_t pool_offset(const Dims& d) { return up256(first_offset(d) + (size_t)d.slices * sizeof(int32_t)); }
size_t flags_offset(const Dims& d) { return up256(pool_offset(d) + (size_t)(d.B * d.L) * sizeof(int32_t)); }
size_t ws_total(const Dims& d) {
  return up256(flags_offset(d) + (size_t)(d.slices * compact_parts(d) * walk_words(max_chunks(d))) * sizeof(uint32_t));
}

ipv_status check_ws(const Dims& d, const void* ws, size_t ws_bytes) {
  if (!ws) return IPV_ERR_WORKSPACE;
  if (!aligned(ws, 256)) return IPV_ERR_ALIGN;
  if (ws_bytes < ws_total(d)) return IPV_ERR_WORKSPACE;
  return IPV_OK;
}

uint32_t* err_word(void* ws) { return reinterpret_cast<uint32_t*>(ws); }
float* ws_table(void* ws) { return reinterpret_cast<float*>(static_cast<char*>(ws) + table_offset()); }
int32_t* ws_prev(void* ws) { return reinterpret_cast<int32_t*>(static_cast<char*>(ws) + table_offset()); }
int32_t* ws_first(void* ws, const Dims& d) {
  return reinterpret_cast<int32_t*>(static_cast<char*>(ws) + first_offset(d));
}
uint32_t* ws_flags(void* ws, const Dims& d) {
  return reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + flags_offset(d));
}
int32_t* ws_pool(void* ws, const Dims& d) {
  return reinterpret_cast<int32_t*>(static_cast<char*>(ws) + pool_offset(d));
}

ipv_status launched() { return hipGetLastError() == hipSuccess ? IPV_OK : IPV_ERR_HIP; }

// blocks: the launch's tile blocks (after any blocks of another role that come first)
TileGrid tile_grid(int32_t col_blocks, int32_t frame_blocks, uint32_t work, uint32_t blocks) {
  return TileGrid{make_fastdiv((uint32_t)col_blocks), make_fastdiv((uint32_t)frame_blocks), work, blocks};
}

// slices of the tile grid (Ragged: padded to a whole number for every XCD)
uint32_t grid_slices(const Dims& d, const Whole&) { return (uint32_t)d.slices; }
uint32_t grid_slices(const Dims&, const Ragged& rows) { return 8u * rows.per_xcd.d; }

uint32_t pad8(uint32_t x) { return (x + 7u) / 8u * 8u; }

// ------------------------------------------------------------ launchers
ipv_status no_mark() { return IPV_OK; }

// K == nullptr: VaN only; V == nullptr: TaR only. With both, the first launch
// builds what TaR needs (the recent-key table, or in the consecutive-frame
// mode the prev rows) with the VaN tiles beside it, and the second scores
// TaR. between(): runs after the first launch (the table, the prev rows, or
// nothing for VaN only), before the sweep that follows.
// zero_chunks > 0: the first kernel also zeroes the compaction flags for a
// compaction of zero_chunks chunks per walk that follows in the same pass.
// adjacent: consecutive-frame TaR (IPV_TAR_ADJACENT)
// cv_tau (may be null): with both scores and the recent-key table, the TaR
// launch also computes the pooling CV and window of every (stream, layer)
// (k_pool_apply must follow); ignored otherwise.
template <typename T, int D, class ST, typename Between>
ipv_status run_scores(const Dims& d, const void* K, const void* V, const int32_t* fr, const int32_t* pa, int32_t n,
                      int32_t r, float* tar, float* van, void* ws, hipStream_t st, Between between,
                      int64_t zero_chunks, bool adjacent, const double* cv_tau, const ST& rows) {
  const uint32_t tile_slices = grid_slices(d, rows);
  const bool do_tar = K != nullptr, do_van = V != nullptr;
  uint32_t* zero = zero_chunks > 0 ? ws_flags(ws, d) : nullptr;
  const int32_t zero_per_slice = (int32_t)(compact_parts(d) * walk_words(zero_chunks));
  if (do_tar && adjacent) {
    if (do_van) {
      // prev-row walks and VaN tiles in one launch
      using C = SweepCfg<T, D>;
      const int32_t col_blocks = (int32_t)((d.p + C::GROUPS - 1) / C::GROUPS);
      const int32_t frame_blocks = (int32_t)(((n + d.p - 1) / d.p + C::U - 1) / C::U);
      const uint32_t work = tile_slices * (uint32_t)(frame_blocks * col_blocks);
      const uint32_t prev_padded = pad8((uint32_t)d.slices);
      k_prev_van<T, D, ST><<<dim3(prev_padded + pad8((work + 3) / 4)), dim3(kPrevThreads), 0, st>>>(
          static_cast<const T*>(V), fr, pa, d.S, n, r, (int32_t)d.p, ws_prev(ws), ws_first(ws, d), err_word(ws),
          zero, zero_per_slice, prev_padded, (uint32_t)d.slices, van,
          tile_grid(col_blocks, frame_blocks, work, pad8((work + 3) / 4)), rows);
    } else {
      k_prev_rows<ST><<<dim3((uint32_t)d.slices), dim3(kPrevThreads), 0, st>>>(
          fr, pa, d.S, n, r, (int32_t)d.p, ws_prev(ws), ws_first(ws, d), err_word(ws), zero, zero_per_slice, rows);
    }
    IPV_TRY(between());
    // then the TaR rows
    constexpr int ROWS = 256 / (D / Lane<T>::EPL) * 4;
    const int32_t bps = (n + ROWS - 1) / ROWS;
    const uint32_t work = tile_slices * (uint32_t)bps;
    k_adjacent_sweep<T, D, ST><<<dim3(pad8(work)), dim3(256), 0, st>>>(static_cast<const T*>(K), ws_prev(ws), d.S, n,
                                                                       ws_first(ws, d), tar, bps, work, rows);
    return launched();
  }
  constexpr int GROUPS = 256 / (D / Lane<T>::EPL);
  const int32_t blocks = (int32_t)((d.p + GROUPS - 1) / GROUPS);
  const size_t lds = (size_t)GROUPS * r * sizeof(int32_t);
  const uint32_t table_real = (uint32_t)(d.slices * blocks);
  using C = SweepCfg<T, D>;
  const int32_t col_blocks = (int32_t)((d.p + C::GROUPS - 1) / C::GROUPS);
  const int32_t frame_blocks = (int32_t)(((n + d.p - 1) / d.p + C::U - 1) / C::U);
  const uint32_t work = tile_slices * (uint32_t)(frame_blocks * col_blocks);
  const dim3 grid(pad8(work)), block(256);
  const T* k = static_cast<const T*>(K);
  const T* v = static_cast<const T*>(V);
  int32_t* first = ws_first(ws, d);
  const int32_t window = (int32_t)((int64_t)r * d.p);  // most rows the recent window can hold
  if (do_tar && do_van) {
    // table and VaN tiles in one launch, then the TaR tiles
    const uint32_t table_padded = pad8(table_real);
    k_table_van<T, D, ST><<<dim3(table_padded + pad8(work)), block, lds, st>>>(
        k, v, fr, pa, d.S, n, r, (int32_t)d.p, blocks, table_padded, table_real, ws_table(ws), first, err_word(ws),
        zero, zero_per_slice, van, tile_grid(col_blocks, frame_blocks, work, pad8(work)), rows);
    IPV_TRY(between());
    if (cv_tau) {
      const uint32_t cv_real = (uint32_t)(d.B * d.L), cv_padded = pad8(cv_real);
      k_tar_sweep_cv<T, D, ST><<<dim3(cv_padded + pad8(work)), block, 0, st>>>(
          k, pa, d.S, n, (int32_t)d.p, ws_table(ws), first, tar, err_word(ws),
          tile_grid(col_blocks, frame_blocks, work, pad8(work)), window, van, (int32_t)d.H, cv_tau[0], cv_tau[1],
          cv_tau[2], ws_pool(ws, d), cv_padded, cv_real, rows);
      return launched();
    }
    k_score_sweep<T, D, true, false, ST><<<grid, block, 0, st>>>(k, v, pa, d.S, n, (int32_t)d.p, ws_table(ws), first,
                                                             tar, van, err_word(ws),
                                                             tile_grid(col_blocks, frame_blocks, work, pad8(work)), window, rows);
    return launched();
  }
  if (do_tar)
    k_recent_table<T, D, ST><<<dim3(table_real), block, lds, st>>>(k, fr, pa, d.S, n, r, (int32_t)d.p, blocks,
                                                                   ws_table(ws), first, err_word(ws), zero,
                                                                   zero_per_slice, rows);
  IPV_TRY(between());
  if (do_tar)
    k_score_sweep<T, D, true, false, ST><<<grid, block, 0, st>>>(k, v, pa, d.S, n, (int32_t)d.p, ws_table(ws), first,
                                                             tar, van, err_word(ws),
                                                             tile_grid(col_blocks, frame_blocks, work, pad8(work)), window, rows);
  else
    k_score_sweep<T, D, false, true, ST><<<grid, block, 0, st>>>(k, v, pa, d.S, n, (int32_t)d.p, ws_table(ws), first,
                                                             tar, van, err_word(ws),
                                                             tile_grid(col_blocks, frame_blocks, work, pad8(work)), 0, rows);
  return launched();
}

template <class ST, typename Between = ipv_status (*)()>
ipv_status scores(const Dims& d, const void* K, const void* V, const int32_t* fr, const int32_t* pa, int32_t n,
                  const ST& rows, int32_t r, float* tar, float* van, void* ws, hipStream_t st, Between between = no_mark,
                  int64_t zero_chunks = 0, bool adjacent = false, const double* cv_tau = nullptr) {
#define IPV_SCORES(T, DD)                                                                                        \
  if (d.D == DD)                                                                                                 \
    return run_scores<T, DD>(d, K, V, fr, pa, n, r, tar, van, ws, st, between, zero_chunks, adjacent, cv_tau, rows);
  if (d.dtype == IPV_BF16) {
    IPV_SCORES(uint16_t, 32) IPV_SCORES(uint16_t, 64) IPV_SCORES(uint16_t, 128) IPV_SCORES(uint16_t, 256)
  } else {
    IPV_SCORES(float, 32) IPV_SCORES(float, 64) IPV_SCORES(float, 128) IPV_SCORES(float, 256)
  }
#undef IPV_SCORES
  return IPV_ERR_SHAPE;
}

// cv_done: the TaR launch has computed the windows already (k_tar_sweep_cv)
template <class ST>
ipv_status pool_d(const Dims& d, const double* tau, float* van, const int32_t* fr, const int32_t* pa, int32_t n,
                  const ST& rows, int32_t* pool_out, void* ws, hipStream_t st, bool cv_done = false) {
  if (!cv_done)
    k_pool_cv<<<dim3((uint32_t)(d.B * d.L)), dim3(kPoolThreads), 0, st>>>(van, d.S, n, (int32_t)d.H, tau[0], tau[1],
                                                                          tau[2], ws_pool(ws, d), pool_out, rows);
  k_pool_apply<<<dim3((uint32_t)d.slices), dim3(kPoolThreads), 0, st>>>(
      van, fr, pa, d.S, n, (int32_t)d.H, d.gh, d.gw, ws_pool(ws, d), make_fastdiv((uint32_t)d.p),
      make_fastdiv((uint32_t)d.gw), rows);
  return launched();
}

__global__ void k_fill_i32(int32_t* p, int64_t count, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

constexpr int kSelThreads = 1024;  // most threads of a selection workgroup
constexpr int64_t kComputeUnits = 256;  // MI355X

// Threads of a selection workgroup: whole waves for the n rows at RPT rows a
// thread, at most kSelThreads (the caller picks RPT >= n / kSelThreads).
uint32_t sel_threads(int32_t n, int RPT) {
  const int32_t t = (n + RPT - 1) / RPT;
  return (uint32_t)std::min(kSelThreads, (t + 63) / 64 * 64);
}

uint32_t flip_bits(uint32_t mode, uint32_t bit) { return (mode & bit) ? 0xffffffffu : 0u; }

// mode: the reverse bits complement a stage's keys; IPV_HEAD_SHARED gives one
// block (and one keep set) to each (stream, layer)
template <int RPT, class ST, class EM>
ipv_status run_select(const Dims& d, const float* tar, const float* van, const int32_t* fr, int32_t n, int32_t budget,
                      int32_t tar_total, int32_t r, int32_t* keep, uint32_t* err, hipStream_t st, uint32_t mode,
                      const ST& rows, const EM& em) {
  const int32_t heads = (mode & IPV_HEAD_SHARED) ? (int32_t)d.H : 1;
  const uint32_t tflip = flip_bits(mode, IPV_TAR_REVERSE);
  const uint32_t vflip = flip_bits(mode, IPV_VAN_REVERSE);
  const dim3 grid((uint32_t)(d.slices / heads)), block(sel_threads(n, RPT));
  // 16-byte row-run loads need every slice to start 16-byte aligned
  if (d.S % 4 == 0)
    k_select<kSelThreads, RPT, true><<<grid, block, 0, st>>>(tar, van, fr, d.S, n, budget, tar_total, r, keep, err,
                                                             heads, tflip, vflip, rows, em);
  else
    k_select<kSelThreads, RPT, false><<<grid, block, 0, st>>>(tar, van, fr, d.S, n, budget, tar_total, r, keep, err,
                                                              heads, tflip, vflip, rows, em);
  return launched();
}

// Uniform Select: one block per slice, or per (stream, layer) with
// IPV_HEAD_SHARED. zero (may be null): the blocks also zero zero_per_slice
// words per slice there (the compaction flags of the pass).
template <int RPT, class ST, class EM>
ipv_status run_uniform(const Dims& d, const int32_t* fr, int32_t n, int32_t budget, int32_t r, int32_t* keep,
                       uint32_t* err, hipStream_t st, uint32_t mode, uint32_t* zero, int32_t zero_per_slice,
                       const ST& rows, const EM& em) {
  const int32_t heads = (mode & IPV_HEAD_SHARED) ? (int32_t)d.H : 1;
  const dim3 grid((uint32_t)(d.slices / heads)), block(sel_threads(n, RPT));
  if (d.S % 4 == 0)
    k_select_uniform<kSelThreads, RPT, true><<<grid, block, 0, st>>>(fr, d.S, n, budget, r, keep, err, heads, zero,
                                                                     zero_per_slice, rows, em);
  else
    k_select_uniform<kSelThreads, RPT, false><<<grid, block, 0, st>>>(fr, d.S, n, budget, r, keep, err, heads, zero,
                                                                      zero_per_slice, rows, em);
  return launched();
}

// zero / zero_per_slice: as for run_uniform (used by Uniform Select only).
// rows / em: a Stretch and its Emit for a pass over rows outside the cache.
template <class ST, class EM = NoEmit>
ipv_status select(const Dims& d, const float* tar, const float* van, const int32_t* fr, int32_t n, const ST& rows,
                  int32_t budget, int32_t tar_total, int32_t r, int32_t* keep, uint32_t* err, hipStream_t st,
                  uint32_t mode, uint32_t* zero = nullptr, int32_t zero_per_slice = 0, const EM& em = EM{}) {
  const int32_t rpt = (n + kSelThreads - 1) / kSelThreads;
  // A block of up to 8 rows a thread (832 threads for 6272 rows) holds a CU
  // alone; with more blocks than CUs, 16 rows a thread (half the threads)
  // lets three blocks share a CU, which ends sooner although each block takes
  // longer (16-stream 7B-class batch: 65 against 93 us).
  const int64_t groups = d.slices / ((mode & IPV_HEAD_SHARED) ? d.H : 1);
  const bool many = groups > kComputeUnits && rpt <= 8;
  // Beyond 32 rows a thread the 128 registers of a 1024-thread block bound it:
  // 64 rows a thread, with both columns loaded together, spilled (640 slices of
  // 32928 rows 391 us, against 142 us for 32768 rows at 32 a thread). With the
  // columns one after the other and 36 rows a thread 150 us; 48 for up to 49152
  // rows 278 us (499 before), 64 beyond 393 us (661 before, 65536 rows).
#define IPV_UNIFORM(RPT) return run_uniform<RPT>(d, fr, n, budget, r, keep, err, st, mode, zero, zero_per_slice, rows, em)
#define IPV_SELECT(RPT) return run_select<RPT>(d, tar, van, fr, n, budget, tar_total, r, keep, err, st, mode, rows, em)
  if (mode & IPV_UNIFORM_SELECT) {
    if (many) IPV_UNIFORM(16);
    if (rpt <= 4) IPV_UNIFORM(4);
    if (rpt <= 8) IPV_UNIFORM(8);
    if (rpt <= 16) IPV_UNIFORM(16);
    if (rpt <= 32) IPV_UNIFORM(32);
    IPV_UNIFORM(64);
  }
  if (many) IPV_SELECT(16);
  if (rpt <= 4) IPV_SELECT(4);
  if (rpt <= 8) IPV_SELECT(8);
  if (rpt <= 12) IPV_SELECT(12);
  if (rpt <= 16) IPV_SELECT(16);
  if (rpt <= 32) IPV_SELECT(32);
  if (rpt <= 36) IPV_SELECT(36);
  if (rpt <= 48) IPV_SELECT(48);
  IPV_SELECT(64);
#undef IPV_UNIFORM
#undef IPV_SELECT
}

int64_t compact_chunks(int32_t budget) { return (budget + kCompactRows - 1) / kCompactRows; }

// flags_zeroed: an earlier kernel of the pass (the table or prev-row launch, or
// the uniform selection) has zeroed the flags already
template <int RB, class ST>
ipv_status run_compact(const Dims& d, void* K, void* V, int32_t* fr, int32_t* pa, int32_t n, const ST& rows,
                       const int32_t* keep, int32_t budget, void* ws, hipStream_t st, bool flags_zeroed) {
  using C = CompactCfg<RB, kCompactThreads, kCompactRows, kCompactColBytes>;
  const uint32_t chunks = (uint32_t)compact_chunks(budget);
  const int64_t total = d.slices * C::PARTS * chunks;
  if (!flags_zeroed) {
    const int64_t words = d.slices * C::PARTS * walk_words(chunks);
    k_clear_flags<<<dim3((uint32_t)((words + 255) / 256)), dim3(256), 0, st>>>(ws_flags(ws, d), words);
  }
  k_compact<RB, kCompactThreads, kCompactRows, kCompactColBytes><<<dim3((uint32_t)total), dim3(kCompactThreads), 0, st>>>(
      static_cast<char*>(K), static_cast<char*>(V), fr, pa, d.S, n, budget, keep, err_word(ws), ws_flags(ws, d),
      chunks, make_fastdiv((uint32_t)(d.slices * C::PARTS)), rows);
  return launched();
}

template <class ST>
ipv_status compact(const Dims& d, void* K, void* V, int32_t* fr, int32_t* pa, int32_t n, const ST& rows,
                   const int32_t* keep, int32_t budget, void* ws, hipStream_t st, bool flags_zeroed = false) {
  switch (d.D * d.elem) {
    case 64: return run_compact<64>(d, K, V, fr, pa, n, rows, keep, budget, ws, st, flags_zeroed);
    case 128: return run_compact<128>(d, K, V, fr, pa, n, rows, keep, budget, ws, st, flags_zeroed);
    case 256: return run_compact<256>(d, K, V, fr, pa, n, rows, keep, budget, ws, st, flags_zeroed);
    case 512: return run_compact<512>(d, K, V, fr, pa, n, rows, keep, budget, ws, st, flags_zeroed);
    case 1024: return run_compact<1024>(d, K, V, fr, pa, n, rows, keep, budget, ws, st, flags_zeroed);
  }
  return IPV_ERR_SHAPE;
}

// ------------------------------------------------------------ passes over a stretch (ipv_stretch.hpp)
// Scores of one pass over a run of slices. norms_known: van holds the old
// rows' norms already. cv_tau: the TaR launch also computes the pooling CV.
// zero_chunks > 0: the first kernel zeroes the flags of a gather that follows.
// ahead: this pass's first launch went out with the selection before it.
template <typename T, int D>
ipv_status stretch_scores_t(const Dims& d, const char* K, const char* V, const Stretch& sr, const int32_t* fr,
                            int32_t* pa, int32_t n, int32_t r, float* tar, float* van, void* ws, hipStream_t st,
                            int64_t zero_chunks, bool adjacent, const double* cv_tau, bool norms_known, bool ahead) {
  using C = SweepCfg<T, D>;
  constexpr uint32_t TILE = C::GROUPS * C::U;
  uint32_t* zero = zero_chunks > 0 ? ws_flags(ws, d) : nullptr;
  const int32_t zero_per_slice = (int32_t)(compact_parts(d) * walk_words(zero_chunks));
  const uint32_t slices = (uint32_t)d.slices;
  const uint32_t v0 = ahead ? (uint32_t)n : norms_known ? sr.n0 : 0u;
  const uint32_t van_tiles = ((uint32_t)n - v0 + TILE - 1) / TILE, van_work = slices * van_tiles;
  const FastDiv van_div = make_fastdiv(std::max(1u, van_tiles));
  int32_t* waiting = ahead ? pa : nullptr;
  int32_t* first = ws_first(ws, d);
  if (adjacent) {
    const uint32_t walks = pad8(slices), quads = pad8((van_work + 3) / 4);
    k_stretch_prev_van<T, D><<<dim3(walks + quads), dim3(kPrevThreads), 0, st>>>(
        V, sr, fr, pa, d.S, n, r, (int32_t)d.p, ws_prev(ws), first, err_word(ws), zero, zero_per_slice, walks, slices,
        van, v0, van_div, van_work, quads);
    const uint32_t tiles = ((uint32_t)n + TILE - 1) / TILE, work = slices * tiles;
    k_stretch_adjacent<T, D><<<dim3(pad8(work)), dim3(256), 0, st>>>(K, sr, ws_prev(ws), d.S, n, first, tar,
                                                                     waiting, van, make_fastdiv(tiles), work, pad8(work));
    return launched();
  }
  const uint32_t blocks = (uint32_t)((d.p + C::GROUPS - 1) / C::GROUPS), table = slices * blocks;
  if (!ahead)
    k_stretch_table_van<T, D><<<dim3(pad8(table) + pad8(van_work)), dim3(256), (size_t)C::GROUPS * r * sizeof(int32_t), st>>>(
        K, V, sr, fr, pa, d.S, n, r, (int32_t)d.p, make_fastdiv(blocks), pad8(table), table, ws_table(ws), first,
        err_word(ws), zero, zero_per_slice, van, v0, van_div, make_fastdiv(slices), van_work, pad8(van_work));
  const uint32_t rows = sr.rows.d, new_frames = ((uint32_t)n - sr.n0) / rows;
  const uint32_t old_tiles = (sr.n0 + TILE - 1) / TILE, cols = (rows + C::GROUPS - 1) / C::GROUPS;
  const uint32_t tiles = old_tiles + (new_frames + C::U - 1) / C::U * cols;
  const uint32_t group = sr.n0 == 0 ? slice_group(slices, (uint32_t)(d.p * d.D) * 4u) : 0u;
  const uint32_t work = ((slices + (1u << group) - 1) >> group << group) * tiles;
  const uint32_t cv = cv_tau ? (uint32_t)(d.B * d.L) : 0u;
  const int32_t sure_past = (int32_t)std::max<int64_t>(0, (int64_t)n - (int64_t)r * d.p);
  k_stretch_tar<T, D><<<dim3(pad8(cv) + pad8(work)), dim3(256), 0, st>>>(
      K, sr, pa, waiting, d.S, n, (int32_t)d.p, ws_table(ws), first, tar, err_word(ws), make_fastdiv(tiles), old_tiles,
      make_fastdiv(cols), work, pad8(work), slices, group, sure_past, van, (int32_t)d.H, cv ? cv_tau[0] : 0.0,
      cv ? cv_tau[1] : 0.0, cv ? cv_tau[2] : 0.0, ws_pool(ws, d), pad8(cv), cv);
  return launched();
}

ipv_status stretch_scores(const Dims& d, const char* K, const char* V, const Stretch& sr, const int32_t* fr,
                          int32_t* pa, int32_t n, int32_t r, float* tar, float* van, void* ws, hipStream_t st,
                          int64_t zero_chunks, bool adjacent, const double* cv_tau, bool norms_known, bool ahead) {
#define IPV_SCORES(T, DD)                                                                                           \
  if (d.D == DD)                                                                                                    \
    return stretch_scores_t<T, DD>(d, K, V, sr, fr, pa, n, r, tar, van, ws, st, zero_chunks, adjacent, cv_tau, norms_known, \
                                   ahead);
  if (d.dtype == IPV_BF16) {
    IPV_SCORES(uint16_t, 32) IPV_SCORES(uint16_t, 64) IPV_SCORES(uint16_t, 128) IPV_SCORES(uint16_t, 256)
  } else {
    IPV_SCORES(float, 32) IPV_SCORES(float, 64) IPV_SCORES(float, 128) IPV_SCORES(float, 256)
  }
#undef IPV_SCORES
  return IPV_ERR_SHAPE;
}

// ------------------------------------------------------------ work of the next pass (ipv_ahead.hpp)
// Whether the next pass's first launch goes out with this pass's selection (n rows;
// new_frames: the next pass's). A selection block fills a CU, so it pays while that
// leaves CUs for the work beside it, the more the longer the rows. A call of five
// passes without / with it, us, 196 rows a frame, bf16 rows of 256 bytes:
//   28 slices of 2156 rows 138 / 119, of 12544 rows 362 / 333; 112 slices 223 / 220 and
//   892 / 853; 128: 245 / 244 and 992 / 957; 144: 264 / 263 and 1092 / 1082; 160:
//   281 / 288 and 1179 / 1169; 192: 319 / 329 and 1393 / 1402; head-shared, 80
//   selections 902 / 894 and 4505 / 4451, 144: 433 / 442 and 2030 / 2033;
//   rows of 128 bytes, 160 slices of 6272 rows 398 / 383; of 512 bytes, 112 slices
//   835 / 818, 144 1035 / 1032 (of 1568 rows 344 / 342); of 1 KB, 64 slices 844 / 825,
//   80 1031 / 1022 (of 2156 rows 418 / 422), 112 1410 / 1410, 144 1786 / 1805.
// Up to 16 rows a thread: longer slices' selections use every register of a CU.
// Only if the recent-key table goes with it (the window lies in the new frames):
// the norms alone save no launch (28 slices of 1568 rows 123 / 128, 128 202 / 209).
// The consecutive-frame mode has the norms beside its walks already, unless the
// walks take most of the CUs and the selections do not: 56 head-shared selections
// of 224 slices of 12544 rows 1808 / 1676, of 2156 rows 349 / 322, 28 of 112 slices
// 1014 / 988 and 226 / 232, 4 of 16 426 / 441; 64 slices, each its own, 551 / 562.
bool ahead_fits(const Dims& d, int32_t n, int32_t r, uint32_t mode, int32_t new_frames) {
  const int64_t groups = d.slices / ((mode & IPV_HEAD_SHARED) ? d.H : 1);
  if (n > 16 * kSelThreads || groups > 192 - d.D * d.elem / 8) return false;
  if (mode & IPV_TAR_ADJACENT) return 2 * groups <= d.slices && d.slices >= 96 && d.slices * n >= 300000;
  return new_frames > r;
}

// The selection of a pass, with the first launch of the next one (next: its
// rows, n_next of them; its new rows all lie in the frames).
ipv_status select_ahead(const Dims& d, const float* tar, const float* van, int32_t* fr, int32_t* pa, int32_t n,
                        const Stretch& sr, int32_t budget, int32_t tar_total, int32_t r, const Emit& em, const char* K,
                        const char* V, const Stretch& next, int32_t n_next, int64_t next_chunks, void* ws,
                        hipStream_t st, uint32_t mode) {
  const uint32_t lpr = (uint32_t)(d.D * d.elem / 16), slices = (uint32_t)d.slices;
  const int32_t heads = (mode & IPV_HEAD_SHARED) ? (int32_t)d.H : 1;
  const uint32_t tile = 256u / lpr * 4u * kAheadTiles, tiles = ((uint32_t)n_next - next.n0 + tile - 1) / tile;
  const uint32_t per_block = kAheadThreads / lpr, blocks = ((uint32_t)d.p + per_block - 1) / per_block;
  Ahead a{};
  a.K = K;
  a.V = V;
  a.kind = kind_of(d.dtype == IPV_BF16, d.D);
  a.st = next;
  a.n = n_next;
  a.r = r;
  a.p = (int32_t)d.p;
  a.norm = reinterpret_cast<float*>(pa);
  a.slices = make_fastdiv(slices);
  a.n_work = slices * tiles;
  a.tile_blocks = pad8((a.n_work + 3) / 4);
  if (!(mode & IPV_TAR_ADJACENT)) {
    a.table = ws_table(ws);
    a.table_blocks = make_fastdiv(blocks);
    a.table_real = slices * blocks;
    a.table_padded = pad8(a.table_real);
    a.first_recent = ws_first(ws, d);
    a.zero = next_chunks > 0 ? ws_flags(ws, d) : nullptr;
    a.zero_per_slice = (int32_t)(compact_parts(d) * walk_words(next_chunks));
  }
  a.sel_real = slices / (uint32_t)heads;
  a.sel_padded = pad8(a.sel_real);
  const dim3 grid(a.sel_padded + a.table_padded + a.tile_blocks), block(kAheadThreads);
  const uint32_t tflip = flip_bits(mode, IPV_TAR_REVERSE), vflip = flip_bits(mode, IPV_VAN_REVERSE);
  const int32_t rpt = (n + kSelThreads - 1) / kSelThreads;
#define IPV_AHEAD(RPT)                                                                                                \
  if (rpt <= RPT) {                                                                                                   \
    if (d.S % 4 == 0)                                                                                                 \
      k_select_ahead<RPT, true><<<grid, block, 0, st>>>(tar, van, fr, pa, d.S, n, budget, tar_total, r, err_word(ws), \
                                                        heads, tflip, vflip, sr, em, a);                              \
    else                                                                                                              \
      k_select_ahead<RPT, false><<<grid, block, 0, st>>>(tar, van, fr, pa, d.S, n, budget, tar_total, r, err_word(ws), \
                                                         heads, tflip, vflip, sr, em, a);                             \
    return launched();                                                                                                \
  }
  IPV_AHEAD(4) IPV_AHEAD(8) IPV_AHEAD(12) IPV_AHEAD(16)
#undef IPV_AHEAD
  return IPV_ERR_SHAPE;
}

// src: places of the budget rows that stay, [slices, S]; n_entry: most rows a
// slice held before the call
template <int RB>
ipv_status stretch_gather_t(const Dims& d, void* K, void* V, const Stretch& sr, const int32_t* src, int32_t n_entry,
                            int32_t budget, void* ws, hipStream_t st) {
  using C = CompactCfg<RB, kCompactThreads, kCompactRows, kCompactColBytes>;
  const uint32_t chunks = (uint32_t)compact_chunks(budget), walks = (uint32_t)(d.slices * 2 * C::NCB);
  const dim3 grid(walks * chunks), block(kCompactThreads);
  if (n_entry > 0)
    k_stretch_gather<RB, kCompactThreads, kCompactRows, kCompactColBytes, true><<<grid, block, 0, st>>>(
        static_cast<char*>(K), static_cast<char*>(V), sr, src, d.S, n_entry, budget, err_word(ws), ws_flags(ws, d),
        chunks, make_fastdiv(walks));
  else
    k_stretch_gather<RB, kCompactThreads, kCompactRows, kCompactColBytes, false><<<grid, block, 0, st>>>(
        static_cast<char*>(K), static_cast<char*>(V), sr, src, d.S, n_entry, budget, err_word(ws), ws_flags(ws, d),
        chunks, make_fastdiv(walks));
  return launched();
}

ipv_status stretch_gather(const Dims& d, void* K, void* V, const Stretch& sr, const int32_t* src, int32_t n_entry,
                          int32_t budget, void* ws, hipStream_t st) {
  switch (d.D * d.elem) {
    case 64: return stretch_gather_t<64>(d, K, V, sr, src, n_entry, budget, ws, st);
    case 128: return stretch_gather_t<128>(d, K, V, sr, src, n_entry, budget, ws, st);
    case 256: return stretch_gather_t<256>(d, K, V, sr, src, n_entry, budget, ws, st);
    case 512: return stretch_gather_t<512>(d, K, V, sr, src, n_entry, budget, ws, st);
    case 1024: return stretch_gather_t<1024>(d, K, V, sr, src, n_entry, budget, ws, st);
  }
  return IPV_ERR_SHAPE;
}

// ------------------------------------------------------------ small slices (ipv_small.hpp)
// Whether a pass over slices of at most n rows goes out as one launch, a
// workgroup per slice: the plain scores (pooling and the other modes couple a
// layer's slices or have steps of their own), slices that run all at once,
// 256 rows and 64 KB of keys at most, and 24 or 32 KB of keys in a frame of the grid. Passes as GPU time alone, four launches
// against one (a graph of ten): 128 rows of 256 bytes 15.3 -> 13.3 us (2 slices),
// 23.9 -> 16.3 (256 slices); 256 rows 18.4 -> 16.4, 32.6 -> 22.2. Beyond, the one
// workgroup's share of the bandwidth counts: 512 rows of 256 bytes 17.8 -> 20.1,
// of 64 bytes 16.5 -> 19.0, 512 slices of 64 bytes 42.8 -> 45.2. A caller that is
// bound by its launches gains more (two passes and a gather of 128 rows: 7
// launches -> 2, 38 -> 27 us a call).
// The recent-key table takes the workgroup a round (with its own scan of the
// window) for every 16 KB of key rows of one frame, and the tiles go over every
// position of the grid, so the grid has to be small too. 256 rows of 256 bytes,
// 2 slices, the same measure with the metadata restored each time: 64 positions (a
// round) 20.0 -> 17.1, 81 (20 KB) 20.7 -> 19.8, 117 (29 KB) 20.6 -> 21.0; 64 rows of
// 1024 bytes: 24 positions (24 KB) 20.6 -> 20.0, 30 20.5 -> 20.7; single calls on
// 144 positions 25 -> 28, on 576 24 -> 49, 64 rows of 1024 bytes on 4096 29 -> 884.
// A call over a stretch is bound by its launches sooner and takes 32 KB (12 passes
// of 250 rows on 128 positions 237 -> 222 us, 10 of 64 rows on 30 194 -> 174).
constexpr int64_t kSmallBytes = 64 << 10, kSmallFrame = 24 << 10, kSmallFrameStretch = 32 << 10;
bool small_pass(const Dims& d, int32_t n, int32_t r, uint32_t mode, const double* cv_tau, int64_t frame = kSmallFrame) {
  return !cv_tau && (mode & ~(uint32_t)(IPV_TAR_REVERSE | IPV_VAN_REVERSE)) == 0 && n <= kSmallRows && r <= 32 &&
         d.slices <= kComputeUnits && n * d.D * d.elem <= kSmallBytes && d.p * d.D * d.elem <= frame;
}

template <typename T, int D, class ST>
ipv_status small_pass_t(const Dims& d, void* K, void* V, int32_t* fr, int32_t* pa, int32_t n, const ST& rows,
                        int32_t budget, int32_t tar_total, int32_t r, uint32_t mode, float* tar, float* van,
                        int32_t* keep, void* ws, hipStream_t st) {
  constexpr int TG = kSmallThreads / (D / Lane<T>::EPL);
  k_small_pass<T, D><<<dim3((uint32_t)d.slices), dim3(kSmallThreads), (size_t)TG * r * sizeof(int32_t), st>>>(
      static_cast<char*>(K), static_cast<char*>(V), fr, pa, d.S, n, r, (int32_t)d.p, budget, tar_total, ws_table(ws),
      ws_first(ws, d), tar, van, keep, err_word(ws), flip_bits(mode, IPV_TAR_REVERSE), flip_bits(mode, IPV_VAN_REVERSE),
      rows);
  return launched();
}

template <typename T, int D>
ipv_status small_stretch_t(const Dims& d, void* K, void* V, const Stretch& sr, int32_t* fr, int32_t* pa, int32_t n,
                           int32_t budget, int32_t tar_total, int32_t r, uint32_t mode, float* tar, float* van,
                           uint32_t v0, const Emit& em, bool gather, void* ws, hipStream_t st) {
  constexpr int TG = kSmallThreads / (D / Lane<T>::EPL);
  k_small_stretch<T, D><<<dim3((uint32_t)d.slices), dim3(kSmallThreads), (size_t)TG * r * sizeof(int32_t), st>>>(
      static_cast<char*>(K), static_cast<char*>(V), sr, fr, pa, d.S, n, r, (int32_t)d.p, budget, tar_total, ws_table(ws),
      ws_first(ws, d), tar, van, v0, err_word(ws), flip_bits(mode, IPV_TAR_REVERSE), flip_bits(mode, IPV_VAN_REVERSE), em,
      gather);
  return launched();
}

// fn(T, D) for the shape's element type and head size
#define IPV_BY_TYPE(d, CALL)                                                          \
  if ((d).dtype == IPV_BF16) {                                                        \
    if ((d).D == 32) CALL(uint16_t, 32);                                              \
    if ((d).D == 64) CALL(uint16_t, 64);                                              \
    if ((d).D == 128) CALL(uint16_t, 128);                                            \
    if ((d).D == 256) CALL(uint16_t, 256);                                            \
  } else {                                                                            \
    if ((d).D == 32) CALL(float, 32);                                                 \
    if ((d).D == 64) CALL(float, 64);                                                 \
    if ((d).D == 128) CALL(float, 128);                                               \
    if ((d).D == 256) CALL(float, 256);                                               \
  }                                                                                   \
  return IPV_ERR_SHAPE

template <class ST>
ipv_status run_small(const Dims& d, void* K, void* V, int32_t* fr, int32_t* pa, int32_t n, const ST& rows, int32_t budget,
                     int32_t tar_total, int32_t r, uint32_t mode, float* tar, float* van, int32_t* keep, void* ws,
                     hipStream_t st) {
#define IPV_SMALL(T, DD) return small_pass_t<T, DD>(d, K, V, fr, pa, n, rows, budget, tar_total, r, mode, tar, van, keep, ws, st)
  IPV_BY_TYPE(d, IPV_SMALL);
#undef IPV_SMALL
}

ipv_status run_small_stretch(const Dims& d, void* K, void* V, const Stretch& sr, int32_t* fr, int32_t* pa, int32_t n,
                             int32_t budget, int32_t tar_total, int32_t r, uint32_t mode, float* tar, float* van,
                             uint32_t v0, const Emit& em, bool gather, void* ws, hipStream_t st) {
#define IPV_SMALL(T, DD) \
  return small_stretch_t<T, DD>(d, K, V, sr, fr, pa, n, budget, tar_total, r, mode, tar, van, v0, em, gather, ws, st)
  IPV_BY_TYPE(d, IPV_SMALL);
#undef IPV_SMALL
}

// ------------------------------------------------------------ append
// `frames` consecutive frames of `rows` rows each into rows
// [n, n + frames * rows) of every slice. Block row blockIdx.y takes slices
// blockIdx.y, + gridDim.y, ...; in a slice, a grid-stride loop over the 16-byte
// pieces of the new rows in destination order (contiguous), then their
// metadata: frame frame_id + j for the rows of frame j, patch first_patch +
// the row's place in its frame. Source frame j of slice s starts at byte
// j * frame_stride + s * rows * RB. The caller keeps frames * rows * RB within
// the slice's 32-bit byte range (n + frames * rows <= S).
__global__ __launch_bounds__(256) void k_append(const char* __restrict__ Kn, const char* __restrict__ Vn,
                                                char* __restrict__ K, char* __restrict__ V,
                                                int32_t* __restrict__ fr, int32_t* __restrict__ pa, int64_t S,
                                                int32_t n, int32_t rows, int32_t frames, int64_t frame_stride,
                                                int64_t RB, int32_t frame_id, int32_t first_patch, int64_t slices) {
  const uint32_t per_frame = (uint32_t)rows * (uint32_t)(RB / 16);
  const uint32_t pieces = (uint32_t)frames * per_frame, meta = (uint32_t)frames * (uint32_t)rows;
  const uint32_t first = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  for (int64_t slice = blockIdx.y; slice < slices; slice += gridDim.y) {
    const char* ks = Kn + slice * rows * RB;
    const char* vs = Vn + slice * rows * RB;
    char* kd = K + (slice * S + n) * RB;
    char* vd = V + (slice * S + n) * RB;
    for (uint32_t e = first; e < pieces; e += step) {
      const uint32_t j = e / per_frame;
      const int64_t src = (int64_t)j * frame_stride + (int64_t)(e - j * per_frame) * 16;
      store16(kd + (int64_t)e * 16, load16(ks + src));
      store16(vd + (int64_t)e * 16, load16(vs + src));
    }
    for (uint32_t e = first; e < meta; e += step) {
      const uint32_t j = e / (uint32_t)rows;
      fr[slice * S + n + e] = frame_id + (int32_t)j;
      pa[slice * S + n + e] = first_patch + (int32_t)(e - j * (uint32_t)rows);
    }
  }
}

int32_t floor_share(double alpha, int32_t budget) { return (int32_t)std::floor(alpha * (double)budget); }

ipv_status check_tau(const double* tau) {
  if (!tau) return IPV_OK;
  for (int i = 0; i < 3; ++i)
    if (!std::isfinite(tau[i])) return IPV_ERR_ARG;
  if (!(tau[0] <= tau[1] && tau[1] <= tau[2])) return IPV_ERR_ARG;
  return IPV_OK;
}

// ------------------------------------------------------------ per-stream row counts
// Every call takes n_tokens as a host array of B row counts. The work is
// launched once per group of consecutive streams: a contiguous sub-batch, the
// same layouts with fewer streams. A group of one count goes out as before the
// counts came apart; streams of different counts share a launch (Ragged) when
// its grid, made for the largest count, has rows for at least half of its
// tiles, so that no short stream pays for a long one. A launch chain per count
// leaves the chip idle between and within its launches: 16 caches of 28 slices
// of up to 6272 rows at 11 fill levels took 880 us in 15 chains, 475 us in one. Groups reuse the
// workspace one after another on the stream; a stream with 0 rows is left alone.
Dims sub_batch(const Dims& d, int64_t nb) {
  Dims s = d;
  s.B = nb;
  s.slices = nb * d.L * d.H;
  return s;
}

template <typename T>
T* at_stream(T* p, int64_t b0, int64_t per_stream_elems) {
  return p ? p + b0 * per_stream_elems : p;
}

// fn(sub-batch dims, first stream, largest row count, Whole or Ragged) for every group
template <typename F>
ipv_status for_each_group(const Dims& d, const int32_t* n_tokens, F fn) {
  auto run_end = [&](int64_t b) {
    int64_t e = b + 1;
    while (e < d.B && n_tokens[e] == n_tokens[b]) ++e;
    return e;
  };
  for (int64_t b = 0, e; b < d.B; b = e) {
    e = run_end(b);
    if (n_tokens[b] == 0) continue;
    int64_t most = n_tokens[b], sum = most * (e - b), end = e;
    while (end < d.B) {
      const int64_t next = run_end(end), n = n_tokens[end];
      most = std::max(most, n);
      sum += n * (next - end);
      if (next - b > kMaxRagged || most * (next - b) > 2 * sum) break;
      end = next;
      if (n > 0) e = end;  // no empty streams at the end of a group
    }
    const Dims s = sub_batch(d, e - b);
    if (run_end(b) >= e) {
      IPV_TRY(fn(s, b, n_tokens[b], Whole{}));
      continue;
    }
    Ragged rows{make_fastdiv((uint32_t)(d.L * d.H)), make_fastdiv((uint32_t)((s.slices + 7) / 8)), (uint32_t)s.slices, {}};
    int32_t n = 0;
    for (int64_t i = b; i < e; ++i) n = std::max(n, rows.n[i - b] = n_tokens[i]);
    IPV_TRY(fn(s, b, n, rows));
  }
  return IPV_OK;
}

// every count in [0, min(S, kMaxRows)]; `each` checks the non-zero ones further
template <typename F>
ipv_status check_counts(const Dims& d, const int32_t* n_tokens, F each) {
  if (!n_tokens) return IPV_ERR_NULL;
  for (int64_t b = 0; b < d.B; ++b) {
    const int32_t n = n_tokens[b];
    if (n < 0 || n > d.S || n > kMaxRows) return IPV_ERR_SHAPE;
    if (n > 0) IPV_TRY(each(n));
  }
  return IPV_OK;
}

ipv_status no_check(int32_t) { return IPV_OK; }

// loop: the budget check of the continual-compression loop (check_loop_budget)
ipv_status check_pass_args(const Dims& d, const int32_t* n_tokens, int32_t budget, double alpha, int32_t r,
                           const double* cv_tau, uint32_t mode, bool loop = false) {
  IPV_TRY(check_recent(d, r));
  if (!(alpha >= 0.0 && alpha <= 1.0)) return IPV_ERR_ARG;
  IPV_TRY(check_counts(d, n_tokens, [&](int32_t n) {
    return loop ? check_loop_budget(d, n, budget, r) : check_budget(n, budget);
  }));
  IPV_TRY(check_tau(cv_tau));
  return check_mode(mode);
}

// the whole pass on one group; events (may be NULL) as in ipv_compress_timed
template <class ST>
ipv_status compress_run(const Dims& d, void* K, void* V, int32_t* fr, int32_t* pa, int32_t n, const ST& rows,
                        int32_t budget, double alpha, int32_t r, uint32_t mode, const double* cv_tau, float* tar, float* van,
                        int32_t* keep, void* ws, hipStream_t st, const ipv_events* events) {
  auto mark = [&](int i) -> ipv_status {
    if (!events || !events->at[i]) return IPV_OK;
    return hipEventRecord(static_cast<hipEvent_t>(events->at[i]), st) == hipSuccess ? IPV_OK : IPV_ERR_HIP;
  };
  const bool uniform = (mode & IPV_UNIFORM_SELECT) != 0;  // no scores: frame ids decide
  const bool adjacent = (mode & IPV_TAR_ADJACENT) != 0;
  // with the recent-key table, the pooling CV runs in the TaR launch
  const bool cv_fused = cv_tau && !uniform && !adjacent;
  if (!events && small_pass(d, n, r, mode, cv_tau))
    return run_small(d, K, V, fr, pa, n, rows, budget, floor_share(alpha, budget), r, mode, tar, van, keep, ws, st);
  IPV_TRY(mark(0));
  if (uniform)
    IPV_TRY(mark(1));
  else
    IPV_TRY(scores(d, K, V, fr, pa, n, rows, r, tar, van, ws, st, [&]() { return mark(1); }, compact_chunks(budget),
                   adjacent, cv_fused ? cv_tau : nullptr));
  IPV_TRY(mark(2));
  if (cv_tau && !uniform) IPV_TRY(pool_d(d, cv_tau, van, fr, pa, n, rows, nullptr, ws, st, cv_fused));
  IPV_TRY(mark(3));
  // the score launches zero the compaction's flags; without them the uniform selection does
  IPV_TRY(select(d, tar, van, fr, n, rows, budget, floor_share(alpha, budget), r, keep, err_word(ws), st, mode,
                 uniform ? ws_flags(ws, d) : nullptr,
                 (int32_t)(compact_parts(d) * walk_words(compact_chunks(budget)))));
  IPV_TRY(mark(4));
  IPV_TRY(compact(d, K, V, fr, pa, n, rows, keep, budget, ws, st, true));
  return mark(5);
}

// per-stream element counts of the arrays
int64_t kv_bytes_per_stream(const Dims& d) { return d.L * d.H * d.S * d.D * d.elem; }
int64_t rows_per_stream(const Dims& d) { return d.L * d.H * d.S; }

// Frames [0, frames) of K_new / V_new (frame j at byte j * frame_stride; in
// a frame the batch's [B, L, H, rows, D] layout) appended after row n of every
// slice of streams [b, e). Arguments checked by the caller.
ipv_status append_run(const Dims& d, int64_t b, int64_t e, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                      int32_t n, const void* K_new, const void* V_new, int32_t rows, int32_t frames,
                      int64_t frame_stride, int32_t frame_id, int32_t first_patch, hipStream_t st) {
  const int64_t RB = d.D * d.elem;
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d), nb = d.L * d.H * (int64_t)rows * RB;
  const int64_t pieces = (int64_t)frames * rows * (RB / 16), slices = (e - b) * d.L * d.H;
  const dim3 grid((uint32_t)std::min<int64_t>((pieces + 255) / 256, 256), (uint32_t)std::min<int64_t>(slices, 65535));
  k_append<<<grid, dim3(256), 0, st>>>(static_cast<const char*>(K_new) + b * nb,
                                       static_cast<const char*>(V_new) + b * nb, static_cast<char*>(K) + b * kb,
                                       static_cast<char*>(V) + b * kb, frame_idx + b * rs, patch_idx + b * rs, d.S, n,
                                       rows, frames, frame_stride, RB, frame_id, first_patch, slices);
  return launched();
}

// A stream's place in a call of the continual-compression loop. Streams with the
// same rows and the same pending frames are alike for the rest of the call,
// whatever counts they entered it with: the passes they have left and, once they
// have had one (pending > 0), where their rows are found follow from these two.
struct LoopStream {
  int32_t n0;       // rows before its pending frames
  int32_t pending;  // first frame of the call that is not in a pass yet
  int32_t left;     // passes left
  bool operator==(const LoopStream& o) const { return n0 == o.n0 && pending == o.pending; }
};

// fn(b, e) for every maximal run [b, e) of streams that are alike and satisfy want
template <typename W, typename F>
ipv_status for_alike(const std::vector<LoopStream>& ls, W want, F fn) {
  for (size_t b = 0; b < ls.size();) {
    size_t e = b + 1;
    while (e < ls.size() && ls[e] == ls[b]) ++e;
    if (want(ls[b])) IPV_TRY(fn((int64_t)b, (int64_t)e));
    b = e;
  }
  return IPV_OK;
}

}  // namespace

extern "C" {

ipv_status ipv_workspace_bytes(const ipv_shape* shape, size_t* bytes) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!bytes) return IPV_ERR_NULL;
  *bytes = ws_total(d);
  return IPV_OK;
}

ipv_status ipv_tar_scores(const ipv_shape* shape, const void* K, const int32_t* frame_idx, const int32_t* patch_idx,
                          const int32_t* n_tokens, int32_t recent_frames, uint32_t mode, float* tar, void* ws,
                          size_t ws_bytes, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!K || !frame_idx || !patch_idx || !tar) return IPV_ERR_NULL;
  if (!aligned(K, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) || !aligned(tar, 16)) return IPV_ERR_ALIGN;
  IPV_TRY(check_counts(d, n_tokens, no_check));
  IPV_TRY(check_recent(d, recent_frames));
  IPV_TRY(check_mode(mode));
  IPV_TRY(check_ws(d, ws, ws_bytes));
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d);
  return for_each_group(d, n_tokens, [&](const Dims& s, int64_t b0, int32_t n, const auto& rows) {
    return scores(s, static_cast<const char*>(K) + b0 * kb, nullptr, frame_idx + b0 * rs, patch_idx + b0 * rs, n,
                  rows, recent_frames, tar + b0 * rs, nullptr, ws, static_cast<hipStream_t>(stream), no_mark, 0,
                  (mode & IPV_TAR_ADJACENT) != 0);
  });
}

ipv_status ipv_van_scores(const ipv_shape* shape, const void* V, const int32_t* frame_idx, const int32_t* patch_idx,
                          const int32_t* n_tokens, const double* cv_tau, float* van, int32_t* pool_size, void* ws,
                          size_t ws_bytes, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!V || !frame_idx || !patch_idx || !van) return IPV_ERR_NULL;
  if (!aligned(V, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) || !aligned(van, 16)) return IPV_ERR_ALIGN;
  if (pool_size && !aligned(pool_size, 4)) return IPV_ERR_ALIGN;
  IPV_TRY(check_counts(d, n_tokens, no_check));
  IPV_TRY(check_tau(cv_tau));
  IPV_TRY(check_ws(d, ws, ws_bytes));
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d);
  return for_each_group(d, n_tokens, [&](const Dims& s, int64_t b0, int32_t n, const auto& rows) -> ipv_status {
    const int32_t* fr = frame_idx + b0 * rs;
    const int32_t* pa = patch_idx + b0 * rs;
    float* vn = van + b0 * rs;
    int32_t* ps = at_stream(pool_size, b0, d.L);
    IPV_TRY(scores(s, nullptr, static_cast<const char*>(V) + b0 * kb, fr, pa, n, rows, 1, nullptr, vn, ws, st));
    if (cv_tau) return pool_d(s, cv_tau, vn, fr, pa, n, rows, ps, ws, st);
    // a window of 1 for every stream with rows
    for (int64_t b = b0, e; ps && b < b0 + s.B; b = e) {
      for (e = b + 1; e < b0 + s.B && (n_tokens[e] > 0) == (n_tokens[b] > 0);) ++e;
      if (n_tokens[b] == 0) continue;
      const int64_t cnt = (e - b) * d.L;
      k_fill_i32<<<dim3((uint32_t)((cnt + 255) / 256)), dim3(256), 0, st>>>(pool_size + b * d.L, cnt, 1);
      IPV_TRY(launched());
    }
    return IPV_OK;
  });
}

ipv_status ipv_select(const ipv_shape* shape, const float* tar, const float* van, const int32_t* frame_idx,
                      const int32_t* n_tokens, int32_t budget, double alpha, int32_t recent_frames, uint32_t mode,
                      int32_t* keep_idx, void* ws, size_t ws_bytes, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!frame_idx || !keep_idx || (scores_needed(mode) && (!tar || !van))) return IPV_ERR_NULL;
  if (!aligned(tar, 16) || !aligned(van, 16) || !aligned(frame_idx, 16) || !aligned(keep_idx, 16)) return IPV_ERR_ALIGN;
  IPV_TRY(check_pass_args(d, n_tokens, budget, alpha, recent_frames, nullptr, mode));
  IPV_TRY(check_ws(d, ws, ws_bytes));
  const int64_t rs = rows_per_stream(d), ks = d.L * d.H * (int64_t)budget;
  return for_each_group(d, n_tokens, [&](const Dims& s, int64_t b0, int32_t n, const auto& rows) {
    return select(s, at_stream(tar, b0, rs), at_stream(van, b0, rs), frame_idx + b0 * rs, n, rows, budget,
                  floor_share(alpha, budget),
                  recent_frames, keep_idx + b0 * ks, err_word(ws), static_cast<hipStream_t>(stream), mode);
  });
}

ipv_status ipv_compact(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                       const int32_t* n_tokens, const int32_t* keep_idx, int32_t budget, void* ws, size_t ws_bytes,
                       void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!K || !V || !frame_idx || !patch_idx || !keep_idx) return IPV_ERR_NULL;
  if (!aligned(K, 16) || !aligned(V, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) ||
      !aligned(keep_idx, 16))
    return IPV_ERR_ALIGN;
  IPV_TRY(check_counts(d, n_tokens, [&](int32_t n) { return budget < 1 || budget > n ? IPV_ERR_BUDGET : IPV_OK; }));
  IPV_TRY(check_ws(d, ws, ws_bytes));
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d), ks = d.L * d.H * (int64_t)budget;
  return for_each_group(d, n_tokens, [&](const Dims& s, int64_t b0, int32_t n, const auto& rows) {
    return compact(s, static_cast<char*>(K) + b0 * kb, static_cast<char*>(V) + b0 * kb, frame_idx + b0 * rs,
                   patch_idx + b0 * rs, n, rows, keep_idx + b0 * ks, budget, ws, static_cast<hipStream_t>(stream));
  });
}

}  // extern "C"

namespace {

// Every host check of a whole pass except the workspace's.
ipv_status check_compress(const ipv_shape* shape, Dims* d, const void* K, const void* V, const int32_t* frame_idx,
                          const int32_t* patch_idx, const int32_t* n_tokens, int32_t budget, double alpha,
                          int32_t recent_frames, uint32_t mode, const double* cv_tau, const float* tar,
                          const float* van, const int32_t* keep_idx) {
  IPV_TRY(check_shape(shape, d));
  if (!K || !V || !frame_idx || !patch_idx || !keep_idx || (scores_needed(mode) && (!tar || !van)))
    return IPV_ERR_NULL;
  if (!aligned(K, 16) || !aligned(V, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) ||
      !aligned(tar, 16) || !aligned(van, 16) || !aligned(keep_idx, 16))
    return IPV_ERR_ALIGN;
  return check_pass_args(*d, n_tokens, budget, alpha, recent_frames, cv_tau, mode);
}

// ------------------------------------------------------------ allocation-free pass
// ipv_compress_noalloc's workspace: one array per GPU, allocated with the
// library's code object when it is loaded on that GPU and held until the
// process ends. Host code never passes `scratch` itself to a kernel (on the
// host the name is only a stand-in): it passes the device address that
// hipGetSymbolAddress returns for the current GPU, looked up on the first
// call on that GPU and kept per device.
constexpr size_t kScratchBytes = (size_t)96 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};

// The scratch array of the current device; the stream must belong to it.
ipv_status scratch_of(hipStream_t st, void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return IPV_ERR_HIP;
  if (st) {
    hipDevice_t sdev = -1;
    if (hipStreamGetDevice(st, &sdev) != hipSuccess) return IPV_ERR_HIP;
    if ((int)sdev != dev) return IPV_ERR_ARG;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return IPV_ERR_HIP;
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return IPV_OK;
}

// Whether a call's only pass of a stream runs in the cache, after an append of its
// new rows, instead of over the frames where they lie. That costs the append's read
// and write of the new rows and saves the TaR tiles over old rows, which fetch an m
// vector for every row; so it wins while few of the rows are new, and with pooling
// (the norms are read three more times) up to a little more. 112 slices of 6272 rows,
// 1 new frame of 32: 182 us over the frames, 167 in the cache; 3: 181, 170; 4: 179,
// 175; 6: 178, 183; 12288 rows, 1 of 48: 311, 286; 4: 308, 300; 5: 307, 304; 6: 307,
// 315, with pooling 351, 343; 80 slices of 32768 rows, 1 of 167: 586, 540; 12: 578,
// 572; 16: 579, 586. The consecutive-frame mode and Uniform Select have no m vectors:
// 1 frame of 32 takes 165 and 166, 94 and 95 us; but in the cache the rows that stay
// are compacted by more workgroups than select them: 48 slices of 50000 rows, half of
// which stay, 1 new frame, 462 over the frames, 422 in the cache, with pooling 783,
// 690, Uniform Select 239, 198.
bool pass_in_cache(int32_t n0, int32_t n, bool pool) { return (int64_t)(n - n0) * (pool ? 8 : 10) <= n; }

// Whether all passes of a call run in the cache, each after an append of its new
// rows, because what they would do besides selecting costs more than they save.
// n: most rows of a pass; passes: most of a stream; fresh: new rows of a pass; saved:
// bytes that its appends and moves in the cache come to. A selection compacts the
// metadata of its slices by one workgroup, a head after another, where the compaction
// in the cache has hundreds; the pooling, a workgroup a slice, finds every row's frame
// through its place, three times. Fitted to 13384 calls of 1 and 3 passes (1 to 8
// selections, 1 to 8 heads, rows of 64 to 512 bytes, 3136 to 60000 rows, budgets of
// 2/5 to 3/4), us a pass over the frames against in the cache: +0.5 a thousand rows
// and head (1500 more a head: a batch's latency), +20 for Uniform Select beyond 32768
// rows (its registers spill there), with pooling +2.5 a thousand rows beyond 8000 and
// +60 beyond 32768 rows, -0.42 a saved MB, -6 for two launches less, +2 a call for the
// gather, and in the consecutive-frame mode -2 a thousand fresh rows, which are not
// walked. Calls of 3 passes, rows of 128 bytes, over the frames / in the cache:
// head-shared on one layer, budget 3/4, 8 heads of 6272 rows 201 / 157, of 60000 1996
// / 1355, 4 heads of 3136 109 / 110, of 6272 139 / 130, 2 of 6272 (not by this rule)
// 113 / 121; Uniform Select, 8 heads of 46000 rows 840 / 571; with pooling, budget
// 1/2, 2 slices of 50000 rows 1833 / 1234, 48 (not by this rule) 2574 / 2599, 1 of
// 9000 (not by this rule) 244 / 242.
bool call_in_cache(const Dims& d, int32_t n, int32_t passes, int32_t budget, uint32_t mode, bool pool, int64_t fresh,
                   int64_t saved) {
  const double heads = (mode & IPV_HEAD_SHARED) ? (double)d.H : 1.0, spill = n > 32768 ? 1.0 : 0.0;
  const double emit = 0.0005 * heads * (budget + 1500) + ((mode & IPV_UNIFORM_SELECT) ? 20.0 * spill : 0.0);
  const double smooth = pool ? 0.0025 * std::max(n - 8000, 0) + 60.0 * spill : 0.0;
  const double walk = (mode & IPV_TAR_ADJACENT) && scores_needed(mode) ? 0.002 * (double)fresh : 0.0;
  return emit + smooth > 6.0 - 2.0 / passes + 0.42e-6 * (double)saved + walk;
}

// Frames [0, n_frames) of a call of the continual-compression loop whose
// arguments are checked: the passes run over the frames where they lie, one
// gather per stream follows its last pass, and the frames after that are
// appended (or in the cache: call_in_cache, pass_in_cache). The places
// of a stream's rows between two passes are kept in its rows of keep_idx, its
// value norms in van (without pooling, which overwrites them); the last pass
// leaves its keep set and scores there, and the places of the rows that stay in
// the workspace's table region, whose contents (the m vectors or prev rows) the
// pass has used by then.
ipv_status stream_part(const Dims& d, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx, int32_t* n_tokens,
                       const char* fk, const char* fv, int32_t n_frames, int32_t rows, int32_t first_frame_id,
                       int32_t mem_cap, int32_t budget, double alpha, int32_t r, uint32_t mode, const double* cv_tau,
                       float* tar, float* van, int32_t* keep_idx, void* ws, int32_t* passes, hipStream_t st) {
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d), ks = d.L * d.H * (int64_t)budget;
  const int64_t nb = d.L * d.H * (int64_t)rows * d.D * d.elem, frame_bytes = d.B * nb;
  const bool uniform = (mode & IPV_UNIFORM_SELECT) != 0, adjacent = (mode & IPV_TAR_ADJACENT) != 0;
  const bool pool = cv_tau && !uniform;
  auto fires_in = [&](int32_t n) { return (mem_cap - n + rows - 1) / rows; };  // frames until the cap, the last included
  std::vector<LoopStream> ls((size_t)d.B);
  int64_t fresh = 0, moved = 0;  // rows of a slice that the streams' passes bring; that those in the cache move
  int64_t fired = 0, firsts = 0, laters = 0;  // streams that fire; groups of them in first passes (alike in their
                                              // rows) and in later ones (in the frame of the first pass)
  int32_t most = 1, n_most = 0;   // most passes of a stream and rows of a pass
  for (int64_t b = 0; b < d.B; ++b) {
    ls[b] = {n_tokens[b], 0, 0};
    // a budget equal to the cap fires once: the checks let no frame follow that pass
    const int64_t later = fires_in(budget);
    for (int64_t f = fires_in(n_tokens[b]); f <= n_frames; f += later) {
      ++ls[b].left;
      if (later < 1) break;
    }
    if (ls[b].left == 0) continue;
    ++fired;
    const bool begins = b == 0 || ls[b - 1].left == 0;
    firsts += begins || n_tokens[b] != n_tokens[b - 1];
    laters += begins || fires_in(n_tokens[b]) != fires_in(n_tokens[b - 1]);
    fresh += (fires_in(n_tokens[b]) + (ls[b].left - 1) * later) * rows;
    moved += (int64_t)(ls[b].left - 1) * budget;
    most = std::max(most, ls[b].left);
    n_most = std::max<int32_t>(n_most, n_tokens[b] + fires_in(n_tokens[b]) * rows);
  }
  const bool in_cache = fired && call_in_cache(d, n_most, most, budget, mode, pool, fresh / (fired * most),
                                               2 * d.L * d.H * (fresh + moved) * d.D * d.elem / (firsts + laters * (most - 1)));
  auto done = [&](int64_t b, int64_t e, int64_t f) {  // streams [b, e) had a pass at frame f
    for (; b < e; ++b) {
      ls[b] = {budget, (int32_t)f + 1, ls[b].left - 1};
      ++passes[b];
    }
  };
  bool ahead = false;  // the next pass's first launch is out
  for (;;) {
    // the next frame at which a stream reaches the cap (frames [pending, f] are its new rows)
    int64_t f = INT64_MAX;
    for (const LoopStream& s : ls)
      if (s.left > 0) f = std::min<int64_t>(f, (int64_t)s.pending + fires_in(s.n0) - 1);
    if (f == INT64_MAX) break;
    auto fires = [&](const LoopStream& s) { return s.left > 0 && (int64_t)s.pending + fires_in(s.n0) - 1 == f; };
    IPV_TRY(for_alike(ls, fires, [&](int64_t b0, int64_t e) -> ipv_status {
      const Dims s = sub_batch(d, e - b0);
      const LoopStream l = ls[b0];
      const bool last = l.left == 1;
      const int32_t n = l.n0 + (int32_t)(f + 1 - l.pending) * rows;
      const int64_t chunks = last ? compact_chunks(budget) : 0;
      char* k = static_cast<char*>(K) + b0 * kb;
      char* v = static_cast<char*>(V) + b0 * kb;
      int32_t* fr = frame_idx + b0 * rs;
      int32_t* pa = patch_idx + b0 * rs;
      int32_t* keep = keep_idx + b0 * ks;
      float* tr = at_stream(tar, b0, rs);
      float* vn = at_stream(van, b0, rs);
      const bool small = small_pass(s, n, r, mode, cv_tau, kSmallFrameStretch);
      if (in_cache || (last && l.pending == 0 && !small && pass_in_cache(l.n0, n, pool))) {
        IPV_TRY(append_run(d, b0, e, K, V, frame_idx, patch_idx, l.n0, fk + l.pending * frame_bytes,
                           fv + l.pending * frame_bytes, rows, (int32_t)f + 1 - l.pending, frame_bytes,
                           first_frame_id + l.pending, 0, st));
        IPV_TRY(compress_run(s, k, v, fr, pa, n, Whole{}, budget, alpha, r, mode, cv_tau, tr, vn, keep, ws, st, nullptr));
        done(b0, e, f);
        return IPV_OK;
      }
      // the pass over l_n0 rows and the frames from `pending` on
      auto stretch = [&](int32_t l_n0, int32_t pending, const int32_t* src) {
        Stretch sr{};
        sr.K = fk + b0 * nb;
        sr.V = fv + b0 * nb;
        sr.stride = frame_bytes;
        sr.src = src;
        sr.src_stride = budget;
        sr.rows = make_fastdiv((uint32_t)rows);
        sr.n0 = (uint32_t)l_n0;
        sr.f0 = (uint32_t)pending;
        sr.eoff = (uint32_t)pending * (uint32_t)rows - (uint32_t)l_n0;
        sr.id0 = first_frame_id;
        return sr;
      };
      const Stretch sr = stretch(l.n0, l.pending, l.pending ? keep : nullptr);
      int32_t* places = reinterpret_cast<int32_t*>(ws_table(ws));
      const int32_t new_frames = (int32_t)fires_in(budget), n_next = budget + new_frames * rows;  // the next pass's
      if (!uniform && !small)
        IPV_TRY(stretch_scores(s, k, v, sr, fr, pa, n, r, tr, vn, ws, st, chunks, adjacent,
                               pool && !adjacent ? cv_tau : nullptr, l.pending > 0 && !pool, ahead));
      if (pool) IPV_TRY(pool_d(s, cv_tau, vn, fr, pa, n, sr, nullptr, ws, st, !adjacent));
      // a group that is the whole batch stays alike, so the next pass is its own
      ahead = s.B == d.B && !last && !uniform && !pool && !small && l.n0 <= budget &&
              ahead_fits(s, n, r, mode, new_frames) && !small_pass(s, n_next, r, mode, cv_tau, kSmallFrameStretch);
      const Emit em{fr,
                    pa,
                    last ? places : keep,
                    last ? s.S : budget,
                    last || pool || uniform ? nullptr : vn,
                    last ? keep : nullptr};
      if (small)
        IPV_TRY(run_small_stretch(s, k, v, sr, fr, pa, n, budget, floor_share(alpha, budget), r, mode, tr, vn,
                                  l.pending > 0 ? sr.n0 : 0u, em, last, ws, st));
      else if (ahead)
        IPV_TRY(select_ahead(s, tr, vn, fr, pa, n, sr, budget, floor_share(alpha, budget), r, em, k, v,
                             stretch(budget, (int32_t)f + 1, nullptr), n_next,
                             l.left == 2 ? compact_chunks(budget) : 0, ws, st, mode));
      else
        IPV_TRY(select(s, tr, vn, fr, n, sr, budget, floor_share(alpha, budget), r, keep, err_word(ws), st, mode,
                       uniform && last ? ws_flags(ws, s) : nullptr, (int32_t)(compact_parts(s) * walk_words(chunks)),
                       em));
      // only the gather asks how many rows the streams entered the call with: the most of them bounds its waits
      const int32_t n_entry = *std::max_element(n_tokens + b0, n_tokens + e);
      if (last && !small) IPV_TRY(stretch_gather(s, k, v, sr, places, n_entry, budget, ws, st));
      done(b0, e, f);
      return IPV_OK;
    }));
  }
  // the frames after a stream's last pass
  IPV_TRY(for_alike(ls, [&](const LoopStream& s) { return s.pending < n_frames; }, [&](int64_t b, int64_t e) {
    const LoopStream l = ls[b];
    return append_run(d, b, e, K, V, frame_idx, patch_idx, l.n0, fk + l.pending * frame_bytes, fv + l.pending * frame_bytes,
                      rows, n_frames - l.pending, frame_bytes, first_frame_id + l.pending, 0, st);
  }));
  for (int64_t b = 0; b < d.B; ++b) n_tokens[b] = ls[b].n0 + (n_frames - ls[b].pending) * rows;
  return IPV_OK;
}

bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + (uintptr_t)b_bytes && y < x + (uintptr_t)a_bytes;
}

__global__ void k_copy_word(uint32_t* dst, const uint32_t* src) {
  if (threadIdx.x == 0) *dst = *src;
}

}  // namespace

extern "C" {

ipv_status ipv_compress_noalloc(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                                const int32_t* n_tokens, int32_t budget, double alpha, int32_t recent_frames,
                                uint32_t mode, const double* cv_tau, float* tar, float* van, int32_t* keep_idx,
                                uint32_t* device_errors, void* stream) {
  Dims d;
  IPV_TRY(check_compress(shape, &d, K, V, frame_idx, patch_idx, n_tokens, budget, alpha, recent_frames, mode,
                         cv_tau, tar, van, keep_idx));
  if (ws_total(d) > kScratchBytes) return IPV_ERR_WORKSPACE;
  if (device_errors && !aligned(device_errors, 4)) return IPV_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  void* ws = nullptr;
  IPV_TRY(scratch_of(st, &ws));
  // the error word starts at zero (a kernel, not a memset, so the call can be
  // captured into a graph); everything else the pass reads it writes first
  k_fill_i32<<<dim3(1), dim3(64), 0, st>>>(static_cast<int32_t*>(ws), 1, 0);
  IPV_TRY(launched());
  IPV_TRY(ipv_compress_timed(shape, K, V, frame_idx, patch_idx, n_tokens, budget, alpha, recent_frames, mode,
                             cv_tau, tar, van, keep_idx, ws, kScratchBytes, stream, nullptr));
  if (device_errors) {
    k_copy_word<<<dim3(1), dim3(64), 0, st>>>(device_errors, err_word(ws));
    return launched();
  }
  return IPV_OK;
}

ipv_status ipv_compress_timed(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                              const int32_t* n_tokens, int32_t budget, double alpha, int32_t recent_frames,
                              uint32_t mode, const double* cv_tau, float* tar, float* van, int32_t* keep_idx,
                              void* ws, size_t ws_bytes, void* stream, const ipv_events* events) {
  Dims d;
  IPV_TRY(check_compress(shape, &d, K, V, frame_idx, patch_idx, n_tokens, budget, alpha, recent_frames, mode,
                         cv_tau, tar, van, keep_idx));
  IPV_TRY(check_ws(d, ws, ws_bytes));
  const int64_t kb = kv_bytes_per_stream(d), rs = rows_per_stream(d), ks = d.L * d.H * (int64_t)budget;
  return for_each_group(d, n_tokens, [&](const Dims& s, int64_t b0, int32_t n, const auto& rows) {
    return compress_run(s, static_cast<char*>(K) + b0 * kb, static_cast<char*>(V) + b0 * kb, frame_idx + b0 * rs,
                        patch_idx + b0 * rs, n, rows, budget, alpha, recent_frames, mode, cv_tau, at_stream(tar, b0, rs),
                        at_stream(van, b0, rs), keep_idx + b0 * ks, ws, static_cast<hipStream_t>(stream), events);
  });
}

ipv_status ipv_compress(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                        const int32_t* n_tokens, int32_t budget, double alpha, int32_t recent_frames, uint32_t mode,
                        const double* cv_tau, float* tar, float* van, int32_t* keep_idx, void* ws, size_t ws_bytes,
                        void* stream) {
  return ipv_compress_timed(shape, K, V, frame_idx, patch_idx, n_tokens, budget, alpha, recent_frames, mode, cv_tau,
                            tar, van, keep_idx, ws, ws_bytes, stream, nullptr);
}

ipv_status ipv_append(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                      const int32_t* n_tokens, const void* K_new, const void* V_new, int32_t rows, int32_t frame_id,
                      int32_t first_patch, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!K || !V || !frame_idx || !patch_idx || !K_new || !V_new || !n_tokens) return IPV_ERR_NULL;
  if (!aligned(K, 16) || !aligned(V, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) ||
      !aligned(K_new, 16) || !aligned(V_new, 16))
    return IPV_ERR_ALIGN;
  if (rows < 1) return IPV_ERR_SHAPE;
  for (int64_t b = 0; b < d.B; ++b)
    if (n_tokens[b] < 0 || (int64_t)n_tokens[b] + rows > d.S) return IPV_ERR_SHAPE;
  if (first_patch < 0 || (int64_t)first_patch + rows > d.p) return IPV_ERR_ARG;
  // one launch per run of equal counts (an empty stream appends at row 0 like any other)
  for (int64_t b = 0, e; b < d.B; b = e) {
    for (e = b + 1; e < d.B && n_tokens[e] == n_tokens[b];) ++e;
    IPV_TRY(append_run(d, b, e, K, V, frame_idx, patch_idx, n_tokens[b], K_new, V_new, rows, 1, 0, frame_id,
                       first_patch, static_cast<hipStream_t>(stream)));
  }
  return IPV_OK;
}

ipv_status ipv_ckv_step(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                        const int32_t* n_tokens, const void* K_new, const void* V_new, int32_t rows, int32_t frame_id,
                        int32_t first_patch, int32_t mem_cap, int32_t budget, double alpha, int32_t recent_frames,
                        uint32_t mode, const double* cv_tau, float* tar, float* van, int32_t* keep_idx, void* ws,
                        size_t ws_bytes, int32_t* n_out, int32_t* compressed, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!n_out || !compressed || !n_tokens) return IPV_ERR_NULL;
  if (mem_cap < 1 || mem_cap > d.S) return IPV_ERR_SHAPE;
  if (budget > mem_cap) return IPV_ERR_BUDGET;
  // the row counts after the append; the streams that reach the cap run the pass
  std::vector<int32_t> after((size_t)d.B), pass((size_t)d.B);
  bool any = false;
  for (int64_t b = 0; b < d.B; ++b) {
    if (n_tokens[b] < 0 || n_tokens[b] >= mem_cap) return IPV_ERR_SHAPE;
    after[b] = n_tokens[b] + rows;
    pass[b] = after[b] >= mem_cap ? after[b] : 0;
    any |= pass[b] > 0;
  }
  if (any) {
    // every argument of the pass is checked before the append is enqueued
    if (!keep_idx || !K || !V || !frame_idx || !patch_idx || (scores_needed(mode) && (!tar || !van)))
      return IPV_ERR_NULL;
    if (!aligned(tar, 16) || !aligned(van, 16) || !aligned(keep_idx, 16)) return IPV_ERR_ALIGN;
    IPV_TRY(check_pass_args(d, pass.data(), budget, alpha, recent_frames, cv_tau, mode, true));
    IPV_TRY(check_ws(d, ws, ws_bytes));
  }
  IPV_TRY(ipv_append(shape, K, V, frame_idx, patch_idx, n_tokens, K_new, V_new, rows, frame_id, first_patch, stream));
  if (any)
    IPV_TRY(ipv_compress(shape, K, V, frame_idx, patch_idx, pass.data(), budget, alpha, recent_frames, mode, cv_tau,
                         tar, van, keep_idx, ws, ws_bytes, stream));
  for (int64_t b = 0; b < d.B; ++b) {
    n_out[b] = pass[b] > 0 ? budget : after[b];
    compressed[b] = pass[b] > 0;
  }
  return IPV_OK;
}

ipv_status ipv_ckv_stream(const ipv_shape* shape, void* K, void* V, int32_t* frame_idx, int32_t* patch_idx,
                          int32_t* n_tokens, const void* frames_K, const void* frames_V, int32_t n_frames,
                          int32_t rows, int32_t first_frame_id, int32_t mem_cap, int32_t budget, double alpha,
                          int32_t recent_frames, uint32_t mode, const double* cv_tau, float* tar, float* van,
                          int32_t* keep_idx, void* ws, size_t ws_bytes, int32_t* passes, void* stream) {
  Dims d;
  IPV_TRY(check_shape(shape, &d));
  if (!n_tokens || !passes || !frames_K || !frames_V || !K || !V || !frame_idx || !patch_idx) return IPV_ERR_NULL;
  if (!aligned(K, 16) || !aligned(V, 16) || !aligned(frame_idx, 16) || !aligned(patch_idx, 16) ||
      !aligned(frames_K, 16) || !aligned(frames_V, 16))
    return IPV_ERR_ALIGN;
  if (n_frames < 0 || rows < 1 || mem_cap < 1 || mem_cap > d.S) return IPV_ERR_SHAPE;
  if (budget > mem_cap) return IPV_ERR_BUDGET;
  if ((int64_t)first_frame_id + n_frames > INT32_MAX || rows > d.p) return IPV_ERR_ARG;
  // every step is checked on the host before the first one is enqueued: the
  // row counts of the whole stretch follow from the counts, rows and cap alone
  std::vector<int32_t> n(n_tokens, n_tokens + d.B), after((size_t)d.B), pass((size_t)d.B);
  bool any_pass = false;
  for (int32_t f = 0; f < n_frames; ++f) {
    bool any = false;
    for (int64_t b = 0; b < d.B; ++b) {
      if (n[b] < 0 || n[b] >= mem_cap || (int64_t)n[b] + rows > d.S) return IPV_ERR_SHAPE;
      after[b] = n[b] + rows;
      pass[b] = after[b] >= mem_cap ? after[b] : 0;
      any |= pass[b] > 0;
    }
    if (any) IPV_TRY(check_pass_args(d, pass.data(), budget, alpha, recent_frames, cv_tau, mode, true));
    any_pass |= any;
    for (int64_t b = 0; b < d.B; ++b) n[b] = pass[b] > 0 ? budget : after[b];
  }
  if (any_pass) {
    if (!keep_idx || (scores_needed(mode) && (!tar || !van))) return IPV_ERR_NULL;
    if (!aligned(tar, 16) || !aligned(van, 16) || !aligned(keep_idx, 16)) return IPV_ERR_ALIGN;
    IPV_TRY(check_ws(d, ws, ws_bytes));
  }
  // a call that the runtime stops halfway reports the counts it came with and no passes
  for (int64_t b = 0; b < d.B; ++b) passes[b] = 0;
  std::vector<int32_t> done((size_t)d.B, 0);
  n.assign(n_tokens, n_tokens + d.B);
  const int64_t frame_bytes = d.slices * rows * d.D * d.elem, cache_bytes = d.B * kv_bytes_per_stream(d);
  const int64_t call_bytes = n_frames * frame_bytes;
  const char* fk = static_cast<const char*>(frames_K);
  const char* fv = static_cast<const char*>(frames_V);
  if (overlap(fk, call_bytes, K, cache_bytes) || overlap(fk, call_bytes, V, cache_bytes) ||
      overlap(fv, call_bytes, K, cache_bytes) || overlap(fv, call_bytes, V, cache_bytes)) {
    // frames in the cache's own memory (written where they will be appended, say) do not stay
    // where they are while passes run: the loop step by step
    for (int32_t f = 0; f < n_frames; ++f) {
      IPV_TRY(ipv_ckv_step(shape, K, V, frame_idx, patch_idx, n.data(), fk + f * frame_bytes, fv + f * frame_bytes, rows,
                           first_frame_id + f, 0, mem_cap, budget, alpha, recent_frames, mode, cv_tau, tar, van,
                           keep_idx, ws, ws_bytes, after.data(), pass.data(), stream));
      for (int64_t b = 0; b < d.B; ++b) {
        n[b] = after[b];
        done[b] += pass[b];
      }
    }
  } else {
    // places of frame rows are 31-bit: longer calls are taken in parts
    const int32_t part = std::max<int32_t>(1, (INT32_MAX - 1) / rows);
    for (int32_t f = 0; f < n_frames; f += std::min(part, n_frames - f)) {
      const int32_t count = std::min(part, n_frames - f);
      IPV_TRY(stream_part(d, K, V, frame_idx, patch_idx, n.data(), fk + f * frame_bytes, fv + f * frame_bytes, count, rows,
                          first_frame_id + f, mem_cap, budget, alpha, recent_frames, mode, cv_tau, tar, van, keep_idx, ws,
                          done.data(), static_cast<hipStream_t>(stream)));
    }
  }
  std::copy(n.begin(), n.end(), n_tokens);
  std::copy(done.begin(), done.end(), passes);
  return IPV_OK;
}

ipv_status ipv_clear_device_errors(void* ws, size_t ws_bytes, void* stream) {
  if (!ws) return IPV_ERR_NULL;
  if (!aligned(ws, 256)) return IPV_ERR_ALIGN;
  if (ws_bytes < kWsHeader) return IPV_ERR_WORKSPACE;
  k_fill_i32<<<dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream)>>>(static_cast<int32_t*>(ws), 1, 0);
  return launched();
}

ipv_status ipv_read_device_errors(const void* ws, size_t ws_bytes, void* stream, uint32_t* flags) {
  if (!ws || !flags) return IPV_ERR_NULL;
  if (!aligned(ws, 256)) return IPV_ERR_ALIGN;
  if (ws_bytes < kWsHeader) return IPV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(flags, ws, sizeof(uint32_t), hipMemcpyDeviceToHost, st) != hipSuccess) return IPV_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return IPV_ERR_HIP;
  return IPV_OK;
}

const char* ipv_status_str(ipv_status s) {
  switch (s) {
    case IPV_OK: return "ok";
    case IPV_ERR_NULL: return "a required pointer is NULL";
    case IPV_ERR_ALIGN: return "a pointer is not aligned as required";
    case IPV_ERR_SHAPE: return "unsupported or inconsistent shape";
    case IPV_ERR_DTYPE: return "unsupported dtype";
    case IPV_ERR_BUDGET: return "budget outside [1, n] (continual-compression loop: [min(n, r*p), n])";
    case IPV_ERR_ARG: return "invalid argument (alpha, recent_frames or cv_tau)";
    case IPV_ERR_WORKSPACE: return "workspace missing or too small";
    case IPV_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

}  // extern "C"
