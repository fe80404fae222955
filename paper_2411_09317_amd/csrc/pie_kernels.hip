// HIP kernels for gfx950 (CDNA4, 64-wide wavefronts): paged-attention decode with a split over the
// context and its reduction, the KV append, the block gather / scatter used by swaps, and the small
// map-maintenance kernels.
//
// What the attention kernels compute is the paged KV-cache attention of the paper's Section 2.3 for the
// per-layer access pattern of Section 3.2:
//   out[b][h] = sum_t softmax_t(scale * <q[b][h], K[b][g][t]>) V[b][g][t],   t < ctx_b,  g = h / (Hq/Hkv).
//
// One block of one layer holds the K tiles of the kv heads, then their V tiles; inside a tile the elements are
// ordered so that a 16-byte lane vector is a matrix-core operand as loaded (see "element types and the layout
// of a block" below).  The decode is bound by HBM bandwidth: every KV byte of the layer is read exactly once,
// with 16-byte loads per lane that cover a tile in contiguous 1 KiB pieces.

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <mutex>

#include <hip/hip_ext.h>

#include "pie_attn_wide.h"
#include "pie_internal.h"

namespace pie {

// ---------------------------------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------------------------------

__global__ void k_fill_i32(int32_t* __restrict__ p, int32_t n, int32_t v) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_map_patch(int32_t* __restrict__ map, const MapPatch patch) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < patch.n) map[patch.handle[i]] = patch.slot[i];
}

// Occupies a stream for about `ticks` ticks of the constant wall clock: one wave that sleeps and looks at
// the clock.  max_iter bounds the loop, so the wave exits whatever the clock does.
__global__ void k_busy(unsigned long long ticks, uint32_t max_iter, unsigned long long* clock) {
  const unsigned long long t0 = wall_clock64();
  for (uint32_t i = 0; i < max_iter; ++i) {
    if (wall_clock64() - t0 >= ticks) break;
    __builtin_amdgcn_s_sleep(16);
  }
  if (clock && threadIdx.x == 0) atomicMax(&clock[kClockLayerEnd], wall_clock64());
}

// ---- device-clock time stamps ---------------------------------------------------------------------------
// With monitoring by device clock a layer's kernels note when they ran, read from the constant-rate wall
// clock all compute units share; nothing is recorded between kernels, so they stay back to back.  Each layer
// has a row of 64-bit words (kClock*).  Atomics on one address cost about 8 ns each and all of it shows in
// the kernel's duration, so the persistent decode kernel's workgroups write their first and last moment to
// words of their own (kClockWgs pairs per layer) and k_clock_fold, once per step, folds them into the row;
// kernels with few workgroups, or few that matter, use atomic min / max on the row directly.  Work on the
// swap streams is bracketed by k_stamp.
__global__ void k_stamp(unsigned long long* slot) {
  if (threadIdx.x == 0) *slot = wall_clock64();
}

// One workgroup per layer: row[KernelStart / KernelEnd] take in the per-workgroup pairs (row[kClockGrid] of
// them), and row[LayerEnd] is at least the kernel's end.
__global__ __launch_bounds__(256) void k_clock_fold(unsigned long long* __restrict__ rows,
                                                    const unsigned long long* __restrict__ per_wg) {
  __shared__ unsigned long long s_lo[256], s_hi[256];
  unsigned long long* row = rows + (size_t)blockIdx.x * kClockRow;
  const unsigned long long* wg = per_wg + (size_t)blockIdx.x * kClockWgs * 2;
  unsigned long long n = row[kClockGrid];
  n = n > (unsigned long long)kClockWgs ? (unsigned long long)kClockWgs : n;
  unsigned long long lo = ~0ull, hi = 0ull;
  for (unsigned long long i = threadIdx.x; i < n; i += 256) {
    const unsigned long long a = wg[2 * i], b = wg[2 * i + 1];
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  s_lo[threadIdx.x] = lo;
  s_hi[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s_lo[threadIdx.x] = s_lo[threadIdx.x + w] < s_lo[threadIdx.x] ? s_lo[threadIdx.x + w] : s_lo[threadIdx.x];
      s_hi[threadIdx.x] = s_hi[threadIdx.x + w] > s_hi[threadIdx.x] ? s_hi[threadIdx.x + w] : s_hi[threadIdx.x];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const unsigned long long ks = row[kClockKernelStart], ke = row[kClockKernelEnd], le = row[kClockLayerEnd];
    const unsigned long long start = s_lo[0] < ks ? s_lo[0] : ks, end = s_hi[0] > ke ? s_hi[0] : ke;
    row[kClockKernelStart] = start;
    row[kClockKernelEnd] = end;
    row[kClockLayerEnd] = le > end ? le : end;
  }
}

int launch_clock_fold(unsigned long long* rows, int32_t n_layers, hipStream_t s) {
  hipLaunchKernelGGL(k_clock_fold, dim3(n_layers), dim3(256), 0, s, rows,
                     rows + ((size_t)n_layers + 1) * kClockRow);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_stamp(unsigned long long* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, s, slot);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_busy(double us, int wall_clock_khz, hipStream_t s, unsigned long long* clock, hipEvent_t done) {
  if (!(us > 0.0)) return PIE_OK;
  const unsigned long long ticks = (unsigned long long)(us * 1e-3 * (double)wall_clock_khz);
  // an iteration takes at least the sleep's 16 x 64 clocks, i.e. well over 0.1 us: 16 iterations per us plus
  // slack always reach the deadline first
  const uint32_t max_iter = (uint32_t)(us * 16.0) + 4096u;
  // `done` completes with the kernel itself: no separate packet on the stream
  if (done) hipExtLaunchKernelGGL(k_busy, dim3(1), dim3(64), 0, s, nullptr, done, 0, ticks, max_iter, clock);
  else hipLaunchKernelGGL(k_busy, dim3(1), dim3(64), 0, s, ticks, max_iter, clock);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_map_fill(int32_t* d_map, int32_t n, int32_t value, hipStream_t s) {
  if (n <= 0) return PIE_OK;
  hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, s, d_map, n, value);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_zero_u32(uint32_t* d, int32_t n, hipStream_t s) {
  return launch_map_fill(reinterpret_cast<int32_t*>(d), n, 0, s);
}

// A layer whose blocks are spread over chunks of `chunk_blocks` consecutive slots: block h lives in slot
// chunks[h / chunk_blocks] * chunk_blocks + h % chunk_blocks; blocks beyond the layer's chunks map to -1.
__global__ void k_chunk_map_fill(int32_t* __restrict__ map, int32_t n_handles, int32_t chunk_blocks, const ChunkList list) {
  const int32_t h = blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= n_handles) return;
  const int32_t c = h / chunk_blocks;
  map[h] = c < list.n ? list.chunk[c] * chunk_blocks + h % chunk_blocks : -1;
}

int launch_chunk_map_fill(int32_t* d_map, int32_t n_handles, int32_t chunk_blocks, const ChunkList& list, hipStream_t s) {
  if (n_handles <= 0) return PIE_OK;
  hipLaunchKernelGGL(k_chunk_map_fill, dim3((n_handles + 255) / 256), dim3(256), 0, s, d_map, n_handles, chunk_blocks, list);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_map_patch(int32_t* d_map, const MapPatch& patch, hipStream_t s) {
  if (patch.n <= 0) return PIE_OK;
  hipLaunchKernelGGL(k_map_patch, dim3((patch.n + 255) / 256), dim3(256), 0, s, d_map, patch);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

// ---------------------------------------------------------------------------------------------------
// block gather / scatter (swap path PIE_SWAP_KERNEL)
//
// Copies pairs.n blocks of block_bytes each: dst_base + dst[i]*block_bytes <- src_base + src[i]*block_bytes.
// Either side may be pinned host memory mapped into the device's address space, so the kernel is bound by
// the host link: what matters is the number of 16-byte requests in flight, not the number of CUs (one compute
// unit sustains about 3.5 GB/s per wavefront with sixteen loads in flight, at most about 14 GB/s).  A fixed,
// small grid strides over pieces of THREADS x UNROLL 16-byte vectors; each lane keeps UNROLL loads in flight.
// ---------------------------------------------------------------------------------------------------

template <int THREADS, int UNROLL>
__global__ __launch_bounds__(THREADS) void k_swap_copy(char* __restrict__ dst_base, const char* __restrict__ src_base,
                                                       size_t block_bytes, const SwapPairs pairs) {
  constexpr size_t kPiece = (size_t)THREADS * 16 * UNROLL;        // bytes per workgroup iteration
  // few instructions, long waits: let them issue ahead of the decode kernel's waves on the same compute unit
  __builtin_amdgcn_s_setprio(3);
  const size_t pieces_per_block = (block_bytes + kPiece - 1) / kPiece;
  const size_t n_pieces = pieces_per_block * (size_t)pairs.n;
  for (size_t piece = blockIdx.x; piece < n_pieces; piece += gridDim.x) {
    const int32_t i = (int32_t)(piece / pieces_per_block);
    const size_t off = (piece % pieces_per_block) * kPiece;
    const u32x4* s = reinterpret_cast<const u32x4*>(src_base + (size_t)pairs.src[i] * block_bytes + off);
    u32x4* d = reinterpret_cast<u32x4*>(dst_base + (size_t)pairs.dst[i] * block_bytes + off);
    const size_t n16 = (block_bytes - off < kPiece ? block_bytes - off : kPiece) / 16;
    u32x4 v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const size_t j = (size_t)u * THREADS + threadIdx.x;
      if (j < n16) v[u] = __builtin_nontemporal_load(s + j);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const size_t j = (size_t)u * THREADS + threadIdx.x;
      if (j < n16) __builtin_nontemporal_store(v[u], d + j);
    }
  }
}

template <int THREADS, int UNROLL>
static int launch_swap_copy_as(char* dst_layer_base, const char* src_layer_base, size_t block_bytes,
                               const SwapPairs& pairs, int n_wgs, hipStream_t s, hipEvent_t done) {
  constexpr size_t kPiece = (size_t)THREADS * 16 * UNROLL;
  const size_t pieces = ((block_bytes + kPiece - 1) / kPiece) * (size_t)pairs.n;
  const int grid = (int)(pieces < (size_t)n_wgs ? pieces : (size_t)n_wgs);
  if (done)
    hipExtLaunchKernelGGL((k_swap_copy<THREADS, UNROLL>), dim3(grid), dim3(THREADS), 0, s, nullptr, done, 0, dst_layer_base,
                          src_layer_base, block_bytes, pairs);
  else
    hipLaunchKernelGGL((k_swap_copy<THREADS, UNROLL>), dim3(grid), dim3(THREADS), 0, s, dst_layer_base, src_layer_base,
                       block_bytes, pairs);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

// shape: threads per workgroup x 16-byte loads in flight per lane, as threads * 100 + loads; 0 = chosen here
// from the size of the transfer.  What was measured beside the decode kernel of the 7B-shaped workload
// (265 us per layer, every compute unit streaming from HBM):
//  - While the decode kernel runs, a gather wave's requests queue behind the decode waves' in the compute
//    unit's memory pipeline and the link rate is set by the number of gather waves, whatever each has in
//    flight: 64 waves move about 28 GB/s, 128 about 45 GB/s; the decode kernel slows by 2-3 %.
//  - A gather that outlasts the layer runs alone part of the time and then reaches 40-55 GB/s with few waves,
//    but at full speed it costs the decode kernel next to it more: workgroups of 256 threads, 8 / 16 / 64 of
//    them: +4-5 % / +15 % / +110 %; one-wave workgroups with sixteen loads in flight, which fit beside the
//    decode kernel's resident workgroups instead of displacing one, 12 / 16 of them: +1-2 % / +2-3 % at
//    39 / 41 GB/s.
// So a transfer small enough to hide behind a layer is moved by n_wgs workgroups of 256 threads (it must finish
// before the layer does), and a larger one, for which the layer will wait in any case, by n_wgs one-wave
// workgroups (it must not slow the layers it runs beside).
constexpr size_t kGatherSmallBytes = (size_t)12 << 20;

int launch_swap_copy(char* dst_layer_base, const char* src_layer_base, size_t block_bytes, const SwapPairs& pairs,
                     int n_wgs, hipStream_t s, int shape, size_t transfer_bytes, hipEvent_t done) {
  if (pairs.n <= 0) return PIE_OK;
  if (block_bytes % 16 || n_wgs < 1) return PIE_EINVAL;
  if (shape == 0) shape = (transfer_bytes ? transfer_bytes : block_bytes * pairs.n) <= kGatherSmallBytes ? 25604 : 6416;
  switch (shape) {
    case 6404: return launch_swap_copy_as<64, 4>(dst_layer_base, src_layer_base, block_bytes, pairs, n_wgs, s, done);
    case 6416: return launch_swap_copy_as<64, 16>(dst_layer_base, src_layer_base, block_bytes, pairs, n_wgs, s, done);
    case 25602: return launch_swap_copy_as<256, 2>(dst_layer_base, src_layer_base, block_bytes, pairs, n_wgs, s, done);
    case 25604: return launch_swap_copy_as<256, 4>(dst_layer_base, src_layer_base, block_bytes, pairs, n_wgs, s, done);
    case 102416: return launch_swap_copy_as<1024, 16>(dst_layer_base, src_layer_base, block_bytes, pairs, n_wgs, s, done);
    default: return PIE_EINVAL;
  }
}

// ---------------------------------------------------------------------------------------------------
// KV append: one workgroup per sequence copies the new token's key and value rows into its tail block
// ---------------------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_kv_append(const AppendArgs a) { append_rows(a, blockIdx.x, blockIdx.y); }

// Appends for n_layers consecutive layers starting at `layer` in one launch.  With n_layers > 1 only modes
// that leave staged copies alone make sense (staging regions hold one layer each).
int append_args(const pie_pool* p, int32_t layer, int32_t n_layers, const void* d_k, const void* d_v, const int32_t* d_table,
                int32_t max_blocks, const int32_t* d_ctx, int32_t batch, int32_t mode, const LayerView* view, AppendArgs* out) {
  if (((uintptr_t)d_k | (uintptr_t)d_v) % 16) return PIE_EINVAL;
  if (n_layers < 1 || (n_layers > 1 && (mode == kAppendPresent || mode == kAppendStaged))) return PIE_EINVAL;
  AppendArgs& a = *out;
  a.kv_layer = p->d_kv + (size_t)layer * p->d_layer_stride;
  a.map = p->d_map[layer & 1];
  a.err = p->d_err;
  a.k_new = (const char*)d_k;
  a.v_new = (const char*)d_v;
  a.table = d_table;
  a.ctx = d_ctx;
  a.block_bytes = p->block_bytes;
  a.kv_layer_stride = p->d_layer_stride;
  a.new_layer_stride = (size_t)batch * p->cfg.n_kv_heads * p->cfg.head_dim * p->elem_bytes;
  a.map_stride = 0;
  a.max_blocks = max_blocks;
  a.n_handles = p->n_handles;
  a.n_gpu_blocks = p->cfg.n_gpu_blocks;
  a.n_slots = p->cfg.n_gpu_blocks + 2 * p->cfg.n_stage_blocks;
  a.n_kv_heads = p->cfg.n_kv_heads;
  a.head_dim = p->cfg.head_dim;
  a.block_tokens = p->cfg.block_tokens;
  a.elem_bytes = p->elem_bytes;
  a.mode = mode;
  if (view) {                                    // the layer's blocks live elsewhere: all of them "GPU-homed" there
    a.kv_layer = view->kv_base;
    a.kv_layer_stride = 0;
    a.map = view->map;
    a.map_stride = a.n_handles = view->n_handles;
    a.n_gpu_blocks = a.n_slots = view->n_slots;
  }
  return PIE_OK;
}

int launch_kv_append(const pie_pool* p, int32_t layer, int32_t n_layers, const void* d_k, const void* d_v,
                     const int32_t* d_table, int32_t max_blocks, const int32_t* d_ctx, int32_t batch,
                     int32_t mode, hipStream_t s, const LayerView* view) {
  if (view && n_layers != 1) return PIE_EINVAL;
  AppendArgs a;
  const int rc = append_args(p, layer, n_layers, d_k, d_v, d_table, max_blocks, d_ctx, batch, mode, view, &a);
  if (rc) return rc;
  hipLaunchKernelGGL(k_kv_append, dim3(batch, n_layers), dim3(256), 0, s, a);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

// ---------------------------------------------------------------------------------------------------
// paged-attention decode
//
// Work is cut into items: `part_tokens` consecutive tokens of one sequence.  A small planning kernel lists
// the non-empty items, full ones first and the sequences' shorter last pieces after them in descending
// size, and a resolve kernel turns the block table (handles) into device slots once per step.
//
// 16-bit caches (fp16 / bf16): k_attn_decode_mfma.  The kernel is persistent: about as many workgroups as
// the GPU can hold resident, each taking (item, kv head) units from an atomic ticket counter until none are
// left.  That evens out the 8 XCDs (which do not stream at the same rate), leaves only small units for the
// end of the launch, and pays the launch ramp once.  A workgroup of kWaves wavefronts handles one unit and
// all G <= 16 query heads that share the kv head; wave w takes blocks w, w + kWaves, ... of the item.
// Per block a wave issues head_dim/32 K loads and head_dim/32 V loads of 16 bytes per lane, each covering
// 1 KiB contiguous, non-temporal (every KV byte is read once).  The loaded
// vectors are matrix-core operands as they are:
//   S[token][head]  = sum_c K[token][c] Q[head][c]      head_dim/32 x  v_mfma_f32_16x16x32   (A = K, B = Q)
//   O[dim][head]   += sum_t V[t][dim] P[t][head]        head_dim/16 x  v_mfma_f32_16x16x16   (A = V, B = P)
// The 16 columns are the query heads of the group (columns >= G carry zeros); for G = 1 the products are
// matrix-vector and most of the matrix core idles, which costs nothing: the kernel is bound by HBM, and what
// the matrix core buys is that no vector-ALU work is spent on unpacking and multiplying the 16-bit elements.
// The accumulator layout of S (lane = 16 (token / 4) + head, register = token % 4) is the B-operand layout
// of the 16x16x16 form, so P goes from the softmax into the second product without leaving its lane.
// The softmax is online, in the log2 domain, with one running maximum per head shared by the wave (two
// cross-lane swaps per block); the accumulators are rescaled only when some maximum moved.  P is rounded
// to the cache's 16-bit type for the second product; for bf16 the rounding residue goes through a second
// MFMA so that P carries 16 significant bits.  At the end the kWaves partial states merge through LDS and
// are written out (single partition) or stored as (m, l, acc) for the reduction kernel.
//
// fp32 caches: k_attn_decode_f32, a plain vector-ALU kernel over the same items, one workgroup per
// (item, query head).  It exists for the fp32 parity configuration, which is latency-bound.
// ---------------------------------------------------------------------------------------------------

constexpr int kMinPartTokens = 256;
constexpr int kMaxPlanBatch = 4096;   // sequences the planning kernel keeps in LDS

// ---- planning: the list of work items ------------------------------------------------------------------
// items[i] = {sequence | part << 16, context length of the sequence}: item `part` covers the tokens
// [part * part_tokens, min((part + 1) * part_tokens, context)).  hdr[0] = number of items.  Full items
// (part_tokens tokens) come first, then one shorter item per sequence whose length is not a multiple of
// part_tokens (or is <= 0, so that its output is still written), longest first.  With minus = 1 "context" is the
// context without its last token.  hdr[1] = part_tokens: the given one, or with min_units > 0 the one chosen
// here; every kernel that follows reads it from there.  Also zeroes the ticket
// counters of all layers and, if a clock table is given, resets its rows and notes the time in the row
// after the last.
//
// One workgroup, so its time is latency: nothing in it may walk the batch one element at a time.  The offsets of the
// full items come from a scan of the workgroup, and the rank of a short item from a count over unique keys (size,
// then sequence) that reads four of them per LDS access; with a serial scan and a scalar rank loop the launch took
// 5.1 / 13.3 / 1 689 us at 64 / 256 / 4 096 sequences, now 3.4 / 5.5 / 280.
constexpr int kPlanThreads = 1024;       // at most; 256 do for up to 256 sequences (launch_attn_plan)
static_assert(kMaxPlanBatch == 4096, "the rank keys hold a sequence index in 12 bits");

__global__ __launch_bounds__(kPlanThreads) void k_attn_plan(const int32_t* __restrict__ ctx, int32_t batch,
                                                            int32_t part_tokens, int32_t min_units, int32_t n_kv_heads,
                                                            int32_t max_blocks, int32_t minus,
                                                            uint2* __restrict__ items, int32_t* __restrict__ hdr,
                                                            uint32_t* __restrict__ counters, int32_t n_counters,
                                                            uint32_t* __restrict__ err,
                                                            unsigned long long* __restrict__ clock) {
  __shared__ int32_t s_ctx[kMaxPlanBatch];   // context length, clamped to [0, what the table can name]
  __shared__ __align__(16) int32_t s_key[kMaxPlanBatch];   // short items: size << 12 | (4095 - sequence), else -1
  __shared__ int32_t s_full[kPlanThreads / 64], s_short[kPlanThreads / 64];   // per wave, of one round of the scan
  __shared__ int32_t s_units[kAutoParts];    // items per candidate item size
  const int32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nt = blockDim.x;
  if (tid < kAutoParts) s_units[tid] = 0;
  __syncthreads();
  int32_t my_units[kAutoParts] = {};
  for (int32_t b = tid; b < batch; b += nt) {
    const int32_t raw = ctx[b];
    const int32_t full = clamp_ctx(raw, max_blocks);
    if (raw > full) atomicOr(err, PIE_DEVERR_BAD_HANDLE);   // the table cannot name that many blocks
    const int32_t c = full > 0 ? full - minus : full;       // minus = 1: the last token is not read from the cache
    s_ctx[b] = c > 0 ? c : 0;
    if (min_units > 0)
#pragma unroll
      for (int i = 0; i < kAutoParts; ++i) my_units[i] += c > 0 ? (c + auto_part(i) - 1) / auto_part(i) : 1;
  }
  // The item size, when it is not given: the largest candidate that still leaves more than min_units units
  // (items x kv heads) for the decode kernel's workgroups to share, the smallest candidate if none does.
  if (min_units > 0) {
#pragma unroll
    for (int i = 0; i < kAutoParts; ++i) {
      const int32_t n = wave_sum(my_units[i]);
      if (lane == 0 && n) atomicAdd(&s_units[i], n);
    }
  }
  for (int32_t i = tid; i < n_counters; i += nt) counters[i] = 0;
  if (clock) {                                   // one row per launch: min / max slots to their neutral values
    for (int32_t i = tid; i < n_counters; i += nt) {
      clock[(size_t)i * kClockRow + kClockKernelStart] = ~0ull;
      clock[(size_t)i * kClockRow + kClockKernelEnd] = 0ull;
      clock[(size_t)i * kClockRow + kClockLayerEnd] = 0ull;
      clock[(size_t)i * kClockRow + kClockGrid] = 0ull;
    }
    if (tid == 0) clock[(size_t)n_counters * kClockRow] = wall_clock64();   // the step begins
  }
  __syncthreads();
  if (min_units > 0) {
    part_tokens = auto_part(0);
    for (int i = 1; i < kAutoParts; ++i)
      if ((long long)s_units[i] * n_kv_heads > min_units) part_tokens = auto_part(i);
  }
  // full items in sequence order, a round of one per thread at a time
  int32_t n_full = 0, n_short = 0;
  for (int32_t b0 = 0; b0 < batch; b0 += nt) {
    const int32_t b = b0 + tid;
    const bool live = b < batch;
    const int32_t c = live ? s_ctx[b] : 0;
    const int32_t nf = c / part_tokens, rem = c - nf * part_tokens;
    const bool has_short = live && (rem > 0 || c <= 0);
    const int32_t incl = wave_scan(nf);
    const unsigned long long shorts = __builtin_amdgcn_ballot_w64(has_short);
    if (lane == 63) {
      s_full[wave] = incl;
      s_short[wave] = __popcll(shorts);
    }
    __syncthreads();
    int32_t off = n_full + incl - nf;
    for (int w = 0; w < nt / 64; ++w) {
      if (w < wave) off += s_full[w];
      n_full += s_full[w];
      n_short += s_short[w];
    }
    if (live) {
      for (int32_t p = 0; p < nf; ++p) items[off + p] = make_uint2((uint32_t)b | ((uint32_t)p << 16), (uint32_t)c);
      s_key[b] = has_short ? (rem << 12) | (kMaxPlanBatch - 1 - b) : -1;
    }
    __syncthreads();                             // the round's sums are read before the next round's are written
  }
  if (tid < 4 && ((batch + 3) & ~3) - 4 + tid >= batch) s_key[((batch + 3) & ~3) - 4 + tid] = -1;   // to a whole vector
  if (tid == 0) {
    hdr[0] = n_full + n_short;
    hdr[1] = part_tokens;
  }
  __syncthreads();
  for (int32_t b = tid; b < batch; b += nt) {
    const int32_t key = s_key[b];
    if (key < 0) continue;
    int32_t rank = 0;                            // longest first, ties by sequence index
    for (int32_t o = 0; o < batch; o += 4) {
      const int4 k = *reinterpret_cast<const int4*>(&s_key[o]);
      rank += (k.x > key ? 1 : 0) + (k.y > key ? 1 : 0) + (k.z > key ? 1 : 0) + (k.w > key ? 1 : 0);
    }
    const int32_t c = s_ctx[b];
    items[n_full + rank] = make_uint2((uint32_t)b | ((uint32_t)(c / part_tokens) << 16), (uint32_t)c);
  }
}

// ---- resolve: the device slots of every item's blocks, for one or both staging regions ---------------------
// slots[r][i * bpi + jj] = slot of block (part * bpi + jj) of item i's sequence, -1 beyond its context.
struct ResolveArgs {
  const int32_t* table;      // [B][max_blocks] handles
  const uint2* items;
  const int32_t* hdr;
  const int32_t* map[2];
  int32_t* slots[2];         // NULL to skip a region
  uint32_t* err;
  int32_t max_blocks, n_handles, n_gpu_blocks, n_slots;
  int32_t stage_valid[2];
};

__global__ __launch_bounds__(64) void k_attn_resolve(const ResolveArgs a) {
  const int32_t i = blockIdx.x;
  if (i >= a.hdr[0]) return;
  const uint2 rec = a.items[i];
  const int32_t b = (int32_t)(rec.x & 0xffffu), part = (int32_t)(rec.x >> 16);
  const int32_t tok1 = (int32_t)rec.y;
  const int32_t jb1 = tok1 > 0 ? (tok1 + kBlockTokens - 1) / kBlockTokens : 0;   // <= max_blocks
  const int32_t bpi = a.hdr[1] / kBlockTokens;   // blocks per item, as planned
  for (int32_t jj = threadIdx.x; jj < bpi; jj += blockDim.x) {
    const int32_t j = part * bpi + jj;
    const bool live = j < jb1;
    const int32_t h = live ? a.table[(size_t)b * a.max_blocks + j] : -1;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (!a.slots[r]) continue;
      a.slots[r][(size_t)i * bpi + jj] =
          live ? resolve_slot(h, a.map[r], a.n_handles, a.n_gpu_blocks, a.n_slots, a.stage_valid[r] != 0, a.err) : -1;
    }
  }
}

struct AttnArgs {
  const char* kv_layer;
  const int32_t* slots;      // per item: device slots of its blocks, for this layer's staging region
  const uint2* items;
  const int32_t* hdr;
  uint32_t* counter;         // ticket counter of this launch (zeroed by the planning kernel)
  const char* q;             // [B][Hq][d]
  char* out;                 // [B][Hq][d]
  float* ws;                 // [B][Hq][n_parts][2 + d]
  const int32_t* ctx;
  size_t block_bytes;
  float scale_log2e;
  int32_t max_blocks, n_kv_heads, group;
  int32_t n_parts;           // partitions the workspace has room for per (sequence, head); the item size is hdr[1]
  int32_t max_items;         // entries the item list has room for (batch x n_parts)
  unsigned long long* clock;    // this launch's row of the clock table, or NULL
  unsigned long long* clock_wg; // with it: a (first, last moment) pair per workgroup, or NULL (atomics on the row)
  // The newest token's key / value rows [B][Hkv][d], or NULL.  With them the items cover the context without
  // its last token (the planning kernel was told so), every partition's state goes to the workspace, and the
  // reduction kernel adds the last token from these rows: the attention then does not depend on the append
  // that writes the rows into the cache.
  const char* new_k;
  const char* new_v;
  // The layers of the launch, `kv_layer`, q, out, the new rows and the workspace being the first one's: bytes (of the
  // workspace: floats) from one to the next.  They share the items and the slots.
  // (All layers of a step at once, where nothing happens between them, have one ramp, one tail and one reduction: 32 layers
  // of 64 sequences of 1 024 to 2 048 tokens, 32 heads, 8 039 us in a launch and a reduction each, 7 924 so.)
  int32_t n_layers;
  size_t kv_stride, q_stride, new_stride, ws_stride;
};

// LDS floats the MFMA kernel needs for `group` query heads per kv head
template <int HD>
constexpr size_t mfma_lds_floats(int group) {
  return (size_t)kWaves * 2 * kMaxGroup + (size_t)kWaves * group * (HD + 4);
}

#ifndef PIE_MFMA_WAVES_PER_EU
#define PIE_MFMA_WAVES_PER_EU 2
#endif

// VALU: the same kernel with both products on the vector ALU instead (group == 1 only, where they are
// matrix-vector products).  Lane (quad, i) then holds, of a K load, eight dims of token i - its share of that
// token's score, summed over the four quads - and of a V load four tokens of two dims, which it multiplies with
// those tokens' weights fetched from the lanes that own them; the output dims are summed over the quads when the
// unit ends.
template <typename E, int HD, bool SPLIT, bool VALU, bool TWO>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(PIE_MFMA_WAVES_PER_EU, 8)))
void k_attn_decode_mfma(const AttnArgs a) {
  using MM = Mfma<E>;
  constexpr int NKC = HD / 32;                    // 1 KiB loads per K tile and per V tile; QK MFMAs per block
  constexpr int NO = HD / 16;                     // output accumulators (16 dims x 16 heads each)
  constexpr int TILE_BYTES = kBlockTokens * HD * 2;
  constexpr int ROW = HD + 4;                     // padded LDS row of one head's accumulator
  static_assert(HD % 32 == 0, "unsupported head_dim");

  extern __shared__ __align__(16) float s_dyn[];
  __shared__ uint32_t s_ticket;
  float* s_m = s_dyn;                             // [kWaves][16]
  float* s_l = s_dyn + kWaves * kMaxGroup;        // [kWaves][16]
  float* s_acc = s_dyn + 2 * kWaves * kMaxGroup;  // [kWaves][G][ROW]

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, quad = lane >> 4;    // MFMA column (query head of the group) and 4-row group
  const int32_t G = a.group;
  const int32_t n_q_heads = a.n_kv_heads * G;
  const uint32_t n_kv = (uint32_t)a.n_kv_heads;
  const uint32_t per_item = n_kv * (uint32_t)a.n_layers;          // units: its kv heads, layer by layer
  const uint32_t max_units = (uint32_t)a.max_items * per_item;    // what the item and slot lists have room for
  const size_t v_off = a.block_bytes / 2;
  const int32_t part_tokens = a.hdr[1];                           // the item size the planning kernel noted
  const int32_t bpi = part_tokens / kBlockTokens;                 // blocks per item, <= 64 * kWaves
  const int32_t my_n = (bpi + kWaves - 1 - wave) / kWaves;        // blocks of an item this wave may own

  // Units are handed out by tickets.  A workgroup's first two are static (its index, and its index plus the
  // grid size); the rest come from an atomic counter.  The ticket for the unit after next is requested
  // behind a unit's stream, so the next unit is always known one unit ahead: its record and slot list are
  // fetched at the start of the current unit, its first block is requested as soon as the current unit's
  // stream ends, and the merge of the current unit runs behind those loads.
  uint32_t unit = blockIdx.x;
  uint32_t next = gridDim.x + blockIdx.x;
  if (a.clock && threadIdx.x == 0) {
    const unsigned long long t = wall_clock64();
    if (a.clock_wg) {
      a.clock_wg[2 * blockIdx.x] = t;
      if (blockIdx.x == 0) a.clock[kClockGrid] = gridDim.x;
    } else {
      atomicMin(&a.clock[kClockKernelStart], t);
    }
  }

  // record and this wave's slot list of unit u; entries beyond the planned items are never used
  auto fetch_meta = [&](uint32_t u, uint2& r, int32_t& sl) {
    r = make_uint2(0, 0);
    sl = -1;
    if (u < max_units) {
      const uint32_t item = u / per_item;
      r = a.items[item];
      if (lane < my_n) sl = a.slots[(size_t)item * bpi + wave + kWaves * lane];
    }
  };
  // this lane's part of the B operand of the first product: head `col` of the group, dims 32 kc + 8 quad ..
  auto load_q = [&](uint4 (&qr)[NKC], int32_t b, int32_t layer, int32_t g) {
    const char* q = a.q + layer * a.q_stride;
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      qr[kc] = make_uint4(0, 0, 0, 0);
      const int head = VALU ? 0 : col;            // on the vector ALU every lane works for the one head
      if (head < G)
        qr[kc] = *reinterpret_cast<const uint4*>(q + (((size_t)b * n_q_heads + g * G + head) * HD + 32 * kc + 8 * quad) * 2);
    }
  };
  // One block of a wave is in flight, all of it requested before any of it is waited for: the other waves keep the memory
  // busy, and more in flight is not faster.  us a call with two and with one: 260 sequences of 1 000 to 3 000 tokens, 32 heads
  // over 8, 337 and 330; 300 of 300 to 2 000, 12 heads of 64, 184 to 192 and 181 to 183; 12 layers of 64 of 1 024 to 2 048, 32
  // heads of 64, 1 525 and 1 495.  TWO: two, on the vector ALU, where a block takes longer to use (the last of these as a call
  // 137.3 and 139.1), under tables that are very wide (launch_mfma), and for items of a size that the caller has set, which may
  // be shorter than the rule's: of 512 tokens, 64 as above, 32 heads of 64, 147.5 and 149.7, one of 32 749, 64 over 8, 39.2 and
  // 39.8.  (260 of 20 to 300, 32 over 8, are left: 48.8 and 49.4.)
  uint4 kA[NKC], vA[NKC], kB[NKC], vB[NKC];
  auto load_to = [&](uint4 (&kr)[NKC], uint4 (&vr)[NKC], int32_t slots, int32_t it, int32_t layer, int32_t g) {
    int32_t slot = __builtin_amdgcn_readlane(slots, it);
    slot = slot < 0 ? 0 : slot;                                    // flagged blocks are masked when consumed
    const char* kp = a.kv_layer + layer * a.kv_stride + (size_t)slot * a.block_bytes + (size_t)g * TILE_BYTES + (size_t)lane * 16;
#pragma unroll
    for (int i = 0; i < NKC; ++i) kr[i] = nt_load16(kp + (size_t)i * 1024);
#pragma unroll
    for (int i = 0; i < NKC; ++i) vr[i] = nt_load16(kp + v_off + (size_t)i * 1024);
    if (!TWO) __builtin_amdgcn_sched_barrier(0);
  };
  auto load_tile = [&](int32_t slots, int32_t it, int32_t layer, int32_t g) { load_to(kA, vA, slots, it, layer, g); };
  // blocks of unit (r, u) this wave handles: j = jb0 + wave + kWaves * it, it < n_it (<= 0: nothing)
  auto wave_blocks = [&](const uint2& r) {
    const int32_t ctx_u = (int32_t)r.y, tok0_u = (int32_t)(r.x >> 16) * part_tokens;
    const int32_t tok1_u = min(ctx_u, tok0_u + part_tokens);
    const int32_t jb1_u = tok1_u > 0 ? (tok1_u + kBlockTokens - 1) / kBlockTokens : 0;
    return (jb1_u - tok0_u / kBlockTokens - wave + kWaves - 1) / kWaves;
  };

  uint2 rec, rec_next;
  int32_t my_slot, my_slot_next;
  uint4 qreg[NKC];
  fetch_meta(unit, rec, my_slot);
  fetch_meta(next, rec_next, my_slot_next);
  const uint32_t n_units = (uint32_t)a.hdr[0] * per_item;          // <= max_units
  auto layer_of = [&](uint32_t u) { return (int32_t)(u % per_item / n_kv); };
  if (unit < n_units) {
    const int32_t layer = layer_of(unit), g = (int32_t)(unit % n_kv);
    load_q(qreg, (int32_t)(rec.x & 0xffffu), layer, g);
    if (wave_blocks(rec) > 0) load_tile(my_slot, 0, layer, g);
  }

  while (unit < n_units) {                       // every workgroup ends on a ticket past the last unit
    const int32_t layer = layer_of(unit), g = (int32_t)(unit % n_kv);
    const int32_t b = (int32_t)(rec.x & 0xffffu), part = (int32_t)(rec.x >> 16);
    const int32_t ctx_b = (int32_t)rec.y;                          // clamped context length of the sequence
    const int32_t tok0 = part * part_tokens;
    const int32_t tok1 = min(ctx_b, tok0 + part_tokens);         // <= tok0 only for an empty sequence
    const int32_t np_b = ctx_b > 0 ? (ctx_b + part_tokens - 1) / part_tokens : 1;   // partitions of the sequence
    const int32_t hq0 = g * G;
    const int32_t jb0 = tok0 / kBlockTokens;
    const int32_t n_it = wave_blocks(rec);                         // <= my_n <= 64

    float m = kNegBig, l = 0.f;                   // running max of head `col`; this lane's share of the sum
    f32x4 o[NO];
#pragma unroll
    for (int n = 0; n < NO; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float ov[NKC][2];                             // VALU: dims 32 i + (lane & 15) and 16 further, this quad's tokens
#pragma unroll
    for (int i = 0; i < NKC; ++i) ov[i][0] = ov[i][1] = 0.f;

    // VALU form of one block: lane (quad, i = lane & 15).  K load kc holds token i, dims 32 kc + 8 quad ..;
    // V load holds tokens 4 quad .. 4 quad + 3 of dims 32 ld + i (x, y) and 32 ld + 16 + i (z, w).
    auto consume_valu = [&](uint4 (&kr)[NKC], uint4 (&vr)[NKC], int32_t it) {
      const int32_t t_first = (jb0 + wave + kWaves * it) * kBlockTokens;
      const bool present = __builtin_amdgcn_readlane(my_slot, it) >= 0;
      const int32_t limit = present ? tok1 : 0;
      float d = 0.f;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        d = Dot2<E>::fma2(kr[kc].x, qreg[kc].x, d);
        d = Dot2<E>::fma2(kr[kc].y, qreg[kc].y, d);
        d = Dot2<E>::fma2(kr[kc].z, qreg[kc].z, d);
        d = Dot2<E>::fma2(kr[kc].w, qreg[kc].w, d);
      }
      float sc = quad16_sum(d) * a.scale_log2e;   // score of token t_first + i, on all four lanes of the token
      if (t_first + col >= limit) sc = -INFINITY;
      if (t_first + kBlockTokens > limit) {       // garbage rows must not reach the sum
        const int32_t t_lane = t_first + 4 * quad;
        uint32_t keep_lo = 0, keep_hi = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t bits = t_lane + r < limit ? (0xffffu << (16 * (r & 1))) : 0u;
          if (r < 2) keep_lo |= bits; else keep_hi |= bits;
        }
#pragma unroll
        for (int i = 0; i < NKC; ++i) {
          vr[i].x &= keep_lo; vr[i].y &= keep_hi; vr[i].z &= keep_lo; vr[i].w &= keep_hi;
        }
      }
      const float m_new = fmaxf(m, row16_max(sc));           // the same on every lane of the wave
      if (m_new > m) {
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
        l *= corr;
#pragma unroll
        for (int i = 0; i < NKC; ++i) { ov[i][0] *= corr; ov[i][1] *= corr; }
        m = m_new;
      }
      const float p = __builtin_amdgcn_exp2f(sc - m);
      l += p;                                     // token i only; summed over the sixteen tokens when the unit ends
      f32x4 pq;                                   // the weights of this quad's four tokens
#pragma unroll
      for (int r = 0; r < 4; ++r) pq[r] = __shfl(p, 4 * quad + r, 64);
      const uint2 p_hi = MM::round(pq);
      uint2 p_lo = make_uint2(0, 0);
      if (SPLIT) {
        const f32x4 back = MM::widen(p_hi);
        f32x4 rest;
#pragma unroll
        for (int r = 0; r < 4; ++r) rest[r] = pq[r] - back[r];
        p_lo = MM::round(rest);
      }
#pragma unroll
      for (int i = 0; i < NKC; ++i) {
        ov[i][0] = Dot2<E>::fma2(vr[i].x, p_hi.x, ov[i][0]);
        ov[i][0] = Dot2<E>::fma2(vr[i].y, p_hi.y, ov[i][0]);
        ov[i][1] = Dot2<E>::fma2(vr[i].z, p_hi.x, ov[i][1]);
        ov[i][1] = Dot2<E>::fma2(vr[i].w, p_hi.y, ov[i][1]);
        if (SPLIT) {
          ov[i][0] = Dot2<E>::fma2(vr[i].x, p_lo.x, ov[i][0]);
          ov[i][0] = Dot2<E>::fma2(vr[i].y, p_lo.y, ov[i][0]);
          ov[i][1] = Dot2<E>::fma2(vr[i].z, p_lo.x, ov[i][1]);
          ov[i][1] = Dot2<E>::fma2(vr[i].w, p_lo.y, ov[i][1]);
        }
      }
    };

    auto consume = [&](uint4 (&kr)[NKC], uint4 (&vr)[NKC], int32_t it) {
      const bool present = __builtin_amdgcn_readlane(my_slot, it) >= 0;   // a missing block contributes nothing
      mfma_block<E, HD, SPLIT>(kr, vr, qreg, (jb0 + wave + kWaves * it) * kBlockTokens, present ? tok1 : 0, quad,
                               a.scale_log2e, m, l, o);
    };

    // The ticket after next is requested half way through the stream: late enough that the counter is not
    // hit by every workgroup at once, early enough that the answer is there when the unit ends.  Block 0 of
    // the unit is already on its way.
    uint32_t after_next = 0;
    const int32_t it_ticket = TWO ? n_it / 2 & ~1 : n_it / 2;
    if constexpr (TWO) {
      for (int32_t it = 0; it < n_it; it += 2) {
        if (it == it_ticket && threadIdx.x == 0) after_next = 2 * gridDim.x + atomicAdd(a.counter, 1u);
        if (it + 1 < n_it) load_to(kB, vB, my_slot, it + 1, layer, g);
        if constexpr (VALU) consume_valu(kA, vA, it); else consume(kA, vA, it);
        if (it + 1 < n_it) {
          if (it + 2 < n_it) load_tile(my_slot, it + 2, layer, g);
          if constexpr (VALU) consume_valu(kB, vB, it + 1); else consume(kB, vB, it + 1);
        }
      }
    } else {
      for (int32_t it = 0; it < n_it; ++it) {
        if (it == it_ticket && threadIdx.x == 0) after_next = 2 * gridDim.x + atomicAdd(a.counter, 1u);
        consume(kA, vA, it);
        if (it + 1 < n_it) load_tile(my_slot, it + 1, layer, g);
      }
    }
    if (n_it <= 0 && threadIdx.x == 0) after_next = 2 * gridDim.x + atomicAdd(a.counter, 1u);

    // behind the stream: the next unit's first block and query rows arrive while this unit's result is merged
    if (next < n_units) {
      const int32_t layer_next = layer_of(next), g_next = (int32_t)(next % n_kv);
      if (wave_blocks(rec_next) > 0) load_tile(my_slot_next, 0, layer_next, g_next);
      load_q(qreg, (int32_t)(rec_next.x & 0xffffu), layer_next, g_next);
    }

    // merge the kWaves partial states: lane (quad, col) holds O[16 n + 4 quad + r][head col]
    if constexpr (VALU) {
      l = row16_sum(l);                           // over the sixteen tokens of a block position
#pragma unroll
      for (int i = 0; i < NKC; ++i) {             // over the four quads' tokens
        ov[i][0] = quad16_sum(ov[i][0]);
        ov[i][1] = quad16_sum(ov[i][1]);
      }
      if (lane == 0) {
        s_m[wave * kMaxGroup] = m;
        s_l[wave * kMaxGroup] = l;
      }
      if (quad == 0) {
        float* row = s_acc + (size_t)wave * G * ROW;
#pragma unroll
        for (int i = 0; i < NKC; ++i) {
          row[32 * i + col] = ov[i][0];
          row[32 * i + 16 + col] = ov[i][1];
        }
      }
    } else {
    l = quad16_sum(l);
    if (col < G) {
      if (quad == 0) {
        s_m[wave * kMaxGroup + col] = m;
        s_l[wave * kMaxGroup + col] = l;
      }
      float* row = s_acc + ((size_t)wave * G + col) * ROW + 4 * quad;
#pragma unroll
      for (int n = 0; n < NO; ++n) *reinterpret_cast<f32x4*>(row + 16 * n) = o[n];
    }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < G * HD; idx += kWaves * 64) {
      const int h = idx / HD, dim = idx % HD;
      float M = s_m[h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w * kMaxGroup + h]);
      float L = 0.f, A = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float wt = __builtin_amdgcn_exp2f(s_m[w * kMaxGroup + h] - M);
        L = fmaf(wt, s_l[w * kMaxGroup + h], L);
        A = fmaf(wt, s_acc[((size_t)w * G + h) * ROW + dim], A);
      }
      const size_t orow = (size_t)b * n_q_heads + hq0 + h;
      if (np_b == 1 && !a.new_k) {               // the only partition of its sequence: this is the result
        store_elem<E>(a.out + layer * a.q_stride, orow * HD + dim, L > 0.f ? A / L : 0.f);
      } else {
        float* w = a.ws + layer * a.ws_stride + (orow * a.n_parts + part) * (HD + 2);
        if (dim == 0) {
          w[0] = M;
          w[1] = L;
        }
        w[2 + dim] = A;
      }
    }
    if (threadIdx.x == 0) s_ticket = after_next;
    __syncthreads();                             // merge buffers free again; the new ticket is visible
    unit = next;
    next = s_ticket;
    rec = rec_next;
    my_slot = my_slot_next;
    __syncthreads();                             // all have read the ticket before it is overwritten
    fetch_meta(next, rec_next, my_slot_next);    // consumed when this unit's stream ends
  }
  if (a.clock && threadIdx.x == 0) {
    const unsigned long long t = wall_clock64();
    if (a.clock_wg) a.clock_wg[2 * blockIdx.x + 1] = t;
    else atomicMax(&a.clock[kClockKernelEnd], t);
  }
}

// The same items, states and sums, read eight kv heads side by side (pie_attn_wide.h): a unit is an item for eight heads, of
// which a wave each takes the four shares that a workgroup's waves take above, and four more waves merge those and store the
// results, two heads each.  For launches of six layers and more (planned_wide): HBM-bound, the tiles read lie in 32 KB pieces and no
// merge stands between two units.  32 layers of 64 sequences of 1 024 to 2 048 tokens, 32 heads: 7 930 us in k_attn_decode_mfma,
// 7 690 here (49.4 GB, 6.6 TB/s without the rows).
struct PlannedItems {
  const AttnArgs& a;
  int32_t part_tokens, bpi, n_items;
  __device__ __forceinline__ void fetch(const WideUnit& u, int lane, WideMeta& x) const {
    const int32_t i = u.place >= 0 && u.place < n_items ? u.place : 0;
    x.rec = reinterpret_cast<const int32_t*>(a.items + i)[lane & 1];
#pragma unroll
    for (int s = 0; s < kWaves; ++s) x.slots[s] = a.slots[(size_t)i * bpi + min(s + kWaves * lane, bpi - 1)];
  }
  __device__ __forceinline__ void read(WideUnit& u, const WideMeta& x) const {
    const uint32_t of = (uint32_t)__builtin_amdgcn_readlane(x.rec, 0);
    const int32_t ctx = __builtin_amdgcn_readlane(x.rec, 1);       // clamped context length of the sequence
    u.b = u.place < n_items ? (int32_t)(of & 0xffffu) : -1;
    u.part = (int32_t)(of >> 16);
    u.tok0 = u.part * part_tokens;
    u.tok1 = min(ctx, u.tok0 + part_tokens);     // <= tok0 only for an empty sequence
    u.np = ctx > 0 ? (ctx + part_tokens - 1) / part_tokens : 1;
    u.first = u.ctx_raw = 0;
  }
  __device__ __forceinline__ void look_up(const WideUnit&, const WideMeta&, int32_t (&)[kWaves]) const {}
  __device__ __forceinline__ void found_out(const WideUnit&, WideMeta&, const int32_t (&)[kWaves]) const {}
};

template <typename E, int HD, bool SPLIT>
__global__ __launch_bounds__((kPlannedWideHeads + kFinishers) * 64) __attribute__((amdgpu_waves_per_eu(3, 8)))
void k_attn_decode_wide(const AttnArgs a) {
  constexpr int ROW = HD + 4, HW = kPlannedWideHeads;
  extern __shared__ __align__(16) float s_dyn[];
  __shared__ WideLds lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t n_items = a.hdr[0], part_tokens = a.hdr[1];
  if (wave < HW) {
    wide_read<Wave16<E, HD, SPLIT>, HW>({a.kv_layer, a.q, a.counter, a.block_bytes, a.kv_stride, a.q_stride, a.scale_log2e,
                                     a.n_kv_heads, a.group, a.n_layers, a.max_items},
                                    PlannedItems{a, part_tokens, part_tokens / kBlockTokens, n_items}, s_dyn, lds);
    return;
  }
  const int32_t G = a.group, n_q_heads = a.n_kv_heads * G;
  wide_finish(lds, [&](int half, int32_t x, int thread) {
    const int32_t b = __builtin_amdgcn_readlane(x, 0), g0 = __builtin_amdgcn_readlane(x, 1);
    const int32_t layer = __builtin_amdgcn_readlane(x, 2), np = __builtin_amdgcn_readlane(x, 3), part = __builtin_amdgcn_readlane(x, 5);
    for (int hw = wave - HW; hw < HW; hw += kFinishers) {
    const int32_t g = g0 + hw;
    const float* const s_m = s_dyn + (half * HW + hw) * wide_head_floats(HD, G);
    const float* const s_l = s_m + kWaves * kMaxGroup;
    const float* const s_acc = s_l + kWaves * kMaxGroup;
    for (int idx = 2 * thread; idx < G * HD; idx += 128) {
      const int h = idx / HD, dim = idx % HD;
      float M = s_m[h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w * kMaxGroup + h]);
      float L = 0.f;
      float2 A = make_float2(0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float wt = __builtin_amdgcn_exp2f(s_m[w * kMaxGroup + h] - M);
        const float2 y = *reinterpret_cast<const float2*>(&s_acc[((size_t)w * G + h) * ROW + dim]);
        L = fmaf(wt, s_l[w * kMaxGroup + h], L);
        A.x = fmaf(wt, y.x, A.x);
        A.y = fmaf(wt, y.y, A.y);
      }
      const size_t orow = (size_t)b * n_q_heads + g * G + h;
      if (np == 1 && !a.new_k) {                 // the only partition of its sequence: this is the result
        store_elem2<E>(a.out + layer * a.q_stride, orow * HD + dim, make_float2(L > 0.f ? A.x / L : 0.f, L > 0.f ? A.y / L : 0.f));
      } else {
        float* w = a.ws + layer * a.ws_stride + (orow * a.n_parts + part) * (HD + 2);
        if (dim == 0) *reinterpret_cast<float2*>(w) = make_float2(M, L);
        *reinterpret_cast<float2*>(w + 2 + dim) = A;
      }
    }
    }
  });
}

// Calibration: reads exactly the K and V tiles the decode kernel reads for the planned items, in the same
// order and with the same loads (units by ticket, wave w takes blocks w, w + kWaves, ..., two blocks in
// flight), and does nothing with them but fold them into a word nobody looks at.  Its rate is what this
// access pattern can stream at; the decode kernel is measured against it as well as against the HBM peak.
template <int NL>                                 // 1 KiB loads per tile
__global__ __launch_bounds__(kWaves * 64) void k_stream_probe(const AttnArgs a, size_t tile_bytes, uint32_t* sink) {
  __shared__ uint32_t s_ticket;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t n_kv = (uint32_t)a.n_kv_heads;
  const uint32_t n_units = (uint32_t)a.hdr[0] * n_kv;
  const size_t v_off = a.block_bytes / 2;
  const int32_t part_tokens = a.hdr[1];
  const int32_t bpi = part_tokens / kBlockTokens;
  const int32_t my_n = (bpi + kWaves - 1 - wave) / kWaves;
  u32x4 acc = {0, 0, 0, 0};
  uint32_t unit = blockIdx.x;
  while (unit < n_units) {                       // every workgroup ends on a ticket past the last unit
    const uint32_t item = unit / n_kv;
    const uint2 rec = a.items[item];
    int32_t my_slot = -1;
    if (lane < my_n) my_slot = a.slots[(size_t)item * bpi + wave + kWaves * lane];
    const int32_t ctx_u = (int32_t)rec.y, tok0 = (int32_t)(rec.x >> 16) * part_tokens;
    const int32_t tok1 = min(ctx_u, tok0 + part_tokens);
    const int32_t jb1 = tok1 > 0 ? (tok1 + kBlockTokens - 1) / kBlockTokens : 0;
    const int32_t n_it = (jb1 - tok0 / kBlockTokens - wave + kWaves - 1) / kWaves;
    const size_t head_off = (size_t)(unit % n_kv) * tile_bytes + (size_t)lane * 16;
    u32x4 ta[2 * NL], tb[2 * NL];
    auto load = [&](u32x4 (&t)[2 * NL], int32_t it) {
      int32_t slot = __shfl(my_slot, it, 64);
      slot = slot < 0 ? 0 : slot;
      const char* kp = a.kv_layer + (size_t)slot * a.block_bytes + head_off;
#pragma unroll
      for (int i = 0; i < NL; ++i) t[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp + (size_t)i * 1024));
#pragma unroll
      for (int i = 0; i < NL; ++i)
        t[NL + i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp + v_off + (size_t)i * 1024));
    };
    auto fold = [&](u32x4 (&t)[2 * NL]) {
#pragma unroll
      for (int i = 0; i < 2 * NL; ++i) acc ^= t[i];
    };
    if (n_it > 0) load(ta, 0);
    for (int32_t it = 0; it < n_it; it += 2) {
      if (it + 1 < n_it) load(tb, it + 1);
      fold(ta);
      if (it + 1 < n_it) {
        if (it + 2 < n_it) load(ta, it + 2);
        fold(tb);
      }
    }
    if (threadIdx.x == 0) s_ticket = gridDim.x + atomicAdd(a.counter, 1u);
    __syncthreads();
    unit = s_ticket;
    __syncthreads();
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) *sink = 1;   // keeps the loads alive
}

// fp32 caches.  One workgroup per (item, query head); wave w takes blocks w, w + kWaves, ...  Lane
// (quad, row) = (lane / 16, lane % 16): for K it holds token `row` of the block and the 4-dim vectors
// 4 i + quad; for V it holds dim 16 n + row and the tokens 4 quad .. 4 quad + 3.
template <int HD>
__global__ __launch_bounds__(kWaves * 64) void k_attn_decode_f32(const AttnArgs a) {
  constexpr int NLD = HD / 16;                    // 1 KiB loads per K tile and per V tile
  constexpr int TILE_BYTES = kBlockTokens * HD * 4;
  __shared__ float s_m[kWaves], s_l[kWaves];
  __shared__ float s_acc[kWaves][HD];

  const int32_t item = blockIdx.x;
  if (item >= a.hdr[0]) return;                   // uniform over the workgroup
  if (a.clock && threadIdx.x == 0) atomicMin(&a.clock[kClockKernelStart], wall_clock64());
  const int32_t hq = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, quad = lane >> 4;
  const int32_t G = a.group;
  const int32_t n_q_heads = a.n_kv_heads * G;
  const int32_t g = hq / G;
  const int32_t part_tokens = a.hdr[1];
  const int32_t bpi = part_tokens / kBlockTokens;
  const int32_t my_n = (bpi + kWaves - 1 - wave) / kWaves;
  const uint2 rec = a.items[item];
  const int32_t b = (int32_t)(rec.x & 0xffffu), part = (int32_t)(rec.x >> 16);
  const int32_t ctx_b = (int32_t)rec.y;           // clamped context length of the sequence
  const int32_t tok0 = part * part_tokens, tok1 = min(ctx_b, tok0 + part_tokens);
  const int32_t np_b = ctx_b > 0 ? (ctx_b + part_tokens - 1) / part_tokens : 1;
  const int32_t jb0 = tok0 / kBlockTokens;
  const int32_t jb1 = tok1 > 0 ? (tok1 + kBlockTokens - 1) / kBlockTokens : 0;
  const int32_t n_it = (jb1 - jb0 - wave + kWaves - 1) / kWaves;
  int32_t my_slot = -1;
  if (lane < my_n) my_slot = a.slots[(size_t)item * bpi + wave + kWaves * lane];

  float qf[NLD][4];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const float4 t = *reinterpret_cast<const float4*>(a.q + (((size_t)b * n_q_heads + hq) * HD + 4 * (4 * i + quad)) * 4);
    qf[i][0] = t.x * a.scale_log2e; qf[i][1] = t.y * a.scale_log2e;
    qf[i][2] = t.z * a.scale_log2e; qf[i][3] = t.w * a.scale_log2e;
  }
  float m = kNegBig, l = 0.f, acc[NLD];
#pragma unroll
  for (int n = 0; n < NLD; ++n) acc[n] = 0.f;
  const size_t v_off = a.block_bytes / 2;
  const size_t head_off = (size_t)g * TILE_BYTES + (size_t)lane * 16;

  for (int32_t it = 0; it < n_it; ++it) {
    int32_t slot = __shfl(my_slot, it, 64);
    const bool present = slot >= 0;
    slot = present ? slot : 0;
    const int32_t limit = present ? tok1 : 0;
    const int32_t t_first = (jb0 + wave + kWaves * it) * kBlockTokens;
    const char* kp = a.kv_layer + (size_t)slot * a.block_bytes + head_off;
    uint4 kr[NLD], vr[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) kr[i] = nt_load16(kp + (size_t)i * 1024);
#pragma unroll
    for (int i = 0; i < NLD; ++i) vr[i] = nt_load16(kp + v_off + (size_t)i * 1024);
    f32_block<HD>(kr, vr, qf, t_first, limit, lane, m, l, acc);
  }
  l = row16_sum(l);
#pragma unroll
  for (int n = 0; n < NLD; ++n) acc[n] = quad16_sum(acc[n]);
  if (lane == 0) {
    s_m[wave] = m;
    s_l[wave] = l;
  }
  if (quad == 0) {
#pragma unroll
    for (int n = 0; n < NLD; ++n) s_acc[wave][16 * n + row] = acc[n];
  }
  __syncthreads();
  for (int dim = threadIdx.x; dim < HD; dim += kWaves * 64) {
    float M = s_m[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w]);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wt = __builtin_amdgcn_exp2f(s_m[w] - M);
      L = fmaf(wt, s_l[w], L);
      A = fmaf(wt, s_acc[w][dim], A);
    }
    const size_t orow = (size_t)b * n_q_heads + hq;
    if (np_b == 1 && !a.new_k) {                 // the only partition of its sequence: this is the result
      store_elem<F32>(a.out, orow * HD + dim, L > 0.f ? A / L : 0.f);
    } else {
      float* w = a.ws + (orow * a.n_parts + part) * (HD + 2);
      if (dim == 0) {
        w[0] = M;
        w[1] = L;
      }
      w[2 + dim] = A;
    }
  }
  if (a.clock && threadIdx.x == 0) atomicMax(&a.clock[kClockKernelEnd], wall_clock64());
}

// Reduction over the partitions of one (sequence, query head): out = sum_s 2^(m_s - M) acc_s / sum_s 2^(m_s - M) l_s.
// With the newest token's rows given, that token is one more partition, (q . k_new, 1, v_new), computed here:
// s = q . k_new in the log2 domain like the partitions' maxima; the rows are requested first and used after the
// partitions have been merged.
//
// Two forms.  k_attn_reduce_heads, for up to eight partitions per sequence: head_dim / 2 threads per query head,
// two dims each, 512 / head_dim heads per workgroup, no LDS and no barrier (the launch is as short as its number
// of workgroups allows: the 8B workload has 8 192 rows).  k_attn_reduce, for long contexts: 256 threads per
// head, thread (sub, dim) = (tid / HD, tid % HD) merging the partitions sub, sub + 256/HD, ... online, four
// loads in flight, and the 256/HD partial merges meet in LDS.

struct ReduceRow {
  int32_t np;        // partitions to merge
  bool add_new;      // and the newest token
  bool skip;         // nothing to do: a lone partition wrote the result itself
};
__device__ __forceinline__ ReduceRow reduce_row(const AttnArgs& a, int32_t b) {
  const int32_t full = clamp_ctx(a.ctx[b], a.max_blocks);
  const bool with_new = a.new_k != nullptr;
  const int32_t ctx = with_new && full > 0 ? full - 1 : full;   // the tokens the partitions covered
  const int32_t part_tokens = a.hdr[1];
  int32_t np = ctx <= 0 ? 1 : (ctx + part_tokens - 1) / part_tokens;
  if (np > a.n_parts) np = a.n_parts;
  return {np, with_new && full > 0, np <= 1 && !with_new};
}

template <typename E, int HD>
__global__ __launch_bounds__(256) void k_attn_reduce_heads(const AttnArgs a, int32_t n_q_heads) {
  constexpr int TPH = HD / 2;                     // threads per head: a wave or half a wave
  constexpr int HPW = 256 / TPH;
  constexpr int UNR = 4;
  static_assert(TPH == 64 || TPH == 32, "a head's threads must be a wave or half a wave");
  const int32_t b = blockIdx.y;
  const int d0 = 2 * (threadIdx.x % TPH);
  const int32_t hq = (int32_t)blockIdx.x * HPW + threadIdx.x / TPH;
  const ReduceRow r = reduce_row(a, b);
  if (r.skip) return;
  const int32_t layer = blockIdx.z;
  const char* q = a.q + layer * a.q_stride;
  char* const out = a.out + layer * a.q_stride;
  const char* const new_k = a.new_k + layer * a.new_stride;       // (followed only if there are any)
  const char* const new_v = a.new_v + layer * a.new_stride;
  const float* const ws = a.ws + layer * a.ws_stride;
  if (hq < n_q_heads) {
    const size_t row = (size_t)b * n_q_heads + hq;
    float qk = 0.f;
    float2 v_new = make_float2(0.f, 0.f);
    if (r.add_new) {
      const size_t kv_row = ((size_t)b * a.n_kv_heads + hq / a.group) * HD;
      const float2 q2 = load_elem2<E>(q, row * HD + d0), k2 = load_elem2<E>(new_k, kv_row + d0);
      qk = fmaf(q2.x, k2.x, q2.y * k2.y);
      v_new = load_elem2<E>(new_v, kv_row + d0);
    }
    const float* w = ws + row * a.n_parts * (HD + 2);
    float M = kNegBig, L = 0.f;
    float2 A = make_float2(0.f, 0.f);
    for (int32_t s0 = 0; s0 < r.np; s0 += UNR) {
      float mi[UNR], li[UNR];
      float2 ai[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const bool live = s0 + u < r.np;
        const float* wp = w + (size_t)(live ? s0 + u : s0) * (HD + 2);
        mi[u] = live ? wp[0] : kNegBig;
        li[u] = live ? wp[1] : 0.f;
        ai[u] = live ? *reinterpret_cast<const float2*>(wp + 2 + d0) : make_float2(0.f, 0.f);
      }
      float m_new = M;
#pragma unroll
      for (int u = 0; u < UNR; ++u) m_new = fmaxf(m_new, mi[u]);
      const float corr = __builtin_amdgcn_exp2f(M - m_new);
      L *= corr;
      A.x *= corr;
      A.y *= corr;
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const float wt = __builtin_amdgcn_exp2f(mi[u] - m_new);
        L = fmaf(wt, li[u], L);
        A.x = fmaf(wt, ai[u].x, A.x);
        A.y = fmaf(wt, ai[u].y, A.y);
      }
      M = m_new;
    }
    if (r.add_new) {
      float d = row16_sum(qk);                    // over the head's threads: rows of 16 lanes, then the rows
      if constexpr (TPH == 64) d = quad16_sum(d);
      else d += __shfl_xor(d, 16, 64);
      const float s_new = d * a.scale_log2e;
      const float m2 = fmaxf(M, s_new);
      const float w_old = __builtin_amdgcn_exp2f(M - m2), w_new = __builtin_amdgcn_exp2f(s_new - m2);
      L = fmaf(L, w_old, w_new);
      A.x = fmaf(A.x, w_old, w_new * v_new.x);
      A.y = fmaf(A.y, w_old, w_new * v_new.y);
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    store_elem2<E>(out, row * HD + d0, make_float2(L > 0.f ? A.x * inv : 0.f, L > 0.f ? A.y * inv : 0.f));
  }
  // the last workgroups dispatched are the last to end, to within a few of them: those of the last sequence
  // and one per 16 sequences note the time
  if (a.clock && threadIdx.x == 0 && (b == (int32_t)gridDim.y - 1 || (blockIdx.x == 0 && (b & 15) == 15)))
    atomicMax(&a.clock[kClockLayerEnd], wall_clock64());
}

template <typename E, int HD>
__global__ __launch_bounds__(256) void k_attn_reduce(const AttnArgs a, int32_t n_q_heads) {
  constexpr int NSUB = 256 / HD;
  constexpr int UNR = 4;
  constexpr int WPH = (HD + 63) / 64;             // waves that hold a head's q . k_new products
  __shared__ float s_M[NSUB], s_L[NSUB], s_A[NSUB][HD];
  __shared__ float s_dot[WPH];
  const int32_t hq = blockIdx.x, b = blockIdx.y;
  const int dim = threadIdx.x % HD, sub = threadIdx.x / HD;
  const ReduceRow r = reduce_row(a, b);
  if (r.skip) return;
  const int32_t layer = blockIdx.z;
  const char* q = a.q + layer * a.q_stride;
  char* const out = a.out + layer * a.q_stride;
  const char* const new_k = a.new_k + layer * a.new_stride;       // (followed only if there are any)
  const char* const new_v = a.new_v + layer * a.new_stride;
  const float* const ws = a.ws + layer * a.ws_stride;
  const size_t row = (size_t)b * n_q_heads + hq;
  float qk = 0.f, v_new = 0.f;
  if (r.add_new && sub == 0) {
    const size_t kv_row = ((size_t)b * a.n_kv_heads + hq / a.group) * HD;
    qk = load_elem<E>(q, row * HD + dim) * load_elem<E>(new_k, kv_row + dim);
    v_new = load_elem<E>(new_v, kv_row + dim);
  }
  const float* w = ws + row * a.n_parts * (HD + 2);
  float M = kNegBig, L = 0.f, A = 0.f;
  for (int32_t s0 = sub; s0 < r.np; s0 += NSUB * UNR) {
    float mi[UNR], li[UNR], ai[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int32_t sp = s0 + u * NSUB;
      const bool live = sp < r.np;
      const float* wp = w + (size_t)(live ? sp : s0) * (HD + 2);
      mi[u] = live ? wp[0] : kNegBig;
      li[u] = live ? wp[1] : 0.f;
      ai[u] = live ? wp[2 + dim] : 0.f;
    }
    float m_new = M;
#pragma unroll
    for (int u = 0; u < UNR; ++u) m_new = fmaxf(m_new, mi[u]);
    const float corr = __builtin_amdgcn_exp2f(M - m_new);
    L *= corr;
    A *= corr;
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const float wt = __builtin_amdgcn_exp2f(mi[u] - m_new);
      L = fmaf(wt, li[u], L);
      A = fmaf(wt, ai[u], A);
    }
    M = m_new;
  }
  if (dim == 0) {
    s_M[sub] = M;
    s_L[sub] = L;
  }
  s_A[sub][dim] = A;
  if (r.add_new && sub == 0) {                   // HD / 64 waves hold the products: each leaves its sum
    const float wave_sum = quad16_sum(row16_sum(qk));
    if ((threadIdx.x & 63) == 0) s_dot[threadIdx.x >> 6] = wave_sum;
  }
  __syncthreads();
  if (sub == 0) {
    float Mt = s_M[0];
#pragma unroll
    for (int i = 1; i < NSUB; ++i) Mt = fmaxf(Mt, s_M[i]);
    float Lt = 0.f, At = 0.f;
#pragma unroll
    for (int i = 0; i < NSUB; ++i) {
      const float wt = __builtin_amdgcn_exp2f(s_M[i] - Mt);
      Lt = fmaf(wt, s_L[i], Lt);
      At = fmaf(wt, s_A[i][dim], At);
    }
    if (r.add_new) {
      float d = s_dot[0];
#pragma unroll
      for (int i = 1; i < WPH; ++i) d += s_dot[i];
      const float s_new = d * a.scale_log2e;
      const float m2 = fmaxf(Mt, s_new);
      const float w_old = __builtin_amdgcn_exp2f(Mt - m2), w_new = __builtin_amdgcn_exp2f(s_new - m2);
      Lt = fmaf(Lt, w_old, w_new);
      At = fmaf(At, w_old, w_new * v_new);
    }
    store_elem<E>(out, row * HD + dim, Lt > 0.f ? At / Lt : 0.f);
  }
  if (a.clock && threadIdx.x == 0 && (b == (int32_t)gridDim.y - 1 || (hq == 0 && (b & 15) == 15)))
    atomicMax(&a.clock[kClockLayerEnd], wall_clock64());
}

// ---- dispatch ----------------------------------------------------------------------------------------

bool attn_config_supported(const pie_config& c) {
  if (c.block_tokens != kBlockTokens || c.dtype < 0 || c.dtype > 2) return false;
  if (c.head_dim != 64 && c.head_dim != 128) return false;
  const int32_t g = c.n_q_heads / c.n_kv_heads;
  if (c.dtype != PIE_DTYPE_F32 && g > kMaxGroup) return false;
  return c.max_batch <= kMaxPlanBatch && c.max_blocks_per_seq <= (1 << 19);
}

static size_t max_parts_for(int32_t max_blocks) {
  const size_t mp = ((size_t)max_blocks * kBlockTokens + kMinPartTokens - 1) / kMinPartTokens;
  return mp ? mp : 1;
}
static size_t max_parts_of(const pie_config& c) { return max_parts_for(c.max_blocks_per_seq); }

size_t attn_workspace_floats(const pie_config& c) {
  const size_t planned = (size_t)c.max_batch * c.n_q_heads * max_parts_of(c) * (c.head_dim + 2);
  const size_t direct = attn_direct_floats(c);
  return planned > direct ? planned : direct;
}

// Blocks of slot lists one region needs: every item lists part_tokens / 16 slots, and a sequence's items
// cover its blocks rounded up to a whole item.
static size_t slot_list_ints(int32_t batch, int32_t max_blocks) {
  return (size_t)batch * ((size_t)max_blocks + kWaves * 64);
}

// int32 words of planning state: header, ticket counters (one per layer of a step), item records (2 words
// each), and the per-item slot lists of the two staging regions
static size_t plan_counter_ints(int32_t n_counters) {
  return (size_t)n_counters + ((size_t)n_counters & 1);    // keeps the item records 8-byte aligned
}

static size_t plan_ints_for(int32_t n_counters, int32_t batch, int32_t max_blocks) {
  return kPlanHdrInts + plan_counter_ints(n_counters) + 2 * (size_t)batch * max_parts_for(max_blocks) +
         2 * slot_list_ints(batch, max_blocks);
}

size_t attn_plan_ints(const pie_config& c) { return plan_ints_for(c.n_layers, c.max_batch, c.max_blocks_per_seq); }

// The pool's own scratch: the planning state and the partials carved from the caller's device buffer, laid out
// for the pool's largest batch and table width.
static AttnWork pool_work(const pie_pool* p) {
  AttnWork w;
  w.plan = p->d_plan;
  w.ws = p->d_ws;
  w.ws_floats = p->ws_floats;
  w.arrive = p->d_arrive;
  w.arrive_launches = &p->arrive_launches;
  w.n_counters = p->cfg.n_layers;
  w.lay_batch = p->cfg.max_batch;
  w.lay_max_blocks = p->cfg.max_blocks_per_seq;
  return w;
}

static int32_t* plan_hdr(const AttnWork& w) { return w.plan; }
static uint32_t* plan_counters(const AttnWork& w) { return reinterpret_cast<uint32_t*>(w.plan + kPlanHdrInts); }
static size_t plan_items_off(const AttnWork& w) { return kPlanHdrInts + plan_counter_ints(w.n_counters); }
static uint2* plan_items(const AttnWork& w) { return reinterpret_cast<uint2*>(w.plan + plan_items_off(w)); }
static int32_t* plan_slots(const AttnWork& w, int region) {
  return w.plan + plan_items_off(w) + 2 * (size_t)w.lay_batch * max_parts_for(w.lay_max_blocks) +
         (size_t)region * slot_list_ints(w.lay_batch, w.lay_max_blocks);
}

// Item size: a multiple of one pass of the workgroup's waves, at most 64 blocks per wave.  With no size set
// (attn_partition 0) the planning kernel chooses one of auto_part(); the host then sizes grids and the
// workspace for the smallest of them, which has the most items.
static int32_t part_tokens_of(const pie_pool* p) {
  int32_t part = p->attn_partition;
  if (part <= 0) return auto_part(0);
  const int32_t quantum = kWaves * kBlockTokens;
  if (part < kMinPartTokens) part = kMinPartTokens;
  part = (part + quantum - 1) / quantum * quantum;
  if (part > quantum * 64) part = quantum * 64;
  return part;
}

int launch_attn_plan(const pie_pool* p, const int32_t* d_ctx, int32_t batch, int32_t max_blocks, hipStream_t s,
                     bool reset_clock, const AttnWork* work, bool without_last) {
  const AttnWork w = work ? *work : pool_work(p);
  if (batch > kMaxPlanBatch || batch > w.lay_batch || max_blocks > w.lay_max_blocks) return PIE_EINVAL;
  // automatic item size: keep more than about eight and a half units per workgroup of the persistent decode grid
  const int32_t min_units = p->attn_partition <= 0 ? attn_min_units(p) : 0;
  hipLaunchKernelGGL(k_attn_plan, dim3(1), dim3(batch > 256 ? kPlanThreads : 256), 0, s, d_ctx, batch, part_tokens_of(p), min_units,
                     p->cfg.n_kv_heads, max_blocks, without_last ? 1 : 0, plan_items(w),
                     plan_hdr(w), plan_counters(w), w.n_counters, p->d_err, reset_clock ? p->d_clock : nullptr);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

int launch_attn_resolve(const pie_pool* p, const int32_t* d_table, const int32_t* d_ctx, int32_t batch,
                        int32_t max_blocks, bool region0, bool valid0, bool region1, bool valid1, hipStream_t s,
                        const LayerView* view, const AttnWork* work) {
  (void)d_ctx;
  const AttnWork w = work ? *work : pool_work(p);
  if (batch > w.lay_batch || max_blocks > w.lay_max_blocks || max_blocks <= 0) return PIE_EINVAL;
  const int32_t part = part_tokens_of(p);
  ResolveArgs a;
  a.table = d_table;
  a.items = plan_items(w);
  a.hdr = plan_hdr(w);
  a.map[0] = p->d_map[0];
  a.map[1] = p->d_map[1];
  a.slots[0] = region0 ? plan_slots(w, 0) : nullptr;
  a.slots[1] = region1 ? plan_slots(w, 1) : nullptr;
  a.err = p->d_err;
  a.max_blocks = max_blocks;
  a.n_handles = p->n_handles;
  a.n_gpu_blocks = p->cfg.n_gpu_blocks;
  a.n_slots = p->cfg.n_gpu_blocks + 2 * p->cfg.n_stage_blocks;
  a.stage_valid[0] = valid0 ? 1 : 0;
  a.stage_valid[1] = valid1 ? 1 : 0;
  if (view) {                                    // one layer's own handle -> slot map, into the slot list of region 0
    if (!region0 || region1) return PIE_EINVAL;
    a.map[0] = view->map;
    a.n_handles = view->n_handles;
    a.n_gpu_blocks = a.n_slots = view->n_slots;
  }
  // one workgroup per possible item; those past the planned count return at once
  const int32_t max_items = batch * ((max_blocks * kBlockTokens + part - 1) / part);
  hipLaunchKernelGGL(k_attn_resolve, dim3(max_items), dim3(64), 0, s, a);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

bool attn_planned_wide(const pie_pool* p, int32_t batch, int32_t layers) {
  const pie_config& c = p->cfg;
  if (c.dtype == PIE_DTYPE_F32 || p->attn_partition > 0 || (p->attn_valu && c.n_q_heads == c.n_kv_heads)) return false;
  return planned_wide(p->n_cu, c.n_kv_heads, c.n_q_heads / c.n_kv_heads, c.head_dim, layers, batch);
}

// done: an event that is to complete with this kernel (it rides on the kernel's own completion signal), or NULL
template <typename E, int HD>
static void launch_reduce(const AttnArgs& a, int32_t batch, int32_t n_q_heads, hipStream_t s, hipEvent_t done) {
  if (a.n_parts <= 8) {                           // few partitions per sequence: several heads per workgroup
    constexpr int HPW = 512 / HD;
    hipExtLaunchKernelGGL((k_attn_reduce_heads<E, HD>), dim3((n_q_heads + HPW - 1) / HPW, batch, a.n_layers), dim3(256), 0, s,
                          nullptr, done, 0, a, n_q_heads);
  } else {
    hipExtLaunchKernelGGL((k_attn_reduce<E, HD>), dim3(n_q_heads, batch, a.n_layers), dim3(256), 0, s, nullptr, done, 0, a,
                          n_q_heads);
  }
}

template <typename E, int HD, bool SPLIT, bool VALU, bool TWO>
static int launch_mfma_as(const pie_pool* p, AttnArgs a, int32_t layer_row, int32_t batch, int32_t n_q_heads,
                       hipStream_t s, hipEvent_t e0, hipEvent_t e1, hipEvent_t done) {
  const size_t lds = mfma_lds_floats<HD>(a.group) * sizeof(float);
  // As many workgroups as fit on the GPU at once, at most two a compute unit (four with head_dim 64): more only ask for more
  // at a time (32 layers of 64 sequences of 1 024 to 2 048 tokens, 32 heads, one / two / three: 8 457 / 7 962 / 7 980 us; 2 of
  // 256 of 128 to 4 096, 32 over 8: 485 / 441 / 454; on the vector ALU a call of the first, two and three: 262 and 268).  The
  // ticket counter hands out the work.
  static int wgs_per_cu[kMaxGroup + 1] = {};
  if (wgs_per_cu[a.group] == 0) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_attn_decode_mfma<E, HD, SPLIT, VALU, TWO>, kWaves * 64, lds) !=
            hipSuccess || n < 1) {
      (void)hipGetLastError();
      n = 2;
    }
    wgs_per_cu[a.group] = n < 256 / HD ? n : 256 / HD;
  }
  const int grid = p->n_cu * wgs_per_cu[a.group];
  if (a.clock && grid <= kClockWgs)
    a.clock_wg = p->d_clock + ((size_t)p->cfg.n_layers + 1) * kClockRow + (size_t)layer_row * kClockWgs * 2;
  if (e0) PIE_HIP(hipEventRecord(e0, s));
  // `done` (an event that completes with the layer's last kernel) rides on that kernel's own completion
  // signal instead of a packet of its own behind it
  const bool reduce = a.n_parts > 1 || a.new_k;
  if (done && !reduce)
    hipExtLaunchKernelGGL((k_attn_decode_mfma<E, HD, SPLIT, VALU, TWO>), dim3(grid), dim3(kWaves * 64), (uint32_t)lds, s,
                          nullptr, done, 0, a);
  else
    hipLaunchKernelGGL((k_attn_decode_mfma<E, HD, SPLIT, VALU, TWO>), dim3(grid), dim3(kWaves * 64), lds, s, a);
  PIE_HIP(hipGetLastError());
  if (e1) PIE_HIP(hipEventRecord(e1, s));
  if (reduce) launch_reduce<E, HD>(a, batch, n_q_heads, s, done);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

template <typename E, int HD, bool SPLIT, bool VALU = false>
static int launch_mfma(const pie_pool* p, const AttnArgs& a, int32_t layer_row, int32_t batch, int32_t n_q_heads,
                       hipStream_t s, hipEvent_t e0, hipEvent_t e1, hipEvent_t done) {
  // Where a table is so wide that for it alone the units do not fit k_attn_direct, the contexts are most likely much shorter
  // than the table: few units, each as fast as its waves ask.  us a call under tables
  // of 131 072 tokens, two blocks and one: 32 sequences of 100 to 1 000, 32 heads over 8, 24.2 and 25.7; 24 of 60 to 600, 32
  // heads, 37.4 and 38.5; 64 of 300 to 1 500, 12 heads of 64, 47.6 and 49.0; 200 of 500 to 3 000, 32 over 8, 251 and 248.
  // (Chosen by the units on the device, with both loops in the kernel: 24.6, 37.9, 48.0, but 1 000 of 20 to 300, which have
  // one, 166.6 and not 161.4.)
  const bool wide_table = a.n_layers == 1 && direct_too_wide(p->n_cu, a.n_kv_heads, a.group, batch, a.max_blocks);
  if constexpr (!VALU && HD == 128)              // (more than one layer: neither events, nor the clock, nor a map of its own)
    if (attn_planned_wide(p, batch, a.n_layers)) {
      hipLaunchKernelGGL((k_attn_decode_wide<E, HD, SPLIT>), dim3(p->n_cu), dim3((kPlannedWideHeads + kFinishers) * 64),
                         (uint32_t)wide_lds(kPlannedWideHeads, a.group, HD), s, a);
      PIE_HIP(hipGetLastError());
      if (a.n_parts > 1 || a.new_k) launch_reduce<E, HD>(a, batch, n_q_heads, s, done);
      else if (done) PIE_HIP(hipEventRecord(done, s));
      PIE_HIP(hipGetLastError());
      return PIE_OK;
    }
  if constexpr (!VALU)
    if (p->attn_partition <= 0 && !wide_table)
      return launch_mfma_as<E, HD, SPLIT, false, false>(p, a, layer_row, batch, n_q_heads, s, e0, e1, done);
  return launch_mfma_as<E, HD, SPLIT, VALU, true>(p, a, layer_row, batch, n_q_heads, s, e0, e1, done);
}

template <int HD>
static int launch_f32(const AttnArgs& a, int32_t batch, int32_t n_q_heads, int32_t max_items, hipStream_t s,
                      hipEvent_t e0, hipEvent_t e1, hipEvent_t done) {
  if (e0) PIE_HIP(hipEventRecord(e0, s));
  // one workgroup per possible item and query head; those past the planned count return at once
  hipLaunchKernelGGL((k_attn_decode_f32<HD>), dim3(max_items, n_q_heads), dim3(kWaves * 64), 0, s, a);
  PIE_HIP(hipGetLastError());
  if (e1) PIE_HIP(hipEventRecord(e1, s));
  if (a.n_parts > 1 || a.new_k) {
    launch_reduce<F32, HD>(a, batch, n_q_heads, s, nullptr);
    PIE_HIP(hipGetLastError());
  }
  if (done) PIE_HIP(hipEventRecord(done, s));     // the fp32 path is not tuned: an ordinary record
  return PIE_OK;
}

// How many layers of a planned step one launch may take: as many as the pool has room for partials of.  (The fp32 kernel,
// which is not tuned, takes them one by one.)
int32_t attn_planned_layers(const pie_pool* p, int32_t batch, int32_t max_blocks) {
  const pie_config& c = p->cfg;
  if (c.dtype == PIE_DTYPE_F32) return 1;
  return planned_step_layers(c, p->ws_floats, part_tokens_of(p), batch, max_blocks);
}

// Needs launch_attn_plan and launch_attn_resolve (for region layer & 1) earlier on the same stream, with the
// same batch, table width and context lengths.  d_k_new / d_v_new: the newest token's rows of this layer, taken
// from there instead of from the cache (the planning launch must have been told: without_last); NULL = the cache
// holds every token.
int launch_attn_decode(const pie_pool* p, int32_t layer, const void* d_q, int32_t max_blocks, const int32_t* d_ctx,
                       int32_t batch, void* d_out, hipStream_t s, hipEvent_t k_start, hipEvent_t k_end,
                       int32_t ticket_index, unsigned long long* clock_row, const LayerView* view, hipEvent_t done,
                       const AttnWork* work, const void* d_k_new, const void* d_v_new, int32_t n_layers) {
  const pie_config& c = p->cfg;
  const AttnWork w = work ? *work : pool_work(p);
  if (((uintptr_t)d_q | (uintptr_t)d_out) % 16) return PIE_EINVAL;
  if (max_blocks <= 0) return PIE_EINVAL;
  if (c.n_gpu_blocks + 2 * c.n_stage_blocks <= 0) return PIE_EINVAL;
  const int32_t g = c.n_q_heads / c.n_kv_heads;
  const int32_t part = part_tokens_of(p);
  const int32_t max_tokens = max_blocks * kBlockTokens;
  const int32_t n_parts = (max_tokens + part - 1) / part;
  const size_t layer_floats = (size_t)batch * c.n_q_heads * n_parts * (c.head_dim + 2);
  if (layer_floats > w.ws_floats) return PIE_ENOMEM;
  if (n_layers < 1 || (n_layers > 1 && (work || view || clock_row || n_layers > attn_planned_layers(p, batch, max_blocks))))
    return PIE_EINVAL;
  if (batch > w.lay_batch || max_blocks > w.lay_max_blocks) return PIE_EINVAL;
  if (!work) p->step_plan = StepPlan{};          // (the partials lie where it does)

  AttnArgs a;
  a.kv_layer = view ? view->kv_base : p->d_kv + (size_t)layer * p->d_layer_stride;
  a.slots = plan_slots(w, view ? 0 : (layer & 1));
  a.items = plan_items(w);
  a.hdr = plan_hdr(w);
  // one ticket counter per launch since the last planning kernel (by default the layer's)
  if (ticket_index < 0) ticket_index = layer;
  if (ticket_index >= w.n_counters) return PIE_EINVAL;
  a.counter = plan_counters(w) + ticket_index;
  a.q = (const char*)d_q;
  a.out = (char*)d_out;
  a.ws = w.ws;
  a.ctx = d_ctx;
  a.block_bytes = p->block_bytes;
  a.scale_log2e = p->scale_log2e;
  a.max_blocks = max_blocks;
  a.n_kv_heads = c.n_kv_heads;
  a.group = g;
  a.n_parts = n_parts;
  a.max_items = batch * n_parts;
  a.clock = clock_row;
  a.clock_wg = nullptr;         // set by the launcher of a persistent grid that fits the per-workgroup words
  if ((d_k_new == nullptr) != (d_v_new == nullptr)) return PIE_EINVAL;
  if (((uintptr_t)d_k_new | (uintptr_t)d_v_new) % 8) return PIE_EINVAL;   // the reduction loads two elements at once
  a.new_k = (const char*)d_k_new;
  a.new_v = (const char*)d_v_new;
  a.n_layers = n_layers;
  a.kv_stride = p->d_layer_stride;
  a.q_stride = (size_t)batch * c.n_q_heads * c.head_dim * p->elem_bytes;
  a.new_stride = (size_t)batch * c.n_kv_heads * c.head_dim * p->elem_bytes;
  a.ws_stride = layer_floats;
  const bool hd128 = c.head_dim == 128;
  const int32_t row = clock_row ? (int32_t)((clock_row - p->d_clock) / kClockRow) : 0;
  switch (c.dtype) {
    case PIE_DTYPE_F32: {
      return hd128 ? launch_f32<128>(a, batch, c.n_q_heads, a.max_items, s, k_start, k_end, done)
                   : launch_f32<64>(a, batch, c.n_q_heads, a.max_items, s, k_start, k_end, done);
    }
    case PIE_DTYPE_F16:
      if (g == 1 && p->attn_valu)
        return hd128 ? launch_mfma<F16, 128, false, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done)
                     : launch_mfma<F16, 64, false, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done);
      return hd128 ? launch_mfma<F16, 128, false>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done)
                   : launch_mfma<F16, 64, false>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done);
    case PIE_DTYPE_BF16:
      if (g == 1 && p->attn_valu)
        return hd128 ? launch_mfma<BF16, 128, true, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done)
                     : launch_mfma<BF16, 64, true, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done);
      return hd128 ? launch_mfma<BF16, 128, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done)
                   : launch_mfma<BF16, 64, true>(p, a, row, batch, c.n_q_heads, s, k_start, k_end, done);
    default: return PIE_EINVAL;
  }
}

// The calibration kernel over the same planning state (launch_attn_plan and launch_attn_resolve first).
int launch_stream_probe(const pie_pool* p, int32_t layer, int32_t max_blocks, int32_t batch, hipStream_t s) {
  const pie_config& c = p->cfg;
  if (max_blocks <= 0 || layer < 0 || layer >= c.n_layers) return PIE_EINVAL;
  const AttnWork w = pool_work(p);
  AttnArgs a = {};
  a.kv_layer = p->d_kv + (size_t)layer * p->d_layer_stride;
  a.slots = plan_slots(w, layer & 1);
  a.items = plan_items(w);
  a.hdr = plan_hdr(w);
  a.counter = plan_counters(w) + layer;
  a.block_bytes = p->block_bytes;
  a.n_kv_heads = c.n_kv_heads;
  const size_t tile_bytes = (size_t)kBlockTokens * c.head_dim * p->elem_bytes;
  uint32_t* sink = p->d_err + 1;                  // a spare word of the error page
  const int grid = p->n_cu * 2;
  switch (tile_bytes / 1024) {
    case 2: hipLaunchKernelGGL((k_stream_probe<2>), dim3(grid), dim3(kWaves * 64), 0, s, a, tile_bytes, sink); break;
    case 4: hipLaunchKernelGGL((k_stream_probe<4>), dim3(grid), dim3(kWaves * 64), 0, s, a, tile_bytes, sink); break;
    case 8: hipLaunchKernelGGL((k_stream_probe<8>), dim3(grid), dim3(kWaves * 64), 0, s, a, tile_bytes, sink); break;
    default: return PIE_EINVAL;
  }
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

// ---- attention without a workspace from the caller ---------------------------------------------------
// For callers that cannot give or allocate scratch memory (code under graph capture, tight serving loops,
// harnesses that forbid allocation): the planning state and the split-context partials of one attention call
// live in a file-scope device array.  Every device the library runs on holds its own copy of the array for the
// life of the process; its address on a device is looked up once, with that device current, and only that
// address is ever handed to kernels (the array's name in host code is a host-side stand-in).

constexpr size_t kStaticScratchBytes = (size_t)40 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kArriveWords * kArriveStride * 8];   // arrival words last

constexpr int kMaxScratchDevices = 64;
static char* g_scratch_ptr[kMaxScratchDevices] = {};
static std::atomic<uint64_t> g_scratch_launches[kMaxScratchDevices];   // launches that have used its arrival words
static std::mutex g_scratch_mutex;

// Device address of the current device's copy of the array.
int attn_static_scratch(char** out, std::atomic<uint64_t>** out_launches) {
  int dev = -1;
  PIE_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxScratchDevices) return PIE_EINVAL;
  std::lock_guard<std::mutex> guard(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    PIE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return PIE_EHIP;
    g_scratch_ptr[dev] = static_cast<char*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  if (out_launches) *out_launches = &g_scratch_launches[dev];
  return PIE_OK;
}

// The scratch of one call over `batch` sequences of up to `max_blocks` blocks, placed in the array: planning
// state first, partials behind it.  PIE_ENOMEM if the call needs more than the array holds.
int attn_static_work(const pie_pool* p, int32_t batch, int32_t max_blocks, AttnWork* out) {
  if (batch < 0 || batch > kMaxPlanBatch || max_blocks < 0 || max_blocks > (1 << 19)) return PIE_EINVAL;
  char* base = nullptr;
  std::atomic<uint64_t>* launches = nullptr;
  const int rc = attn_static_scratch(&base, &launches);
  if (rc) return rc;
  const int32_t part = part_tokens_of(p);
  const size_t n_parts = ((size_t)max_blocks * kBlockTokens + part - 1) / part;
  const size_t plan_bytes = (plan_ints_for(2, batch, max_blocks) * 4 + kAlign - 1) / kAlign * kAlign;
  const size_t ws_floats = (size_t)batch * p->cfg.n_q_heads * n_parts * (p->cfg.head_dim + 2);
  if (plan_bytes > kStaticScratchBytes || ws_floats * 4 > kStaticScratchBytes - plan_bytes) return PIE_ENOMEM;
  out->plan = reinterpret_cast<int32_t*>(base);
  out->ws = reinterpret_cast<float*>(base + plan_bytes);
  out->ws_floats = ws_floats;
  out->arrive = reinterpret_cast<uint64_t*>(base + kStaticScratchBytes);
  out->arrive_launches = launches;
  out->n_counters = 2;          // one is used; two keep the item records 8-byte aligned
  out->lay_batch = batch;
  out->lay_max_blocks = max_blocks;
  return PIE_OK;
}

}  // namespace pie
