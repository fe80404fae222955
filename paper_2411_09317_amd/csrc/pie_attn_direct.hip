// Paged-attention decode in one launch, for calls too small to fill the GPU for long.
//
// The planned path (pie_kernels.hip) costs four launches a call - plan, resolve, decode, reduce - or two a layer inside
// a step, and cuts contexts into items of at least 512 tokens.  Below a few hundred MB of keys and values per layer its
// time is launches, the gaps between them and a grid that mostly idles, not bytes.  Here every workgroup works out the
// whole split for itself from the context lengths (at most four per lane, one scan), looks its blocks up through table
// and map, streams them, and the workgroup that finishes a (sequence, kv head) last merges the partial states, adds the
// newest token and writes the result; with new rows it can also store them.
//
// The layers of a step start from a plan, and where nothing has to happen between them they share a launch too (n_layers),
// behind one that works the plan out: then the chain of accesses, the tail and the gap behind it, 7 of 11 us a layer of a
// small step, come once a step and not once a layer.  us a step, a launch a layer before and one of k_attn_direct for all: 32
// layers of 8 sequences of 128 to 4 096 tokens, 32 heads over 8, 358 and 162 (888 MB, 5.5 TB/s); 16 of 24 of 100 to 1 100, 32
// heads, 613 and 525; 16 growing caches of 48 sequences, 685 and 573.  The last two have units enough to be read four heads side
// by side (k_attn_direct_wide, below), 518 and 556.
//
// What bounds it: for small calls a chain of dependent accesses, about 7 us from the first workgroup's start (context
// lengths and split 1.4 us, table and map 0.7, a block 0.9, the part's state stored 1.0 and counted 0.4 to 1.3, the
// merge 1.4); so short contexts are not cut (attn_whole) and need neither split nor merge.  For large ones HBM bounds it.  us
// a call among others, planned before and in one launch now: one sequence of 700 tokens, 32 heads over 8: 24.6 and 6.5; one
// of 32 749, 64 over 8: 48.6 and 26.4 (134 MB, 5.1 TB/s); 32 of 32 768, 64 over 8: 671 and 656 (4.3 GB, 6.5 TB/s).

#include <hip/hip_ext.h>

#include <atomic>

#include "pie_attn_wide.h"

namespace pie {

// Where the arrival word of a pair in a launch's layer lies: sixteen layers of a pair share a line.
__device__ __forceinline__ size_t arrive_word(int32_t lines, int32_t layer, size_t pair) {
  return ((size_t)(layer / kArriveStride) * lines + pair) * kArriveStride + layer % kArriveStride;
}

struct SplitIn {             // what the split of a call follows from
  const int32_t* ctx;
  uint32_t* err;
  int32_t* hdr;              // plan header, to note the nominal item size in, or NULL
  int32_t batch, max_blocks, n_kv_heads;
  int32_t minus;             // 1: the newest token is not read from the cache
  int32_t min_units;         // as in k_attn_plan; 0: the size is the smallest whatever the lengths
  int32_t max_items;         // items (all sequences' parts) the split may make
};

struct SplitArgs : SplitIn { // the plan of a step
  const int32_t* table;
  const int32_t* map[2];     // per staging region: handle -> slot, or NULL for no region or no slots
  int32_t* plan[2];
  int32_t n_handles, n_gpu_blocks, n_slots, stage_valid;
  int32_t append;            // kAppend*, where each layer's launch stores its rows, or -1
  int32_t places;            // items there may be: a workgroup each; those behind them store the new rows
  uint32_t* counters;        // of k_attn_direct_wide, to clear: tickets, one a layer of the pool,
  uint64_t* arrive;          // and the arrival words of the layers of a launch, or NULL
  int32_t n_counters, arrive_lines, n_layers;
};

struct DirectArgs : SplitIn {
  const char* kv_layer;
  const int32_t* table;      // [B][max_blocks] handles
  const int32_t* map;        // handle -> slot
  const char* q;             // [B][Hq][d]
  char* out;                 // [B][Hq][d]
  const char* new_k;         // newest token's rows [B][Hkv][d] (see AttnArgs), or NULL
  const char* new_v;
  float* ws;                 // partial states: [unit][group][d + 4]
  uint64_t* arrive;          // per (sequence, head unit): workgroups of which launch have stored their part
  uint64_t launch;           // this launch's number << kArriveShift
  int32_t* plan;             // records and slot lists of the items (kPlan*): read where PLAN says so, else written; or NULL
  unsigned long long* clock;    // the layer's row of the clock table and its workgroups' pairs, or NULL
  unsigned long long* clock_wg;
  size_t block_bytes;
  size_t kv_stride, q_stride, new_stride;   // bytes between the layers of the launch: caches, q and out, new rows
  int32_t map_stride;        // entries between their maps: 0 where they share one
  int32_t ws_bytes;          // of one layer's partial states
  int32_t arrive_lines;      // lines of arrival words, a pair's for sixteen layers each, between those of layer l and l + 16
  float scale_log2e;
  int32_t group, n_q_heads;
  int32_t n_handles, n_gpu_blocks, n_slots, stage_valid;
  int32_t append;            // kAppend*: store the new rows into the tail blocks this says, or -1
  int32_t n_layers, places;  // k_attn_direct_wide: layers of the launch, items there may be,
  uint32_t* counter;         // its ticket counter, cleared ahead of it like the arrival words it uses
};

// ---- one wave's share of a unit ------------------------------------------------------------------------

template <int HD_>
struct Wave32 {              // fp32 caches: one query head, on the vector ALU
  using E = F32;
  static constexpr int HD = HD_, NL = HD / 16, EB = 4, kWavesPerEu = 2;
  float q[NL][4];
  float m, l, acc[NL];
  __device__ __forceinline__ void load_q(const char* base, size_t row0, int, int lane, float scale) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const float4 t = *reinterpret_cast<const float4*>(base + (row0 * HD + 4 * (4 * i + (lane >> 4))) * 4);
      q[i][0] = t.x * scale; q[i][1] = t.y * scale; q[i][2] = t.z * scale; q[i][3] = t.w * scale;
    }
  }
  __device__ __forceinline__ void reset() {
    m = kNegBig;
    l = 0.f;
#pragma unroll
    for (int n = 0; n < NL; ++n) acc[n] = 0.f;
  }
  __device__ __forceinline__ void block(uint4 (&kr)[NL], uint4 (&vr)[NL], int32_t t_first, int32_t limit, int lane, float) {
    f32_block<HD>(kr, vr, q, t_first, limit, lane, m, l, acc);
  }
  __device__ __forceinline__ void to_lds(float* s_m, float* s_l, float* s_acc, int row_floats, int wave, int, int lane) {
    l = row16_sum(l);
#pragma unroll
    for (int n = 0; n < NL; ++n) acc[n] = quad16_sum(acc[n]);
    if (lane == 0) {
      s_m[wave * kMaxGroup] = m;
      s_l[wave * kMaxGroup] = l;
    }
    if (lane < 16) {
#pragma unroll
      for (int n = 0; n < NL; ++n) s_acc[wave * row_floats + 16 * n + lane] = acc[n];
    }
  }
};

// ---- partial states between workgroups -------------------------------------------------------------------
// They may run on different XCDs, whose L2 caches do not see each other's lines.  So a part is written through and
// read past them (the sc1 accesses an agent-scope atomic uses, sixteen bytes at a time): a part is complete when the
// writer's stores have been counted down, which every writing wave waits for before its workgroup is counted in, and
// the reader starts when all are in.  No cache is written back or invalidated for it: a release and an acquire fence
// at agent scope instead cost 20 to 100 us here, since each makes a whole L2 do so.
constexpr int kAuxAgent = 16;                    // sc1
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t parts_rsrc(float* base, int32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
}
__device__ __forceinline__ void put4(__amdgpu_buffer_rsrc_t r, int32_t off, const float4& x) {
  __builtin_amdgcn_raw_buffer_store_b128(bits_as<u32x4>(x), r, off, 0, kAuxAgent);
}
__device__ __forceinline__ float4 get4(__amdgpu_buffer_rsrc_t r, int32_t off, int32_t wave_off) {
  return bits_as<float4>(__builtin_amdgcn_raw_buffer_load_b128(r, off, wave_off, kAuxAgent));
}
__device__ __forceinline__ void put2(__amdgpu_buffer_rsrc_t r, int32_t off, float x, float y) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(x), __float_as_uint(y)}, r, off, 0, kAuxAgent);
}
__device__ __forceinline__ float2 get2(__amdgpu_buffer_rsrc_t r, int32_t off) {
  return bits_as<float2>(__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kAuxAgent));
}
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// four consecutive elements
template <typename E>
__device__ __forceinline__ float4 load_elem4(const char* base, size_t idx) {
  const float2 a = load_elem2<E>(base, idx), b = load_elem2<E>(base, idx + 2);
  return make_float4(a.x, a.y, b.x, b.y);
}
__device__ __forceinline__ void axpy(float4& y, float w, const float4& x) {
  y.x = fmaf(w, x.x, y.x); y.y = fmaf(w, x.y, y.y); y.z = fmaf(w, x.z, y.z); y.w = fmaf(w, x.w, y.w);
}

// max / sum over a head's threads, one or two rows of sixteen lanes; every one of them gets it
template <int TPH>
__device__ __forceinline__ float head_max(float x) {
  x = row16_max(x);
  if constexpr (TPH == 32) x = fmaxf(x, __shfl_xor(x, 16, 64));
  return x;
}
template <int TPH>
__device__ __forceinline__ float head_sum(float x) {
  x = row16_sum(x);
  if constexpr (TPH == 32) x += __shfl_xor(x, 16, 64);
  return x;
}

// ---- states into one ---------------------------------------------------------------------------------------
// What k_attn_direct's workgroups and k_attn_direct_wide's finishing waves sum, a column (four dims of a head) to a thread, in
// one order: a step's results are the same bits whichever its layers run in.

// n states in LDS (the waves', or the merging groups'): head h, dims d0 ..  (By reference: given the pointers themselves the compiler
// orders k_attn_direct's tail otherwise, 6.23 us and not 6.21 for one sequence of 700 tokens.)
template <int ROW>
__device__ __forceinline__ void merge_states(const float* const& s_m, const float* const& s_l, const float* const& s_acc, const int& G,
                                             int n, int h, int d0, float& M, float& L, float4& A) {
  M = s_m[h];
  for (int i = 1; i < n; ++i) M = fmaxf(M, s_m[i * kMaxGroup + h]);
  L = 0.f;
  A = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i = 0; i < n; ++i) {
    const float wt = __builtin_amdgcn_exp2f(s_m[i * kMaxGroup + h] - M);
    L = fmaf(wt, s_l[i * kMaxGroup + h], L);
    axpy(A, wt, *reinterpret_cast<const float4*>(&s_acc[((size_t)i * G + h) * ROW + d0]));
  }
}

// The newest token's part, (q . k, 1, v), to the others'.
template <int TPH>
__device__ __forceinline__ void add_newest(float4 q, float4 k, float4 v, float scale_log2e, float M, float& L, float4& A) {
  const float dot = fmaf(q.x, k.x, q.y * k.y) + fmaf(q.z, k.z, q.w * k.w);
  const float s_new = head_sum<TPH>(dot) * scale_log2e;
  const float m2 = fmaxf(M, s_new);
  const float w_old = __builtin_amdgcn_exp2f(M - m2), w_new = __builtin_amdgcn_exp2f(s_new - m2);
  L = fmaf(L, w_old, w_new);
  A = make_float4(A.x * w_old, A.y * w_old, A.z * w_old, A.w * w_old);
  axpy(A, w_new, v);
}

// A head's threads take TPH stored parts at a time: thread i has part i's (M, L), if there is one, and works out its weight ...
template <int TPH>
__device__ __forceinline__ float weigh_parts(float2 ml, bool live, float& M, float& L, float4& A) {
  const float m_new = fmaxf(M, head_max<TPH>(ml.x));
  const float corr = __builtin_amdgcn_exp2f(M - m_new);
  const float wt = live ? __builtin_amdgcn_exp2f(ml.x - m_new) : 0.f;
  L = fmaf(L, corr, head_sum<TPH>(wt * ml.y));
  A = make_float4(A.x * corr, A.y * corr, A.z * corr, A.w * corr);
  M = m_new;
  return wt;
}
// ... then every thread sums its four dims over them (those beyond the last weigh 0).
template <int UNR>
__device__ __forceinline__ void sum_parts(const float* weights, const float4 (&ai)[UNR], float4& A) {
#pragma unroll
  for (int u = 0; u < UNR; u += 4) {
    const float4 wu = *reinterpret_cast<const float4*>(&weights[u]);
    axpy(A, wu.x, ai[u]);
    axpy(A, wu.y, ai[u + 1]);
    axpy(A, wu.z, ai[u + 2]);
    axpy(A, wu.w, ai[u + 3]);
  }
}
// A round that is not full reads its last part several times, with weights of zero for all but one.  If that part holds an
// infinity, or any other, the sum is made once more part by part.
__device__ __forceinline__ void sum_again_if_infinite(__amdgpu_buffer_rsrc_t parts, int32_t part0, int32_t step, int ml_off, int d0,
                                                      int32_t s_begin, int32_t s_end, float M, float4& A) {
  if (!(fmaf(A.x, 0.f, fmaf(A.y, 0.f, fmaf(A.z, 0.f, A.w * 0.f))) == 0.f)) {
    A = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t s = s_begin; s < s_end; ++s)
      axpy(A, __builtin_amdgcn_exp2f(get2(parts, part0 + s * step + ml_off).x - M), get4(parts, part0 + d0 * 4, s * step));
  }
}

struct FastRcp {
  __device__ __forceinline__ float operator()(float y) const { return __builtin_amdgcn_rcpf(y); }
};

constexpr int kDirectLaneSeqs = kDirectSeqs / 64;   // sequences per lane in the split
constexpr int32_t kEarlyParts = 32;

// A step's layers share the split and, per staging region, the slots: k_step_begin works them out for every item ahead of
// the layers, or, where they do not share launches, the first layer of each region leaves what it has worked out, and the
// others start from that, one access deep instead of four.  Where every layer has a map of its own (the growing caches) they
// share the split alone.  PLAN: kDirectPlanReplay, kDirectPlanReplaySplit, kDirectPlanWrite for those that leave it, or
// kDirectPlanNone.
constexpr int kPlanRec = 8;                      // b, tok0, tok1, parts, first item, part, tail slot, raw context length
constexpr int kPlanInts = kPlanRec + kDirectMaxQuanta * kWaves;   // a record, then the slots of each wave's blocks

struct Item {
  int32_t b, tok0, tok1, np, first, part;         // one part of sequence b, of np from item `first`; b < 0: there is none
  int32_t at;                                     // where in the plan its record stands (ranked)
};
// The item size the planning kernel would have chosen, as asked for by pie_get_attn_partition_sync, worked out by one wave
// whose lane i has the lengths of the sequences i, i + 64, ...
template <int SEQS>
__device__ __forceinline__ void note_item_size(const SplitIn& a, const int32_t (&c4)[SEQS]) {
  const int lane = threadIdx.x & 63;
  int32_t size = auto_part(0);
  if (a.min_units > 0) {
#pragma unroll 1
    for (int t = 1; t < kAutoParts; ++t) {
      int32_t n = 0;
#pragma unroll
      for (int i = 0; i < SEQS; ++i)
        if (64 * i + lane < a.batch) n += c4[i] > 0 ? (c4[i] + auto_part(t) - 1) / auto_part(t) : 1;
      if ((long long)wave_sum(n) * a.n_kv_heads > a.min_units) size = auto_part(t);
    }
  }
  if (threadIdx.x == 0) a.hdr[1] = size;
}

// The split, by one wave: lane i has the sequences i, i + 64, ...  lead: the one workgroup that reports errors and the size.
template <int SEQS>
__device__ __forceinline__ Item split_item(const SplitIn& a, int32_t place, bool lead, bool ranked) {
  const int lane = threadIdx.x & 63;
  int32_t c4[SEQS], q4[SEQS], n4[SEQS], k4[SEQS], end4[SEQS];
  int32_t total = 0;
#pragma unroll
  for (int i = 0; i < SEQS; ++i) {
    c4[i] = q4[i] = 0;
    if (64 * i < a.batch) {
      const int32_t b = 64 * i + lane;
      if (b < a.batch) {
        const int32_t raw = a.ctx[b];
        const int32_t full = clamp_ctx(raw, a.max_blocks);
        if (raw > full && lead) atomicOr(a.err, PIE_DEVERR_BAD_HANDLE);
        c4[i] = full > a.minus ? full - a.minus : 0;
        q4[i] = quanta_of(c4[i]);
      }
      total += wave_sum(q4[i]);
    }
  }
  if (a.hdr && lead) note_item_size(a, c4);
  auto items_of = [&](int32_t k) {
    int32_t n = 0;
#pragma unroll
    for (int i = 0; i < SEQS; ++i)
      if (64 * i < a.batch) n += div_up(q4[i], k, FastRcp());   // (0 beyond the batch)
    return wave_sum(n);
  };
  const int32_t k = quanta_per_part(total, a.max_items, items_of);
  int32_t n_items = 0;
#pragma unroll
  for (int i = 0; i < SEQS; ++i) {
    n4[i] = k4[i] = end4[i] = 0;
    if (64 * i < a.batch) {
      if (q4[i] > 0) {
        const SeqParts parts = seq_parts(q4[i], k, FastRcp());
        k4[i] = parts.each;
        n4[i] = parts.n;
      }
      end4[i] = n_items + wave_scan(n4[i]);       // items up to and including the lane's sequence
      n_items = __builtin_amdgcn_readlane(end4[i], 63);
    }
  }
  const int32_t item = place;
  // one unit a workgroup: the launch has at least as many workgroups as the split can make units
  int32_t b = 0;                                  // sequences whose items all come before this one
#pragma unroll
    for (int i = 0; i < SEQS; ++i)
      if (64 * i < a.batch) b += __popcll(__builtin_amdgcn_ballot_w64(64 * i + lane < a.batch && end4[i] <= item));
  int32_t ctx_b = 0, kq = 1, end = 1, np = 1, at = place;
#pragma unroll
    for (int i = 0; i < SEQS; ++i)
      if (b >> 6 == i) {
        ctx_b = __builtin_amdgcn_readlane(c4[i], b & 63);
        kq = __builtin_amdgcn_readlane(k4[i], b & 63);
        np = __builtin_amdgcn_readlane(n4[i], b & 63);
        end = __builtin_amdgcn_readlane(end4[i], b & 63);
      }
  const int32_t first = end - np, part = item - first;
  const int32_t tok0 = part * kq * kQuantum;
  const int32_t tok1 = min(ctx_b, tok0 + kq * kQuantum);       // <= tok0 only for an empty sequence
  if (item >= n_items) b = -1;
  // The plan lists the items by size, largest first, so that the layers that start from it spread the large parts over
  // the compute units and end on small ones: 639 -> 617 us for 16 layers of 24 sequences of 100 to 1 100 tokens.
  if (ranked && b >= 0) {
    int32_t before = 0;
#pragma unroll
    for (int i = 0; i < SEQS; ++i)
      if (64 * i < a.batch) before += k4[i] > kq || (k4[i] == kq && 64 * i + lane < b) ? n4[i] : 0;
    at = wave_sum(before) + part;
  }
  return {b, tok0, tok1, np, first, part, at};
}

// Ahead of a step's layers: their plan, a workgroup to an item and a lane to a block, and the new rows of all layers.
__global__ __launch_bounds__(kWaves * 64) void k_step_begin(const SplitArgs a, const AppendArgs rows) {
  if ((int32_t)blockIdx.x >= a.places) {
    const int32_t i = blockIdx.x - a.places;
    append_rows(rows, i % a.batch, i / a.batch);
    return;
  }
  const int32_t place = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Item it = split_item<kDirectLaneSeqs>(a, place, place == 0, true);
  if (a.arrive && place == 0)
    for (int32_t i = threadIdx.x; i < a.n_counters; i += kWaves * 64) a.counters[i] = 0;
  if (a.arrive && it.b >= 0 && it.np > 1 && it.part == 0)
    for (int32_t i = threadIdx.x; i < a.n_layers * a.n_kv_heads; i += kWaves * 64) {
      const int32_t l = i / a.n_kv_heads, g = i - l * a.n_kv_heads;
      a.arrive[arrive_word(a.arrive_lines, l, (size_t)it.b * a.n_kv_heads + g)] = 0;
    }
  const int32_t jb = it.tok0 / kBlockTokens + wave + kWaves * lane;
  const bool live = it.b >= 0 && jb * kBlockTokens < it.tok1;
  const int32_t ctx_raw = it.b >= 0 ? a.ctx[it.b] : 0, jt = (ctx_raw - 1) / kBlockTokens;
  const bool has_tail = a.append >= 0 && it.part == it.np - 1 && ctx_raw > 0;
  const int32_t* row = a.table + (size_t)(it.b >= 0 ? it.b : 0) * a.max_blocks;
  const int32_t handle = live ? row[jb] : -1, tail = has_tail && jt < a.max_blocks ? row[jt] : -1;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (!a.plan[r]) continue;
    int32_t* rec = a.plan[r] + (size_t)it.at * kPlanInts;
    int32_t tail_slot = -1;
    if (a.map[r] && has_tail)
      tail_slot = append_slot(tail, a.map[r], a.n_handles, a.n_gpu_blocks, a.n_slots, a.append, threadIdx.x == 0, a.err);
    if (live)
      rec[kPlanRec + wave * kDirectMaxQuanta + lane] =
          a.map[r] ? resolve_slot(handle, a.map[r], a.n_handles, a.n_gpu_blocks, a.n_slots, a.stage_valid != 0, a.err) : handle;
    if (threadIdx.x == 0) {
      *reinterpret_cast<int4*>(rec) = make_int4(it.b, it.tok0, it.tok1, it.np);
      *reinterpret_cast<int4*>(rec + 4) = make_int4(it.first, it.part, tail_slot, ctx_raw);
    }
  }
}

// SEQS: sequences to a lane in the split.  A small call runs its code once, so every instruction of it is a wait: with one to a
// lane, for up to 64 sequences, the split is a quarter as long.  us a call, four and one: one sequence of 700 tokens, 32 heads over
// 8, 6.48 and 6.24; 8 of 100 to 1 000 7.67 and 7.42; 30 of 100 to 1 000 16.2 and 15.8; 64 of 200 to 1 800, 12 heads of 64, 37.9
// and 37.1; one of 32 749, 64 over 8, 24.5 and 24.2.  (To look the whole of a small table up beside the lengths, and not behind the
// split, saves two accesses and costs more than those in code: 6.48 and 7.29.)
template <typename W, int NW, int PLAN, bool TWO, int SEQS>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW > kWaves ? NW / 4 : W::kWavesPerEu, 8)))
void k_attn_direct(const DirectArgs a) {
  using E = typename W::E;
  constexpr int HD = W::HD, NL = W::NL, EB = W::EB;
  constexpr int NT = NW * 64;
  constexpr bool WHOLE = NW == kWholeWaves;       // nothing is cut: a workgroup to a (sequence, kv head)
  static_assert(NW == kWaves || (WHOLE && PLAN == kDirectPlanNone), "the split is in quanta of so many waves");
  constexpr int TILE_BYTES = kBlockTokens * HD * EB;
  constexpr int ROW = HD + 4;                     // padded LDS row of one head's accumulator
  constexpr int TPH = HD / 4;                     // threads per head when states are merged, four dims each
  constexpr int PART = (HD + 4) * 4;              // bytes of a head's partial state: accumulator, max, sum, padding

  constexpr bool SLOTS = PLAN == kDirectPlanReplay, REPLAY = SLOTS || PLAN == kDirectPlanReplaySplit;
  constexpr bool LEAVES = PLAN == kDirectPlanWrite;

  extern __shared__ __align__(16) float s_dyn[];
  __shared__ bool s_last;
  __shared__ __align__(16) float s_w[NT];         // weights of the parts being merged, a thread each
  float* s_m = s_dyn;                             // [NW][16]
  float* s_l = s_dyn + NW * kMaxGroup;            // [NW][16]
  float* s_acc = s_dyn + 2 * NW * kMaxGroup;      // [NW][G][ROW]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t G = a.group, H = a.n_kv_heads;
  // (no store comes before the uniform loads below: they are then scalar loads)
  const unsigned long long t_start = a.clock ? wall_clock64() : 0ull;
  // kv heads innermost: their tiles lie side by side; then the layers, so that all of them come with their largest items
  const int32_t g = blockIdx.x, layer = blockIdx.y, place = blockIdx.z;
  const bool lead = (g | layer | place) == 0;
  const char* kv_layer = a.kv_layer + layer * a.kv_stride;
  const int32_t* map = a.map + (size_t)layer * a.map_stride;
  const char* q_in = a.q + layer * a.q_stride;
  char* const out = a.out + layer * a.q_stride;
  const char* new_k = a.new_k ? a.new_k + layer * a.new_stride : nullptr;
  const char* new_v = a.new_k ? a.new_v + layer * a.new_stride : nullptr;
  int32_t b, ctx_raw, tok0, tok1, np, first, part, tail = -1;   // this unit: one part of sequence b, of np from item `first`
  int32_t slots = -1, handle = -1;                // of this wave's blocks, one to a lane
  int32_t at = 0;                                 // where in the plan this item's record stands
  if constexpr (SLOTS) slots = a.plan[(size_t)place * kPlanInts + kPlanRec + wave * kDirectMaxQuanta + lane];
  if constexpr (REPLAY) {
    const int32_t* rec = a.plan + (size_t)place * kPlanInts;
    b = rec[0]; tok0 = rec[1]; tok1 = rec[2]; np = rec[3]; first = rec[4]; part = rec[5]; tail = rec[6]; ctx_raw = rec[7];
  } else if constexpr (WHOLE) {                   // (place: the sequence)
    const int32_t j = wave + NW * lane;           // its blocks, as many as the table has, looked up beside its length
    if (j < a.max_blocks) handle = a.table[(size_t)place * a.max_blocks + j];
    if (handle >= 0 && handle < a.n_handles) slots = map[handle];
    b = place;
    ctx_raw = a.ctx[b];
    const int32_t full = clamp_ctx(ctx_raw, a.max_blocks);
    if (ctx_raw > full && g == 0) atomicOr(a.err, PIE_DEVERR_BAD_HANDLE);
    tok0 = 0;
    tok1 = full > a.minus ? full - a.minus : 0;
    np = 1;
    first = place;
    part = 0;
  } else {
    const Item it = split_item<SEQS>(a, place, lead, LEAVES);
    b = it.b; tok0 = it.tok0; tok1 = it.tok1; np = it.np; first = it.first; part = it.part; at = it.at;
    ctx_raw = b >= 0 ? a.ctx[b] : 0;
  }
  if constexpr (!SLOTS) {                         // where this sequence's newest token goes, if its last part's
    tail = -1;                                    // workgroups store it
    if (a.append >= 0 && b >= 0 && part == np - 1 && ctx_raw > 0) {
      const int32_t j = (ctx_raw - 1) / kBlockTokens;
      tail = append_slot(j < a.max_blocks ? a.table[(size_t)b * a.max_blocks + j] : -1, map, a.n_handles, a.n_gpu_blocks,
                         a.n_slots, a.append, tid == 0, a.err);
    }
  }
  if (b >= 0) {
    const int32_t jb0 = tok0 / kBlockTokens;
    const int32_t jb1 = tok1 > 0 ? (tok1 + kBlockTokens - 1) / kBlockTokens : 0;
    const int32_t n_it = (jb1 - jb0 - wave + NW - 1) / NW;  // blocks of this wave: jb0 + wave + NW * it; <= 64
    const size_t row0 = (size_t)b * a.n_q_heads + (size_t)g * G;

    if (WHOLE)
      slots = lane < n_it ? check_slot(handle, slots, a.n_handles, a.n_gpu_blocks, a.n_slots, a.stage_valid != 0, a.err) : -1;
    else if (!SLOTS && lane < n_it)               // (with SLOTS the lanes beyond n_it hold what nobody uses)
      slots = resolve_slot(a.table[(size_t)b * a.max_blocks + jb0 + wave + NW * lane], map, a.n_handles, a.n_gpu_blocks,
                           a.n_slots, a.stage_valid != 0, a.err);
    W w;
    w.load_q(q_in, row0, G, lane, a.scale_log2e);
    w.reset();
    uint4 kr[NL], vr[NL];
    auto load_tile = [&](uint4 (&kr)[NL], uint4 (&vr)[NL], int32_t it) {
      int32_t slot = __builtin_amdgcn_readlane(slots, it);
      slot = slot < 0 ? 0 : slot;                 // flagged blocks are masked when consumed
      const char* kp = kv_layer + (size_t)slot * a.block_bytes + (size_t)g * TILE_BYTES + (size_t)lane * 16;
#pragma unroll
      for (int i = 0; i < NL; ++i) kr[i] = nt_load16(kp + (size_t)i * 1024);
#pragma unroll
      for (int i = 0; i < NL; ++i) vr[i] = nt_load16(kp + a.block_bytes / 2 + (size_t)i * 1024);
      if (EB == 2) __builtin_amdgcn_sched_barrier(0);   // (or the value loads sink below the keys' products)
    };
    auto consume = [&](uint4 (&kr)[NL], uint4 (&vr)[NL], int32_t it) {
      const bool present = __builtin_amdgcn_readlane(slots, it) >= 0;
      w.block(kr, vr, (jb0 + wave + NW * it) * kBlockTokens, present ? tok1 : 0, lane, a.scale_log2e);
    };
    // One block of a wave in flight, all of it requested before any of it is waited for, or two (direct_two_blocks).  (Keys,
    // then values when the keys are there: 16 layers of 256 sequences 3 505 us and not 3 340, 32 of eight 182 and not 162.)
    // fp32, on the vector ALU, has two (6 sequences of 100 to 4 000 tokens, 8 heads of 128: 23.7 and, with one, 24.3).
    if constexpr (!TWO) {
      for (int32_t it = 0; it < n_it; ++it) {
        load_tile(kr, vr, it);
        consume(kr, vr, it);
      }
    } else {
      uint4 kB[NL], vB[NL];
      if (n_it > 0) load_tile(kr, vr, 0);
      for (int32_t it = 0; it < n_it; it += 2) {
        if (it + 1 < n_it) load_tile(kB, vB, it + 1);
        consume(kr, vr, it);
        if (it + 1 < n_it) {
          if (it + 2 < n_it) load_tile(kr, vr, it + 2);
          consume(kB, vB, it + 1);
        }
      }
    }
    if (LEAVES && g == 0)
      a.plan[(size_t)at * kPlanInts + kPlanRec + wave * kDirectMaxQuanta + lane] = slots;
    // The last arrival leaves its word zero.  What calls that must not overlap have left in it is the number of a launch
    // that was enqueued before this one: every workgroup puts this launch's in its place before it counts itself.  With
    // few parts right before (the accesses to a word are served one after another, 10 ns each), with many here, before the
    // waves' states are merged (the wave's wait for its stores covers it).
    uint64_t* word = a.arrive + ((size_t)(layer / kArriveStride) * a.arrive_lines + (size_t)b * H + g) * kArriveStride +
                     layer % kArriveStride;
    if (!WHOLE && np > kEarlyParts && wave == NW - 1 && lane == 0)
      (void)__hip_atomic_fetch_max(word, a.launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool stores = a.append >= 0 && tail >= 0;
    uint4 k_piece;
    uint32_t v_el = 0;
    if (stores) {
      const size_t row = ((size_t)b * H + g) * HD * EB;
      if (tid < HD * EB / 16) k_piece = *reinterpret_cast<const uint4*>(new_k + row + (size_t)tid * 16);
      if (tid < HD) v_el = EB == 2 ? *reinterpret_cast<const uint16_t*>(new_v + row + (size_t)tid * 2)
                                   : *reinterpret_cast<const uint32_t*>(new_v + row + (size_t)tid * 4);
    }
    w.to_lds(s_m, s_l, s_acc, ROW, wave, G, lane);
    if (stores) {                                 // rows at or beyond tok1 are masked by index wherever they are read
      char* blk = const_cast<char*>(kv_layer) + (size_t)tail * a.block_bytes + (size_t)g * TILE_BYTES;
      const int32_t t = (ctx_raw - 1) % kBlockTokens, v = 16 / EB;
      if (tid < HD * EB / 16) *reinterpret_cast<uint4*>(blk + (size_t)k_tile_index(t, tid * v, v) * EB) = k_piece;
      if (tid < HD) {
        char* dst = blk + a.block_bytes / 2 + (size_t)v_tile_index(t, tid, v) * EB;
        if (EB == 2) *reinterpret_cast<uint16_t*>(dst) = (uint16_t)v_el;
        else *reinterpret_cast<uint32_t*>(dst) = v_el;
      }
    }
    __syncthreads();

    // thread t has head t / TPH, dims 4 (t % TPH) ..
    const int32_t cols = G * TPH;
    // The newest token's part is (q . k, 1, v).  Its rows are read here, for the thread's first column, so that they
    // have arrived when the last step needs them.
    const bool add_new = new_k && ctx_raw > 0;
    const size_t kv_row = ((size_t)b * H + g) * HD;
    float4 qd, kd, vd;
    auto read_new = [&](int c) {
      const int d0 = 4 * (c % TPH);
      qd = load_elem4<E>(q_in, (row0 + c / TPH) * HD + d0);
      kd = load_elem4<E>(new_k, kv_row + d0);
      vd = load_elem4<E>(new_v, kv_row + d0);
    };
    if (add_new && tid < cols) read_new(tid);
    auto finish = [&](int c, float M, float L, float4 A) {
      const int d0 = 4 * (c % TPH);
      const size_t row = row0 + c / TPH;
      if (add_new) {
        if (c >= NT) read_new(c);
        add_newest<TPH>(qd, kd, vd, a.scale_log2e, M, L, A);
      }
      const bool some = L > 0.f;
      store_elem2<E>(out, row * HD + d0, make_float2(some ? A.x / L : 0.f, some ? A.y / L : 0.f));
      store_elem2<E>(out, row * HD + d0 + 2, make_float2(some ? A.z / L : 0.f, some ? A.w / L : 0.f));
    };
    const __amdgpu_buffer_rsrc_t parts = parts_rsrc(a.ws + (size_t)layer * (a.ws_bytes / 4), a.ws_bytes);
    for (int c = tid; c < cols; c += NT) {
      const int h = c / TPH, d0 = 4 * (c % TPH);
      float M, L;
      float4 A;
      merge_states<ROW>(s_m, s_l, s_acc, G, NW, h, d0, M, L, A);
      if (WHOLE || np == 1) {
        finish(c, M, L, A);
      } else {
        const int32_t off = (((first + part) * H + g) * G + h) * PART;
        put4(parts, off + d0 * 4, A);
        if (d0 == 0) put2(parts, off + HD * 4, M, L);
      }
    }
    if (!WHOLE && np > 1) {
      wait_stores();
      __syncthreads();
      if (tid == 0) {
        if (np <= kEarlyParts) (void)__hip_atomic_fetch_max(word, a.launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = __hip_atomic_fetch_add(word, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                 a.launch + (uint64_t)(np - 1);
      }
      __syncthreads();
      if (s_last) {                               // every part is stored: merge them, in order
        if (tid == 0) __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // TPH parts at a time, sixteen loads in flight, the weights fetched from LDS.  With few heads and many parts, groups of
        // threads take a share of the parts each and meet in LDS.
        const int pitch = (cols + 63) & ~63;      // threads of a group: whole waves
        const int nsub = np > 16 ? max(1, NT / pitch) : 1;
        const int sub = nsub > 1 ? wave * 64 / pitch : 0;
        constexpr int UNR = 16;
        const int32_t step = H * G * PART;
        for (int c = tid - sub * pitch; c < cols && sub < nsub; c += NT) {
          const int h = c / TPH, t = c % TPH, d0 = 4 * t;
          const int32_t part0 = ((first * H + g) * G + h) * PART;
          const int32_t s_end = np * (sub + 1) / nsub;
          float M = kNegBig, L = 0.f;
          float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
          for (int32_t s0 = np * sub / nsub; s0 < s_end; s0 += TPH) {
            const int32_t n = min(s_end - s0, TPH);
            float2 ml = make_float2(kNegBig, 0.f);
            if (t < n) ml = get2(parts, part0 + (s0 + t) * step + HD * 4);
            for (int32_t u0 = 0; u0 < n; u0 += UNR) {
              float4 ai[UNR];
#pragma unroll
              for (int u = 0; u < UNR; ++u) ai[u] = get4(parts, part0 + d0 * 4, (s0 + min(u0 + u, n - 1)) * step);
              if (u0 == 0) {
                s_w[tid] = weigh_parts<TPH>(ml, t < n, M, L, A);   // read by this wave only
                __builtin_amdgcn_wave_barrier();
              }
              sum_parts<UNR>(&s_w[(tid & ~(TPH - 1)) + u0], ai, A);   // (TPH is a multiple of UNR)
            }
          }
          sum_again_if_infinite(parts, part0, step, HD * 4, d0, np * sub / nsub, s_end, M, A);
          if (nsub == 1) {
            finish(c, M, L, A);
          } else {
            if (d0 == 0) {
              s_m[sub * kMaxGroup + h] = M;
              s_l[sub * kMaxGroup + h] = L;
            }
            *reinterpret_cast<float4*>(&s_acc[((size_t)sub * G + h) * ROW + d0]) = A;
          }
        }
        if (nsub > 1) {
          __syncthreads();
          if (tid < cols) {
            const int h = tid / TPH, d0 = 4 * (tid % TPH);
            float M, L;
            float4 A;
            merge_states<ROW>(s_m, s_l, s_acc, G, nsub, h, d0, M, L, A);
            finish(tid, M, L, A);
          }
        }
      }
    }
  }
  if (LEAVES && g == 0 && tid < kPlanRec) {
    const int32_t rec[kPlanRec] = {b, tok0, tok1, np, first, part, tail, ctx_raw};
    int32_t x = rec[0];
#pragma unroll
    for (int i = 1; i < kPlanRec; ++i) x = tid == i ? rec[i] : x;
    a.plan[(size_t)at * kPlanInts + tid] = x;
  }
  if (WHOLE && lead && a.hdr) {                   // (ahead of the rest the code alone cost every workgroup: 137 of 61
    // tokens, 12 heads of 64, 8.8 us and not 7.9)
    int32_t c4[kDirectLaneSeqs] = {};
    if (a.min_units > 0) {                        // (many heads of 64: else the rule's smallest size is its choice)
#pragma unroll
      for (int i = 0; i < kDirectLaneSeqs; ++i)
        if (64 * i + lane < a.batch) c4[i] = max(0, clamp_ctx(a.ctx[64 * i + lane], a.max_blocks) - a.minus);
    }
    note_item_size(a, c4);
  }
  if (a.clock && tid == 0) {
    const int32_t wg = place * H + g;              // (a launch that notes its times has one layer)
    a.clock_wg[2 * wg] = t_start;
    a.clock_wg[2 * wg + 1] = wall_clock64();
    if (wg == 0) a.clock[kClockGrid] = gridDim.x * gridDim.z;
  }
}

// ---- layers that share a launch, four kv heads side by side -------------------------------------------------
// The same parts, states and sums as k_attn_direct's, with the work dealt out otherwise.  There a workgroup's four waves take the
// four shares of one head's part, and three workgroups a compute unit keep 96 KB in flight that lie 4 KB here and 4 KB there.
// HBM bounds both, and gives more when less is asked for at a time and what is asked for lies together: reads alone, of 4 KB
// tiles of blocks of 64 KB, 6.82 TB/s so and 7.24 with four waves a compute unit on four neighbouring heads of one block; of
// blocks of 256 KB 6.68 and 6.91.  So a workgroup stays on a compute unit and takes units by ticket, the largest parts first, of
// four heads each: a wave a head, which takes the four shares one after another.  A block's eight loads go out together behind
// the block before (the keys' behind its keys' product, the values' behind its values': 3 352 us and not 3 093 for 16 layers of
// 256 sequences of 128 to 4 096 tokens, 32 heads over 8).
//
// With one wave in flight a SIMD nothing may come between two blocks.  What a unit needs beyond them is asked for a unit ahead;
// and what is left to do when its blocks have been read - the merge of the shares, and, where the context is cut, the part's
// stores, the count and the merge of the parts, 5 us in all - is another four waves', out of LDS, one half of which the first
// four fill while the others work on what the other half holds.  us a step, launches of k_attn_direct, the reading waves doing
// all of it, and so: the above 3 330, 3 079, 3 075 (21.5 GB, 7.0 TB/s); 8 layers of 120 of 500 to 2 500, 32 over 8, 937, 900,
// 889; 32 of 8 of 128 to 4 096 162, 180, 162; 16 of 24 of 100 to 1 100, 32 heads, 525, 518, 518.
struct PartOf { int32_t b, g, layer, np, first, part, ctx_raw; };

// What k_attn_direct's workgroup does when its waves have streamed their shares of a part, by one wave for a kv head: the four
// states in LDS become one; a lone part's is finished, another's stored, counted and, by the last to arrive, merged with the
// others'.
template <typename W>
struct PartEnd {
  using E = typename W::E;
  static constexpr int HD = W::HD;
  static constexpr int NW = kWaves, NT = 64;
  static constexpr int ROW = HD + 4;
  static constexpr int TPH = HD / 4;              // threads per head when states are merged, four dims each
  static constexpr int PART = (HD + 4) * 4;       // bytes of a head's partial state: accumulator, max, sum, padding
  const DirectArgs& a;
  PartOf p;
  float *s_m, *s_l, *s_acc, *s_w;                 // s_w: 2 NT floats
  int tid;
  uint64_t* word;                                 // its pair's arrival word
  __amdgpu_buffer_rsrc_t ws;                      // the layer's parts
  size_t row0;                                    // first row among the queries and results
  float4 qd, kd, vd;                              // the newest token's part is (q . k, 1, v)

  __device__ __forceinline__ PartEnd(const DirectArgs& a_, const PartOf& p_, float* s_state, float* s_weights, int thread)
      : a(a_), p(p_), s_m(s_state), s_l(s_state + NW * kMaxGroup), s_acc(s_state + 2 * NW * kMaxGroup), s_w(s_weights),
        tid(thread), word(a_.arrive + arrive_word(a_.arrive_lines, p_.layer, (size_t)p_.b * a_.n_kv_heads + p_.g)),
        ws(parts_rsrc(a_.ws + (size_t)p_.layer * (a_.ws_bytes / 4), a_.ws_bytes)),
        row0((size_t)p_.b * a_.n_q_heads + (size_t)p_.g * a_.group) {}
  __device__ __forceinline__ static void sync() {   // what its threads have left in LDS can be read
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // thread t has head t / TPH, dims 4 (t % TPH) ..
  __device__ __forceinline__ int cols() const { return a.group * TPH; }
  __device__ __forceinline__ bool add_new() const { return a.new_k && p.ctx_raw > 0; }
  // The newest token's rows are read here, for the thread's first column, so that they have arrived when the last step needs
  // them.
  __device__ __forceinline__ void read_q(int c) { qd = load_elem4<E>(a.q + p.layer * a.q_stride, (row0 + c / TPH) * HD + 4 * (c % TPH)); }
  __device__ __forceinline__ void read_new() {
    if (!add_new() || tid >= cols()) return;
    const size_t at = ((size_t)p.b * a.n_kv_heads + p.g) * HD + 4 * (tid % TPH);
    read_q(tid);
    kd = load_elem4<E>(a.new_k + p.layer * a.new_stride, at);   // (NT is a multiple of TPH: the same dims in all columns)
    vd = load_elem4<E>(a.new_v + p.layer * a.new_stride, at);
  }
  __device__ __forceinline__ void finish(int c, float M, float L, float4 A) {   // a column
    const int d0 = 4 * (c % TPH);
    const size_t row = row0 + c / TPH;
    if (add_new()) {
      if (c >= NT) read_q(c);
      add_newest<TPH>(qd, kd, vd, a.scale_log2e, M, L, A);
    }
    const bool some = L > 0.f;
    char* const out = a.out + p.layer * a.q_stride;
    store_elem2<E>(out, row * HD + d0, make_float2(some ? A.x / L : 0.f, some ? A.y / L : 0.f));
    store_elem2<E>(out, row * HD + d0 + 2, make_float2(some ? A.z / L : 0.f, some ? A.w / L : 0.f));
  }
  __device__ __forceinline__ void merge_lds(int n, int h, int d0, float& M, float& L, float4& A) const {
    merge_states<ROW>(s_m, s_l, s_acc, a.group, n, h, d0, M, L, A);
  }
  // the states into one, which is finished (the newest token's rows have been read) or stored
  __device__ __forceinline__ void leave() {
    for (int c = tid; c < cols(); c += NT) {
      const int h = c / TPH, d0 = 4 * (c % TPH);
      float M, L;
      float4 A;
      merge_lds(NW, h, d0, M, L, A);
      if (p.np == 1) {
        finish(c, M, L, A);
      } else {
        const int32_t off = (((p.first + p.part) * a.n_kv_heads + p.g) * a.group + h) * PART;
        put4(ws, off + d0 * 4, A);
        if (d0 == 0) put2(ws, off + HD * 4, M, L);
      }
    }
  }
  // One more part stored, the word having been cleared ahead of the launch; the last arrival leaves it zero again.
  __device__ __forceinline__ uint32_t count() const { return add_one(word, tid); }
  __device__ __forceinline__ bool is_last(uint32_t counted) const {
    return __builtin_amdgcn_readfirstlane(counted) == (uint32_t)(p.np - 1);
  }
  // NC columns of a thread from c0 on, of the parts [s_begin, s_end), UNR parts' loads in flight for each column, the weights
  // fetched from LDS.  sub: whose group's result it is, or -1: the only one's.
  template <int NC, int UNR>
  __device__ __forceinline__ void merge_columns(int sub, int32_t s_begin, int32_t s_end, int c0) {
    const int32_t G = a.group, H = a.n_kv_heads, step = H * G * PART;
    const int t = c0 % TPH, d0 = 4 * t;
    int32_t part0[NC];
    float M[NC], L[NC];
    float4 A[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int c = NC == 1 ? c0 : min(c0 + NT * j, cols() - TPH + t);
      part0[j] = ((p.first * H + p.g) * G + c / TPH) * PART;
      M[j] = kNegBig;
      L[j] = 0.f;
      A[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int32_t s0 = s_begin; s0 < s_end; s0 += TPH) {
      const int32_t n = min(s_end - s0, TPH);
      float2 ml[NC];
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        ml[j] = make_float2(kNegBig, 0.f);
        if (t < n) ml[j] = get2(ws, part0[j] + (s0 + t) * step + HD * 4);
      }
      for (int32_t u0 = 0; u0 < n; u0 += UNR) {
        float4 ai[NC][UNR];
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
          for (int u = 0; u < UNR; ++u) ai[j][u] = get4(ws, part0[j] + d0 * 4, (s0 + min(u0 + u, n - 1)) * step);
        if (u0 == 0) {
#pragma unroll
          for (int j = 0; j < NC; ++j) s_w[j * NT + tid] = weigh_parts<TPH>(ml[j], t < n, M[j], L[j], A[j]);   // read by this wave only
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) sum_parts<UNR>(&s_w[j * NT + (tid & ~(TPH - 1)) + u0], ai[j], A[j]);   // (TPH is a multiple of UNR)
      }
    }
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      sum_again_if_infinite(ws, part0[j], step, HD * 4, d0, s_begin, s_end, M[j], A[j]);
      const int c = c0 + NT * j, h = c / TPH;
      if (NC > 1 && c >= cols()) continue;
      if (sub < 0) {
        finish(c, M[j], L[j], A[j]);
      } else {
        if (d0 == 0) {
          s_m[sub * kMaxGroup + h] = M[j];
          s_l[sub * kMaxGroup + h] = L[j];
        }
        *reinterpret_cast<float4*>(&s_acc[((size_t)sub * G + h) * ROW + d0]) = A[j];
      }
    }
  }
  // By the last to arrive: every part is stored; merge them, in order, in as many groups as a workgroup's threads would make.
  __device__ __forceinline__ void merge() {
    if (tid == 0) __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int32_t np = p.np;
    const int pitch = (cols() + 63) & ~63;        // threads of a group: whole waves
    const int nsub = np > 16 ? max(1, NW * 64 / pitch) : 1;
    auto merge_share = [&](int sub, int from) {
      const int32_t s_begin = np * sub / nsub, s_end = np * (sub + 1) / nsub;
      if (np <= 8) {                              // few parts: no more loads than there are, and two columns' at a time
        for (int c = from; c < cols(); c += 2 * NT) merge_columns<2, 8>(-1, s_begin, s_end, c);
        return;
      }
      for (int c = from; c < cols(); c += NT) merge_columns<1, 16>(nsub > 1 ? sub : -1, s_begin, s_end, c);
    };
    for (int sub = 0; sub < nsub; ++sub) merge_share(sub, tid);   // one group's share after another
    if (nsub > 1) {
      sync();
      for (int c = tid; c < cols(); c += NT) {
        const int d0 = 4 * (c % TPH);
        float M, L;
        float4 A;
        merge_lds(nsub, c / TPH, d0, M, L, A);
        finish(c, M, L, A);
      }
    }
  }
};

// Where k_step_begin has left the parts.  SLOTS: with their slots; else, every layer having a map of its own, with handles.
template <bool SLOTS>
struct StepParts {
  const DirectArgs& a;
  __device__ __forceinline__ void fetch(const WideUnit& u, int lane, WideMeta& x) const {
    const int32_t* rec = a.plan + (size_t)(u.place < 0 ? 0 : u.place) * kPlanInts;
    x.rec = rec[lane & (kPlanRec - 1)];
#pragma unroll
    for (int s = 0; s < kWaves; ++s) x.slots[s] = rec[kPlanRec + s * kDirectMaxQuanta + lane];
  }
  __device__ __forceinline__ void read(WideUnit& u, const WideMeta& x) const {
    u.b = __builtin_amdgcn_readlane(x.rec, 0);
    u.tok0 = __builtin_amdgcn_readlane(x.rec, 1);
    u.tok1 = __builtin_amdgcn_readlane(x.rec, 2);
    u.np = __builtin_amdgcn_readlane(x.rec, 3);
    u.first = __builtin_amdgcn_readlane(x.rec, 4);
    u.part = __builtin_amdgcn_readlane(x.rec, 5);
    u.ctx_raw = __builtin_amdgcn_readlane(x.rec, 7);
  }
  __device__ __forceinline__ void look_up(const WideUnit& u, const WideMeta& x, int32_t (&found)[kWaves]) const {
    if constexpr (!SLOTS) {
      const int32_t* map = a.map + (size_t)u.layer * a.map_stride;
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int s = 0; s < kWaves; ++s) {
        const bool live = u.b >= 0 && lane < share_blocks(u, s) && x.slots[s] >= 0 && x.slots[s] < a.n_handles;
        found[s] = map[live ? x.slots[s] : 0];
      }
    }
  }
  __device__ __forceinline__ void found_out(const WideUnit& u, WideMeta& x, const int32_t (&found)[kWaves]) const {
    if constexpr (!SLOTS) {
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int s = 0; s < kWaves; ++s)
        x.slots[s] = u.b >= 0 && lane < share_blocks(u, s)
                         ? check_slot(x.slots[s], found[s], a.n_handles, a.n_gpu_blocks, a.n_slots, a.stage_valid != 0, a.err)
                         : -1;
    }
  }
};

template <typename W, bool SLOTS>
__global__ __launch_bounds__((kWideHeads + kFinishers) * 64) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_attn_direct_wide(const DirectArgs a) {
  using End = PartEnd<W>;
  extern __shared__ __align__(16) float s_dyn[];
  __shared__ __align__(16) float s_wts[kFinishers * 128];   // weights of parts being merged, of two columns a lane
  __shared__ WideLds lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= kWideHeads) {                       // finishes, a head
    const int w = wave - kWideHeads;
    wide_finish(lds, [&](int half, int32_t x, int thread) {
      PartOf p;
      p.b = __builtin_amdgcn_readlane(x, 0);
      p.g = __builtin_amdgcn_readlane(x, 1) + w;
      p.layer = __builtin_amdgcn_readlane(x, 2);
      p.np = __builtin_amdgcn_readlane(x, 3);
      p.first = __builtin_amdgcn_readlane(x, 4);
      p.part = __builtin_amdgcn_readlane(x, 5);
      p.ctx_raw = __builtin_amdgcn_readlane(x, 6);
      End end(a, p, s_dyn + (half * kWideHeads + w) * wide_head_floats(W::HD, a.group), s_wts + w * 128, thread);
      if (p.np == 1) end.read_new();
      end.leave();
      if (p.np > 1) {
        wait_stores();
        if (end.is_last(end.count())) {
          end.read_new();
          End::sync();
          end.merge();
        }
      }
    });
    return;
  }
  wide_read<W, kWideHeads>({a.kv_layer, a.q, a.counter, a.block_bytes, a.kv_stride, a.q_stride, a.scale_log2e, a.n_kv_heads, a.group,
                a.n_layers, a.places},
               StepParts<SLOTS>{a}, s_dyn, lds);
}

// ---- dispatch --------------------------------------------------------------------------------------------

// Its scratch in a pool: the parts, then the items' records and slot lists of the two staging regions, for as many units
// as the pool's largest batch and widest table can make (a call's own scratch has room for any).
static size_t parts_floats(const pie_config& c) { return direct_step_rows(c) * (c.head_dim + 4); }
static size_t plan_region_ints(const pie_config& c) { return direct_pool_items(c) * kPlanInts; }
size_t attn_arrive_lines(const pie_config& c) { return direct_arrive_lines(c); }
size_t attn_direct_floats(const pie_config& c) { return parts_floats(c) + 2 * plan_region_ints(c); }

// How many units the split of a call may make; 0: the call is left to the planned path, which has what this one lacks -
// an item size set by the caller, the vector-ALU variant, fp32 with grouped queries (every query head reads the keys
// and values again: many small items share them in the caches, 80 us against 95 to 104 for six sequences of 100 to
// 4 000 tokens, 32 heads over 8), more sequences than the in-kernel split covers - or for which the units do not fit.
static int32_t direct_max_units(const pie_pool* p, int32_t batch, int32_t max_blocks) {
  const pie_config& c = p->cfg;
  const int32_t group = c.n_q_heads / c.n_kv_heads;
  if (p->attn_partition > 0 || p->attn_valu || (c.dtype == PIE_DTYPE_F32 && group > 1)) return 0;
  return direct_units(p->n_cu, c.n_kv_heads, group, batch, max_blocks);
}

bool attn_direct(const pie_pool* p, int32_t batch, int32_t max_blocks) { return direct_max_units(p, batch, max_blocks) > 0; }

// A step's layers.  Without grouped queries, more than three (sequence, kv head) pairs per compute unit over long contexts
// stay planned.  One launch a layer does not pay there (64 sequences of 1 024 to 2 048 tokens, 32 heads, 32 layers, us
// planned and in one launch each: 8 041 and 8 101, apart 8 088 and 8 005, in a first pass 8 148 and 8 267, with host blocks
// 8 155 and 8 329; 40 of 300 to 1 700, 40 heads, 32 layers 4 624 and 4 644), and fewer, longer parts have fewer weights of
// exactly one, so that rounding the weights to f16 costs more (2.24e-4 from 64 bits against 2.19e-4).  With grouped queries it
// gains from about 8 layers on (256 sequences of 128 to 4 096 tokens, 32 heads over 8: 8 layers 1 776 and 1 752, 16 layers 3 614
// and 3 517; with host blocks, 0.5 %, 16 layers 3 631 and 3 585, 32 layers 7 100 and 7 098).
//
// Layers that share launches have the rows of all stored by the one ahead of them.  What they cost is the lines they touch, 24
// a pair, each of them 110 to 250 ps of memory time, more the more they come among reads: us a step with them in every
// layer's part of the launch, in a launch beside it on another stream, and ahead of it (without any): 16 layers of 24
// sequences of 100 to 1 100 tokens, 32 heads 569, 563 and 527 (490); 16 of 256 of 128 to 4 096, 32 over 8 3 518, 3 390 and
// 3 383 (3 303); 8 of 60 of 60 to 300, 32 over 8 296, 307 and 292 (259); 8 of 30 of 60 to 300, 32 heads 168, 181 and 171
// (144).  Stored as whole lines, what else is in them read first, they cost the same.  Layers in a launch each store theirs
// there or have them stored ahead (step_body has the rule, with times); layers that move store their rows a layer at a time:
// in its launch, or in big steps (kStepDirectAppendApart) ahead of it, 8 layers as above with grouping 1 808 and 1 785 us
// planned and so, 16 layers 3 703 and 3 580, 32 layers 7 169 and 7 094.
int attn_step_path(const pie_pool* p, int32_t n_layers, int32_t batch, int32_t max_blocks) {
  if (!attn_direct(p, batch, max_blocks)) return kStepPlanned;
  const int64_t pairs = (int64_t)batch * p->cfg.n_kv_heads;
  if (pairs <= 3 * (int64_t)p->n_cu || pairs * max_blocks * kBlockTokens <= (int64_t)8192 * p->n_cu) return kStepDirect;
  return p->cfg.n_q_heads > p->cfg.n_kv_heads && n_layers >= 8 ? kStepDirectAppendApart : kStepPlanned;
}

bool attn_whole(const pie_pool* p, int32_t batch, int32_t max_blocks, int32_t layers) {
  return attn_direct(p, batch, max_blocks) && direct_whole(p->n_cu, (int64_t)batch * p->cfg.n_kv_heads, layers, max_blocks,
                                                           p->block_bytes / p->cfg.n_kv_heads);
}

// How many layers of a step one launch may take: as many as the pool has room for parts of.
int32_t attn_step_layers(const pie_pool* p, int32_t batch, int32_t max_blocks, bool whole) {
  const pie_config& c = p->cfg;
  if (whole) return c.n_layers;                   // (no parts)
  const int32_t units = direct_max_units(p, batch, max_blocks);
  return units > 0 ? direct_step_layers(c, units, batch, max_blocks) : 0;
}

// Whether so many layers of a step share a launch of k_attn_direct_wide.
bool attn_wide(const pie_pool* p, int32_t batch, int32_t max_blocks, int32_t layers) {
  const pie_config& c = p->cfg;
  const int32_t units = direct_max_units(p, batch, max_blocks), H = c.n_kv_heads;
  return units > 0 && direct_wide(p->n_cu, H, c.n_q_heads / H, c.head_dim, p->elem_bytes, layers,
                                  direct_grid(units, H, batch, max_blocks) / H, max_blocks);
}

// A launch in a graph has the same number in every replay, so there the words it uses are cleared ahead of it.
__global__ __launch_bounds__(256) void k_arrive_clear(uint64_t* __restrict__ words, int32_t n) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < n) words[i] = 0;
}

template <typename W, int NW, int PLAN, bool TWO, int SEQS = kDirectLaneSeqs>
static int launch_direct_as(const DirectArgs& a, dim3 grid, hipStream_t s, hipEvent_t done, size_t min_lds) {
  size_t lds = ((size_t)NW * 2 * kMaxGroup + (size_t)NW * a.group * (W::HD + 4)) * sizeof(float);
  if (lds < min_lds) lds = min_lds;
  if (done) hipExtLaunchKernelGGL((k_attn_direct<W, NW, PLAN, TWO, SEQS>), grid, dim3(NW * 64), (uint32_t)lds, s, nullptr, done, 0, a);
  else hipLaunchKernelGGL((k_attn_direct<W, NW, PLAN, TWO, SEQS>), grid, dim3(NW * 64), (uint32_t)lds, s, a);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}

template <typename W, bool SLOTS>
static int launch_wide(const pie_pool* p, const DirectArgs& a, hipStream_t s, hipEvent_t done) {
  const uint32_t lds = (uint32_t)wide_lds(kWideHeads, a.group, W::HD);
  const dim3 grid(p->n_cu), block((kWideHeads + kFinishers) * 64);
  if (done) hipExtLaunchKernelGGL((k_attn_direct_wide<W, SLOTS>), grid, block, lds, s, nullptr, done, 0, a);
  else hipLaunchKernelGGL((k_attn_direct_wide<W, SLOTS>), grid, block, lds, s, a);
  PIE_HIP(hipGetLastError());
  return PIE_OK;
}
template <typename W>
static int launch_wide(const pie_pool* p, const DirectArgs& a, hipStream_t s, hipEvent_t done, int32_t plan) {
  return plan == kDirectPlanReplay ? launch_wide<W, true>(p, a, s, done) : launch_wide<W, false>(p, a, s, done);
}

template <typename W, bool TWO>
static int launch_cut(const DirectArgs& a, dim3 grid, hipStream_t s, hipEvent_t done, int32_t plan, size_t min_lds) {
  switch (plan) {
    case kDirectPlanReplay: return launch_direct_as<W, kWaves, kDirectPlanReplay, TWO>(a, grid, s, done, min_lds);
    case kDirectPlanReplaySplit: return launch_direct_as<W, kWaves, kDirectPlanReplaySplit, TWO>(a, grid, s, done, min_lds);
    case kDirectPlanWrite: return launch_direct_as<W, kWaves, kDirectPlanWrite, TWO>(a, grid, s, done, min_lds);
    default:
      return a.batch <= 64 ? launch_direct_as<W, kWaves, kDirectPlanNone, TWO, 1>(a, grid, s, done, min_lds)
                           : launch_direct_as<W, kWaves, kDirectPlanNone, TWO>(a, grid, s, done, min_lds);
  }
}

static int32_t* plan_region(const pie_pool* p, int region) {
  return reinterpret_cast<int32_t*>(p->d_ws + parts_floats(p->cfg)) + region * plan_region_ints(p->cfg);
}

static void fill_split(const pie_pool* p, const int32_t* d_ctx, int32_t batch, int32_t max_blocks, int32_t max_units,
                       bool without_last, SplitIn* a) {
  const int32_t H = p->cfg.n_kv_heads;
  a->ctx = d_ctx;
  a->err = p->d_err;
  a->hdr = p->d_plan;
  a->batch = batch;
  a->max_blocks = max_blocks;
  a->n_kv_heads = H;
  a->minus = without_last ? 1 : 0;
  const int64_t second = ((int64_t)max_blocks * kBlockTokens + auto_part(1) - 1) / auto_part(1);
  a->min_units = batch * second * H > attn_min_units(p) ? attn_min_units(p) : 0;
  a->max_items = max_units / H;
}

int launch_step_begin(const pie_pool* p, const int32_t* d_table, int32_t max_blocks, const int32_t* d_ctx, int32_t batch,
                      bool stage_valid, bool without_last, int32_t append, int32_t regions, hipStream_t s,
                      const AppendArgs* rows, int32_t n_layers) {
  const pie_config& c = p->cfg;
  const int32_t H = c.n_kv_heads, max_units = direct_max_units(p, batch, max_blocks);
  if (max_units <= 0 || regions < 0 || regions > 2) return PIE_EINVAL;
  SplitArgs a = {};
  fill_split(p, d_ctx, batch, max_blocks, max_units, without_last, &a);
  a.table = d_table;
  for (int r = 0; r < 2; ++r) {
    a.map[r] = r < regions ? p->d_map[r] : nullptr;
    a.plan[r] = r < (regions ? regions : 1) ? plan_region(p, r) : nullptr;
  }
  a.n_handles = p->n_handles;
  a.n_gpu_blocks = c.n_gpu_blocks;
  a.n_slots = c.n_gpu_blocks + 2 * c.n_stage_blocks;
  a.stage_valid = stage_valid ? 1 : 0;
  a.append = append;
  a.places = direct_grid(max_units, H, batch, max_blocks) / H;
  const int32_t most = attn_step_layers(p, batch, max_blocks, false), together = n_layers < most ? n_layers : most;
  const bool wide = regions < 2 && attn_wide(p, batch, max_blocks, together);
  if (wide) {
    a.counters = reinterpret_cast<uint32_t*>(p->d_plan + kPlanHdrInts);
    a.n_counters = c.n_layers;
    a.arrive = p->d_arrive;
    a.arrive_lines = (int32_t)direct_pool_words(c);
    a.n_layers = together;
  }
  const int64_t grid = a.places + (rows ? (int64_t)batch * n_layers : 0);
  if (grid > INT32_MAX) return PIE_EINVAL;
  hipLaunchKernelGGL(k_step_begin, dim3((uint32_t)grid), dim3(kWaves * 64), 0, s, a, rows ? *rows : AppendArgs{});
  PIE_HIP(hipGetLastError());
  p->step_plan = StepPlan{};
  for (int r = 0; r < 2; ++r)
    if (a.plan[r]) p->step_plan.add(batch, max_blocks, without_last, r, a.map[r] != nullptr, append);
  p->step_plan.shared = wide ? together : 0;
  return PIE_OK;
}

// CUT, WHOLE: one wave's share of a part, and of a context that is not cut
template <typename CUT, typename WHOLE>
static int launch_direct(const DirectArgs& a, dim3 grid, dim3 pairs, hipStream_t s, hipEvent_t done, int32_t plan, size_t min_lds,
                         bool two) {
  // (fp32 with 128 dims: two blocks of 16 KB a wave leave a compute unit registers for one workgroup.  us a call with two and
  // with one, and cut: 20 sequences of 256 tokens, 32 heads, 30.8 26.7 28.3; of 128 18.1 14.7 16.3; one of 256, 2 heads, 6.0
  // 5.8 6.8)
  if (plan == kDirectWhole)
    return launch_direct_as<WHOLE, kWholeWaves, kDirectPlanNone, WHOLE::EB == 4 && WHOLE::HD == 64>(a, pairs, s, done, min_lds);
  if constexpr (CUT::EB == 2 && CUT::HD == 128)
    if (!two) return launch_cut<CUT, false>(a, grid, s, done, plan, min_lds);
  return launch_cut<CUT, true>(a, grid, s, done, plan, min_lds);
}

int launch_attn_direct(const pie_pool* p, int32_t layer, const void* d_q, const int32_t* d_table, int32_t max_blocks,
                       const int32_t* d_ctx, int32_t batch, void* d_out, bool stage_valid, hipStream_t s,
                       const void* d_k_new, const void* d_v_new, int32_t append, const LayerView* view,
                       const AttnWork* work, hipEvent_t k_start, hipEvent_t k_end, unsigned long long* clock_row,
                       hipEvent_t done, int32_t plan, bool leave_room, int32_t n_layers, int32_t region) {
  // How many workgroups a compute unit holds, by the LDS they ask for: three, where head_dim 128 in 16 bits leaves registers
  // for four (16 layers as above 3 392 us with four, 3 340 with three; it is 3 300 with two, but 32 layers of eight sequences
  // take 170 then and not 162, and the lengths are not known here).  Two where a gather beside them needs room to start
  // before one ends (step_body says when that pays, with the times).
  const bool wide16 = p->cfg.head_dim == 128 && p->cfg.dtype != PIE_DTYPE_F32;
  const size_t min_lds = leave_room ? (size_t)56 << 10 : wide16 ? (size_t)41 << 10 : 0;
  const bool planned = plan == kDirectPlanReplay || plan == kDirectPlanReplaySplit, leaves = plan == kDirectPlanWrite;
  if ((planned || leaves) && work) return PIE_EINVAL;   // the plan lies in the pool's scratch, by region
  if (leaves && n_layers != 1) return PIE_EINVAL;
  if (region < 0) region = view ? 0 : layer & 1;
  if (region > 1 || (view && region)) return PIE_EINVAL;
  if (planned && !p->step_plan.serves(batch, max_blocks, d_k_new != nullptr, region, plan == kDirectPlanReplay, append))
    return PIE_EINVAL;
  const pie_config& c = p->cfg;
  if (((uintptr_t)d_q | (uintptr_t)d_out) % 16) return PIE_EINVAL;
  if (c.n_gpu_blocks + 2 * c.n_stage_blocks <= 0) return PIE_EINVAL;
  if ((d_k_new == nullptr) != (d_v_new == nullptr)) return PIE_EINVAL;
  if (((uintptr_t)d_k_new | (uintptr_t)d_v_new) % 16) return PIE_EINVAL;
  const int32_t group = c.n_q_heads / c.n_kv_heads, H = c.n_kv_heads, max_units = direct_max_units(p, batch, max_blocks);
  if (max_units <= 0) return PIE_EINVAL;
  const int32_t places = direct_grid(max_units, H, batch, max_blocks) / H;   // the items there may be, at most max_units / H
  const bool whole = plan == kDirectWhole;
  if (n_layers < 1) return PIE_EINVAL;
  if (n_layers > 1 && (work || clock_row || n_layers > attn_step_layers(p, batch, max_blocks, whole))) return PIE_EINVAL;
  if (whole && max_blocks > 64 * kWholeWaves) return PIE_EINVAL;   // (a lane looks up a block of its wave's)
  DirectArgs a;
  a.kv_layer = view ? view->kv_base : p->d_kv + (size_t)layer * p->d_layer_stride;
  a.table = d_table;
  a.map = view ? view->map : p->d_map[region];
  fill_split(p, d_ctx, batch, max_blocks, max_units, d_k_new != nullptr, &a);
  if (work) a.hdr = nullptr;
  a.q = (const char*)d_q;
  a.out = (char*)d_out;
  a.new_k = (const char*)d_k_new;
  a.new_v = (const char*)d_v_new;
  a.ws = work ? reinterpret_cast<float*>(work->plan) : p->d_ws;   // a call's own scratch from its start
  a.arrive = work ? work->arrive : p->d_arrive;
  a.launch = ((work ? work->arrive_launches : &p->arrive_launches)->fetch_add(1, std::memory_order_relaxed) + 1) << kArriveShift;
  a.block_bytes = p->block_bytes;
  a.kv_stride = view ? 0 : p->d_layer_stride;     // (the caches that grow share their memory and have a map each)
  a.map_stride = view ? view->n_handles : 0;
  a.q_stride = (size_t)batch * c.n_q_heads * c.head_dim * p->elem_bytes;
  a.new_stride = (size_t)batch * H * c.head_dim * p->elem_bytes;
  a.ws_bytes = places * c.n_q_heads * (c.head_dim + 4) * (int32_t)sizeof(float);
  a.arrive_lines = work ? kArriveWords : (int32_t)direct_pool_words(c);
  a.plan = planned || leaves ? plan_region(p, region) : nullptr;
  a.scale_log2e = p->scale_log2e;
  a.group = group;
  a.n_q_heads = c.n_q_heads;
  a.n_handles = view ? view->n_handles : p->n_handles;
  a.n_gpu_blocks = view ? view->n_slots : c.n_gpu_blocks;
  a.n_slots = view ? view->n_slots : c.n_gpu_blocks + 2 * c.n_stage_blocks;
  a.stage_valid = stage_valid ? 1 : 0;
  a.append = append;
  const dim3 grid(H, n_layers, places);
  a.n_layers = n_layers;
  a.places = places;
  a.counter = reinterpret_cast<uint32_t*>(p->d_plan + kPlanHdrInts) + layer;   // (a launch a counter: the first layer's)
  // (By the launch's own layers: a step's last one may have too few.  us with both side by side and with the last in k_attn_direct:
  // 24 layers of 39 sequences of up to 1 024 tokens, 32 heads over 8, 20 and 4, 204.9 and 198.2; 16 of 38 of 542, 64 over 8, 10 and
  // 6, 285 and 279; growing caches, 10 of 60 of 122 to 3 912, 64 over 8, 8 and 2, 585 and 575.)
  const bool wide = planned && n_layers > 1 && n_layers <= p->step_plan.shared && layer >= 0 && layer < c.n_layers &&
                    attn_wide(p, batch, max_blocks, n_layers);
  a.clock = clock_row;
  a.clock_wg = nullptr;
  if (clock_row) {                                // (a pair for every workgroup: kDirectMaxUnits <= kClockWgs)
    const size_t row = (size_t)(clock_row - p->d_clock) / kClockRow;
    a.clock_wg = p->d_clock + ((size_t)c.n_layers + 1) * kClockRow + row * kClockWgs * 2;
  }
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
    (void)hipGetLastError();                      // (the default stream beside another's capture: the launch says so)
    capture = hipStreamCaptureStatusNone;
  }
  if (capture == hipStreamCaptureStatusActive) {
    const int32_t n = ((n_layers - 1) / kArriveStride * a.arrive_lines + batch * H) * kArriveStride;
    hipLaunchKernelGGL(k_arrive_clear, dim3((n + 255) / 256), dim3(256), 0, s, a.arrive, n);
    PIE_HIP(hipGetLastError());
  }
  if (wide)
    return c.dtype == PIE_DTYPE_F16 ? launch_wide<Wave16<F16, 128, false>>(p, a, s, done, plan)
                                    : launch_wide<Wave16<BF16, 128, true>>(p, a, s, done, plan);
  if (k_start) PIE_HIP(hipEventRecord(k_start, s));
  int rc = PIE_EINVAL;
  const bool hd128 = c.head_dim == 128;
  const dim3 pairs(H, n_layers, batch);
  const bool two = direct_two_blocks(c.head_dim, (int64_t)H * n_layers * places, p->n_cu, (int64_t)batch * H, H, planned);
  switch (c.dtype) {
    case PIE_DTYPE_F32:
      rc = hd128 ? launch_direct<Wave32<128>, Wave32<128>>(a, grid, pairs, s, done, plan, min_lds, two)
                 : launch_direct<Wave32<64>, Wave32<64>>(a, grid, pairs, s, done, plan, min_lds, two);
      break;
    case PIE_DTYPE_F16:                           // (whole contexts have fewer weights of exactly one: both products there)
      rc = hd128 ? launch_direct<Wave16<F16, 128, false>, Wave16<F16, 128, true>>(a, grid, pairs, s, done, plan, min_lds, two)
                 : launch_direct<Wave16<F16, 64, false>, Wave16<F16, 64, true>>(a, grid, pairs, s, done, plan, min_lds, two);
      break;
    case PIE_DTYPE_BF16:
      rc = hd128 ? launch_direct<Wave16<BF16, 128, true>, Wave16<BF16, 128, true>>(a, grid, pairs, s, done, plan, min_lds, two)
                 : launch_direct<Wave16<BF16, 64, true>, Wave16<BF16, 64, true>>(a, grid, pairs, s, done, plan, min_lds, two);
      break;
  }
  if (rc) return rc;
  if (leaves) p->step_plan.add(batch, max_blocks, d_k_new != nullptr, region, !view, append);
  if (k_end) PIE_HIP(hipEventRecord(k_end, s));
  return PIE_OK;
}

}  // namespace pie
