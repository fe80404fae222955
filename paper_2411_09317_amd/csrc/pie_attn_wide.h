// Reading keys and values several kv heads side by side: what k_attn_direct_wide (four) and k_attn_decode_wide (eight) have in
// common.
//
// A workgroup stays on its compute unit and takes units by ticket: a part of a sequence for that many neighbouring heads.  As
// many waves read, a head each, the four shares of the part that a workgroup's waves would take (blocks s, s + 4, ...) one after
// another, and leave a state of each in LDS; four more finish what those have read (wide_finish), out of one half of the LDS
// while the readers fill the other.  k_attn_direct_wide's comment says why, with what it gives.
#pragma once

#include "pie_attn_device.h"

namespace pie {

constexpr int kFinishers = 4;                    // waves that finish what the others, one a head, have read

struct WideUnit {            // one part of sequence b (b < 0: none), tokens [tok0, tok1), for head g of a launch's layer
  int32_t b, tok0, tok1, np, first, part, ctx_raw, layer, g, place;
};
struct WideMeta {            // a record as fetched, a word to a lane, and the slots (or handles) of the four shares' blocks
  int32_t rec, slots[kWaves];
};
struct WideLds {             // what the waves of a workgroup tell each other
  uint32_t ticket[2];
  int32_t part[2][8];        // what the states in either half are of: b, g of the first wave, layer, np, first, part, ctx_raw
};
struct WideArgs {
  const char* kv_layer;
  const char* q;             // [B][Hq][d], a layer's
  uint32_t* counter;         // tickets, cleared ahead of the launch
  size_t block_bytes, kv_stride, q_stride;
  float scale_log2e;
  int32_t n_kv_heads, group, n_layers, places;    // places: records there may be
};

__device__ __forceinline__ int wide_head_floats(int HD, int G) { return 2 * kWaves * kMaxGroup + kWaves * G * (HD + 4); }

// One more in a word of which the first thread of a wave gets the old value, the others nothing: for the others it lies out of
// the buffer's range, so there is no branch around it and nobody waits for the answer before it is used (an atomic by one
// thread is waited for where the branches meet).
__device__ __forceinline__ uint32_t add_one(void* word, int32_t thread) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(word, 0, 4, 0x00027000);
  return (uint32_t)__builtin_amdgcn_raw_ptr_buffer_atomic_add_i32(1, r, 4 * thread, 0, 0);
}

// By the kFinishers waves behind those that read: finish(half, words of WideLds::part, a lane each, thread) for every unit.
template <typename Finish>
__device__ __forceinline__ void wide_finish(WideLds& lds, Finish finish) {
  int thread = threadIdx.x & 63;
  for (int half = 0;; half ^= 1) {
    __syncthreads();                              // the states are there (and those of the part before have been read)
    asm volatile("" : "+v"(thread));              // (or all addresses are worked out ahead of the loop, and spill)
    const int32_t x = lds.part[half][thread & 7];
    if (__builtin_amdgcn_readlane(x, 0) < 0) return;
    finish(half, x, thread);
  }
}

__device__ __forceinline__ int32_t wide_blocks(const WideUnit& u) {
  return (u.tok1 > 0 ? (u.tok1 + kBlockTokens - 1) / kBlockTokens : 0) - u.tok0 / kBlockTokens;
}
__device__ __forceinline__ int32_t share_blocks(const WideUnit& u, int s) { return (wide_blocks(u) - s + kWaves - 1) / kWaves; }

// By the first HW waves.  Src: where the records and slots of the parts are -
//   fetch(unit, lane, meta)      asks for those of unit.place (any, if that is < 0)
//   read(unit, meta)             the unit from the record, once it has arrived
//   look_up, found_out           a second access, where the slots fetched are handles: asked for, and arrived
template <typename W, int HW, typename Src>
__device__ __forceinline__ void wide_read(const WideArgs& a, const Src& src, float* s_dyn, WideLds& lds) {
  constexpr int HD = W::HD, NL = W::NL, EB = W::EB;
  constexpr int TILE_BYTES = kBlockTokens * HD * EB;
  constexpr int ROW = HD + 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t G = a.group, H = a.n_kv_heads, L = a.n_layers;
  int half = 0;
  auto unit_of = [&](uint32_t t) {                // what ticket t stands for: place < 0 beyond the last
    WideUnit u = {};
    const uint32_t hg = H / HW, i = t / hg;
    u.g = (int32_t)(t - i * hg) * HW + wave;
    u.place = (int32_t)(i / (uint32_t)L);
    u.layer = (int32_t)(i - (uint32_t)u.place * L);
    u.b = -1;
    if (u.place >= a.places) u.place = -1;
    return u;
  };
  auto settle = [&](WideUnit& u, WideMeta& x) {   // what was fetched has arrived
    asm volatile("" : "+v"(x.rec), "+v"(x.slots[0]), "+v"(x.slots[1]), "+v"(x.slots[2]), "+v"(x.slots[3]));
    src.read(u, x);
    if (u.place < 0) u.b = -1;
  };
  auto slots_of = [&](const WideMeta& x, int s) { return s == 0 ? x.slots[0] : s == 1 ? x.slots[1] : s == 2 ? x.slots[2] : x.slots[3]; };
  auto tile = [&](const WideUnit& u, int32_t slot) {
    slot = slot < 0 ? 0 : slot;                   // flagged blocks are masked when consumed
    return a.kv_layer + u.layer * a.kv_stride + (size_t)slot * a.block_bytes + (size_t)u.g * TILE_BYTES + (size_t)lane * 16;
  };
  W w;
  uint4 kr[NL], vr[NL], q_next[NL];
  auto load_tile = [&](const char* p) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NL; ++i) kr[i] = nt_load16(p + (size_t)i * 1024);
#pragma unroll
    for (int i = 0; i < NL; ++i) vr[i] = nt_load16(p + a.block_bytes / 2 + (size_t)i * 1024);
    __builtin_amdgcn_sched_barrier(0);
  };
  // where the first block of a unit lies (anywhere in the caches, if it has none)
  auto first_tile = [&](const WideUnit& u, const WideMeta& x) {
    const bool some = u.b >= 0 && wide_blocks(u) > 0;
    WideUnit v = u;
    if (u.b < 0) { v.layer = 0; v.g = 0; }
    return tile(v, some ? __builtin_amdgcn_readlane(x.slots[0], 0) : 0);
  };
  // the query rows: lanes beyond the group read the last one's, and are cleared once it has arrived
  auto load_q = [&](const WideUnit& u) {
    const int32_t b = u.b < 0 ? 0 : u.b;
    const size_t row = (size_t)b * H * G + (size_t)(u.b < 0 ? 0 : u.g) * G + min(lane & 15, G - 1);
    const char* q = a.q + (u.b < 0 ? 0 : u.layer) * a.q_stride + (row * HD + 8 * (lane >> 4)) * 2;
#pragma unroll
    for (int kc = 0; kc < NL; ++kc) q_next[kc] = *reinterpret_cast<const uint4*>(q + 64 * kc);
  };
  auto settle_q = [&] {
    const bool mine = (lane & 15) < G;
#pragma unroll
    for (int kc = 0; kc < NL; ++kc) {
      asm volatile("" : "+v"(q_next[kc].x), "+v"(q_next[kc].y), "+v"(q_next[kc].z), "+v"(q_next[kc].w));
      w.q[kc] = make_uint4(mine ? q_next[kc].x : 0u, mine ? q_next[kc].y : 0u, mine ? q_next[kc].z : 0u, mine ? q_next[kc].w : 0u);
    }
  };

  WideUnit u = unit_of(blockIdx.x), n = unit_of(gridDim.x + blockIdx.x), nn = n;
  uint32_t t2 = 2 * gridDim.x + blockIdx.x, drawn = 0;
  WideMeta mu, mn, mm;
  int32_t found[kWaves] = {};
  src.fetch(u, lane, mu);
  src.fetch(n, lane, mn);
  settle(u, mu);
  src.look_up(u, mu, found);
  src.found_out(u, mu, found);
  load_q(u);
  load_tile(first_tile(u, mu));
  mm = mn;
  while (u.b >= 0) {
    settle_q();
    settle(n, mn);
    const int32_t jb0 = u.tok0 / kBlockTokens;
    float* const state = s_dyn + (half * HW + wave) * wide_head_floats(HD, G);
    // what the units behind this one need is asked for behind its first block, ahead of its second: then no block waits for it
    bool ahead = false;
    auto ask_ahead = [&] {
      ahead = true;
      drawn = add_one(a.counter, threadIdx.x);
      src.look_up(n, mn, found);
      load_q(n);
      nn = unit_of(t2);
      src.fetch(nn, lane, mm);
    };
    if (wide_blocks(u) <= 0) ask_ahead();
#pragma unroll 1
    for (int s = 0; s < kWaves; ++s) {
      const int32_t n_it = share_blocks(u, s), slots = slots_of(mu, s);
      w.reset();
      for (int32_t it = 0; it < n_it; ++it) {
        const bool present = __builtin_amdgcn_readlane(slots, it) >= 0;
        w.block(kr, vr, (jb0 + s + kWaves * it) * kBlockTokens, present ? u.tok1 : 0, lane, a.scale_log2e);
        if (!ahead) ask_ahead();
        const char* p;
        if (it + 1 < n_it) {
          p = tile(u, __builtin_amdgcn_readlane(slots, it + 1));
        } else if (s + 1 < kWaves && share_blocks(u, s + 1) > 0) {
          p = tile(u, __builtin_amdgcn_readlane(slots_of(mu, s + 1), 0));
        } else {
          src.found_out(n, mn, found);
          p = first_tile(n, mn);
        }
        load_tile(p);
      }
      w.to_lds(state, state + kWaves * kMaxGroup, state + 2 * kWaves * kMaxGroup, ROW, s, G, lane);
    }
    if (wide_blocks(u) <= 0) {
      src.found_out(n, mn, found);
      load_tile(first_tile(n, mn));
    }
    if (threadIdx.x == 0) {
      lds.ticket[half] = 3 * gridDim.x + drawn;
      int32_t* const x = lds.part[half];
      x[0] = u.b; x[1] = u.g; x[2] = u.layer; x[3] = u.np; x[4] = u.first; x[5] = u.part; x[6] = u.ctx_raw;
    }
    __syncthreads();                              // the states and the new ticket are there
    t2 = __builtin_amdgcn_readfirstlane(lds.ticket[half]);
    half ^= 1;
    u = n;
    mu = mn;
    n = nn;
    mn = mm;
  }
  if (threadIdx.x == 0) lds.part[half][0] = -1;
  __syncthreads();
}

}  // namespace pie
