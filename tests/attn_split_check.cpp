// The one-launch attention's split and the sizes of its scratch (csrc/pie_attn_split.h, the header the kernel and its
// launcher use), run on the CPU: for random calls on random pools every part, plan record, arrival word and workgroup is
// in range and the parts cover every context exactly once, whichever way the reciprocal's last place falls; so are the
// parts, words and units of the layers of a step that share a launch.  Built and
// run by tests/test_attn_split_host.py.  Prints "split ok" and exits 0.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#include "pie_attn_split.h"
using namespace pie;
#define REQUIRE(c) do { if (!(c)) { printf("FAILED line %d: %s\n", __LINE__, #c); exit(1); } } while (0)

static std::mt19937_64 rng(1);
static int32_t ri(int64_t lo, int64_t hi) { return (int32_t)(lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1))); }
template <size_t N> static int32_t pick(const int32_t (&v)[N]) { return v[rng() % N]; }

struct Rcp {                                     // the correctly rounded reciprocal, or a neighbour
  int ulp;
  float operator()(float y) const {
    const float r = 1.0f / y;
    return ulp ? std::nextafter(r, ulp > 0 ? 2.0f : 0.0f) : r;
  }
};

static void check_div_up() {
  const int32_t end = 1 << 20;
  auto same = [](int32_t x, int32_t y) {
    for (const int ulp : {-1, 0, 1}) REQUIRE(div_up(x, y, Rcp{ulp}) == (x + y - 1) / y);
  };
  for (int32_t y = 1; y < end; y = y < 5000 ? y + 1 : y + ri(1, 997)) {
    const int32_t top = end - 1 - y;             // x + y < 2^20
    same(0, y);
    same(top, y);
    for (int i = 0; i < 24; ++i) {
      const int32_t m = (int32_t)((int64_t)y * ri(0, top / y));   // multiples and their neighbours, where it turns over
      for (int32_t x = m - 1; x <= m + 1; ++x)
        if (x >= 0 && x <= top) same(x, y);
    }
    same(ri(0, top), y);
  }
}

// The layers of a step that share a launch: their parts, side by side, lie in the scratch, their arrival words in the pool's
// lines, one to a layer and pair, and what a capture clears ahead of them covers the words without leaving the lines.
static void check_step(pie_config c, int32_t units, int32_t batch, int32_t width, int32_t items) {
  const int32_t H = c.n_kv_heads, n = direct_step_layers(c, units, batch, width), places = direct_grid(units, H, batch, width) / H;
  REQUIRE(n >= 1 && n <= c.n_layers);                                        // (a loop over launches ends)
  const size_t layer_floats = (size_t)places * c.n_q_heads * (c.head_dim + 4);
  REQUIRE(items <= places && layer_floats * 4 <= (size_t)INT32_MAX);
  REQUIRE(n * layer_floats <= direct_step_rows(c) * (c.head_dim + 4));
  REQUIRE(direct_step_rows(c) >= direct_pool_rows(c) && direct_step_rows(c) <= direct_pool_rows(c) * c.n_layers);
  const size_t lines = direct_pool_words(c), words = direct_arrive_lines(c) * kArriveStride;
  const int32_t layers = ri(0, 1) ? n : c.n_layers;                          // (whole contexts: all layers, no parts)
  const size_t cleared = ((size_t)(layers - 1) / kArriveStride * lines + (size_t)batch * H) * kArriveStride;
  REQUIRE(cleared <= words);
  for (const int32_t l : {0, layers - 1, ri(0, layers - 1), ri(0, layers - 1)})
    for (const int32_t pair : {0, batch * H - 1, ri(0, batch * H - 1)}) {
      const size_t w = ((size_t)(l / kArriveStride) * lines + pair) * kArriveStride + l % kArriveStride;
      REQUIRE(w < cleared && w / kArriveStride / lines == (size_t)(l / kArriveStride));
      REQUIRE(w / kArriveStride % lines == (size_t)pair && w % kArriveStride == (size_t)(l % kArriveStride));
    }
}

// and the planned ones
static void check_planned() {
  pie_config c; memset(&c, 0, sizeof c);
  c.n_kv_heads = pick({1, 2, 8, 12, 32, 64, 300});
  c.n_q_heads = c.n_kv_heads * pick({1, 2, 4, 8, 16});
  c.head_dim = pick({64, 128});
  c.n_layers = ri(1, 100);
  const int32_t part = 64 * ri(4, 64), batch = ri(1, ri(0, 3) ? 300 : 16384), width = (int32_t)std::exp2(std::uniform_real_distribution<double>(0, 17)(rng));
  const size_t items = (size_t)batch * ((width * 16 + part - 1) / part), layer = items * c.n_q_heads * (c.head_dim + 2);
  if (items > INT32_MAX) return;
  const size_t floats = (size_t)(layer * std::uniform_real_distribution<double>(1, 200)(rng));
  const int32_t n = planned_step_layers(c, floats, part, batch, width);
  REQUIRE(n >= 1 && n <= c.n_layers && n * layer <= floats);
  REQUIRE(n == 1 || items * c.n_kv_heads * n <= (size_t)1 << 31);            // units and the grid's tickets in 32 bits
  REQUIRE(planned_step_layers(c, layer, part, batch, width) == 1);
}

static bool check_call() {
  pie_config c; memset(&c, 0, sizeof c);
  c.n_layers = ri(1, 100);
  c.head_dim = pick({64, 128});
  c.block_tokens = kBlockTokens;
  c.dtype = pick({PIE_DTYPE_F32, PIE_DTYPE_F16, PIE_DTYPE_BF16});
  c.n_gpu_blocks = (int32_t)std::exp2(std::uniform_real_distribution<double>(0, 24)(rng));
  c.n_kv_heads = pick({1, 2, 3, 4, 8, 12, 16, 32, 40, 64, 300});
  const int32_t group = pick({1, 2, 3, 4, 7, 8, 16}), n_cu = pick({32, 64, 128, 256, 304});
  c.n_q_heads = c.n_kv_heads * group;
  c.max_batch = ri(1, 400);
  c.max_blocks_per_seq = (int32_t)std::exp2(std::uniform_real_distribution<double>(0, ri(0, 3) ? 10 : 19)(rng));
  const int32_t batch = ri(1, c.max_batch), width = ri(0, 1) ? ri(1, c.max_blocks_per_seq) : c.max_blocks_per_seq;
  const int32_t H = c.n_kv_heads;
  const int32_t units = direct_units(n_cu, H, group, batch, width);
  if (units == 0) return false;
  REQUIRE(batch <= kDirectSeqs && units <= kDirectMaxUnits && (int64_t)units * group <= kDirectRows);
  const int32_t grid = direct_grid(units, H, batch, width), max_items = units / H;
  std::vector<int32_t> ctx(batch);
  const int kind = ri(0, 3);
  int32_t total = 0;
  for (int32_t& x : ctx) {
    const int32_t most = width * kBlockTokens;
    x = kind == 0 ? most : kind == 1 ? ri(0, most) : kind == 2 ? ri(0, std::min(most, 200)) : ri(0, 7) ? ri(0, std::min(most, 64)) : most;
    total += quanta_of(x);
  }
  const Rcp rcp{ri(-1, 1)};
  const int32_t k = quanta_per_part(total, max_items, [&](int32_t q) {
    int32_t n = 0;
    for (const int32_t x : ctx) n += div_up(quanta_of(x), q, rcp);
    return n;
  });
  REQUIRE(k >= 1 && k <= kDirectMaxQuanta);
  int32_t items = 0;
  for (const int32_t x : ctx) {
    const SeqParts p = seq_parts(quanta_of(x), k, rcp);
    REQUIRE(p.n >= 1 && p.each >= 1 && p.each <= kDirectMaxQuanta);          // a lane of the slot list for every block of a wave
    REQUIRE((int64_t)p.n * p.each * kQuantum >= x);                          // the parts reach the end
    REQUIRE((int64_t)(p.n - 1) * p.each * kQuantum < std::max(x, 1));        // and none lies beyond it
    REQUIRE(p.n < (1 << kArriveShift));                                      // what an arrival word counts
    items += p.n;
  }
  REQUIRE(items <= max_items);
  REQUIRE((int64_t)items * H <= grid);                                       // a workgroup for every unit
  REQUIRE((size_t)items * c.n_q_heads <= direct_pool_rows(c));               // a partial state for every row of every part
  REQUIRE((size_t)items * c.n_q_heads <= (size_t)kDirectRows);               // (also in a call's own scratch)
  REQUIRE((size_t)((grid - 1) / H) < direct_pool_items(c));                  // a record for every place, used or not
  REQUIRE((size_t)batch * H <= direct_pool_words(c));                        // a word for every (sequence, head)
  REQUIRE(batch * H <= kArriveWords && grid <= kClockWgs);
  check_step(c, units, batch, width, items);
  return true;
}

// Which launches keep two blocks of a wave in flight, and which steps are planned ahead.
static void check_rules() {
  const int32_t n_cu = pick({64, 256, 304});
  const int64_t pairs = ri(1, 3000), wgs = ri(1, 5000);
  const int32_t heads = pick({1, 4, 8, 32});
  for (const bool plan : {false, true}) {
    REQUIRE(direct_two_blocks(64, wgs, n_cu, pairs, heads, plan));
    if (wgs > 3 * n_cu) REQUIRE(!direct_two_blocks(128, wgs, n_cu, pairs, heads, plan));
    REQUIRE(direct_two_blocks(128, n_cu, n_cu, n_cu, heads, plan));
  }
  REQUIRE(direct_two_blocks(128, 256, 256, 30, 8, false) && !direct_two_blocks(128, 256, 256, 30, 8, true));
  REQUIRE(!direct_two_blocks(128, 256, 256, 8, 8, false) && direct_two_blocks(128, 256, 256, 8, 4, false));
  const int32_t batch = ri(1, 300), group = pick({1, 4, 8, 16}), blocks = ri(1, 9000);
  if (direct_too_wide(n_cu, heads, group, batch, blocks)) {
    REQUIRE(batch <= kDirectSeqs && blocks > kDirectMaxQuanta * kWaves && batch * heads <= kDirectRows / group);
    REQUIRE(direct_too_wide(n_cu, heads, group, batch, 2 * blocks));
  }
  REQUIRE(direct_too_wide(256, 8, 4, 32, 8192) && !direct_too_wide(256, 32, 1, 190, 5) && !direct_too_wide(256, 8, 4, 300, 8192));
  for (const int32_t layers : {0, 1, 2}) REQUIRE(!direct_plan_ahead(n_cu, pairs, layers));
  REQUIRE(direct_plan_ahead(n_cu, 2 * n_cu + 1, 3) && !direct_plan_ahead(n_cu, 2 * n_cu, 80));
}

// Four heads side by side: only what the kernel is written for, what its LDS holds, and units numbered in 32 bits.
static void check_wide() {
  const int32_t n_cu = pick({64, 256, 304}), H = pick({1, 2, 4, 8, 12, 32, 40, 300}), group = pick({1, 3, 4, 8, 16}), hd = pick({64, 128});
  const int32_t bytes = pick({2, 4}), layers = ri(0, 100), places = ri(1, 4096), blocks = ri(1, 2000), batch = ri(1, 4096);
  if (planned_wide(n_cu, H, group, hd, layers, batch)) {
    REQUIRE(hd == 128 && H % kPlannedWideHeads == 0 && layers > 1 && wide_lds(kPlannedWideHeads, group, hd) + 4096 <= (size_t)160 << 10);
    REQUIRE(planned_wide(n_cu, H, group, hd, layers + 1, batch));
  }
  if (!direct_wide(n_cu, H, group, hd, bytes, layers, places, blocks)) return;
  REQUIRE(bytes == 2 && hd == 128 && H % kWaves == 0 && layers > 1 && group <= 8);
  REQUIRE(wide_lds(kWideHeads, group, hd) + 4096 <= (size_t)160 << 10);
  for (const int32_t heads : {kWideHeads, kPlannedWideHeads}) REQUIRE(2 * wide_lds(heads, group, hd) > (size_t)160 << 10);   // one a compute unit
  REQUIRE((int64_t)places * (H / kWaves) * layers + 3 * n_cu <= INT32_MAX);
  REQUIRE(direct_wide(n_cu, H, group, hd, bytes, layers + 1, places, blocks));
}

// Which launches are read so, of 256 compute units: those that measured faster, down to nine units a compute unit.
static void check_wide_shapes() {
  struct Shape { int32_t H, group, batch, blocks, layers; bool wide; };
  for (const Shape& s : {Shape{8, 4, 256, 256, 16, true}, Shape{8, 4, 48, 256, 16, true}, Shape{32, 1, 24, 69, 16, true},
                         Shape{8, 4, 30, 500, 13, true}, Shape{16, 2, 12, 445, 12, true}, Shape{40, 1, 44, 3, 12, true},
                         Shape{8, 4, 8, 316, 32, false}, Shape{8, 8, 45, 46, 8, false}, Shape{12, 2, 192, 20, 3, false},
                         Shape{40, 1, 9, 46, 10, false}, Shape{32, 1, 11, 80, 9, false}, Shape{8, 4, 39, 64, 4, false}}) {
    const int32_t units = direct_units(256, s.H, s.group, s.batch, s.blocks);
    REQUIRE(units > 0);
    const int32_t places = direct_grid(units, s.H, s.batch, s.blocks) / s.H;
    REQUIRE(direct_wide(256, s.H, s.group, 128, 2, s.layers, places, s.blocks) == s.wide);
  }
  // planned ones, from six layers on and, a unit a sequence, four units a compute unit
  REQUIRE(planned_wide(256, 32, 1, 128, 16, 64) && planned_wide(256, 32, 1, 128, 6, 64) && planned_wide(256, 8, 4, 128, 12, 300));
  REQUIRE(planned_wide(256, 32, 1, 128, 9, 30) && !planned_wide(256, 32, 1, 128, 8, 30) && !planned_wide(256, 32, 1, 128, 5, 300));
  REQUIRE(!planned_wide(256, 8, 4, 128, 16, 40) && !planned_wide(256, 8, 8, 128, 16, 300) && !planned_wide(256, 32, 1, 64, 16, 64));
}

// Contexts are left whole only where a workgroup's waves can list their blocks, never more than 256 KB of them; a few pairs
// not beyond six passes, whichever way the pairs of a step are divided into layers.
static void check_whole() {
  const int32_t n_cu = pick({64, 256, 304}), layers = ri(0, 40), blocks = ri(1, 200);
  const int64_t pairs = ri(1, ri(0, 1) ? 50 : 5000);
  const size_t head_block = (size_t)32 * pick({64, 128}) * pick({2, 4});
  const bool whole = direct_whole(n_cu, pairs, layers, blocks, head_block);
  if (whole) REQUIRE(blocks * head_block <= (size_t)256 << 10 && blocks <= 64 * kWholeWaves);
  if (whole && layers) REQUIRE(pairs <= 4 * n_cu && direct_whole(n_cu, pairs, layers + 1, blocks, head_block));
  if (blocks * head_block <= (size_t)256 << 10 && blocks <= 48 && (layers == 0 || pairs <= 4 * n_cu)) REQUIRE(whole);
  REQUIRE(direct_whole(256, 24, 0, 64, 4096) == false && direct_whole(256, 48, 0, 64, 4096) && direct_whole(256, 12, 0, 48, 4096));
}

int main() {
  check_div_up();
  int taken = 0;
  for (int i = 0; i < 60000; ++i) taken += check_call() ? 1 : 0;
  REQUIRE(taken > 5000);
  for (int i = 0; i < 60000; ++i) check_planned();
  for (int i = 0; i < 60000; ++i) check_whole();
  for (int i = 0; i < 60000; ++i) check_wide();
  check_wide_shapes();
  for (int i = 0; i < 1000; ++i) check_rules();
  printf("split ok (%d calls)\n", taken);
  return 0;
}
