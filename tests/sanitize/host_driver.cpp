// Drives the C-ABI host code under AddressSanitizer / UndefinedBehaviorSanitizer
// (with the device side replaced by kernel_stubs.cpp): map construction for
// every Table 2 configuration and the 7B-like map, general-map validation,
// argument validation of every entry point, and the planning / workspace
// layout that runs before a launch (which the stubs then refuse).  Exits 0
// when every expectation holds.
#include <cstdio>
#include <cstdint>
#include <utility>
#include <vector>

#include "kernels.h"
#include "mlkv.h"

static int g_failures = 0;
#define EXPECT(cond)                                                      \
  do {                                                                    \
    if (!(cond)) {                                                        \
      std::fprintf(stderr, "FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); \
      ++g_failures;                                                       \
    }                                                                     \
  } while (0)

static void* addr(uintptr_t a) { return reinterpret_cast<void*>(a); }
static const int32_t* lens(uintptr_t a) { return reinterpret_cast<const int32_t*>(a); }

static void maps() {
  // (l, h, m, g) of Table 2 (Pythia-160M variants) and the 7B-like map.
  const int cfg[][4] = {{12, 12, 12, 12}, {12, 12, 12, 4}, {12, 12, 4, 12}, {12, 12, 12, 1},
                        {12, 12, 4, 3},   {12, 12, 6, 1},  {12, 12, 4, 1},  {12, 12, 2, 1},
                        {12, 12, 1, 1},   {32, 32, 8, 8}};
  for (const auto& c : cfg) {
    mlkv_map* m = nullptr;
    EXPECT(mlkv_map_create_uniform(c[0], c[1], c[2], c[3], &m) == MLKV_OK && m);
    if (!m) continue;
    EXPECT(mlkv_map_num_kv_heads(m) == c[2] * c[3]);
    for (int n = 0; n < c[0]; ++n)
      for (int i = 0; i < c[1]; ++i) {
        const int kv = mlkv_map_kv_head(m, n, i);
        EXPECT(kv == (n / (c[0] / c[2])) * c[3] + i / (c[1] / c[3]));
        EXPECT(mlkv_map_owner_layer(m, kv) <= n);
      }
    EXPECT(mlkv_map_kv_head(m, c[0], 0) == -1 && mlkv_map_owner_layer(m, -1) == -1);
    EXPECT(mlkv_cache_bytes(m, 3, 64, 64) == 2ull * 3 * 64 * c[2] * c[3] * 64 * 2);
    mlkv_map_destroy(m);
  }
  mlkv_map* m = nullptr;
  EXPECT(mlkv_map_create_uniform(12, 12, 5, 1, &m) == MLKV_ERR_INVALID_ARG && !m);
  EXPECT(mlkv_map_create_uniform(12, 12, 4, 5, &m) == MLKV_ERR_INVALID_ARG && !m);
  EXPECT(mlkv_map_create_uniform(0, 12, 4, 1, &m) == MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_map_create_uniform(12, 12, 4, 1, nullptr) == MLKV_ERR_INVALID_ARG);
  // general maps: a valid cross-layer pattern, then rule violations
  const int32_t kv_ok[4 * 4] = {0, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 1};
  const int32_t own_ok[2] = {0, 2};
  EXPECT(mlkv_map_create(4, 4, 2, kv_ok, own_ok, &m) == MLKV_OK && m);
  mlkv_map_destroy(m);
  const int32_t own_late[2] = {1, 2};  // head 0 read by layer 0 before its owner
  EXPECT(mlkv_map_create(4, 4, 2, kv_ok, own_late, &m) == MLKV_ERR_BAD_MAP && !m);
  const int32_t kv_bad[4 * 4] = {0, 1, 0, 1, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 1};
  EXPECT(mlkv_map_create(4, 4, 2, kv_bad, own_ok, &m) == MLKV_ERR_BAD_MAP);
  const int32_t kv_range[4 * 4] = {0, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 2, 2, 2, 2};
  EXPECT(mlkv_map_create(4, 4, 2, kv_range, own_ok, &m) == MLKV_ERR_BAD_MAP);
  const int32_t kv_unread[4 * 4] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  EXPECT(mlkv_map_create(4, 4, 2, kv_unread, own_ok, &m) == MLKV_ERR_BAD_MAP);
  EXPECT(mlkv_map_create(4, 4, 2, nullptr, own_ok, &m) == MLKV_ERR_INVALID_ARG);
  mlkv_map_destroy(nullptr);
}

static void entry_points() {
  mlkv_map* mp = nullptr;
  EXPECT(mlkv_map_create_uniform(12, 12, 4, 1, &mp) == MLKV_OK);
  const uintptr_t K = 0x100000, V = 0x200000, Q = 0x300000, LEN = 0x400000, OUT = 0x500000,
                  WS = 0x600000;
  mlkv_cache c{addr(K), addr(V), 4, 2, 64, 64};
  const size_t big = size_t(1) << 30;
  // argument errors, reported before anything else
  EXPECT(mlkv_decode_attention(0, addr(Q), &c, nullptr, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_decode_attention(12, addr(Q), &c, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_decode_attention(0, addr(Q + 4), &c, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_ALIGNMENT);
  EXPECT(mlkv_decode_attention(0, addr(Q), &c, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 65,
                               addr(WS), big, nullptr) == MLKV_ERR_CAPACITY);
  mlkv_cache bad = c;
  bad.capacity = 48;
  EXPECT(mlkv_decode_attention(0, addr(Q), &bad, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_CAPACITY);
  bad = c;
  bad.head_dim = 96;
  EXPECT(mlkv_decode_attention(0, addr(Q), &bad, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_UNSUPPORTED);
  mlkv_cache large{addr(K), addr(V), 4, 2, 4096, 64};
  EXPECT(mlkv_decode_attention(0, addr(Q), &large, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), 16, nullptr) == MLKV_ERR_WORKSPACE);
  // valid arguments: planning and the workspace layout run, the stub refuses the launch
  EXPECT(mlkv_decode_attention(0, addr(Q), &large, mp, lens(LEN), addr(OUT), MLKV_OUT_F32, 0,
                               addr(WS), big, nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_decode_step(addr(Q), addr(Q), addr(Q), &large, mp, lens(LEN), addr(OUT),
                          MLKV_OUT_BF16, 0, addr(WS), big, nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_decode_step_rope(addr(Q), addr(Q), addr(Q), &large, mp, lens(LEN), 8, 1e4,
                               addr(OUT), MLKV_OUT_F32, 0, addr(WS), big, nullptr) ==
         MLKV_ERR_UNSUPPORTED);
  EXPECT(mlkv_decode_step_rope(addr(Q), addr(Q), addr(Q), &large, mp, lens(LEN), 16, 1e4,
                               addr(OUT), MLKV_OUT_F32, 0, addr(WS), 64, nullptr) ==
         MLKV_ERR_WORKSPACE);
  EXPECT(mlkv_decode_step_rope(addr(Q), addr(Q), addr(Q), &large, mp, lens(LEN), 16, 1e4,
                               addr(OUT), MLKV_OUT_F32, 0, addr(WS), big, nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_cache_append(0, mp, &c, addr(Q), addr(Q), 64, lens(LEN), nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_cache_append(0, mp, &c, addr(Q), addr(Q), 60, lens(LEN), nullptr) ==
         MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_cache_append(1, mp, &c, nullptr, nullptr, 0, nullptr, nullptr) == MLKV_OK);
  EXPECT(mlkv_cache_write_rows(&c, 0, 4, addr(Q), addr(Q), nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_cache_read_rows(&c, 3, 2, addr(Q), addr(Q), nullptr) == MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_prefill_step(addr(Q), addr(Q), addr(Q), &large, mp, lens(LEN), 100, addr(OUT),
                           MLKV_OUT_F32, nullptr) == MLKV_ERR_HIP);
  EXPECT(mlkv_prefill_attention(0, addr(Q), &c, mp, lens(LEN), 65, addr(OUT), MLKV_OUT_F32,
                                nullptr) == MLKV_ERR_CAPACITY);
  EXPECT(mlkv_workspace_init(addr(WS), 4096, nullptr) == MLKV_ERR_HIP);
  // planning and workspace sizes over batches, capacities and head sizes
  for (int B : {1, 2, 7, 128, 2048, 5000})
    for (int S : {32, 96, 2112, 32800})
      for (int D : {64, 128}) {
        const size_t ws = mlkv_workspace_bytes(mp, B, S, D);
        EXPECT(mlkv_workspace_bytes_rope(mp, B, S, D, 16) >= ws + size_t(B) * 8 * 16);
        int wg = 0, parts = 0;
        for (int layer = 0; layer < 12; ++layer) {
          EXPECT(mlkv_plan(mp, layer, B, S, D, S, &wg, &parts) == MLKV_OK);
          EXPECT(wg >= 1 && parts >= 1);
          EXPECT(mlkv_plan_merge_kernel(mp, layer, B, S, D, S) >= 0);
        }
      }
  EXPECT(mlkv_plan_merge_kernel(mp, 12, 2, 64, 64, 0) == -1);
  mlkv_map_destroy(mp);
}

extern long stub_prefills, stub_prefill_threads;

// A prefill takes every layer in one launch only where the device takes the
// grid (fewer than 2^32 threads); beyond, layer by layer as other maps do.
static void prefill_grids() {
  for (const auto& c : {std::pair<int, long>{4, 1}, std::pair<int, long>{40000, 512}}) {
    mlkv_map* mp = nullptr;
    EXPECT(mlkv_map_create_uniform(512, 1, 512, 1, &mp) == MLKV_OK);
    mlkv_cache big{addr(0x100000), addr(0x200000), 512, c.first, 32, 64};
    stub_prefills = stub_prefill_threads = 0;
    EXPECT(mlkv_prefill_step(addr(0x300000), addr(0x300000), addr(0x300000), &big, mp,
                             lens(0x400000), 1, addr(0x500000), MLKV_OUT_F32, nullptr) == MLKV_OK);
    EXPECT(stub_prefills == c.second);
    EXPECT(stub_prefill_threads < (1L << 32));
    stub_prefills = -1;
    mlkv_map_destroy(mp);
  }
}

extern int stub_prefill_form;

// The form of a prefill (0 plain, 1 split over the tokens, 2 wide blocks) at
// the sizes at which the GPU tests check the forms' results, and where a form
// was chosen that was slower than the plain one: few tokens on short contexts.
static void prefill_forms() {
  const struct { int l, h, m, g, D, B, T, S, form; } cases[] = {
      {4, 8, 2, 4, 64, 24, 50, 160, 0},   {4, 8, 2, 4, 128, 24, 50, 160, 0},
      {6, 12, 3, 4, 128, 43, 33, 320, 2}, {2, 12, 2, 1, 64, 2, 80, 544, 1},
      {2, 12, 2, 1, 128, 2, 80, 544, 1},
      {1, 32, 1, 32, 128, 101, 1, 64, 0},  {1, 12, 1, 12, 128, 80, 1, 64, 0},
      {12, 12, 12, 12, 128, 126, 2, 64, 0}, {1, 32, 1, 32, 128, 41, 26, 64, 0},
      {1, 32, 1, 8, 64, 5, 129, 256, 0},   {1, 12, 1, 4, 64, 21, 75, 128, 0},
      {1, 12, 1, 1, 64, 2, 822, 832, 1},   {1, 12, 1, 1, 64, 4, 500, 512, 0},
      {1, 12, 1, 1, 128, 1, 800, 832, 1},
  };
  for (const auto& c : cases) {
    mlkv_map* mp = nullptr;
    EXPECT(mlkv_map_create_uniform(c.l, c.h, c.m, c.g, &mp) == MLKV_OK);
    mlkv_cache cache{addr(0x100000), addr(0x200000), c.m * c.g, c.B, c.S, c.D};
    stub_prefills = 0;
    EXPECT(mlkv_prefill_step(addr(0x300000), addr(0x300000), addr(0x300000), &cache, mp,
                             lens(0x400000), c.T, addr(0x500000), MLKV_OUT_F32, nullptr) == MLKV_OK);
    EXPECT(stub_prefills == 1 && stub_prefill_form == c.form);
    stub_prefills = -1;
    mlkv_map_destroy(mp);
  }
}

extern long stub_steps;
extern mlkv::StepParams stub_step;

// Few long sequences: a unit's runs grow with the square root of its tiles
// (16 at least), leave a grid of at most one workgroup per compute unit, and
// fit any workspace that is handed in; a map of one layer on up to three very
// long units keeps the layer's own kernel.
static void step_runs() {
  const struct { int l, h, m, g, D, B, len, runs; } cases[] = {
      {2, 8, 1, 1, 64, 1, 131072, 64},  {2, 8, 1, 1, 64, 1, 8192, 16},
      {2, 8, 1, 1, 64, 1, 500000, 125}, {2, 8, 1, 1, 64, 8, 131072, 16},
      {2, 8, 1, 1, 64, 8, 500000, 32},  {12, 12, 4, 1, 128, 1, 500000, 20},
      {12, 12, 1, 1, 64, 2, 2048, 8},   {1, 8, 1, 1, 64, 1, 131072, 0},
      {1, 8, 1, 1, 128, 3, 32768, 0},   {1, 8, 1, 1, 64, 1, 32768, 32},
      {1, 8, 1, 1, 64, 4, 131072, 32},
  };
  for (const auto& c : cases) {
    mlkv_map* mp = nullptr;
    EXPECT(mlkv_map_create_uniform(c.l, c.h, c.m, c.g, &mp) == MLKV_OK);
    mlkv_cache cache{addr(0x100000), addr(0x200000), c.m * c.g, c.B, c.len, c.D};
    const size_t full = mlkv_workspace_bytes(mp, c.B, c.len, c.D);
    int last = c.runs;
    for (size_t ws = full; ws > 0; ws = ws * 4 / 5) {
      stub_steps = 0;
      const mlkv_status s = mlkv_decode_step(addr(0x300000), addr(0x300000), addr(0x300000),
                                             &cache, mp, lens(0x400000), addr(0x500000),
                                             MLKV_OUT_F32, 0, addr(0x600000), ws, nullptr);
      const long steps = stub_steps;
      stub_steps = -1;
      if (s == MLKV_ERR_WORKSPACE && ws < full) break;
      EXPECT(s == MLKV_OK && steps == (c.runs > 0 ? 1 : 0));
      if (steps != 1) continue;
      const mlkv::StepParams& p = stub_step;
      if (ws == full) EXPECT(p.runs == c.runs);
      EXPECT(p.runs >= 1 && p.runs <= last);
      last = p.runs;
      if (p.runs == 1) continue;
      EXPECT((p.items + 7) / 8 * 8 * p.chunks <= 256);
      const size_t rows = size_t(c.B) * c.m * c.g * p.chunks * p.runs * p.chunk_rows;
      const char* base = static_cast<char*>(addr(0x600000));
      EXPECT(reinterpret_cast<char*>(p.part_acc + rows * c.D) <=
             reinterpret_cast<char*>(p.part_ml));
      EXPECT(reinterpret_cast<char*>(p.part_ml + rows * 2) <= base + ws);
    }
    mlkv_map_destroy(mp);
  }
}

// Every map of four layers of two heads on up to three KV heads: a step takes
// all layers in one launch exactly where the launch's arithmetic (KV head from
// layer group and place in it, the group's first layer appending) is the map's.
static void one_launch_maps() {
  long one = 0, by_layer = 0;
  for (int n_kv = 1; n_kv <= 3; ++n_kv) {
    std::vector<std::pair<int, int>> reads;  // (first KV head, count) of a layer
    for (int c = 1; c <= 2; ++c)
      for (int lo = 0; lo + c <= n_kv; ++lo) reads.push_back({lo, c});
    const int nr = static_cast<int>(reads.size()), tables = nr * nr * nr * nr;
    for (int t = 0; t < tables; ++t)
      for (int o = 0; o < 1 << (2 * n_kv); ++o) {
        int32_t kv_of[8], owner_of[3];
        for (int n = 0, x = t; n < 4; ++n, x /= nr)
          for (int i = 0; i < 2; ++i) kv_of[2 * n + i] = reads[x % nr].first + i * (reads[x % nr].second - 1);
        for (int kv = 0; kv < n_kv; ++kv) owner_of[kv] = o >> (2 * kv) & 3;
        mlkv_map* mp = nullptr;
        if (mlkv_map_create(4, 2, n_kv, kv_of, owner_of, &mp) != MLKV_OK) continue;
        mlkv_cache cache{addr(0x100000), addr(0x200000), n_kv, 1, 32, 64};
        stub_steps = 0;
        EXPECT(mlkv_decode_step(addr(0x300000), addr(0x300000), addr(0x300000), &cache, mp,
                                lens(0x400000), addr(0x500000), MLKV_OUT_F32, 0, addr(0x600000),
                                1 << 20, nullptr) == MLKV_OK);
        bool grouped = false;  // some group size for which the arithmetic is the map's
        for (int per = 1; per <= 4; per *= 2) {
          const int g = n_kv * per / 4;  // KV heads of a layer
          if (g * 4 != n_kv * per || g < 1 || g > 2) continue;
          bool same = true;
          for (int n = 0; n < 4; ++n)
            for (int i = 0; i < 2; ++i)
              same = same && kv_of[2 * n + i] == n / per * g + i / (2 / g);
          for (int kv = 0; kv < n_kv; ++kv) same = same && owner_of[kv] == kv / g * per;
          grouped = grouped || same;
          if (same && stub_steps == 1)
            EXPECT(stub_step.layers == per && stub_step.kv_per_layer == g &&
                   stub_step.G == 2 / g && stub_step.n_kv == n_kv);
        }
        EXPECT(stub_steps == (grouped ? 1 : 0));
        (stub_steps == 1 ? one : by_layer) += 1;
        stub_steps = -1;
        mlkv_map_destroy(mp);
      }
  }
  EXPECT(one >= 3 && by_layer > 100);
}

// Several rounds of whole units: eight waves only where the caller's own bound
// allows long sequences; a long cache may hold short ones.
static void step_waves() {
  mlkv_map* mp = nullptr;
  EXPECT(mlkv_map_create_uniform(1, 32, 1, 8, &mp) == MLKV_OK);
  mlkv_cache cache{addr(0x100000), addr(0x200000), 8, 142, 4096, 128};
  for (const auto& c : {std::pair<int, int>{0, 4}, std::pair<int, int>{40, 4},
                        std::pair<int, int>{4096, 8}}) {
    stub_steps = 0;
    EXPECT(mlkv_decode_step(addr(0x300000), addr(0x300000), addr(0x300000), &cache, mp,
                            lens(0x400000), addr(0x500000), MLKV_OUT_F32, c.first, addr(0x600000),
                            mlkv_workspace_bytes(mp, 142, 4096, 128), nullptr) == MLKV_OK);
    EXPECT(stub_steps == 1 && stub_step.waves == c.second);
    stub_steps = -1;
  }
  mlkv_map_destroy(mp);
}

static void model() {
  mlkv_map* mp = nullptr;
  EXPECT(mlkv_map_create_uniform(2, 4, 1, 1, &mp) == MLKV_OK);
  mlkv_model* model = nullptr;
  std::vector<mlkv_layer_weights> w(2);
  EXPECT(mlkv_model_create(mp, 256, 256, 64, 16, 1e4, 1e-5, w.data(), &model) ==
         MLKV_ERR_INVALID_ARG && !model);
  EXPECT(mlkv_model_create(mp, 250, 256, 64, 16, 1e4, 1e-5, w.data(), &model) ==
         MLKV_ERR_INVALID_ARG);
  EXPECT(mlkv_model_create(mp, 256, 256, 96, 16, 1e4, 1e-5, w.data(), &model) ==
         MLKV_ERR_UNSUPPORTED);
  EXPECT(mlkv_model_workspace_bytes(nullptr, 2, 64) == 0);
  mlkv_map_destroy(mp);
}

int main() {
  maps();
  entry_points();
  prefill_grids();
  prefill_forms();
  step_runs();
  step_waves();
  one_launch_maps();
  model();
  std::printf("host driver: %d failure(s)\n", g_failures);
  return g_failures == 0 ? 0 : 1;
}
