// Checks of the GEMM launchers' choices, of the few-token path's limits, of the pooling kernels' and of top-K's bucket map, without a GPU: this program
// is linked with the launchers' object files and defines hipLaunchKernel itself, so every launch is recorded instead of made.
// Swept over shapes, list lengths and options, every launch must fit what its kernel assumes.  Exit code 0 = all hold.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <set>
#include <vector>

#include "ff_internal.h"

struct Launch {
  const void *fn;
  unsigned grid, threads;
  size_t lds;
  Gemm1Params g1;
  Gemm2Params g2;
  dim3 dims;
  const double *pooled;     // where a pooling kernel writes
};
static std::vector<Launch> g_log;
static int g_fail = 0, g_calls = 0;
static bool g_down = false, g_few = false, g_pred = false;   // whose launches are being recorded
static size_t g_pool_at = 0;                                 // which of the predictor's is the pooling kernel

extern "C" hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
  Launch l = {fn, grid.x * grid.y * grid.z, block.x, lds, {}, {}, grid, nullptr};
  if (g_pred && g_log.size() == g_pool_at) memcpy(&l.pooled, args[3], sizeof(l.pooled));
  if (g_few || g_pred) {}                                                  // (the grid says enough)
  else if (g_down) memcpy(static_cast<void *>(&l.g2), args[0], sizeof(l.g2));
  else memcpy(static_cast<void *>(&l.g1), args[0], sizeof(l.g1));
  g_log.push_back(l);
  return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
// (what a launch with <<< >>> hands to hipLaunchKernel)
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } g_config;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = {grid, block, lds, stream};
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
  return hipSuccess;
}

#define CHECK(cond, ...)                                  \
  do {                                                    \
    static int printed_ = 0;                              \
    if (!(cond) && ++g_fail && printed_++ < 4) {          \
      fprintf(stderr, "line %d: %s: ", __LINE__, #cond);  \
      fprintf(stderr, __VA_ARGS__);                       \
      fprintf(stderr, "\n");                              \
    }                                                     \
  } while (0)

constexpr int kLds = 160 * 1024;
static int32_t g_idx[1];      // stands for a list: the launchers only ask whether there is one

// n_heavy: how many blocks have k_heavy positions instead of k; -1: lengths that only the device knows, k bounds them (merged
// lists), about k_heavy
struct Shape { int T, block, d_model, d_ffn, rc, k, k_heavy, n_heavy; };

static KSpec lists(const Shape &s, int n_blocks) {
  KSpec k;
  k.uniform = k.k_max = k.k_base = s.k;
  if (s.n_heavy < 0) k.per_block = g_idx;
  if (s.n_heavy > 0 && s.k_heavy > s.k && n_blocks > s.n_heavy) {
    k.per_block = g_idx;
    k.k_max = s.k_heavy;
    k.n_heavy = s.n_heavy;
    for (int i = 0; i < s.n_heavy; ++i) k.heavy[i] = i;
  }
  return k;
}
static hipError_t gemm1(const Shape &s, bool list, int variant, int split, int heavy_tiles) {
  Gemm1Params p = {};
  p.T = s.T; p.d_model = s.d_model; p.d_ffn = s.d_ffn; p.block = s.block; p.n_blocks = (s.T + s.block - 1) / s.block;
  p.rc = s.rc; p.idx = list ? g_idx : nullptr; p.k_stride = s.d_ffn;
  p.k = lists(s, p.n_blocks);
  p.hs = (p.k.k_max + s.rc + 63) / 64 * 64;
  g_log.clear();
  g_down = false;
  ++g_calls;
  return ff_launch_gemm1(p, variant, split, heavy_tiles, s.n_heavy < 0 ? s.k_heavy : 0, nullptr);
}
struct DownOptions { int variant = -1, split = -1, row_mode = -1, ksplit = -1, nsplit = -1; };
static float g_room[1];       // stands for the workspace's room for partial sums: never touched
static hipError_t gemm2(const Shape &s, bool list, const DownOptions &o, bool room) {
  Gemm2Params p = {};
  p.T = s.T; p.d_model = s.d_model; p.d_ffn = s.d_ffn; p.block = s.block; p.n_blocks = (s.T + s.block - 1) / s.block;
  p.rc = s.rc; p.idx = list ? g_idx : nullptr; p.k_stride = s.d_ffn;
  p.k = lists(s, p.n_blocks);
  p.hs = (p.k.k_max + s.rc + 63) / 64 * 64;
  if (room) {
    p.part_bytes = ff_gemm2_part_bytes(s.T, s.block, s.d_model);
    p.split_bytes = ff_gemm2_split_bytes(s.T, s.d_model);
    if (p.part_bytes) p.part = g_room;
    if (p.split_bytes) p.split_part = g_room;
  }
  g_log.clear();
  g_down = true;
  ++g_calls;
  return ff_launch_gemm2(p, o.variant, o.split, o.row_mode, o.ksplit, o.nsplit, nullptr);
}

// Gate/up: the kernel leaves H zero up to the next multiple of 64 behind a block's list.  Where the list's end goes to a
// launch of its own, that launch has to start on a multiple of 64 (what it finds complete there it leaves alone).
static void check_gemm1(const Shape &s) {
  for (int variant = -1; variant < ff_gemm1_num_variants(); ++variant)
    for (int split = -1; split <= 1; ++split)
      for (int list = s.n_heavy != 0; list < 2; ++list) {
        const hipError_t e = gemm1(s, list, variant, split, -1);
        CHECK(e == hipSuccess && !g_log.empty(), "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
        for (const Launch &l : g_log) {
          CHECK(l.lds <= kLds && l.grid > 0, "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
          CHECK(l.g1.rem_bn % 64 == 0, "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
        }
      }
}

// Gate/up: the tiles with the weights in registers (11 and 12) form 32-bit offsets into a matrix.  Where those do not reach,
// the library takes another tile and a forced one is an error.
static void check_gemm1_addresses() {
  std::set<const void *> in_registers;
  for (int variant : {11, 12}) {
    CHECK(gemm1({700, 128, 256, 1024, 32, 512, 0, 0}, true, variant, 0, -1) == hipSuccess && g_log.size() == 1, "tile %d", variant);
    for (const Launch &l : g_log) in_registers.insert(l.fn);
  }
  struct { Shape s; bool ok; } sizes[] = {{{9000, 128, 65536, 32768, 32, 7168, 0, 0}, false}, {{9000, 64, 65536, 32768, 32, 7168, 0, 0}, false},
                                         {{9000, 128, 65536, 32760, 32, 7168, 0, 0}, true},   {{9000, 64, 65536, 32760, 32, 7168, 0, 0}, true},
                                         {{20, 10, 16777216, 8, 0, 8, 0, 0}, false},          {{20, 10, 4194304, 8, 0, 8, 0, 0}, true}};
  for (const auto &z : sizes) {
    CHECK(gemm1(z.s, true, -1, -1, -1) == hipSuccess, "d_model %d d_ffn %d", z.s.d_model, z.s.d_ffn);
    int used = 0;
    for (const Launch &l : g_log) used += in_registers.count(l.fn);
    CHECK(z.s.T < 9000 ? z.ok || !used : (used > 0) == z.ok, "d_model %d d_ffn %d block %d", z.s.d_model, z.s.d_ffn, z.s.block);
    for (int variant : {11, 12})
      CHECK((gemm1(z.s, true, variant, 0, -1) == hipSuccess) == z.ok && g_log.empty() == !z.ok, "d_model %d d_ffn %d tile %d", z.s.d_model, z.s.d_ffn, variant);
  }
}

// Gate/up: positions beyond the last full tile get a launch of their own where the tile that they would need starts a further
// round of workgroups, one per CU; not where it fits into the last one.  Compensator units and nothing else: workgroups of 32
// tokens, of 64 from 256 such on.
static void check_gemm1_splits() {
  struct { Shape s; size_t launches; unsigned rem_grid; } calls[] = {
      {{4096, 64, 4096, 14336, 64, 7168, 0, 0}, 2, 128}, {{4096, 64, 4096, 14336, 64, 5120, 0, 0}, 2, 128},   // 7 and 5 whole rounds
      {{2126, 64, 4096, 14336, 64, 7168, 0, 0}, 2, 67}, {{3000, 64, 2048, 8192, 64, 4096, 0, 0}, 2, 94},    // by the busiest XCD's count
      {{4096, 64, 4096, 14336, 64, 3584, 0, 0}, 1, 0},  {{3000, 64, 4096, 14336, 64, 7168, 0, 0}, 1, 0},    // 3.5 and 5.1 rounds
      {{1845, 128, 2048, 8192, 32, 4096, 8192, 2}, 1, 0},  {{3732, 64, 2048, 8192, 32, 4096, 8192, 2}, 1, 0},    // two longer lists
      {{1907, 64, 4096, 14336, 64, 10752, 14336, 2}, 1, 0},
      {{8192, 128, 4096, 14336, 64, 7168, 0, 0}, 2, 256}, {{9153, 128, 4096, 14336, 64, 7168, 0, 0}, 2, 144},
      {{2126, 64, 4096, 14336, 64, 7160, 0, 0}, 2, 67},   // units from the ninth on
      {{2126, 64, 4096, 14336, 64, 7180, 0, 0}, 2, 72}, {{8192, 128, 4096, 14336, 64, 7180, 0, 0}, 2, 256}};   // lists that end inside a tile
  for (const auto &c : calls) {
    CHECK(gemm1(c.s, true, -1, -1, -1) == hipSuccess && g_log.size() == c.launches, "T %d block %d K %d: %zu launches", c.s.T, c.s.block, c.s.k, g_log.size());
    if (c.launches > 1 && g_log.size() > 1) CHECK(g_log[1].g1.rem_bn == 256 && g_log[1].grid == c.rem_grid, "T %d K %d: grid %u", c.s.T, c.s.k, g_log[1].grid);
  }
}

// Gate/up: the 128 x 256 tile (11) against the 128 x 128 one (0) goes by the rounds of the busiest XCD, lists whole or their
// ends in a launch of their own.
static void check_gemm1_wide() {
  struct { Shape s; bool wide; size_t launches; } calls[] = {
      {{2200, 128, 4096, 14336, 64, 3584, 0, 0}, false, 2},   // 252 tiles that no split over the XCDs takes in one round
      {{2000, 128, 4096, 14336, 64, 7168, 0, 0}, true, 1},    // two rounds either way: whole
      {{1000, 128, 4096, 14336, 64, 7168, 0, 0}, true, 1},   {{1200, 128, 4096, 14336, 64, 7168, 0, 0}, false, 1},
      {{900, 128, 2048, 8192, 32, 4096, 0, 0}, true, 2},      // half a tile of units: cut
      {{4500, 128, 4096, 14336, 64, 7168, 0, 0}, true, 2},    // whole: a fifth round
      {{2800, 200, 4096, 14336, 64, 7168, 0, 0}, false, 1},   // two token tiles to a block
      {{9312, 128, 3584, 18944, 64, 9472, 0, 0}, true, 1}, {{8401, 128, 3584, 18944, 64, 9472, 0, 0}, true, 1}};   // 12 rounds against 22 of half the size
  for (const auto &c : calls) {
    gemm1(c.s, true, 11, 0, -1);
    const void *fn = g_log.empty() ? nullptr : g_log[0].fn;
    CHECK(gemm1(c.s, true, -1, -1, -1) == hipSuccess && (g_log[0].fn == fn) == c.wide && g_log.size() == c.launches, "T %d K %d", c.s.T, c.s.k);
    for (int split : {0, 1}) CHECK(gemm1(c.s, true, -1, split, -1) == hipSuccess && g_log.size() <= (split ? 2u : 1u), "T %d K %d split %d", c.s.T, c.s.k, split);
  }
}

// Gate/up: tiles of one short block, which reads every row of its list once: two rounds of 64 x 64 tiles lose to one of 128 x 128
// that is half empty; not so with a second block.
static void check_gemm1_short_block() {
  struct { Shape s; int variant; } calls[] = {
      {{61, 128, 3584, 18944, 64, 18944, 17760, -1}, 0}, {{61, 128, 3584, 18944, 64, 18944, 14208, -1}, 7}, {{64, 64, 3584, 18944, 64, 18944, 0, 0}, 0},
      {{40, 64, 128, 17024, 64, 17000, 0, 0}, 0},
      {{61, 128, 128, 17024, 64, 17024, 16896, -1}, 0}, {{64, 64, 3584, 18944, 64, 9472, 0, 0}, 7},  {{30, 128, 4096, 14336, 64, 7168, 0, 0}, 10}};
  for (const auto &c : calls) {
    gemm1(c.s, true, c.variant, 0, -1);
    const void *fn = g_log.empty() ? nullptr : g_log[0].fn;
    CHECK(gemm1(c.s, true, -1, -1, -1) == hipSuccess && g_log.size() == 1 && g_log[0].fn == fn, "T %d block %d K %d", c.s.T, c.s.block, c.s.k);
  }
  gemm1({64, 64, 3584, 18944, 64, 18944, 0, 0}, true, 0, 0, -1);
  const void *fn = g_log[0].fn;
  CHECK(gemm1({122, 64, 3584, 18944, 64, 18944, 0, 0}, true, -1, -1, -1) == hipSuccess && g_log[0].fn != fn, "two blocks");
}

// Down: the tiles with the weights in registers (5 to 9) form 32-bit offsets into W_down and H.  Where those do not
// reach, the library takes another tile and a forced one is an error, cut along the list or not.
static void check_gemm2_addresses() {
  std::set<const void *> in_registers;
  for (int variant : {5, 6, 7, 8, 9})
    for (bool list : {false, true}) {
      DownOptions o;
      o.variant = variant;
      CHECK(gemm2({700, 128, 256, 1024, 32, 512, 0, 0}, list, o, true) == hipSuccess && g_log.size() == 1, "tile %d", variant);
      for (const Launch &l : g_log) in_registers.insert(l.fn);
    }
  CHECK(in_registers.size() == 10, "%zu kernels", in_registers.size());
  // rows of 16 MiB; a matrix of 4 GiB, and just below; H of 2^24 positions
  struct { Shape s; bool ok, ok_list; } sizes[] = {{{20, 10, 8388608, 8, 0, 8, 0, 0}, false, false},
                                                  {{20, 10, 8388608 - 128, 8, 0, 8, 0, 0}, true, true},
                                                  {{20, 10, 65536, 32768, 0, 700, 0, 0}, true, false},
                                                  {{300, 128, 65536, 32768, 32, 700, 0, 0}, true, false},
                                                  {{300, 128, 65536, 32760, 0, 700, 0, 0}, true, true},
                                                  {{300, 128, 128, 1 << 24, 0, 1 << 24, 0, 0}, false, false}};
  for (const auto &z : sizes)
    for (bool list : {false, true})
      for (int nsplit : {-1, 0, 3}) {
        DownOptions o;
        o.nsplit = nsplit;
        CHECK(gemm2(z.s, list, o, true) == hipSuccess, "d_model %d d_ffn %d", z.s.d_model, z.s.d_ffn);
        const bool may = list ? z.ok_list : z.ok;
        for (const Launch &l : g_log)
          CHECK(may || !in_registers.count(l.fn), "d_model %d d_ffn %d list %d", z.s.d_model, z.s.d_ffn, list);
        for (int variant : {5, 6, 7, 8, 9}) {
          o.variant = variant;
          const hipError_t e = gemm2(z.s, list, o, true);
          CHECK((e == hipSuccess) == may && g_log.empty() == !may, "d_model %d d_ffn %d list %d tile %d nsplit %d", z.s.d_model, z.s.d_ffn, list, variant, nsplit);
        }
      }
}

// Calls that the GPU tests take for a route of their own: the library's choice has to be that kernel.
static void check_gemm2_routes() {
  struct { Shape s; bool list; int variant, row_mode; bool cut; } routes[] = {
      {{9000, 256, 1024, 1064, 24, 1064, 0, 0}, false, 5, -1, false},   // the identity list with compensator rows behind it
      {{150, 256, 4096, 4096, 24, 4096, 0, 0}, false, 8, -1, true},
      {{160, 256, 4096, 8192, 24, 8192, 0, 0}, false, 6, -1, true},
      {{60, 256, 2048, 4096, 24, 4096, 0, 0}, false, 9, -1, true},
      {{256, 256, 256, 344, 24, 344, 0, 0}, false, 9, -1, false},
      {{3000, 64, 512, 65536, 16, 3000, 0, 0}, true, 3, 2, true}};     // ids of more than 16 bits: scalar loads
  for (const auto &r : routes) {
    CHECK(gemm2(r.s, r.list, DownOptions(), true) == hipSuccess && !g_log.empty(), "T %d", r.s.T);
    const std::vector<Launch> chosen = g_log;
    DownOptions o;
    o.variant = r.variant;
    o.row_mode = r.row_mode;
    CHECK(gemm2(r.s, r.list, o, true) == hipSuccess && g_log[0].fn == chosen[0].fn && (chosen[0].g2.n_split > 1) == r.cut,
          "T %d d_model %d d_ffn %d", r.s.T, r.s.d_model, r.s.d_ffn);
  }
}

// Down: which tile the prices choose.
static void check_gemm2_prices() {
  struct { Shape s; bool list; int variant; } calls[] = {
      // two token tiles of 64, one list longer: priced for two like lists of equal length
      {{90, 48, 4096, 14336, 64, 3584, 14336, 1}, true, 9}, {{100, 50, 3584, 18944, 64, 4736, 18944, 1}, true, 9},
      // W_down in an XCD's L2: 64 x 64, then 64 x 256; with three steps or dense on to the longest calls, with more steps and blocks of 128 tokens or
      // more 128 x 256 there
      {{5000, 128, 256, 688, 0, 688, 0, 0}, false, 9}, {{7000, 128, 256, 688, 0, 688, 0, 0}, false, 9}, {{9500, 128, 256, 688, 0, 688, 0, 0}, false, 8},
      {{5000, 128, 256, 688, 16, 344, 0, 0}, true, 9}, {{7000, 256, 256, 688, 0, 344, 0, 0}, true, 9}, {{14000, 128, 256, 688, 16, 344, 0, 0}, true, 4},
      {{14000, 128, 256, 688, 16, 172, 0, 0}, true, 8},
      {{2000, 128, 256, 688, 16, 344, 688, 2}, true, 9}, {{5000, 128, 256, 688, 16, 344, 688, 2}, true, 8}, {{7000, 128, 256, 688, 16, 344, 688, 2}, true, 8},
      {{9000, 128, 256, 688, 16, 344, 688, 2}, true, 8}, {{11582, 128, 256, 688, 16, 688, 0, -1}, true, 4},   // (the last of merged lists)
      // ... and where it is not; a few longer lists' pieces beside more than a round of common tiles, and beside less
      {{2909, 64, 4096, 14336, 64, 3584, 14336, 2}, true, 6}, {{3000, 64, 3584, 18944, 64, 4736, 18944, 2}, true, 6},
      {{11490, 256, 2048, 8192, 32, 2327, 8192, 2}, true, 5}, {{11609, 128, 2048, 8192, 32, 2048, 8192, 2}, true, 5},
      {{2062, 256, 4096, 14336, 64, 7168, 14336, 2}, true, 5},
      {{2909, 160, 3584, 18944, 64, 9472, 18944, 2}, true, 6}, {{2300, 64, 3584, 18944, 64, 9472, 18944, 2}, true, 8},
      {{1700, 64, 2048, 8192, 32, 2048, 8192, 2}, true, 6}, {{2048, 64, 2048, 8192, 32, 2048, 8192, 2}, true, 6},
      {{4096, 128, 2048, 8192, 32, 4096, 0, 0}, true, 7}, {{1350, 128, 2048, 8192, 32, 4096, 0, 0}, true, 7}};
  for (const auto &c : calls) {
    DownOptions o;
    o.variant = c.variant;
    gemm2(c.s, c.list, o, true);
    const void *fn = g_log.empty() ? nullptr : g_log[0].fn;
    CHECK(gemm2(c.s, c.list, DownOptions(), true) == hipSuccess && !g_log.empty() && g_log[0].fn == fn,
          "T %d block %d d_model %d K %d, not tile %d", c.s.T, c.s.block, c.s.d_model, c.s.k, c.variant);
  }
  // no tile of 512 columns for 256 or fewer, whatever the lists
  std::set<const void *> wide;
  for (int variant : {5, 6})
    for (bool list : {false, true}) {
      DownOptions o;
      o.variant = variant;
      gemm2({700, 128, 256, 688, 16, 344, 0, 0}, list, o, true);
      for (const Launch &l : g_log) wide.insert(l.fn);
    }
  for (int T = 9; T < 20000; T += T / 8 + 1)
    for (int block : {16, 64, 128, 200, 256})
      for (int dm : {128, 256})
        for (int df : {688, 4096, 14336})
          for (int k : {df / 4, df / 2, df})
            for (int heavy : {-1, 0, 1, 2}) {
              const Shape s = {T, block, dm, df, 16, k, df, heavy};
              CHECK(gemm2(s, true, DownOptions(), true) == hipSuccess && !wide.count(g_log[0].fn), "T %d block %d d_model %d K %d, %d dense", T, block, dm, k, heavy);
            }
}

// Down: the longest list whose row-id table fits beside the ring of a tile with the weights in registers.  One position more and
// the tile is refused where it is forced, and not taken where it is not.
static void check_gemm2_row_table() {
  const int tiles[][2] = {{5, 49152}, {6, 65536}, {7, 16384}, {8, 49152}, {9, 49152}};
  for (const auto &t : tiles)
    for (int more = 0; more <= (t[1] < 65536); ++more)
      for (int T : {24, 300, 4096}) {
        const Shape s = {T, 128, 1024, 65528, 8, t[1] - 8 + more, 0, 0};
        DownOptions o;
        o.variant = t[0];
        o.nsplit = o.ksplit = 0;
        const hipError_t e = gemm2(s, true, o, true);
        CHECK((e == hipSuccess) == !more && g_log.empty() == (more != 0), "tile %d, list of %d", t[0], s.k + 8);
        for (const Launch &l : g_log) CHECK(l.lds <= kLds, "tile %d, list of %d", t[0], s.k + 8);
        const void *fn = g_log.empty() ? nullptr : g_log[0].fn;
        if (more) { Shape s0 = s; --s0.k; gemm2(s0, true, o, true); fn = g_log[0].fn; }
        o.variant = -1;
        CHECK(gemm2(s, true, o, true) == hipSuccess && !g_log.empty(), "T %d, list of %d", T, s.k + 8);
        for (const Launch &l : g_log) CHECK(l.lds <= kLds && !(more && l.fn == fn), "T %d, list of %d", T, s.k + 8);
      }
}

// A forced source of the row ids: the library chooses among the tiles that have it, and refuses only where none does.
static void check_gemm2_row_sources() {
  for (int T : {9, 300, 2000, 8192, 20000})
    for (int block : {16, 64, 128, 300})
      for (int dm : {256, 2048, 4096})
        for (int df : {14336, 65536})
          for (int k : {100, 7168, 14336})
            for (int heavy : {-1, 0, 2})
              for (int row_mode = 1; row_mode <= 3; ++row_mode)
                for (int nsplit : {-1, 0, 3}) {
                  const Shape s = {T, block, dm, df, 32, k, df, heavy};
                  DownOptions o;
                  o.row_mode = row_mode;
                  o.nsplit = nsplit;
                  const hipError_t e = gemm2(s, true, o, true);
                  bool any = false;
                  for (o.variant = 0; o.variant < ff_gemm2_num_variants() && !any; ++o.variant) any = gemm2(s, true, o, true) == hipSuccess;
                  CHECK(e == hipSuccess || !any, "T %d block %d d_model %d d_ffn %d K %d, %d dense, source %d, nsplit %d", T, block, dm, df, k, heavy, row_mode, nsplit);
                }
}

// The room that ff_workspace_bytes asks for to cut every list: no more pieces than the launcher would take by itself on the
// tile with the fewest tiles (two rounds of the chip), and room for every cut that it makes.
static void check_gemm2_room() {
  const int tiles[][2] = {{128, 512}, {64, 512}, {128, 256}, {256, 256}};
  for (int T : {9, 100, 700, 2000, 3000, 4500, 16000, 60000, 400000})
    for (int dm : {128, 256, 640, 1024, 4096, 8320}) {
      long fewest = 1 << 30;
      for (const auto &t : tiles) fewest = std::min(fewest, (long)((T + t[0] - 1) / t[0]) * ((dm + t[1] - 1) / t[1]));
      const size_t piece = (size_t)T * dm * 4, room = ff_gemm2_split_bytes(T, dm);
      CHECK(room % piece == 0 && room <= ((size_t)96 << 20) && room / piece != 1 && room / piece <= 16, "T %d d_model %d: %zu bytes", T, dm, room);
      CHECK((long)(room / piece) * fewest <= 512, "T %d d_model %d: room for %zu pieces of %ld tiles", T, dm, room / piece, fewest);
      for (int k : {500, 4000, 14336})
        for (bool list : {false, true}) {
          CHECK(gemm2({T, 128, dm, 14336, 0, list ? k : 14336, 0, 0}, list, DownOptions(), true) == hipSuccess, "T %d d_model %d", T, dm);
          for (const Launch &l : g_log) CHECK(l.g2.n_split <= 1 || (size_t)l.g2.n_split * piece <= room, "T %d d_model %d: %d pieces", T, dm, l.g2.n_split);
        }
    }
}

// Few tokens: the path takes a call wherever its tokens, as they are, fit into LDS.
static void check_few_tokens() {
  g_few = true;
  for (int nt = 1; nt <= kGemvMaxTokens + 1; ++nt)
    for (int dm = 128; dm <= 90112; dm += 128) {
      const bool fits = nt <= kGemvMaxTokens && (size_t)nt * dm * 2 <= kLds;
      CHECK(ff_gemv_eligible(nt, nt, dm, kLds) == fits, "%d tokens of %d", nt, dm);
      GemvParams p = {};
      p.T = p.block = nt; p.n_blocks = 1; p.d_model = dm; p.d_ffn = p.k_stride = 4096; p.idx = g_idx; p.part = g_room;
      p.k.uniform = p.k.k_max = p.k.k_base = 2048;
      g_log.clear();
      ++g_calls;
      CHECK((ff_launch_gemv(p, kLds, nullptr, nullptr) == hipSuccess) == fits && g_log.size() == (fits ? 2 : 0), "%d tokens of %d: %zu launches", nt, dm, g_log.size());
      for (const Launch &l : g_log) CHECK(l.lds <= kLds && l.grid > 0, "%d tokens of %d", nt, dm);
      // (the first kernel's copy of the tokens, then 1 KB of sums per wavefront)
      if (fits) CHECK(g_log[0].lds >= (size_t)nt * dm * 2 && g_log[0].lds >= g_log[0].threads * 16, "%d tokens of %d", nt, dm);
    }
  // wavefronts of the first kernel by its workgroups, one for 16 positions of a list, and the rows' length; workgroups of the
  // second: two per CU, else as many as have 512 positions each, up to one per CU
  struct { int T, block, dm, k; unsigned threads, grid2; } calls[] = {
      {1, 1, 4096, 7168, 256, 256}, {1, 1, 4096, 3584, 512, 224}, {1, 1, 4096, 1434, 1024, 96}, {1, 1, 4096, 14336, 512, 512},
      {1, 1, 2048, 2048, 512, 64}, {1, 1, 2048, 8192, 256, 256}, {1, 1, 2048, 16385, 256, 512}, {1, 1, 3584, 4736, 256, 252},
      {8, 8, 4096, 7168, 256, 256}, {8, 8, 4096, 14336, 512, 512}, {8, 8, 8192, 14336, 1024, 512}, {4, 1, 8192, 2048, 256, 512},
      {8, 1, 16384, 2048, 1024, 1024}, {1, 1, 256, 18944, 256, 74}};
  for (const auto &c : calls) {
    GemvParams p = {};
    p.T = c.T; p.block = c.block; p.n_blocks = (c.T + c.block - 1) / c.block; p.d_model = c.dm; p.d_ffn = p.k_stride = 18944; p.idx = g_idx; p.part = g_room;
    p.k.uniform = p.k.k_max = p.k.k_base = c.k;
    g_log.clear();
    CHECK(ff_launch_gemv(p, kLds, nullptr, nullptr) == hipSuccess && g_log[0].threads == c.threads && g_log[1].grid == c.grid2,
          "%d tokens of %d, K %d: %u threads, then %u workgroups", c.T, c.dm, c.k,
          g_log[0].threads, g_log[1].grid);
  }
  g_few = false;
}

// The predictor: which calls pool in narrow slices, and how narrow, given the room that ff_pool_fine_bytes asks for; without it the same
// slices with a launch that adds them, or one workgroup for all of a block's where the scores' place does not hold them either.
static void check_pooling() {
  g_pred = true;
  struct { int T, block, dm, r; bool softmax; unsigned slices; } calls[] = {      // slices: 0 = of 512 channels
      {64, 64, 4096, 128, true, 32}, {63, 128, 4096, 128, true, 0}, {700, 63, 4096, 128, true, 0}, {96, 96, 4096, 128, false, 32}, {95, 128, 4096, 128, false, 0},
      {128, 128, 4096, 136, false, 16}, {128, 128, 4096, 132, false, 0}, {100, 128, 2048, 64, true, 16},      // 4096 partial sums and more; r no multiple of 8
      {257, 128, 2048, 64, true, 16}, {257, 128, 2048, 72, true, 8}, {257, 128, 4096, 128, false, 16},        // three blocks: the scores kernel adds for four
      {16 * 128, 128, 4096, 64, false, 16}, {17 * 128, 128, 4096, 64, false, 0}, {128 * 128, 128, 512, 8, false, 4}, {129 * 128, 128, 512, 8, false, 0},
      {4096, 4096, 65536, 8, true, 512}, {4096, 4096, 65664, 8, true, 0}};
  for (const auto &c : calls)
    for (int room : {0, 1, 2}) {                   // none and too few neurons, none and enough of them, all that is asked for
      PredictParams p = {};
      p.T = c.T; p.block = c.block; p.d_model = c.dm; p.d_ffn = room == 1 ? c.slices * c.r + 8 : 24; p.r = c.r; p.n_blocks = (c.T + c.block - 1) / c.block;
      p.q_pred = c.softmax ? reinterpret_cast<const bf16_t *>(g_idx) : nullptr;
      p.k_stride = p.k.uniform = p.k.k_max = p.k.k_base = 8;
      double at[3];
      p.hpart = at; p.scores = at + 1; p.hpart_fine = at + 2;
      const size_t bytes = ff_pool_fine_bytes(c.T, c.block, c.dm, c.r, c.softmax), n = (size_t)p.n_blocks * c.r * sizeof(double);
      CHECK(bytes == c.slices * n && ff_pool_fine_bytes(c.T, c.block, c.dm, c.r, true) >= bytes,
            "T %d block %d d_model %d r %d: %zu bytes", c.T, c.block, c.dm, c.r, bytes);
      p.hpart_fine_bytes = room == 2 ? bytes : bytes - (bytes > 0);
      g_log.clear();
      g_pool_at = c.softmax;
      ++g_calls;
      const bool fine = c.slices > 0, sum = fine && room == 1;
      CHECK(ff_launch_predict(p, kLds, nullptr, nullptr) == hipSuccess && g_log.size() == 3u + c.softmax + sum, "T %d: %zu launches", c.T, g_log.size());
      const Launch &pool = g_log[c.softmax], &after = g_log[c.softmax + 1];
      const unsigned x = !fine ? (c.dm + 511) / 512 : room == 0 ? 1 : c.slices;
      CHECK(pool.threads == (fine ? 512u : 256u) && pool.dims.x == x && pool.dims.y == (unsigned)p.n_blocks &&
                pool.pooled == (!fine || room == 0 ? p.hpart : room == 1 ? p.scores : p.hpart_fine),
            "T %d block %d d_model %d r %d softmax %d: %u x %u workgroups of %u", c.T, c.block, c.dm, c.r, c.softmax, pool.dims.x, pool.dims.y, pool.threads);
      CHECK(!sum || (after.threads == 64 && after.dims.x == (unsigned)(c.r + 63) / 64 && after.dims.y == (unsigned)p.n_blocks), "T %d: sums", c.T);
    }
  g_pred = false;
}

// Top-K's bucket map: monotone over the scores, and scores spread evenly over their range fill the buckets evenly, however
// narrow the range is against the scores' size and however small or large they are.  (A bucket of more than TOPK_CAND keys
// sends the whole block to eight passes over its scores.)
static void check_topk_map() {
  constexpr int n = 16384;
  for (int centre = -1; centre <= 1; ++centre)
    for (int e = 0; e <= 36; ++e)
      for (double size : {1.0, 0x1p-140, 0x1p-40, 0x1p40, 0x1p140}) {
        ++g_calls;
        double s[n];
        std::vector<int> hist(TOPK_BUCKETS, 0);
        for (int i = 0; i < n; ++i) s[i] = size * (centre + ldexp((double)i / n, -e));
        const TopkMap m = topk_map(s[0], s[n - 1]);
        int last = 0, most = 0;
        for (int i = 0; i < n && !m.none; ++i) {
          const int b = m.fine ? m.bucket64(s[i]) : m.bucket((float)s[i]);
          CHECK(b >= last && b < TOPK_BUCKETS, "size %g centre %d range 2^-%d: score %d", size, centre, e, i);
          last = b;
          if (++hist[b] > most) most = hist[b];
        }
        CHECK(!m.none && most <= 8, "size %g centre %d range 2^-%d: %d in one bucket", size, centre, e, most);
      }
  CHECK(topk_map(1.0, 1.0).none && topk_map(0.0, INFINITY).none && topk_map(-INFINITY, 0.0).none && topk_map(0.0, NAN).none && topk_map(NAN, 0.0).none, "no range");
}

int main() {
  if (ff_gemm_init(kLds) != hipSuccess) return 1;
  for (int T : {9, 70, 300, 700, 2000, 8192})
    for (int block : {16, 64, 96, 128, 300})
      for (int dm : {256, 2048, 4096})
        for (int k : {33, 96, 160, 1000, 3584, 7168})
          for (int rc : {0, 32, 64})
            for (int heavy : {-1, 0, 2}) check_gemm1({T, block, dm, 14336, rc, k, 14336, heavy});
  check_gemm1_addresses();
  check_gemm1_splits();
  check_gemm1_wide();
  check_gemm1_short_block();
  check_gemm2_addresses();
  check_gemm2_routes();
  check_gemm2_prices();
  check_gemm2_row_table();
  check_gemm2_row_sources();
  check_gemm2_room();
  check_few_tokens();
  check_pooling();
  check_topk_map();
  printf("launch checks: %d calls, %d wrong\n", g_calls, g_fail);
  return g_fail != 0;
}
