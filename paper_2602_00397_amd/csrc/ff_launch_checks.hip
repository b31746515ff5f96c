// Checks of the GEMM launchers' choices, without a GPU: this program is linked with the launchers' object file and defines
// hipLaunchKernel itself, so every launch is recorded instead of made.  Swept over shapes, list lengths and options, every
// launch must fit what its kernel assumes.  Exit code 0 = all hold.
#include <stdio.h>
#include <string.h>

#include <vector>

#include "ff_internal.h"

struct Launch {
  const void *fn;
  unsigned grid, threads;
  size_t lds;
  Gemm1Params g1;
};
static std::vector<Launch> g_log;
static int g_fail = 0, g_calls = 0;

extern "C" hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
  Launch l = {fn, grid.x, block.x, lds, {}};
  memcpy(&l.g1, args[0], sizeof(l.g1));
  g_log.push_back(l);
  return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }

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

struct Shape { int T, block, d_model, d_ffn, rc, k, k_heavy, n_heavy; };

static KSpec lists(const Shape &s, int n_blocks) {
  KSpec k;
  k.uniform = k.k_max = k.k_base = s.k;
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
  ++g_calls;
  return ff_launch_gemm1(p, variant, split, heavy_tiles, nullptr);
}

// Gate/up: the kernel leaves H zero up to the next multiple of 64 behind a block's list.  Where the list's end goes to a
// launch of its own, that launch has to start on a multiple of 64 (what it finds complete there it leaves alone).
static void check_gemm1(const Shape &s) {
  for (int variant = -1; variant < ff_gemm1_num_variants(); ++variant)
    for (int split = -1; split <= 1; ++split)
      for (int list = s.n_heavy > 0; list < 2; ++list) {
        const hipError_t e = gemm1(s, list, variant, split, -1);
        CHECK(e == hipSuccess && !g_log.empty(), "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
        for (const Launch &l : g_log) {
          CHECK(l.lds <= kLds && l.grid > 0, "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
          CHECK(l.g1.rem_bn % 64 == 0, "T %d block %d K %d tile %d split %d", s.T, s.block, s.k, variant, split);
        }
      }
}

int main() {
  if (ff_gemm_init(kLds) != hipSuccess) return 1;
  for (int T : {9, 70, 300, 700, 2000, 8192})
    for (int block : {16, 64, 96, 128, 300})
      for (int dm : {256, 2048, 4096})
        for (int k : {33, 96, 160, 1000, 3584, 7168})
          for (int rc : {0, 32, 64})
            check_gemm1({T, block, dm, 14336, rc, k, 14336, (T + block - 1) / block > 2 ? 2 : 0});
  printf("launch checks: %d calls, %d wrong\n", g_calls, g_fail);
  return g_fail != 0;
}
