// Few-token path of the sparse FFN (Eq. 15-18, 20-21 for prompts of at most kGemvMaxTokens
// tokens: the generation-time regime, where a block is a handful of tokens or a single one).
// With so few rows the work is a gather of 3 K weight rows per block read exactly once, i.e.
// bound by HBM, and the tiles of the prefill kernels would leave most of the chip idle
// (one block gives the down GEMM only d_model / 512 workgroups).  Two kernels:
//   gemv1: H[t][p] = bf16( SiLU(x_t . Wgate[r]) * (x_t . Wup[r]) ), r = idx_b[p]   (p <  K_b)
//          H[t][p] = bf16( act(x_t . Wc1[p - K_b]) )                                (compensator units)
//          H[t][p] = 0                                                      up to the next multiple of 32
//   gemv2: Y[t] = sum_p H[t][p] * R_b[p][:], the list in chunks whose fp32 partial sums the last workgroup of a column
//          group adds in chunk order; rounded once (or added to the residual stream).
// Same rounding points as the prefill kernels (H in bf16, fp32 accumulation); every reduction has
// a fixed order, so results are reproducible.
// The products are MFMAs with weight rows on one side and the tokens, repeated to fill an operand, on the
// other: with multiply-adds the arithmetic of several tokens and its lane reductions took longer than the loads.
#include <algorithm>

#include "ff_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kGemvWaves = 8;      // wavefronts per workgroup of gemv2
constexpr int kGemv1Pos = 16;      // list positions per workgroup of gemv1
constexpr int kGemv2Cols = 128;    // output columns per workgroup of gemv2
constexpr int kGemv1Red = 16 * 16 * 4;  // bytes of gemv1's reduction, per wavefront

__device__ __forceinline__ f32x4_t mfma16(const u32x4_t &a, const u32x4_t &b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mfma32(const u32x4_t &a, const u32x4_t &b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
// list length of block b, at most cap
__device__ __forceinline__ int gv_block_k(const int32_t *per_block, int uniform, int cap, int b) {
  return max(1, min(per_block ? per_block[b] : uniform, cap));
}
__device__ __forceinline__ float gv_act(int act, float g) {
  if (act == FF_ACT_SILU) return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
  if (act == FF_ACT_RELU) return fmaxf(g, 0.0f);
  return g;
}

// What a kernel gets: first what its first loads' addresses need, as plain arguments, two vectors of four and three pointers, in
// scalar registers at the start (five tokens on a kept list of 2048/8192, both kernels 19.6 -> 19.1 us); then a struct of what it needs
// besides.  Few arguments and bytes, for the launches: the smallest calls last as long as the host takes to send them (256/688, kept list, a
// token, us: the whole parameter block and eleven plain arguments 8.62, the block alone 8.38, this 8.50; a dense one 8.30, 8.95 and 8.18).
typedef int32_t __attribute__((ext_vector_type(4))) i32x4_t;
struct Gemv1Args {
  const bf16_t *wg, *wu, *wc1;
  bf16_t *h;
  int32_t *counter;      // [n_blocks][column groups] of the next kernel, how many chunks are done
  const uint8_t *mask;
  int32_t sub_block, comp_act, d_ffn, hs;
};
struct Gemv2Args {
  const bf16_t *wd, *wc2;
  float *part;
  int32_t *counter;
  void *y;
  bf16_t *res;
  int32_t d_ffn, d_model, out_f32;
};

// One workgroup per 16 list positions; its wavefronts split the channels (steps steps of 64 each), every wavefront with a ring
// of 2 steps on their way, and their sums are added in wavefront order.  The 32 rows of an MFMA (32x32x16) are the 16 gate rows
// and the 16 up rows; they are loaded by fours of lanes and exchanged as in the gate/up GEMM (lane by lane, as the operand wants
// them, the address unit made it 54.9 us for a dense token of 4096/14336).  The block's tokens go through LDS, each
// wavefront its own channels, 16-byte chunks swizzled by the token; the tokens repeat past the last one.
// Bound by HBM.  Few steps of each wavefront on their way and small workgroups: what counts is that workgroups start and
// end next to each other (a dense token, 8 wavefronts: with 4 steps 54.5 us, with 2 52.6).  How many wavefronts: gemv1_waves.
// With multiply-adds, a wavefront per position, a dense token of 4096/14336 took 44.5 us (now 45.5), one on a list of 7168 23.2
// (22.6), one on 4096 positions of 8192/28672 86.1 (87.5), five tokens on 4096 positions of 2048/8192 19.5 (12.3).
// grid (groups of 16 positions, n_blocks), LDS = gemv1_lds.
template <int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW == 16 ? 4 : 6)))
void ff_gemv1_kernel(i32x4_t lists, i32x4_t sizes, const int32_t *idx, const int32_t *per_block, const bf16_t *x, Gemv1Args p) {
  const int uniform = lists[0], cap = lists[1], k_stride = lists[2], rc = lists[3], T = sizes[0], block = sizes[1], d_model = sizes[2], steps = sizes[3];
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, half = lane >> 5;
  const int b = blockIdx.y;
  const int t0 = b * block;
  const int nt = min(T, t0 + block) - t0;          // <= kGemvMaxTokens by the launcher's check
  const int Kb = gv_block_k(per_block, uniform, cap, b);
  const int ntot = Kb + rc;
  const int pos0 = blockIdx.x * kGemv1Pos;
  // (the counters of the next kernel's column groups start at zero)
  if (blockIdx.x == 0)
    for (int i = tid; i < d_model / kGemv2Cols; i += NW * 64) p.counter[b * (d_model / kGemv2Cols) + i] = 0;
  if (pos0 >= (ntot + 31) / 32 * 32) return;
  // load j of a step: chunk (lane mod 4) + 4 (lane / 32) of row j + 4 (lane / 4 mod 8), gate rows in front of the up rows
  // (positions past the list's end: the last one's rows again; H is written as zero there)
  const bool up = (lane >> 4) & 1;
  int entry[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int pos = min(pos0 + j + 4 * ((lane >> 2) & 3), ntot - 1);
    entry[j] = idx ? idx[(size_t)b * k_stride + min(pos, Kb - 1)] : pos;
  }
  const int ch0 = wave * steps * 64;                             // this wavefront's first channel
  const int n = max(0, min(d_model - ch0, steps * 64)) / 64;   // its steps
  const int pitch = n * 128;                                     // bytes per token in LDS
  uint8_t *xs = smem + (size_t)nt * min(ch0, d_model) * 2;
  const int nc = n * 8;                                          // 16-byte chunks per token
  for (int t = 0; t < nt; ++t)
    for (int c0 = 0; c0 < nc; c0 += 64)
      if (c0 + lane < nc)
        gload_lds16(x + (size_t)(t0 + t) * d_model + ch0 + ((c0 + lane) ^ t) * 8, lds_addr_of(xs) + (uint32_t)(t * pitch + c0 * 16));
  __builtin_amdgcn_sched_barrier(0);
  const bf16_t *rows[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int pos = min(pos0 + j + 4 * ((lane >> 2) & 3), ntot - 1);
    const bf16_t *row = pos < Kb ? (up ? p.wu : p.wg) + (size_t)min(max(entry[j], 0), p.d_ffn - 1) * d_model
                                 : p.wc1 + (size_t)(pos - Kb) * d_model;
    rows[j] = row + ch0 + ((lane & 3) + 4 * half) * 8;
  }
  constexpr int U = 2;
  u32x4_t w[U][4];
  if (n > 0) {
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) w[i][j] = *reinterpret_cast<const u32x4_t *>(rows[j] + min(i, n - 1) * 64);
  }
  __builtin_amdgcn_sched_barrier(0);
  // the tokens are older than the weights: they have landed by the time that one step of those is all that is on its way
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"((U - 1) * 4) : "memory");
  // (a wavefront reads what it copied itself: no barrier)
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  const int tok = min(c & 7, nt - 1);
  for (int s0 = 0; s0 < n; s0 += U) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int s = s0 + i;
      if (s < n) {
#pragma unroll
        for (int d = 0; d < 4; ++d) transpose4<true>(w[i], d);
#pragma unroll
        for (int g = 0; g < 4; ++g)
          acc = mfma32(w[i][g], *reinterpret_cast<const u32x4_t *>(xs + tok * pitch + (((8 * s + g + 4 * half) ^ tok) << 4)), acc);
      }
      if (s + U < n) {
#pragma unroll
        for (int j = 0; j < 4; ++j) w[i][j] = *reinterpret_cast<const u32x4_t *>(rows[j] + (s + U) * 64);
      }
    }
  }
  // lane (c, half) holds rows 8 (e / 4) + 4 half + e mod 4 of token c
  __syncthreads();                                               // the tokens' LDS is free
  float *red = reinterpret_cast<float *>(smem);
  if (c < 8) {
#pragma unroll
    for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 16 + 8 * half + c] = acc[e];
  }
  __syncthreads();
  const int pp = tid & 15, t = tid >> 4;                         // position and token of this thread
  static_assert(NW * 64 >= 16 * kGemvMaxTokens, "a thread for every output");
  if (t >= nt) return;
  const int at = ((pp & 3) + 4 * (pp >> 3)) * 16 + 8 * ((pp >> 2) & 1) + t;
  float g = 0.0f, u = 0.0f;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    g += red[v * 256 + at];
    u += red[v * 256 + 128 + at];
  }
  const int pos = pos0 + pp;
  float hv = pos < Kb ? gv_act(FF_ACT_SILU, g) * u : (pos < ntot ? gv_act(p.comp_act, g) : 0.0f);
  if (p.mask != nullptr && pos < Kb && !(((uint32_t)p.mask[(size_t)b * k_stride + pos] >> (t / p.sub_block)) & 1u)) hv = 0.0f;   // not selected for this token
  p.h[(size_t)(t0 + t) * p.hs + pos] = f32_to_bf16(hv);
}

// One workgroup per 128 output columns and chunk of the list; a wavefront takes every eighth group of 32 positions of the
// chunk, two groups on their way.  Lane (c, q) loads columns 8 c .. 8 c + 7 of rows 8 q .. 8 q + 7, which one byte permute per
// dword turns into the operands of eight MFMAs (tile f: column 8 c + f).  The wavefronts' sums are added in order through
// LDS, the chunks' through memory by the workgroup of the column group that is last to finish.  They are stored and loaded as
// relaxed atomics of device scope, hence past the L2 that this XCD does not share with the others, and counted when they have
// arrived (vmcnt); a release fence would write back the whole L2 instead (13.7 us become 28.4, a dense token's 27 become 140).
// Bound by HBM.  (Multiply-adds and a third launch for the sum: five tokens on 4096 positions of 2048/8192 20.0 us, now 13.7; one
// token on 7168 of 4096/14336 19.0 and 15.9, dense 31.2 and 27.0; eight tokens of a list each 39.2 and 23.7.)
// grid (d_model / 128, n_chunks, n_blocks)
__global__ __launch_bounds__(kGemvWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
void ff_gemv2_kernel(i32x4_t lists, i32x4_t sizes, const int32_t *idx, const int32_t *per_block, const bf16_t *h, Gemv2Args p) {
  const int uniform = lists[0], cap = lists[1], k_stride = lists[2], rc = lists[3], T = sizes[0], block = sizes[1], hs = sizes[2], n_chunks = sizes[3];
  constexpr int PITCH = kGemv2Cols + 4;
  __shared__ __align__(16) float red[kGemvWaves][kGemvMaxTokens][PITCH];
  __shared__ int last_s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4;
  const int b = blockIdx.z, ch = blockIdx.y;
  const int t0 = b * block;
  const int nt = min(T, t0 + block) - t0;
  const int Kb = gv_block_k(per_block, uniform, cap, b);
  const int ntot = Kb + rc;
  const int n_groups = (ntot + 31) / 32;
  const int per = (n_groups + n_chunks - 1) / n_chunks;
  const int g_end = min(n_groups, (ch + 1) * per);
  const int col0 = blockIdx.x * kGemv2Cols;
  const int32_t *list = idx ? idx + (size_t)b * k_stride : nullptr;
  const bf16_t *hrow = h + (size_t)(t0 + min(c & 7, nt - 1)) * hs + 8 * q;
  const size_t lane_col = (size_t)(col0 + 8 * c);
  f32x4_t acc[8];
#pragma unroll
  for (int f = 0; f < 8; ++f) acc[f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  // rows of this lane in group g (positions past the list's end: the last one again, next to zeros of H)
  auto ids = [&](int g, int (&id)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int pos = min(g * 32 + 8 * q + i, ntot - 1);
      id[i] = list ? list[min(pos, Kb - 1)] : pos;
    }
  };
  auto load = [&](int g, const int (&id)[8], u32x4_t (&w)[8], u32x4_t &hf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int pos = min(g * 32 + 8 * q + i, ntot - 1);
      const bf16_t *row = pos < Kb ? p.wd + (size_t)min(max(id[i], 0), p.d_ffn - 1) * p.d_model : p.wc2 + (size_t)(pos - Kb) * p.d_model;
      w[i] = *reinterpret_cast<const u32x4_t *>(row + lane_col);
    }
    hf = *reinterpret_cast<const u32x4_t *>(hrow + g * 32);
  };
  auto fma_group = [&](const u32x4_t (&w)[8], const u32x4_t &hf) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      u32x4_t ev, od;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ev[i] = __builtin_amdgcn_perm(w[2 * i + 1][d], w[2 * i][d], 0x05040100u);
        od[i] = __builtin_amdgcn_perm(w[2 * i + 1][d], w[2 * i][d], 0x07060302u);
      }
      acc[2 * d] = mfma16(ev, hf, acc[2 * d]);
      acc[2 * d + 1] = mfma16(od, hf, acc[2 * d + 1]);
    }
  };
  for (int g = ch * per + wave; g < g_end; g += 2 * kGemvWaves) {
    const int g2 = g + kGemvWaves;
    int ida[8], idb[8];
    u32x4_t wa[8], wb[8], ha, hb;
    ids(g, ida);
    ids(min(g2, g_end - 1), idb);
    __builtin_amdgcn_sched_barrier(0);
    load(g, ida, wa, ha);
    if (g2 < g_end) load(g2, idb, wb, hb);
    __builtin_amdgcn_sched_barrier(0);
    fma_group(wa, ha);
    if (g2 < g_end) fma_group(wb, hb);
  }
  // lane (c, q): columns 8 (4 q + e) + f of token c
  if (c < nt) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float *o = &red[wave][c][8 * (4 * q + e)];
      *reinterpret_cast<float4 *>(o) = make_float4(acc[0][e], acc[1][e], acc[2][e], acc[3][e]);
      *reinterpret_cast<float4 *>(o + 4) = make_float4(acc[4][e], acc[5][e], acc[6][e], acc[7][e]);
    }
  }
  __syncthreads();
  auto store = [&](int t, int col, float s) __attribute__((always_inline)) {
    const size_t o = (size_t)(t0 + t) * p.d_model + col;
    if (p.res) {
      p.res[o] = f32_to_bf16(bf16_to_f32(p.res[o]) + bf16_to_f32(f32_to_bf16(s)));
    } else if (p.out_f32) {
      reinterpret_cast<float *>(p.y)[o] = s;
    } else {
      reinterpret_cast<bf16_t *>(p.y)[o] = f32_to_bf16(s);
    }
  };
  for (int v = tid; v < nt * kGemv2Cols; v += kGemvWaves * 64) {
    const int t = v / kGemv2Cols, col = v % kGemv2Cols;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kGemvWaves; ++w) s += red[w][t][col];
    if (n_chunks == 1) store(t, col0 + col, s);
    else __hip_atomic_store(p.part + ((size_t)ch * T + t0 + t) * p.d_model + col0 + col, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (n_chunks == 1) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // this wavefront's sums have arrived
  __syncthreads();
  if (tid == 0)
    last_s = __hip_atomic_fetch_add(p.counter + b * (p.d_model / kGemv2Cols) + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_chunks - 1;
  __syncthreads();
  if (!last_s) return;
  for (int v = tid; v < nt * kGemv2Cols; v += kGemvWaves * 64) {
    const int t = v / kGemv2Cols, col = v % kGemv2Cols;
    float *src = p.part + (size_t)(t0 + t) * p.d_model + col0 + col;
    float s = 0.0f;
    for (int j0 = 0; j0 < n_chunks; j0 += 8) {                 // eight loads in flight, added in chunk order
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        x[j] = __hip_atomic_load(src + (size_t)min(j0 + j, n_chunks - 1) * T * p.d_model, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j0 + j < n_chunks) s += x[j];
    }
    store(t, col0 + col, s);
  }
}

int g_gemv_lds_raised = 0;

// gemv1: its wavefronts per workgroup.  One workgroup's channels are a chain of loads, steps / wavefronts long, and a CU wants
// some sixteen wavefronts with loads on their way.  Four where the groups of 16 positions give it those; eight where there is
// about one workgroup per CU or LDS holds no more of them, sixteen where there are half as many or LDS holds one; eight again
// for long rows in so many workgroups that these follow each other, sixteen for the longest.  One token, us with 4 / 8 / 16:
// 4096/14336, K 1434 15.1 / 11.5 / 10.4, K 3584 15.7 / 14.4 / 15.2, K 7168 22.6 / 23.9 / 24.1, dense 46.4 / 45.5 / 49.2;
// 2048/8192, K 2048 9.9 / 8.3 / 8.2, K 4096 11.9 / 11.7 / 13.5; 3584/18944, K 4736 17.2 / 18.1 / 20.2, dense 54.0 / 51.2 / 57.4;
// 8192/4096, K 2048 25.2 / 18.5 / 16.6; 16384/16384, dense 276 / 266 / 211; 1024/4096, K 1024 7.1 / 6.7 / 7.3.  Eight tokens:
// 3584/18944, K 9472 34.7 / 29.9 / 32.8; 8192/28672, K 14336 135 / 99 / 101.
int gemv1_waves(long groups, int nt, int d_model, int lds_limit) {
  constexpr int kCU = 256;
  const int steps = d_model / 64, per_cu = lds_limit / (nt * d_model * 2);
  if (groups <= kCU * 9 / 16) return steps >= 48 ? 16 : 8;
  if (groups <= kCU * 9 / 8) return per_cu <= 1 ? 16 : 8;
  if (groups > (long)per_cu * kCU || (groups > 3 * kCU && steps >= 48)) return per_cu <= 1 || steps >= 192 ? 16 : 8;
  return 4;
}
// gemv1: steps of 64 channels per wavefront (the last ones may have fewer), and LDS for nt tokens
int gemv1_steps(int nw, int d_model) { return (d_model / 64 + nw - 1) / nw; }
size_t gemv1_lds(int nw, int nt, int d_model) {
  const size_t x = (size_t)nt * d_model * 2, red = (size_t)nw * kGemv1Red;
  return x > red ? x : red;
}

}  // namespace

// (the chunks' sums, and behind them a counter for every column group of every block)
size_t ff_gemv_part_bytes(int n_tokens, int d_model) {
  return n_tokens <= kGemvMaxTokens ? (size_t)(kGemvChunks + 1) * n_tokens * d_model * sizeof(float) : 0;
}

bool ff_gemv_eligible(int n_tokens, int block, int d_model, int lds_limit) {
  const int nt = block < n_tokens ? block : n_tokens;
  return n_tokens <= kGemvMaxTokens && gemv1_lds(16, nt, d_model) <= (size_t)lds_limit;
}

hipError_t ff_launch_gemv(const GemvParams &p, int lds_limit, hipStream_t s, Profiler *prof) {
  if (!ff_gemv_eligible(p.T, p.block, p.d_model, lds_limit)) return hipErrorInvalidValue;
  if (!g_gemv_lds_raised) {
    for (const auto k : {ff_gemv1_kernel<4>, ff_gemv1_kernel<8>, ff_gemv1_kernel<16>}) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit);
      if (e != hipSuccess) return e;
    }
    g_gemv_lds_raised = 1;
  }
  const int nt = p.block < p.T ? p.block : p.T;
  const int n_extent = p.k.k_max + p.rc;
  int32_t *counter = reinterpret_cast<int32_t *>(p.part + (size_t)kGemvChunks * p.T * p.d_model);
  // gemv2: two workgroups per CU where each of their wavefronts then has two groups of 32 positions, the number that it keeps on
  // their way, else at most one: more chunks are more partial sums to add up.  One token, two workgroups per CU down to one group
  // for a wavefront, us -> this: 2048/8192 dense 16.3 -> 13.1, K 4096 11.9 -> 9.9; 4096/14336, K 7168 15.7 -> 14.8, K 3584 12.1 ->
  // 11.1; 3584/18944, K 4736 13.0 -> 12.3 (with two groups and 280 workgroups 13.6)
  const int cols = p.d_model / kGemv2Cols, groups = (n_extent + 31) / 32;
  const int most = 512 / (cols * p.n_blocks), full = (groups + 2 * kGemvWaves - 1) / (2 * kGemvWaves);
  const int nc = most <= full ? most : std::min(full, 256 / (cols * p.n_blocks));
  const int n_chunks = nc < 1 ? 1 : (nc > kGemvChunks ? kGemvChunks : nc);
  const int groups1 = (n_extent + 31) / 32 * (32 / kGemv1Pos);
  const int cap = p.idx ? std::min(p.d_ffn, p.k_stride) : p.d_ffn;   // (without a list position p is row p, and the pitch bounds nothing)
  const i32x4_t lists = {p.k.uniform, cap, p.k_stride, p.rc};
  const int nw = gemv1_waves((long)groups1 * p.n_blocks, nt, p.d_model, lds_limit);
  const auto fn = nw == 4 ? ff_gemv1_kernel<4> : nw == 8 ? ff_gemv1_kernel<8> : ff_gemv1_kernel<16>;
  prof_begin(prof, FF_STAGE_GEMM1, s);
  hipLaunchKernelGGL(fn, dim3(groups1, p.n_blocks), dim3(nw * 64),
                     gemv1_lds(nw, nt, p.d_model), s, lists, (i32x4_t{p.T, p.block, p.d_model, gemv1_steps(nw, p.d_model)}), p.idx, p.k.per_block, p.x,
                     (Gemv1Args{p.wg, p.wu, p.wc1, p.h, counter, p.mask, p.sub_block, p.comp_act, p.d_ffn, p.hs}));
  prof_end(prof, s);
  prof_begin(prof, FF_STAGE_GEMM2, s);
  hipLaunchKernelGGL(ff_gemv2_kernel, dim3(cols, n_chunks, p.n_blocks), dim3(kGemvWaves * 64), 0, s, lists, (i32x4_t{p.T, p.block, p.hs, n_chunks}),
                     p.idx, p.k.per_block, p.h, (Gemv2Args{p.wd, p.wc2, p.part, counter, p.y, p.res, p.d_ffn, p.d_model, p.out_f32}));
  prof_end(prof, s);
  return hipGetLastError();
}
