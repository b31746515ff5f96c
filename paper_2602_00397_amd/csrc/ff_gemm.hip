// Gathered SwiGLU GEMMs on bf16 MFMA (v_mfma_f32_32x32x16_bf16), fp32 accumulate.
//
//   gemm1 (Eq. 15, 16, 18 and the first half of Eq. 20):
//       H[t][p] = bf16( SiLU(x_t . Wgate[idx_b[p]]) * (x_t . Wup[idx_b[p]]) )   p <  K_b
//       H[t][p] = bf16( act(x_t . Wc1[p - K_b]) )                    K_b <= p <  K_b + rc
//       H[t][p] = 0                                                   up to the next multiple of 64
//   gemm2 (Eq. 17, 18 and the second half of Eq. 20, the sum of Eq. 21):
//       Y[t][:] = sum_p H[t][p] * R_b[p][:],  R_b[p] = Wdown[idx_b[p]] for p < K_b,
//                                              R_b[p] = Wc2[p - K_b] for the compensator units.
// The compensator is thus rc extra, always selected, un-gated "neurons" appended to
// every block's list, and its add happens in the accumulator of gemm2.
// With idx == nullptr the list is 0..d_ffn-1 and the pair computes Eq. 10.
//
// Weight rows are gathered straight from the neuron-major matrices by per-thread row
// pointers; nothing is packed per block.  A workgroup owns all tokens of one block
// (or an M-slice of it) and a range of list positions (gemm1) or of output columns
// (gemm2).  Workgroup ids are mapped so that the ids one XCD receives (id mod 8) walk
// its position/column ranges in the same order over its group of blocks: blocks that
// selected the same weight rows then hit them in that XCD's L2.
#include "ff_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

// MFMA groups over which a two-stage ring spreads a stage's copies (all of them would leave the
// last copies no time to land before the next barrier; measured 1, 2, 3 of 4: 2 is best)
constexpr int kSpreadGroupsTwoStage = 2;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

__device__ __forceinline__ f32x16_t mfma32(const u32x4_t &a, const u32x4_t &b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// Workgroup id -> (virtual block, n tile).  The 8 XCDs (id mod 8) form a grid of XV = 2^xs groups of virtual
// blocks by 8 / XV groups of n tiles: XCD (xv, xn) owns virtual blocks xv, xv + XV, ... and n tiles xn,
// xn + 8/XV, ...; its ids enumerate its n tiles outermost, its blocks innermost.
struct TileCoord { int vb, nt; bool valid; };
__device__ __forceinline__ TileCoord map_tile(int w, int V, int N, int xs) {
  const int cnt = (V + (1 << xs) - 1) >> xs;
  const int xcd = w & 7, l = w >> 3;
  const int nl = l / cnt, j = l - nl * cnt;
  const int vb = (xcd & ((1 << xs) - 1)) + (j << xs), nt = (xcd >> xs) + (nl << (3 - xs));
  TileCoord t = {vb, nt, vb < V && nt < N};
  return t;
}

// Lists of unequal length.  The few blocks longer than the common length ("heavy": the first
// and last block when those stay dense) would otherwise leave their extra tiles for the end of
// the launch, all on the one XCD that owns the block, sharing weight rows with nobody.  Their
// tiles get the first ids instead (they start at once, next to everybody else's), and
// consecutive ids go to consecutive XCDs.
__device__ __forceinline__ int heavy_block(const KSpec &k, int h) {
  int b = k.heavy[0];
#pragma unroll
  for (int i = 1; i < kMaxHeavy; ++i) b = __builtin_amdgcn_readfirstlane((h == i) ? k.heavy[i] : b);   // keeps the chain scalar
  return b;
}
__device__ __forceinline__ bool is_heavy(const KSpec &k, int b) {
  bool r = false;
#pragma unroll
  for (int i = 0; i < kMaxHeavy; ++i) r = r || (i < k.n_heavy && k.heavy[i] == b);
  return r;
}

// which entry of heavy[] block b is, or -1
__device__ __forceinline__ int heavy_index(const KSpec &k, int b) {
  int r = -1;
#pragma unroll
  for (int i = 0; i < kMaxHeavy; ++i) r = (i < k.n_heavy && k.heavy[i] == b) ? i : r;
  return r;
}

// 16-byte chunk swizzle of a k-contiguous tile row: logical chunk q of row r is stored
// at chunk q ^ swz(r).  A ds_read_b128 of one chunk column over consecutive rows must
// spread over all banks both for 8 rows (128-byte bank window) and for 16 rows
// (256-byte window); rows of 64 B hold 4 chunks, rows of 128 B hold 8.  Period 16 rows.
template <int BK>
__device__ __forceinline__ int swz(int row) {
  return BK == 32 ? (((row >> 1) & 3) ^ ((row >> 3) & 1)) : (((row >> 1) & 7) ^ ((row & 1) << 2));
}

__device__ __forceinline__ int block_k(const KSpec &k, int b, int d_ffn, int k_stride, bool has_idx) {
  int K = k.per_block ? k.per_block[b] : k.uniform;
  K = max(1, min(K, d_ffn));
  if (has_idx) K = min(K, k_stride);
  return K;
}

__device__ __forceinline__ float act_apply(int act, float g) {
  if (act == FF_ACT_SILU) return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));   // 1-ulp reciprocal: far below bf16 rounding
  if (act == FF_ACT_RELU) return fmaxf(g, 0.0f);
  return g;
}

__device__ __forceinline__ u32x4_t mk4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  u32x4_t v = {a, b, c, d};
  return v;
}

// ---- asynchronous global -> LDS staging (gload_lds16, in the internal header) ----
// from a wave-uniform base plus a 32-bit byte offset per lane
__device__ __forceinline__ void gload_lds16_off(uint64_t base, uint32_t off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(lds_addr)
               : "memory");
}
// the 4-byte form: lane l lands at +4 l (256 bytes per wavefront instruction)
__device__ __forceinline__ void gload_lds4(const void *gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :
               : "v"(gptr), "s"(lds_addr)
               : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  // lgkmcnt(0): this wavefront's own LDS reads of the slot about to be refilled have completed
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// ============================ gemm1 =========================================
// The tile of gemm1 that a workgroup owns: BM tokens from t0 (rows_valid of them there), BN list positions from n0.
struct Gemm1Tile { int b, m, t0, rows_valid, Kb, ntot, n0; bool valid; };
template <int BM, int BN>
__device__ __forceinline__ Gemm1Tile gemm1_tile(const Gemm1Params &p, int V, int mt, int N, int xs, int NX) {
  Gemm1Tile t;
  t.valid = false;
  // ids [0, heavy virtual blocks x NX): the NX tiles beyond the common N of the heavy blocks;
  // then the common region, N tiles for every block
  TileCoord tc;
  const int n_first = p.k.n_heavy * mt * NX;
  if ((int)blockIdx.x < n_first) {
    const int h = __builtin_amdgcn_readfirstlane((int)blockIdx.x / NX);
    const int hb = __builtin_amdgcn_readfirstlane(h / mt);
    tc.vb = heavy_block(p.k, hb) * mt + (h - hb * mt);
    tc.nt = N + ((int)blockIdx.x - h * NX);
    tc.valid = true;
  } else {
    tc = map_tile((int)blockIdx.x - n_first, V, N, xs);
  }
  if (!tc.valid) return t;
  // wave-uniform by construction; say so, so that everything derived from it stays scalar
  tc.vb = __builtin_amdgcn_readfirstlane(tc.vb);
  tc.nt = __builtin_amdgcn_readfirstlane(tc.nt);
  t.b = tc.vb / mt;
  t.m = tc.vb - t.b * mt;
  t.t0 = t.b * p.block + t.m * BM;
  t.rows_valid = min(p.T, (t.b + 1) * p.block) - t.t0;
  if (t.rows_valid <= 0) return t;
  t.Kb = __builtin_amdgcn_readfirstlane(block_k(p.k, t.b, p.d_ffn, p.k_stride, p.idx != nullptr));
  const int ntot = t.ntot = t.Kb + p.rc;
  const int n0 = t.n0 = __builtin_amdgcn_readfirstlane(p.rem_bn ? min(ntot / p.rem_bn * p.rem_bn, p.rem_cap) : 0) + tc.nt * BN;
  // (H is zero up to the next multiple of 64: a tile narrower than that may hold nothing but zeros)
  if (n0 >= (BN < 64 ? (ntot + 63) / 64 * 64 : ntot)) return t;
  if (p.full_only && n0 + BN > ntot) return t;   // the remainder launch takes this part-filled tile
  if (p.skip_heavy && is_heavy(p.k, t.b)) return t;  // a launch of their own has covered the heavy blocks' ends
  t.valid = true;
  return t;
}

// KG groups of WM x WN wavefronts; a wavefront computes 32*TM tokens x 32*TN list positions
// for the gate and the up projection at once (the SiLU(g)*u epilogue is lane-local); with
// KG = 2 the two groups split each stage's k range and exchange halves of their
// accumulators through LDS at the end (fixed order, so results stay reproducible).
// Position p = wave_base + TN*c + f is held by MFMA tile f, column c, so a lane owns TN
// consecutive positions of a token row and H is written in contiguous runs.
// Operands stream through a ring of S LDS stages filled by asynchronous copies issued S-1
// k-steps ahead, one barrier per k-step.  A wave-load covers 1 KiB of a stage = 1024 / (2 BK)
// tile rows; lane l fills 16-byte slot l of it, and fetches the chunk that the read-side
// swizzle expects there.  BK = 64 makes every request a whole 128-byte line.
template <int WM, int WN, int TM, int TN, int BK, int S, int KG = 1>
__global__ __launch_bounds__(WM * WN * KG * 64) __attribute__((amdgpu_waves_per_eu(TM * TN * 2 <= 8 ? 2 : 1)))
void ff_gemm1_kernel(Gemm1Params p, int V, int mt, int N, int xs, int NX) {
  constexpr int NW = WM * WN * KG;                 // KG groups of WM x WN wavefronts split each stage's k range
  constexpr int BM = WM * TM * 32;
  constexpr int WNn = TN * 32;
  constexpr int BNn = WN * WNn;
  constexpr int CPR = BK / 8;
  constexpr int ROWB = BK * 2;
  constexpr int A_BYTES = BM * ROWB;
  constexpr int B_BYTES = 2 * BNn * ROWB;
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int RPL = 1024 / ROWB;                 // tile rows per wave-load
  constexpr int NL = STAGE / 1024;                 // wave-loads per stage
  constexpr int L = NL / NW;                       // wave-loads per wavefront per stage
  static_assert(NL % NW == 0, "stage must split evenly over the wavefronts");
  static_assert(A_BYTES % 1024 == 0 && BNn % RPL == 0, "A and B tiles must be whole wave-loads");
  extern __shared__ __align__(16) uint8_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = wave / (WM * WN), wq = wave % (WM * WN);
  const int wm = wq / WN, wn = wq % WN;
  const int c = lane & 31, half = lane >> 5;

  const Gemm1Tile tl = gemm1_tile<BM, BNn>(p, V, mt, N, xs, NX);
  if (!tl.valid) return;
  const int b = tl.b, m = tl.m, t0 = tl.t0, rows_valid = tl.rows_valid, Kb = tl.Kb, ntot = tl.ntot, n0 = tl.n0;

  // wave-load j = wave + i * NW of a stage covers stage bytes [1024 j, 1024 j + 1024)
  // list position of the B row that copy i of a stage fills (-1: an A row)
  auto b_pos = [&](int i) __attribute__((always_inline)) -> int {
    const int trow = (wave + i * NW) * RPL + lane / CPR;
    if (trow < BM) return -1;
    const int rp = (trow - BM) % BNn;
    return n0 + rp / WNn * WNn + TN * (rp & 31) + ((rp % WNn) >> 5);
  };
  // the list entries first, all loads in flight at once (from a clamped position, so that none is
  // conditional: left inside the branches below, every load is waited for before the next is issued)
  int entry[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int pos = b_pos(i);
    entry[i] = (p.idx != nullptr && pos >= 0) ? p.idx[(size_t)b * p.k_stride + min(pos, Kb - 1)] : pos;
  }
  __builtin_amdgcn_sched_barrier(0);
  // A wave-load is of X or of one matrix (RPL divides both tiles): where its rows start, and which row and chunk this lane takes
  uint64_t from[L];
  int row[L];
  uint32_t is_comp = 0;                              // bit i: a compensator unit's row instead
  auto chunk_of = [&](int i) __attribute__((always_inline)) -> int {
    const int trow = (wave + i * NW) * RPL + lane / CPR;
    return (lane % CPR) ^ swz<BK>(trow);             // BM is a multiple of 32: the B rows keep the swizzle phase
  };
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int trow0 = (wave + i * NW) * RPL;         // row within the stage (A rows, then B rows) of lane 0
    if (trow0 < BM) {
      from[i] = (uint64_t)(uintptr_t)(p.x + (size_t)t0 * p.d_model);
      row[i] = min(trow0 + lane / CPR, rows_valid - 1);
    } else {
      from[i] = (uint64_t)(uintptr_t)((trow0 - BM) / BNn ? p.wu : p.wg);
      const int pos = b_pos(i);
      row[i] = 0;
      if (pos < Kb) {
        row[i] = min(max(entry[i], 0), p.d_ffn - 1);
      } else if (pos < ntot) {
        row[i] = pos - Kb;
        is_comp |= 1u << i;
      }
    }
  }
  const uint32_t lds0 = lds_addr_of(smem);
  f32x16_t accg[TM][TN], accu[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) { accg[i][j][e] = 0.0f; accu[i][j][e] = 0.0f; }

  // Pipeline.  Stage kt+1 is waited for (and the workgroup synchronised) in front of the LAST
  // MFMA group of stage kt, and the first fragments of stage kt+1 are requested from LDS there, so
  // the matrix pipe has work while they arrive.  After that barrier every wavefront is done reading
  // stage kt, so its ring slot takes the copies of stage kt+S: they are issued one at a time
  // between the MFMAs of the next KQ groups (a burst would park the wavefront on a full
  // memory-issue queue with its matrix pipe idle).
  // FAST: all rows are list rows, and their offsets have 32 bits (p.off32): a scalar address and the lane's offset per copy.
  // (Added up in 64 bits in the loop: a dense gate/up launch of 4096 tokens 785 us, this way 755.)
  auto run = [&](auto fast_tag) __attribute__((always_inline)) {
  constexpr bool FAST = decltype(fast_tag)::value;
  uint32_t off[L];
  uint64_t base[L];
  const bf16_t *src[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    if (FAST) {
      off[i] = (uint32_t)row[i] * ((uint32_t)p.d_model * 2u) + (uint32_t)chunk_of(i) * 16u;
      base[i] = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)from[i]) |
                (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(from[i] >> 32)) << 32;   // wave-uniform by construction
    } else src[i] = reinterpret_cast<const bf16_t *>((is_comp >> i) & 1u ? (uint64_t)(uintptr_t)p.wc1 : from[i]) + (size_t)row[i] * p.d_model + chunk_of(i) * 8;
  }
  // (p.spread: the workgroups walk the channels from different places)
  const int first = p.spread ? __builtin_amdgcn_readfirstlane((int)(blockIdx.x >> 3) * 5 % (p.d_model / BK)) : 0;
  // slot: which stage of the ring (kt mod S)
  auto issue_one = [&](int kt, int slot, int i) __attribute__((always_inline)) {
    const uint32_t st = lds0 + (uint32_t)slot * STAGE + (uint32_t)(wave + i * NW) * 1024u;
    const int at = kt + first;
    int k = at >= p.d_model / BK ? at - p.d_model / BK : at;
    asm("" : "+s"(k));                                 // (a scalar: the choice is not made lane by lane, offset by offset)
    if (FAST) gload_lds16_off(base[i], off[i] + (uint32_t)(k * BK * 2), st);
    else gload_lds16(src[i] + k * BK, st);
  };
  auto issue = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < L; ++i) issue_one(kt, kt % S, i);
  };
  constexpr int KQ = BK / 16 / KG;                     // MFMA groups (16 k each) per stage and k-group
  static_assert(KQ % 2 == 0, "fragment double buffer needs an even number of groups per stage");
  constexpr int NMF = TM * TN;                         // gate/up MFMA pairs per group
  constexpr int NSP = S == 2 ? (kSpreadGroupsTwoStage < KQ ? kSpreadGroupsTwoStage : KQ) : KQ;  // groups the copies of a stage are spread over
  constexpr int LQ = (L + NSP - 1) / NSP;              // copies issued during one group
  constexpr int PER = (LQ + NMF - 1) / NMF;            // copies behind one MFMA pair
  constexpr int EVERY = NMF / LQ > 0 ? NMF / LQ : 1;
  constexpr int SLOTS = (NMF + EVERY - 1) / EVERY * PER;  // copy slots between the MFMAs of a group
  const int nk = p.d_model / BK;
  u32x4_t af[2][TM], bg[2][TN], bu[2][TN];
  auto frags = [&](int slot, int kq, int buf) __attribute__((always_inline)) {
    const uint8_t *cur = smem + slot * STAGE;
    const int q = 2 * (kgrp * KQ + kq) + half;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = (wm * TM + i) * 32 + c;
      af[buf][i] = *reinterpret_cast<const u32x4_t *>(cur + row * ROWB + ((q ^ swz<BK>(row)) << 4));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int rho = wn * WNn + j * 32 + c;
      const int off = rho * ROWB + ((q ^ swz<BK>(rho)) << 4);
      bg[buf][j] = *reinterpret_cast<const u32x4_t *>(cur + A_BYTES + off);
      bu[buf][j] = *reinterpret_cast<const u32x4_t *>(cur + A_BYTES + BNn * ROWB + off);
    }
  };
  // MFMA group kq of the current stage from fragment buffer kq & 1, with part `part` (of KQ) of
  // stage `st`'s copies issued in between when `load` is set
  auto group = [&](int kq, int st, int slot, int part, bool load) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        accg[i][j] = mfma32(af[kq & 1][i], bg[kq & 1][j], accg[i][j]);
        accu[i][j] = mfma32(af[kq & 1][i], bu[kq & 1][j], accu[i][j]);
        if ((i * TN + j) % EVERY == 0) {
#pragma unroll
          for (int r = 0; r < PER; ++r) {
            const int n = (i * TN + j) / EVERY * PER + r;
            if (n < LQ && part * LQ + n < L) {
              if (load) issue_one(st, slot, part * LQ + n);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
#pragma unroll
    for (int n = SLOTS; n < LQ; ++n)
      if (load && part * LQ + n < L) issue_one(st, slot, part * LQ + n);
    __builtin_amdgcn_sched_barrier(0);
  };
  // MAIN: stages kt+S-1 and kt+S both exist (no conditions in the loop body).  slot = kt mod S, a constant in the main loop of
  // rings of three, which is unrolled (1000 tokens of 4096/14336 in blocks of 128, K 7168: 127.7 -> 125.5 us; a ring of two
  // has stages of 64 KB, beyond what an LDS address adds at once: 760 -> 765 for 4096 dense tokens).
  auto step = [&](int kt, auto main_tag, auto slot_) __attribute__((always_inline)) {
    constexpr bool MAIN = decltype(main_tag)::value;
    const int slot = slot_, next = (slot + 1) % S, prev = (slot + S - 1) % S;
    const bool la = MAIN || kt + S - 1 < nk;
    const bool lb = MAIN || kt + S < nk;
#pragma unroll
    for (int kq = 0; kq < KQ - 1; ++kq) {
      frags(slot, kq + 1, (kq + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      group(kq, kt + S - 1, prev, kq + 1, la);
    }
    if (MAIN || kt + 1 < nk) {
      // stage kt+1 must have landed; stages kt+2 .. kt+S-1 may still be in flight
      if (MAIN || kt + S - 1 < nk) wait_vm_barrier<(S - 2) * L>(); else wait_vm_barrier<0>();
      frags(next, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    group(KQ - 1, kt + S, slot, 0, lb);
  };
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) issue(s);
  if (S - 1 <= nk) wait_vm_barrier<(S - 2) * L>(); else wait_vm_barrier<0>();
  if (S - 1 < nk) {
#pragma unroll
    for (int i = 0; i < (LQ < L ? LQ : L); ++i) issue_one(S - 1, S - 1, i);
  }
  frags(0, 0, 0);
  const int n_main = max(nk - S, 0);
  int kt = 0;
  if (S == 3) {
    for (; kt + S <= n_main; kt += S) {
      step(kt, std::true_type{}, std::integral_constant<int, 0>{});
      step(kt + 1, std::true_type{}, std::integral_constant<int, 1>{});
      step(kt + 2, std::true_type{}, std::integral_constant<int, 2>{});
    }
  } else {
    for (; kt < n_main; ++kt) step(kt, std::true_type{}, kt % S);
  }
  for (; kt < nk; ++kt) step(kt, std::false_type{}, kt % S);
  };
  if (p.off32 && n0 + BNn <= Kb) run(std::true_type{}); else run(std::false_type{});

  // k-groups: group g keeps token tiles i with i % KG == g and hands the others over through LDS
  if (KG > 1) {
    static_assert(KG == 1 || (KG == 2 && TM % 2 == 0), "two k-groups need an even number of token tiles per wavefront");
    static_assert(KG == 1 || S * STAGE >= WM * WN * 2 * (TM / 2) * TN * 2 * 16 * 64 * 4, "ring too small for the hand-over");
    __syncthreads();                                    // everyone is done with the ring
    float *red = reinterpret_cast<float *>(smem);
    constexpr int PER = (TM / 2) * TN * 2 * 4;          // float4 slots a wavefront hands over
    const int slot0 = ((kgrp * (WM * WN) + wq) * PER) * 64 + lane;
    int sl = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if ((i & 1) != kgrp) {                            // token tiles the other group keeps
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            reinterpret_cast<float4 *>(red)[slot0 + (sl++) * 64] = make_float4(accg[i][j][4 * e4], accg[i][j][4 * e4 + 1], accg[i][j][4 * e4 + 2], accg[i][j][4 * e4 + 3]);
            reinterpret_cast<float4 *>(red)[slot0 + (sl++) * 64] = make_float4(accu[i][j][4 * e4], accu[i][j][4 * e4 + 1], accu[i][j][4 * e4 + 2], accu[i][j][4 * e4 + 3]);
          }
      }
    __syncthreads();
    const int other0 = (((1 - kgrp) * (WM * WN) + wq) * PER) * 64 + lane;
    sl = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if ((i & 1) == kgrp) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            const float4 g4 = reinterpret_cast<const float4 *>(red)[other0 + (sl++) * 64];
            const float4 u4 = reinterpret_cast<const float4 *>(red)[other0 + (sl++) * 64];
            accg[i][j][4 * e4] += g4.x; accg[i][j][4 * e4 + 1] += g4.y; accg[i][j][4 * e4 + 2] += g4.z; accg[i][j][4 * e4 + 3] += g4.w;
            accu[i][j][4 * e4] += u4.x; accu[i][j][4 * e4 + 1] += u4.y; accu[i][j][4 * e4 + 2] += u4.z; accu[i][j][4 * e4 + 3] += u4.w;
          }
      }
  }

  const int pos0 = n0 + wn * WNn + TN * c;
  // the usual tile: every position a selected neuron of every token row (no compensator unit, no padding, no masks)
  const bool plain = p.mask == nullptr && n0 + BNn <= Kb;
  if (pos0 < p.hs) {
    // merged lists: which sub-blocks' rows each of this lane's positions belongs to (all of them otherwise)
    uint32_t member[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
      member[j] = (p.mask != nullptr && pos0 + j < Kb) ? (uint32_t)p.mask[(size_t)b * p.k_stride + pos0 + j] : 0xffffffffu;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if (KG == 1 || (i & 1) == kgrp)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rowl = (wm * TM + i) * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
        if (rowl < rows_valid) {
          const int sub = p.mask != nullptr ? ((m * BM + rowl) >> p.sub_shift) : 0;
          float hv[TN];
          if (plain) {
#pragma unroll
            for (int j = 0; j < TN; ++j) hv[j] = act_apply(FF_ACT_SILU, accg[i][j][e]) * accu[i][j][e];
          } else {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              const int pos = pos0 + j;
              const float g = accg[i][j][e], u = accu[i][j][e];
              hv[j] = pos < Kb ? act_apply(FF_ACT_SILU, g) * u : (pos < ntot ? act_apply(p.comp_act, g) : 0.0f);
              if (!((member[j] >> sub) & 1u)) hv[j] = 0.0f;
            }
          }
          bf16_t *dst = p.h + (size_t)(t0 + rowl) * p.hs + pos0;
          if (TN == 1) {
            dst[0] = f32_to_bf16(hv[0]);
          } else {
#pragma unroll
            for (int j = 0; j < TN; j += 2)
              *reinterpret_cast<uint32_t *>(dst + j) = pack_bf16x2(hv[j], hv[j + 1]);
          }
        }
      }
  }
}

// The same product with the gathered rows loaded straight into registers.  With both operands in LDS a step's LDS traffic
// (272 KB per 64 k of a 128 x 256 tile) took three quarters of the time of its MFMAs and did not overlap with them to the full
// (the chip is at its power limit); here only X passes through LDS (144 KB).  Eight wavefronts side by side, 32 positions of
// both projections each for all 128 tokens: nobody else in the workgroup wants a wavefront's weights.
// The k-loop walks along the gathered rows, so an MFMA operand (32x32x16: lane (c, half) holds eight k of row c) loaded as it
// is has every lane at a row of its own, and the address unit takes one lane per cycle then; four lanes that ask for 64
// contiguous bytes go together (L2-resident rows, 256 workgroups: 30 TB/s by fours, 18 by twos, 9 one by one).  So load j of a
// step (64 k) takes rows j + 4 ((lane / 4) mod 8), lanes 0 .. 3 and 32 .. 35 the eight 16-byte chunks of one, and two rounds
// of exchanges inside the fours (transpose4) turn the four loads of 32 rows into the operands of four MFMA groups: group g
// has chunk g in the lower half of the wavefront and chunk g + 4 in the upper.  The order of k inside a step is free as long
// as X is read in the same one.
// Measured, both operands in LDS against this (one MI355X, 4096/14336): 64 blocks of 128, K 7168, both launches 839 -> 809 us;
// 64 blocks of 64, K 3584 398 -> 325, K 7168 698 -> 645; 16384 tokens of 3584/18944, four layers 7640 -> 7410.  With 128 tokens
// the chip's power and the issue of instructions bind: without the weights' loads 8% less, without X's copies 6%, without the
// exchanges 3%, MFMAs alone three quarters; 64-bit additions for the loads' addresses cost 3%, two idle cycles around every
// exchange 0.7%.  With 64 tokens the loads from beyond L2 do: each row serves 64 tokens.
// Tiles whose 32 rows of a wavefront are all list rows take 32-bit offsets from the two matrices; compensator units and
// padding find their matrix lane by lane.
constexpr int kDirectStages = 4, kDirectWaves = 8;
template <int MT, int WN, int NBUF>
__global__ __launch_bounds__(WN * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ff_gemm1_direct_kernel(Gemm1Params p, int V, int mt, int N, int xs, int NX) {
  constexpr int BM = MT * 32, BN = WN * 32, S = kDirectStages, STAGE = BM * 128, D = 4, LA = BM / 8 / WN;
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, half = lane >> 5;
  const Gemm1Tile tl = gemm1_tile<BM, BN>(p, V, mt, N, xs, NX);
  if (!tl.valid) return;
  const int Kb = tl.Kb, ntot = tl.ntot, rows_valid = tl.rows_valid;
  const int nk = p.d_model / 64, last = nk - 1;
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;

  // X: copy i of a stage covers rows 8 (wave + i WN) .. + 7
  const uint64_t a_base = (uint64_t)(uintptr_t)(p.x + (size_t)tl.t0 * p.d_model);
  uint32_t a_off[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int trow = (wave + i * WN) * 8 + lane / 8;
    a_off[i] = (uint32_t)min(trow, rows_valid - 1) * row_bytes + (uint32_t)((lane & 7) ^ swz<64>(trow)) * 16u;
  }
  const uint32_t lds0 = lds_addr_of(smem);
  // (no conditions in the loop: past the end the last step is requested again, into a slot nobody reads any more)
  auto issue_a = [&](int st, int i) __attribute__((always_inline)) {
    gload_lds16_off(a_base + (uint64_t)(uint32_t)min(st, last) * 128u, a_off[i], lds0 + (uint32_t)(st % S) * STAGE + (uint32_t)(wave + i * WN) * 1024u);
  };
#pragma unroll
  for (int st = 0; st < NBUF; ++st)
#pragma unroll
    for (int i = 0; i < LA; ++i) issue_a(st, i);

  // this lane's rows: position nw + j + 4 lr in load j
  const int nw = tl.n0 + wave * 32;
  const int lr = (lane >> 2) & 7, chunk = (lane & 3) + 4 * half;
  const bool fast = nw + 32 <= Kb;
  uint32_t w_off[4];            // fast, or a list row: offset into both matrices; else into wc1 (or, past the lists' end, of row 0)
  uint32_t is_comp = 0;         // bit j: row j is a compensator unit's
  {
    int entry[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int pos = nw + j + 4 * lr;
      entry[j] = p.idx != nullptr ? p.idx[(size_t)tl.b * p.k_stride + min(pos, Kb - 1)] : pos;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int pos = nw + j + 4 * lr;
      int row = 0;
      if (pos < Kb) {
        row = min(max(entry[j], 0), p.d_ffn - 1);
      } else if (pos < ntot) {
        row = pos - Kb;
        is_comp |= 1u << j;
      }
      w_off[j] = (uint32_t)row * row_bytes + (uint32_t)chunk * 16u;
    }
  }

  f32x16_t acc[MT][2];                        // [token tile][gate, up]
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][f][e] = 0.0f;

  typedef const __attribute__((address_space(1))) u32x4_t *gptr_t;
  u32x4_t wb[NBUF][2][4];                     // [step mod NBUF][gate, up]: loads j, then (transposed) the operands of group g
  u32x4_t af[D];                              // ring of token fragments
  auto load_w = [&](int kt, int buf, int f, int j, auto fast_tag) __attribute__((always_inline)) {
    const uint32_t ko = (uint32_t)min(kt, last) * 128u;
    uintptr_t base = (uintptr_t)(f ? p.wu : p.wg) + ko;
    if (decltype(fast_tag)::value) {
      uint32_t off = w_off[j];
      asm("" : "+v"(off));                    // a scalar base and the lane's 32-bit offset: no address arithmetic in the loop
      wb[buf][f][j] = *(gptr_t)(base + off);
    } else {
      if ((is_comp >> j) & 1u) base = (uintptr_t)p.wc1 + ko;
      wb[buf][f][j] = *(gptr_t)(base + w_off[j]);
    }
  };
  uint32_t aoff[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) aoff[g] = (uint32_t)(c * 128 + (((g + 4 * half) ^ swz<64>(c)) << 4));
  // fragment n of a step: group n / MT, token tile n % MT
  auto frag = [&](int kt, int n) __attribute__((always_inline)) {
    af[n % D] = *reinterpret_cast<const u32x4_t *>(smem + (kt % S) * STAGE + aoff[n / MT] + (n % MT) * 4096);
  };
  // One step of 64 k from buffer kt mod NBUF.  As a group's MFMAs are out, loads of step kt + NBUF take its registers; in the
  // second half the next buffer's loads (step kt + 1) are transposed; in front of the last D fragments the workgroup makes
  // sure that X of step kt + 1 has landed, and behind that X of step kt + NBUF is requested, in front of the step's last two
  // loads.  Requests complete in order, so the wait for X names how many younger ones may still be on their way: all of them.
  // The slot of X requested in a step was last read in step kt + NBUF - S, hence by nobody who has passed this step's barrier.
  constexpr int NF = 4 * MT, TR0 = NF / 2;
  constexpr int NEWER = 2 + 2 * ((NF - D) / MT) + (NBUF - 2) * (8 + LA);
  static_assert(NBUF < S && (NF - D) % MT == 0, "ring of X");
  // END: the steps behind the unrolled loop of three buffers.  Their loads would be for steps that do not exist, so there are none, and the wait
  // for X cannot count on them.
  auto step = [&](int kt, auto buf_tag, auto fast_tag, auto end_tag) __attribute__((always_inline)) {
    constexpr int buf = decltype(buf_tag)::value;
    constexpr bool END = decltype(end_tag)::value;
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      const int g = n / MT, i = n % MT;
      if (n == NF - D) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(END ? 0 : NEWER) : "memory");
      const u32x4_t a = af[n % D];
#pragma unroll
      for (int f = 0; f < 2; ++f) acc[i][f] = mfma32(a, wb[buf][f][g], acc[i][f]);
      __builtin_amdgcn_sched_barrier(0);
      if (n + D < NF) frag(kt, n + D); else frag(kt + 1, n + D - NF);
      if (n >= NF - 1 - LA && n < NF - 1) issue_a(kt + NBUF, n - (NF - 1 - LA));
      if (n >= TR0) {
        constexpr int PER = 8 / (NF - TR0);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
          const int x = (n - TR0) * PER + q;
          if (x < 7) transpose4<false>(wb[(buf + 1) % NBUF][x / 4], x % 4); else transpose4<true>(wb[(buf + 1) % NBUF][x / 4], x % 4);
        }
      }
      if (!END && i == MT - 1) {
        load_w(kt + NBUF, buf, 0, g, fast_tag);
        load_w(kt + NBUF, buf, 1, g, fast_tag);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto run = [&](auto fast_tag) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < NBUF; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        load_w(st, st, 0, j, fast_tag);
        load_w(st, st, 1, j, fast_tag);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < 8; ++x) transpose4<true>(wb[0][x / 4], x % 4);
    asm volatile("s_barrier" ::: "memory");            // (the copies of the first two steps are older than those loads)
#pragma unroll
    for (int n = 0; n < D; ++n) frag(0, n);
    __builtin_amdgcn_sched_barrier(0);
    int kt = 0;
    constexpr std::integral_constant<int, 0> b0{};
    constexpr std::integral_constant<int, 1> b1{};
    constexpr std::integral_constant<int, NBUF - 1> b2{};
    for (; kt + NBUF <= nk; kt += NBUF) {
      step(kt, b0, fast_tag, std::false_type{});
      step(kt + 1, b1, fast_tag, std::false_type{});
      if (NBUF == 3) step(kt + 2, b2, fast_tag, std::false_type{});
    }
    if constexpr (NBUF == 3) {                         // (d_model is a multiple of 128: two buffers leave no step over)
      if (kt < nk) step(kt, b0, fast_tag, std::true_type{});
      if (kt + 1 < nk) step(kt + 1, b1, fast_tag, std::true_type{});
    }
  };
  if (fast) run(std::true_type{}); else run(std::false_type{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies requested past the end

  // Lane (c, half) holds position nw + c of rows 8 (e / 4) + 4 half + e mod 4.  Neighbouring lanes exchange one of two
  // rows, so that each stores two adjacent positions of one row.
  const int pos = nw + c, odd = c & 1;
  if (nw >= p.hs) return;                     // (hs is a multiple of 64)
  const bool plain = p.mask == nullptr && fast;
  const uint32_t member = (p.mask != nullptr && pos < Kb) ? (uint32_t)p.mask[(size_t)tl.b * p.k_stride + pos] : 0xffffffffu;
  const uint32_t pick = odd ? 0x03020706u : 0x05040100u;
  bf16_t *dst0 = p.h + (size_t)tl.t0 * p.hs + (pos - odd);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const int row0 = i * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
      float hv[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const float gt = acc[i][0][e + r], up = acc[i][1][e + r];
        if (plain) {
          hv[r] = act_apply(FF_ACT_SILU, gt) * up;
        } else {
          hv[r] = pos < Kb ? act_apply(FF_ACT_SILU, gt) * up : (pos < ntot ? act_apply(p.comp_act, gt) : 0.0f);
          if (p.mask != nullptr && !((member >> ((tl.m * BM + row0 + r) >> p.sub_shift)) & 1u)) hv[r] = 0.0f;
        }
      }
      const uint32_t mine = pack_bf16x2(hv[0], hv[1]);
      const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xf, 0xf, true);   // lane c ^ 1
      if (row0 + odd < rows_valid)
        *reinterpret_cast<uint32_t *>(dst0 + (size_t)(row0 + odd) * p.hs) = __builtin_amdgcn_perm(other, mine, pick);
    }
}

// The compensator's first layer (Eq. 20) where the units start a tile of their own behind lists of equal length: then they are the
// same columns of H for every token, and blocks mean nothing.
//     H[t][K + u] = act(x_t . Wc1[u]), u0 <= u < rc; zero up to the next multiple of 64.
// A workgroup takes 32 MT tokens and BU units, its eight wavefronts an eighth of the channels each, so that a wavefront has only
// few steps to wait for, two on their way; their sums are added in wavefront order.  The workgroups start at different steps,
// for rows that lie a multiple of 4 KB apart keep all lines of a step in one channel of the L2.  Rows are loaded by fours of lanes
// and exchanged, as in ff_gemm1_direct_kernel.  Bound by the exchanges and the rows' way from L2.
// (As 64 x 64 tiles of the gate/up kernel, half of whose products nobody wants, us -> this: 4096 tokens of 2048, 32 units 16.8 -> 8.8;
// 8192 of 4096, 64 units 28.9 -> 21.2.)
// grid (ceil(T / (32 MT)), tiles of BU units)
template <int MT, int BU>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void ff_comp_kernel(Gemm1Params p, int K, int u0) {
  constexpr int NW = 8, NU = BU / 32, U = 2, BM = 32 * MT;
  __shared__ __align__(16) float red[NW][BM][BU];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, half = lane >> 5;
  const int lr = (lane >> 2) & 7, chunk = (lane & 3) + 4 * half;
  const int t0 = (int)blockIdx.x * BM, unit0 = u0 + (int)blockIdx.y * BU;
  const int rows_valid = min(BM, p.T - t0);
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const int nk = p.d_model / 64, per = (nk + NW - 1) / NW, s0 = min(wave * per, nk), n = min(per, nk - s0);   // this wavefront's steps
  const int rot = n > 0 ? ((int)blockIdx.x >> 3) % n : 0;
  typedef const __attribute__((address_space(1))) u32x4_t *gptr_t;
  const uintptr_t xbase = (uintptr_t)(p.x + (size_t)t0 * p.d_model), wbase = (uintptr_t)p.wc1;
  uint32_t x_off[MT][4], w_off[NU][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int i = 0; i < MT; ++i) x_off[i][j] = (uint32_t)min(32 * i + j + 4 * lr, rows_valid - 1) * row_bytes + (uint32_t)chunk * 16u;
#pragma unroll
    for (int f = 0; f < NU; ++f) w_off[f][j] = (uint32_t)min(unit0 + 32 * f + j + 4 * lr, p.rc - 1) * row_bytes + (uint32_t)chunk * 16u;   // past the end: not stored
  }
  u32x4_t xb[U][MT][4], wb[U][NU][4];
  auto load = [&](int i, int buf) __attribute__((always_inline)) {
    const uint32_t ko = (uint32_t)(s0 + (i + rot < n ? i + rot : i + rot - n)) * 128u;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int j = 0; j < 4; ++j) xb[buf][m][j] = *(gptr_t)(xbase + ko + x_off[m][j]);
#pragma unroll
    for (int f = 0; f < NU; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) wb[buf][f][j] = *(gptr_t)(wbase + ko + w_off[f][j]);
  };
  f32x16_t acc[MT][NU];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int f = 0; f < NU; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[m][f][e] = 0.0f;
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (i < n) load(i, i);
  for (int i0 = 0; i0 < n; i0 += U) {
#pragma unroll
    for (int b = 0; b < U; ++b)
      if (i0 + b < n) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int d = 0; d < 4; ++d) transpose4<true>(xb[b][m], d);
#pragma unroll
        for (int f = 0; f < NU; ++f)
#pragma unroll
          for (int d = 0; d < 4; ++d) transpose4<true>(wb[b][f], d);
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int f = 0; f < NU; ++f) acc[m][f] = mfma32(xb[b][m][g], wb[b][f][g], acc[m][f]);
        if (i0 + b + U < n) load(i0 + b + U, b);
      }
  }
  // lane (c, half) holds unit 32 f + c of tokens 32 m + 8 (e / 4) + 4 half + e mod 4
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int f = 0; f < NU; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave][32 * m + 8 * (e >> 2) + 4 * half + (e & 3)][32 * f + c] = acc[m][f][e];
  __syncthreads();
  constexpr int PER = BU / 16;                                          // adjacent units per thread
  const int u = (tid & 15) * PER;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int t = 32 * m + (tid >> 4);
    if (t >= rows_valid) return;
    float v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) v[q] = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int q = 0; q < PER; ++q) v[q] += red[w][t][u + q];
    bf16_t *dst = p.h + (size_t)(t0 + t) * p.hs + K + unit0 + u;
#pragma unroll
    for (int q = 0; q < PER; ++q) v[q] = unit0 + u + q < p.rc ? act_apply(p.comp_act, v[q]) : 0.0f;
#pragma unroll
    for (int q = 0; q < PER; q += 2) *reinterpret_cast<uint32_t *>(dst + q) = pack_bf16x2(v[q], v[q + 1]);
    if (BU == 32) *reinterpret_cast<uint32_t *>(dst + 32) = 0u;          // (the other half of the 64 that H has behind the lists)
  }
}

// Four adjacent outputs of one token row on their way out of the down projection: Y in fp32, Y in
// bf16, or the stack's residual add (the same two roundings as a bf16 Y followed by a separate add;
// every element of res is read and written by one lane only).  o = element offset of the first.
__device__ __forceinline__ void store_out4(const Gemm2Params &p, size_t o, float4 v) {
  if (p.res) {
    uint2 *hp = reinterpret_cast<uint2 *>(p.res + o);
    const uint2 hv = *hp;
    const float y0 = bf16_to_f32(f32_to_bf16(v.x)), y1 = bf16_to_f32(f32_to_bf16(v.y));
    const float y2 = bf16_to_f32(f32_to_bf16(v.z)), y3 = bf16_to_f32(f32_to_bf16(v.w));
    *hp = make_uint2(pack_bf16x2(bf16_to_f32((bf16_t)(hv.x & 0xffffu)) + y0, bf16_to_f32((bf16_t)(hv.x >> 16)) + y1),
                     pack_bf16x2(bf16_to_f32((bf16_t)(hv.y & 0xffffu)) + y2, bf16_to_f32((bf16_t)(hv.y >> 16)) + y3));
  } else if (p.out_f32) {
    *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.y) + o) = v;
  } else {
    *reinterpret_cast<uint2 *>(reinterpret_cast<bf16_t *>(p.y) + o) =
        make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
  }
}

// The pieces of the lists that were cut along k, added in piece order (Eq. 17, 21: the same sum in a
// fixed, documented order).  One workgroup per token row of a heavy block and 1024 columns; a thread takes
// four columns and has all pieces' loads in flight before the first add.
constexpr int kMaxPieces = 17;
__global__ __launch_bounds__(256) void ff_gemm2_reduce_kernel(Gemm2Params p) {
  const bool all = p.n_split > 1;
  const int hslot = all ? 0 : (int)blockIdx.x / p.block, r = (int)blockIdx.x - hslot * p.block;
  const int t = all ? r : heavy_block(p.k, hslot) * p.block + r;
  if (t >= p.T) return;
  const int n_pieces = all ? p.n_split : p.n_pieces;
  const size_t piece_stride = (size_t)(all ? p.T : p.block) * p.d_model;
  const float *src = p.part + ((size_t)hslot * p.n_pieces * p.block + r) * p.d_model;
  const int c = p.col0 + 1024 * (int)blockIdx.y + 4 * (int)threadIdx.x;
  if (c < p.d_model) {
    float4 v[kMaxPieces];
#pragma unroll
    for (int j = 0; j < kMaxPieces; ++j)
      if (j < n_pieces) v[j] = *reinterpret_cast<const float4 *>(src + j * piece_stride + c);
    __builtin_amdgcn_sched_barrier(0);
    float4 s = v[0];
#pragma unroll
    for (int j = 1; j < kMaxPieces; ++j)
      if (j < n_pieces) { s.x += v[j].x; s.y += v[j].y; s.z += v[j].z; s.w += v[j].w; }
    store_out4(p, (size_t)t * p.d_model + c, s);
  }
}

// ============================ gemm2 =========================================
// The tile of gemm2 that a workgroup owns: BM tokens from t0, BN output columns from n0, nk steps of BK list positions
// from kofs (a multiple of 64; no steps gives zeros).  piece: which piece of a cut list (-1: a whole list), hslot:
// which heavy block.
struct Gemm2Tile { int b, m, t0, rows_valid, Kb, ntot, n0, kofs, nk, piece, hslot; bool valid; };
template <int BM, int BN, int BK>
__device__ __forceinline__ Gemm2Tile gemm2_tile(const Gemm2Params &p, int V, int mt, int N, int xs) {
  Gemm2Tile t;
  t.valid = false;
  // The heavy blocks' tiles (the longest k loops) take the first ids, then everybody else's.  With
  // n_pieces > 0 a heavy block's list is cut along k instead: its first cut0 positions are a tile like
  // everybody else's (piece 0, in the common region), the rest goes to n_pieces - 1 short tiles of
  // piece_len positions with the first ids, and every piece writes fp32 partial sums that
  // ff_gemm2_reduce_kernel adds up in a fixed order.
  TileCoord tc;
  const int n_surplus = p.n_pieces > 0 ? p.n_pieces - 1 : 1;
  const int n_first = p.k.n_heavy * mt * N * n_surplus;
  int piece = -1, hslot = 0;   // piece of a cut list (-1: a whole list), and which heavy block
  if ((int)blockIdx.x < n_first) {
    // id = ((surplus piece * heavy virtual blocks) + heavy virtual block) * N + column tile
    const int hv = p.k.n_heavy * mt;
    const int hn = __builtin_amdgcn_readfirstlane((int)blockIdx.x / N);
    const int sp = __builtin_amdgcn_readfirstlane(hn / hv);
    const int h = hn - sp * hv;
    hslot = __builtin_amdgcn_readfirstlane(h / mt);
    tc.vb = heavy_block(p.k, hslot) * mt + (h - hslot * mt);
    tc.nt = (int)blockIdx.x - hn * N;
    tc.valid = true;
    if (p.n_pieces > 0) piece = 1 + sp;
  } else {
    tc = map_tile((int)blockIdx.x - n_first, V, N, xs);
    if (p.n_split > 1) {   // every list is cut: N counts (piece, column tile) pairs
      piece = tc.nt / p.n_cols;
      tc.nt -= piece * p.n_cols;
    }
    if (tc.valid && p.k.n_heavy > 0) {
      const int hi = heavy_index(p.k, tc.vb / mt);
      if (hi >= 0) {
        if (p.n_pieces == 0) return t;
        piece = 0;
        hslot = hi;
      }
    }
  }
  if (!tc.valid) return t;
  tc.vb = __builtin_amdgcn_readfirstlane(tc.vb);   // wave-uniform by construction
  tc.nt = __builtin_amdgcn_readfirstlane(tc.nt);
  piece = __builtin_amdgcn_readfirstlane(piece);
  hslot = __builtin_amdgcn_readfirstlane(hslot);
  t.b = tc.vb / mt;
  t.m = tc.vb - t.b * mt;
  t.t0 = t.b * p.block + t.m * BM;
  t.rows_valid = min(p.T, (t.b + 1) * p.block) - t.t0;
  if (t.rows_valid <= 0) return t;
  t.Kb = __builtin_amdgcn_readfirstlane(block_k(p.k, t.b, p.d_ffn, p.k_stride, p.idx != nullptr));
  t.ntot = t.Kb + p.rc;
  const int ntot = t.ntot;
  t.n0 = p.col0 + tc.nt * BN;
  // list positions [kofs, kend) of this tile (kofs a multiple of 64; an empty range gives zeros)
  int kofs = 0, kend = ntot;
  if (p.n_split > 1) {
    const int len = ((ntot + p.n_split - 1) / p.n_split + 63) / 64 * 64;
    kofs = min(piece * len, (ntot + 63) / 64 * 64);
    kend = min(ntot, (piece + 1) * len);
  } else if (piece == 0) {
    kend = min(ntot, p.cut0);
  } else if (piece > 0) {
    kofs = min(p.cut0 + (piece - 1) * p.piece_len, (ntot + 63) / 64 * 64);
    kend = min(ntot, p.cut0 + piece * p.piece_len);
  }
  t.kofs = __builtin_amdgcn_readfirstlane(kofs);
  t.nk = __builtin_amdgcn_readfirstlane(max(kend - kofs + BK - 1, 0) / BK);
  t.piece = piece;
  t.hslot = hslot;
  t.valid = true;
  return t;
}
// four adjacent columns of row rowl of the tile: a piece's partial sums, or the output
template <int BM>
__device__ __forceinline__ void gemm2_store(const Gemm2Params &p, const Gemm2Tile &t, int rowl, int col, float4 v) {
  if (t.piece >= 0) {
    const size_t prow = p.n_split > 1 ? (size_t)t.piece * p.T + (t.t0 + rowl)
                                      : ((size_t)t.hslot * p.n_pieces + t.piece) * p.block + (t.m * BM + rowl);
    *reinterpret_cast<float4 *>(p.part + prow * p.d_model + col) = v;
  } else {
    store_out4(p, (size_t)(t.t0 + rowl) * p.d_model + col, v);
  }
}

// WM x WN wavefronts; a wavefront computes 32*TM tokens x 128 output columns.  The B
// operand tile is [BK list positions][BN columns] as it lies in memory (a gathered row is
// contiguous along the columns); the k-contiguous MFMA fragments are formed by reading
// 8 rows x 4 columns per lane (ds_read_b64) and interleaving row pairs with one byte
// permute per dword.  MFMA tile f, column c holds output column wave_base + 4c + f: a lane
// ends up with 4 consecutive columns of a row.
// Same S-stage asynchronous LDS ring as gemm1.  A B wave-load is 1 KiB of gathered rows
// (1024 / (2 BN) rows).  Where the row ids come from is a template parameter RM, so that the
// loop has no branches on it: 0 = identity list (Eq. 10, or K = all), computed; 1 = the block's
// whole list (Wdown rows, then the compensator units as ids d_ffn + u, then 0 padding) is
// copied once into an LDS table of 16-bit ids behind the ring and each lane reads the id of
// the row it fills from there, one k-step ahead; 2 = scalar loads of the list through the
// constant address space, the fallback when the table does not fit; 3 = the list streams through
// a small LDS ring of raw entries, one asynchronous 256-byte copy per k-step issued three steps
// before its entries are read (any list length, 2 KB of LDS).  Nothing in the loop is tracked by
// vmcnt except the asynchronous copies themselves.
// With KG = 2 two groups of WM x WN wavefronts split each stage's k range, as in gemm1, and exchange
// halves of their accumulators through LDS at the end (fixed order): eight wavefronts on a 128 x 256
// tile, for launches that give every CU one workgroup at most.
template <int WM, int WN, int TM, int BK, int S, int RM, int KG = 1>
__global__ __launch_bounds__(WM * WN * KG * 64) __attribute__((amdgpu_waves_per_eu(TM * 4 <= 8 ? 2 : 1)))
void ff_gemm2_kernel(Gemm2Params p, int V, int mt, int N, int xs) {
  constexpr int NW = WM * WN * KG;
  constexpr int BM = WM * TM * 32;
  constexpr int BN = WN * 128;
  constexpr int CPR = BK / 8;
  constexpr int ROWB = BK * 2;
  constexpr int A_BYTES = BM * ROWB;
  constexpr int ROWB_B = BN * 2;
  constexpr int B_BYTES = BK * ROWB_B;
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int RPLA = 1024 / ROWB;     // A rows per wave-load
  constexpr int RPLB = 1024 / ROWB_B;   // B rows per wave-load
  constexpr int LPR = 64 / RPLB;        // lanes per B row in a wave-load
  constexpr int LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW;
  constexpr int L = LA + LB;
  static_assert(ROWB_B <= 1024, "a B tile row must fit one wave-load");
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "tiles must split evenly over the wavefronts");
  extern __shared__ __align__(16) uint8_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = wave / (WM * WN), wq = wave % (WM * WN);
  const int wm = wq / WN, wn = wq % WN;
  const int c = lane & 31, half = lane >> 5;

  const Gemm2Tile tl = gemm2_tile<BM, BN, BK>(p, V, mt, N, xs);
  if (!tl.valid) return;
  const int b = tl.b, t0 = tl.t0, rows_valid = tl.rows_valid, Kb = tl.Kb, ntot = tl.ntot, n0 = tl.n0, kofs = tl.kofs, nk = tl.nk;

  const bf16_t *a_src[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int trow = (wave + i * NW) * RPLA + lane / CPR;
    const int ch = (lane % CPR) ^ swz<BK>(trow);
    const int tok = t0 + min(trow, rows_valid - 1);
    a_src[i] = p.h + (size_t)tok * p.hs + kofs + ch * 8;
  }
  const int b_sub = lane / LPR;                                   // which of the wave-load's rows this lane fills
  const int b_col = min(n0 + (lane % LPR) * 8, p.d_model - 8);
  typedef const __attribute__((address_space(4))) int32_t *cidx_t;
  const cidx_t idx_row = RM == 2 ? (cidx_t)(p.idx + (size_t)b * p.k_stride) : (cidx_t) nullptr;
  // source row id of list position pos: < d_ffn -> Wdown row, else compensator unit
  auto src_row = [&](int pos, auto load) __attribute__((always_inline)) -> int {
    if (pos < Kb) return min(max(load(pos), 0), p.d_ffn - 1);
    return pos < ntot ? p.d_ffn + (pos - Kb) : 0;
  };
  uint16_t *tab = reinterpret_cast<uint16_t *>(smem + S * STAGE);
  if (RM == 1) {
    // eight list entries per thread in flight at a time (left to itself the loop waits for every load)
    const int32_t *gl = p.idx + (size_t)b * p.k_stride;
    constexpr int U = 8;
    for (int i0 = tid; i0 < nk * BK; i0 += U * NW * 64) {
      int raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = gl[min(kofs + i0 + u * NW * 64, Kb - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * NW * 64;
        if (i < nk * BK) tab[i] = (uint16_t)src_row(kofs + i, [&](int) { return raw[u]; });
      }
    }
    __syncthreads();
  }
  // RM 3: ring of kIdSlots stages' raw list entries behind the operand ring.  Every wavefront issues
  // the same copy (identical bytes to the same place), so all of them count the same number of
  // outstanding loads.  Lane l fetches entry st * BK + l % BK, clamped into the list.
  constexpr int kIdSlots = 8;
  static_assert(RM != 3 || S + 2 <= kIdSlots - 2, "id ring too short for the ring depth");
  const int32_t *idring = reinterpret_cast<const int32_t *>(smem + S * STAGE);
  const uint32_t idring_lds = lds_addr_of(smem) + (uint32_t)(S * STAGE);
  const int32_t *id_src = p.idx + (size_t)b * p.k_stride;
  auto issue_ids = [&](int st) __attribute__((always_inline)) {
    const int q = min(kofs + st * BK + lane % BK, Kb - 1);
    gload_lds4(id_src + q, idring_lds + (uint32_t)(st % kIdSlots) * 256u);
  };
  if (RM == 3) {
    // stages 0 .. S+1 up front; stage j+S+2 follows in step j, right behind that step's barrier
#pragma unroll
    for (int st = 0; st < S + 2; ++st) issue_ids(st);
    wait_vm_barrier<0>();
  }
  // A VGPR zero the compiler cannot see through: keeps the table reads per-lane LDS reads
  // (a wave-uniform address would be turned into a read + wait + readfirstlane in the loop).
  int lane_zero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(lane_zero));
  // rows_v: row id of the B row this lane fills in copy i of the stage issued next; rows_n: the
  // same for the stage after it, fetched a whole step before it is needed
  int rows_v[LB], rows_n[LB];
  auto fetch_rows = [&](int st, int (&dst)[LB]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int rel0 = st * BK + (wave + i * NW) * RPLB;   // within this tile's k range
      const int pos0 = kofs + rel0;
      if (RM == 0) {
        dst[i] = src_row(pos0 + b_sub, [](int q) { return q; });
      } else if (RM == 1) {
        dst[i] = (int)tab[rel0 + b_sub + lane_zero];
      } else if (RM == 3) {
        const int raw = idring[(st % kIdSlots) * 64 + (wave + i * NW) * RPLB + b_sub + lane_zero];
        dst[i] = src_row(pos0 + b_sub, [&](int) { return raw; });
      } else {
        int r = src_row(pos0, [&](int q) { return idx_row[q]; });
#pragma unroll
        for (int u = 1; u < RPLB; ++u) {
          const int ru = src_row(pos0 + u, [&](int q) { return idx_row[q]; });
          r = (b_sub == u) ? ru : r;
        }
        dst[i] = r;
      }
    }
  };
  const uint32_t lds0 = lds_addr_of(smem);
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const uint64_t base_w = reinterpret_cast<uint64_t>(p.wd + b_col);
  const uint64_t base_c = reinterpret_cast<uint64_t>(p.wc2 + b_col) - (uint64_t)p.d_ffn * row_bytes;
  // copy i of stage st (uses rows == row ids of stage st): i < LA -> A tile, else gathered B rows
  auto issue_one = [&](int st, int i) __attribute__((always_inline)) {
    const uint32_t base = lds0 + (uint32_t)(st % S) * STAGE + (uint32_t)wave * 1024u;
    if (i < LA) {
      gload_lds16(a_src[i] + st * BK, base + (uint32_t)i * (NW * 1024u));
    } else {
      const int ib = i - LA;
      // row id r < d_ffn: Wdown row r; else compensator unit r - d_ffn.  One compare, one 64-bit
      // select and one 32 x 32 + 64 multiply-add per copy (this arithmetic sits between the MFMAs).
      const uint32_t r = (uint32_t)rows_v[ib];
      const uint64_t src = (uint64_t)r * row_bytes + (r < (uint32_t)p.d_ffn ? base_w : base_c);
      gload_lds16(reinterpret_cast<const void *>(src), base + A_BYTES + (uint32_t)ib * (NW * 1024u));
    }
  };
  auto issue = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < L; ++i) issue_one(st, i);
  };

  f32x16_t acc[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][f][e] = 0.0f;

  // Same pipeline as gemm1: stage kt+1 is waited for in front of the last MFMA group of stage
  // kt, its first fragments are requested there, and the copies of stage kt+S go out one at a
  // time between the MFMAs of the following KQ groups.  The row ids of stage kt+S are fetched
  // at the start of step kt and take the place of stage kt+S-1's once its last copy is out.
  constexpr int KQ = BK / 16 / KG;                     // MFMA groups (16 k each) per stage and k-group
  static_assert(KQ % 2 == 0, "fragment double buffer needs an even number of groups per stage");
  constexpr int NMF = TM * 4;
  constexpr int LQ = (L + KQ - 1) / KQ;
  constexpr int PER = (LQ + NMF - 1) / NMF;
  constexpr int EVERY = NMF / LQ > 0 ? NMF / LQ : 1;
  constexpr int SLOTS = (NMF + EVERY - 1) / EVERY * PER;
  u32x4_t af[2][TM];
  u32x2_t d[2][8];
  auto frags = [&](int kt, int kk, int buf) __attribute__((always_inline)) {
    const uint8_t *cur = smem + (kt % S) * STAGE;
    const int kg = kgrp * KQ + kk;                     // 16-k group within the stage
    const int q = 2 * kg + half;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = (wm * TM + i) * 32 + c;
      af[buf][i] = *reinterpret_cast<const u32x4_t *>(cur + row * ROWB + ((q ^ swz<BK>(row)) << 4));
    }
    const uint8_t *bb = cur + A_BYTES + (kg * 16 + 8 * half) * ROWB_B + (wn * 128 + 4 * c) * 2;
#pragma unroll
    for (int i = 0; i < 8; ++i) d[buf][i] = *reinterpret_cast<const u32x2_t *>(bb + i * ROWB_B);
  };
  auto group = [&](int kk, int st, int part, bool load) __attribute__((always_inline)) {
    const u32x2_t *dd = d[kk & 1];
    u32x4_t bf[4];
    // One byte permute per dword: low halves (even columns) or high halves (odd columns) of the
    // rows (2j, 2j+1), lower row in the low half.  The four permutes of column tile f are issued
    // right in front of its first MFMA, so all but the first four hide under the previous MFMA.
#define FF_LO(e, o) __builtin_amdgcn_perm((o), (e), 0x05040100u)
#define FF_HI(e, o) __builtin_amdgcn_perm((o), (e), 0x07060302u)
    auto make_bf = [&](int f) __attribute__((always_inline)) {
      if (f == 0) bf[0] = mk4(FF_LO(dd[0].x, dd[1].x), FF_LO(dd[2].x, dd[3].x), FF_LO(dd[4].x, dd[5].x), FF_LO(dd[6].x, dd[7].x));
      if (f == 1) bf[1] = mk4(FF_HI(dd[0].x, dd[1].x), FF_HI(dd[2].x, dd[3].x), FF_HI(dd[4].x, dd[5].x), FF_HI(dd[6].x, dd[7].x));
      if (f == 2) bf[2] = mk4(FF_LO(dd[0].y, dd[1].y), FF_LO(dd[2].y, dd[3].y), FF_LO(dd[4].y, dd[5].y), FF_LO(dd[6].y, dd[7].y));
      if (f == 3) bf[3] = mk4(FF_HI(dd[0].y, dd[1].y), FF_HI(dd[2].y, dd[3].y), FF_HI(dd[4].y, dd[5].y), FF_HI(dd[6].y, dd[7].y));
    };
    // (with a gathered list the copies' address arithmetic already fills those slots, and spreading
    //  the permutes as well measured 5% slower; with the identity list it is 6% faster)
    constexpr bool SPREAD_PERM = RM == 0;
    make_bf(0);
    if (!SPREAD_PERM) { make_bf(1); make_bf(2); make_bf(3); }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        acc[i][f] = mfma32(af[kk & 1][i], bf[f], acc[i][f]);
        if (SPREAD_PERM && i == 0 && f < 3) make_bf(f + 1);
        bool fenced = false;
        if ((i * 4 + f) % EVERY == 0) {
#pragma unroll
          for (int r = 0; r < PER; ++r) {
            const int n = (i * 4 + f) / EVERY * PER + r;
            if (n < LQ && part * LQ + n < L) {
              if (load) issue_one(st, part * LQ + n);
              __builtin_amdgcn_sched_barrier(0);
              fenced = true;
            }
          }
        }
        if (SPREAD_PERM && i == 0 && !fenced) __builtin_amdgcn_sched_barrier(0);
      }
#undef FF_LO
#undef FF_HI
#pragma unroll
    for (int n = SLOTS; n < LQ; ++n)
      if (load && part * LQ + n < L) issue_one(st, part * LQ + n);
    __builtin_amdgcn_sched_barrier(0);
  };
  // MAIN: stages kt+S-1 and kt+S both exist (no conditions in the loop body)
  auto step = [&](int kt, auto main_tag) __attribute__((always_inline)) {
    constexpr bool MAIN = decltype(main_tag)::value;
    const bool la = MAIN || kt + S - 1 < nk;
    const bool lb = MAIN || kt + S < nk;
    if (lb) fetch_rows(kt + S, rows_n);
#pragma unroll
    for (int kk = 0; kk < KQ - 1; ++kk) {
      frags(kt, kk + 1, (kk + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      group(kk, kt + S - 1, kk + 1, la);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) rows_v[i] = rows_n[i];   // the last copy of stage kt+S-1 is out
    if (MAIN || kt + 1 < nk) {
      // stage kt+1 must have landed; stages kt+2 .. kt+S-1 may still be in flight
      if (MAIN || kt + S - 1 < nk) wait_vm_barrier<(S - 2) * L>(); else wait_vm_barrier<0>();
      frags(kt + 1, 0, 0);
      // older than every copy the next wait lets stay in flight, so it has landed by then, one
      // step before fetch_rows reads it
      if (RM == 3) issue_ids(kt + S + 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    group(KQ - 1, kt + S, 0, lb);
  };
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) {
      fetch_rows(s, rows_v);
      issue(s);
    }
  if (S - 1 < nk) fetch_rows(S - 1, rows_v);
#pragma unroll
  for (int i = 0; i < LB; ++i) rows_n[i] = rows_v[i];
  if (S - 1 <= nk) wait_vm_barrier<(S - 2) * L>(); else wait_vm_barrier<0>();
  if (S - 1 < nk) {
#pragma unroll
    for (int i = 0; i < (LQ < L ? LQ : L); ++i) issue_one(S - 1, i);
  }
  frags(0, 0, 0);
  const int n_main = max(nk - S, 0);
  for (int kt = 0; kt < n_main; ++kt) step(kt, std::true_type{});
  for (int kt = n_main; kt < nk; ++kt) step(kt, std::false_type{});
  if (RM == 3) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last id copies (nobody reads them)

  // k-groups: group g keeps token tiles i with i % KG == g and hands the others over through LDS
  if (KG > 1) {
    static_assert(KG == 1 || (KG == 2 && TM % 2 == 0), "two k-groups need an even number of token tiles per wavefront");
    static_assert(KG == 1 || S * STAGE >= WM * WN * 2 * (TM / 2) * 4 * 16 * 64 * 4, "ring too small for the hand-over");
    __syncthreads();                                    // everyone is done with the ring
    float4 *red = reinterpret_cast<float4 *>(smem);
    constexpr int XPER = (TM / 2) * 4 * 4;              // float4 slots a wavefront hands over
    const int slot0 = ((kgrp * (WM * WN) + wq) * XPER) * 64 + lane;
    int sl = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if ((i & 1) != kgrp) {                            // token tiles the other group keeps
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4)
            red[slot0 + (sl++) * 64] = make_float4(acc[i][f][4 * e4], acc[i][f][4 * e4 + 1], acc[i][f][4 * e4 + 2], acc[i][f][4 * e4 + 3]);
      }
    __syncthreads();
    const int other0 = (((1 - kgrp) * (WM * WN) + wq) * XPER) * 64 + lane;
    sl = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if ((i & 1) == kgrp) {
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            const float4 o4 = red[other0 + (sl++) * 64];
            acc[i][f][4 * e4] += o4.x; acc[i][f][4 * e4 + 1] += o4.y; acc[i][f][4 * e4 + 2] += o4.z; acc[i][f][4 * e4 + 3] += o4.w;
          }
      }
  }

  const int col = n0 + wn * 128 + 4 * c;
  if (col < p.d_model) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if (KG == 1 || (i & 1) == kgrp)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rowl = (wm * TM + i) * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
        if (rowl < rows_valid) {
          const float4 v = make_float4(acc[i][0][e], acc[i][1][e], acc[i][2][e], acc[i][3][e]);
          gemm2_store<BM>(p, tl, rowl, col, v);
        }
      }
  }
}

// The same product with the gathered rows loaded straight into registers.  A row of W_down is contiguous along the
// output columns, so 16 lanes of a load instruction ask for 128 contiguous bytes of one row, and the transposition that
// MFMA wants (eight list positions of one column in a lane) is one byte permute per dword of eight rows' pieces.  Eight
// wavefronts side by side, 64 columns each for all tokens of the tile: nobody else in the workgroup wants a wavefront's
// weights, only H passes through LDS.  KG = 2: two groups of four wavefronts take the steps in turn and exchange halves of
// their accumulators at the end (fixed order), for calls with few columns and blocks.
// v_mfma_f32_16x16x32_bf16: lane (c, q) holds list positions 8 q .. 8 q + 7 of a step's half of 32; MFMA tile f, column c
// is output column 8 (c mod 8) + 4 (c / 8) + f of the wavefront's 64, so a lane ends with four adjacent columns.
// RM 0: the identity list; 1: the tile's list in an LDS table of 16-bit ids, as above.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
__device__ __forceinline__ f32x4_t mfma16(const u32x4_t &a, const u32x4_t &b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
template <int MT, int RM, int KG>
__global__ __launch_bounds__(kDirectWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ff_gemm2_direct_kernel(Gemm2Params p, int V, int mt, int N, int xs) {
  constexpr int NW = kDirectWaves, WN = NW / KG, BM = MT * 16, BN = WN * 64, S = kDirectStages, D = 4;
  constexpr int STAGE = BM * 128, LA = BM * KG / 8 / NW;   // a stage: H of 64 positions; a round of the loop takes KG of them
  constexpr int NB = MT == 8 ? 2 : 4;         // halves of a step whose weights are on their way (as many as registers allow)
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = KG == 1 ? 0 : wave / WN, wn = KG == 1 ? wave : wave % WN;
  const int c = lane & 15, q = lane >> 4;
  const Gemm2Tile tl = gemm2_tile<BM, BN, 64>(p, V, mt, N, xs);
  if (!tl.valid) return;
  const int Kb = tl.Kb, ntot = tl.ntot, kofs = tl.kofs, nk = tl.nk;
  const int last = max(nk - 1, 0), rounds = (nk + KG - 1) / KG;

  // H: copy i of a round covers rows 8 (wave + i NW) .. + 7 of its KG stages
  const uint64_t a_base = (uint64_t)(uintptr_t)(p.h + (size_t)tl.t0 * p.hs + kofs);
  uint32_t a_off[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int trow = ((wave + i * NW) * 8 + lane / 8) % (KG == 1 ? 1 << 30 : BM);
    a_off[i] = (uint32_t)(min(trow, tl.rows_valid - 1) * p.hs + ((lane & 7) ^ swz<64>(trow)) * 8) * 2u;
  }
  const uint32_t lds0 = lds_addr_of(smem);
  // (no conditions in the loop: past the end the last step is requested again, into a slot nobody reads any more, or next to
  // weights that are not multiplied)
  auto issue_a = [&](int rd, int i) __attribute__((always_inline)) {
    const int st = KG == 1 ? rd : rd * KG + (wave + i * NW) * 8 / BM;
    gload_lds16_off(a_base + (uint64_t)(uint32_t)min(st, last) * 128u, a_off[i], lds0 + (uint32_t)(rd % S) * (KG * STAGE) + (uint32_t)(wave + i * NW) * 1024u);
  };
  if (nk > 0) {
#pragma unroll
    for (int st = 0; st < S - 2; ++st)
#pragma unroll
      for (int i = 0; i < LA; ++i) issue_a(st, i);
  }
  uint16_t *tab = reinterpret_cast<uint16_t *>(smem + S * KG * STAGE);
  if (RM == 1) {
    // eight list entries per thread in flight at a time (left to itself the loop waits for every load)
    const int32_t *gl = p.idx + (size_t)tl.b * p.k_stride;
    constexpr int U = 8;
    for (int i0 = tid; i0 < nk * 64; i0 += U * NW * 64) {
      int raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = gl[min(kofs + i0 + u * NW * 64, Kb - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * NW * 64, pos = kofs + i;
        if (i < nk * 64) tab[i] = (uint16_t)(pos < Kb ? min(max(raw[u], 0), p.d_ffn - 1) : (pos < ntot ? p.d_ffn + (pos - Kb) : 0));
      }
    }
    __syncthreads();
  }
  const int colw = tl.n0 + wn * 64;                              // d_model is a multiple of 64: a wavefront is in or out
  const int hi = c >> 3;                                           // which of a pair of rows this lane loads
  const int col4 = 8 * (c & 7) + 4 * hi;                           // this lane's four columns, once the pairs have swapped
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const uint32_t col_bytes = (uint32_t)(min(colw, p.d_model - 64) + 8 * (c & 7)) * 2u;
  const uint32_t lane_off = (8u * (uint32_t)q + (uint32_t)hi) * row_bytes + col_bytes;

  f32x4_t acc[MT][4];                         // [token tile][f]
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[i][f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

  typedef const __attribute__((address_space(1))) u32x4_t *gptr_t;
  typedef const __attribute__((address_space(1))) uint8_t *gbyte_t;
  u32x4_t wb[NB][4];                          // [half of a step mod NB][i]: eight columns of row 8 q + 2 i + hi
  u32x4_t ids[2];                             // ids of rows 8 q .. 8 q + 7 of the half requested next (by its parity)
  u32x4_t af[D];                              // ring of token fragments
  u32x4_t bf[2][4];                           // operands of the half at hand and of the next
  // (halves are counted through the wavefront's own steps: half hh is half hh % 2 of its step hh / 2)
  auto half_at = [&](int hh) __attribute__((always_inline)) -> int { return KG == 1 ? min(hh, 2 * last + 1) : 2 * min((hh >> 1) * KG + kgrp, last) + (hh & 1); };
  auto fetch_ids = [&](int hh, int par) __attribute__((always_inline)) {
    if (RM == 1) ids[par] = *reinterpret_cast<const u32x4_t *>(tab + half_at(hh) * 32 + 8 * q);
  };
  // load i of half hh.  FAST: all of its positions are W_down rows, whose offsets fit 32 bits (the launcher's check);
  // else each row's matrix is found lane by lane.
  auto load_w = [&](int hh_, int par, int buf, int i, auto fast_tag) __attribute__((always_inline)) {
    const int hh = half_at(hh_);
    const uint32_t id = RM == 1 ? (ids[par][i] >> (16 * hi)) & 0xffffu : 0u;
    if (decltype(fast_tag)::value) {
      if (RM == 1) {
        wb[buf][i] = *(gptr_t)((uintptr_t)p.wd + (__umul24(id, row_bytes) + col_bytes));
      } else {
        const gbyte_t row0 = (gbyte_t)(uintptr_t)p.wd + (size_t)(uint32_t)(kofs + hh * 32 + 2 * i) * row_bytes;   // scalar
        wb[buf][i] = *(gptr_t)(row0 + lane_off);
      }
    } else {
      const int pos = kofs + hh * 32 + 8 * q + 2 * i + hi;
      const uint32_t r = RM == 1 ? id : (uint32_t)(pos < Kb ? min(pos, p.d_ffn - 1) : (pos < ntot ? p.d_ffn + (pos - Kb) : 0));
      const uintptr_t base = r < (uint32_t)p.d_ffn ? (uintptr_t)p.wd : (uintptr_t)p.wc2 - (size_t)p.d_ffn * row_bytes;
      wb[buf][i] = *(gptr_t)(base + (size_t)r * row_bytes + col_bytes);
    }
  };
  // Rows 2 i and 2 i + 1 lie in lanes c and c ^ 8, eight columns each.  Those lanes swap halves (DPP rotation by 8 within
  // 16 lanes, written to eight of them), so that each holds both rows' pieces of its own four columns; one byte permute
  // per dword then pairs the two rows.
  auto make_bf = [&](int h, int buf, int i) __attribute__((always_inline)) {
    constexpr int ROR8 = 0x128;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const uint32_t lo = wb[buf][i][d], up = wb[buf][i][2 + d];
      const uint32_t ev = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)up, ROR8, 0xf, 0xc, false);
      const uint32_t od = (uint32_t)__builtin_amdgcn_update_dpp((int)up, (int)lo, ROR8, 0xf, 0x3, false);
      bf[h][2 * d][i] = __builtin_amdgcn_perm(od, ev, 0x05040100u);
      bf[h][2 * d + 1][i] = __builtin_amdgcn_perm(od, ev, 0x07060302u);
    }
  };
  uint32_t aoff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) aoff[h] = (uint32_t)(c * 128 + (((4 * h + q) ^ swz<64>(c)) << 4));
  // fragment n of a step: half n / MT, token tile n % MT
  auto frag = [&](int kt, int n) __attribute__((always_inline)) {
    af[n % D] = *reinterpret_cast<const u32x4_t *>(smem + ((kt % S) * KG + kgrp) * STAGE + aoff[n / MT] + (n % MT) * 2048);
  };
  // One step of 64 positions in each k-group.  During a half the next one's weights are permuted into operands, and those of half
  // hh + 1 + NB take their registers; H of step kt + S - 2 is requested in the first half; in front of the last D
  // fragments the workgroup makes sure that H of step kt + 1 has landed (its copies are older than the last 8
  // requests).  The slot of H requested in a step was last read two steps before, hence by nobody who has passed the
  // barrier in between.  PH: 2 kt mod NB.
  // (Spreading the permutes over the half and taking the wait for LDS reads out of the barrier: 412 -> 376 us.)
  auto step = [&](int kt, auto ph_tag, auto fast_tag) __attribute__((always_inline)) {
    constexpr int PH = decltype(ph_tag)::value;
#pragma unroll
    for (int n = 0; n < 2 * MT; ++n) {
      const int h = n / MT, r = n % MT;
      if (n == 2 * MT - D) asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
      const u32x4_t a = af[n % D];
      if (KG == 1 || decltype(fast_tag)::value || kt * KG + kgrp < nk) {      // (an odd number of steps: one group has one less)
#pragma unroll
        for (int f = 0; f < 4; ++f) acc[r][f] = mfma16(a, bf[h][f], acc[r][f]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (n + D < 2 * MT) frag(kt, n + D); else frag(kt + 1, n + D - 2 * MT);
      if (n < LA) issue_a(kt + S - 2, n);
      if (r == 1) fetch_ids(2 * kt + h + 2 + NB, h);
      if (r >= MT - 4) {
        const int i = r - (MT - 4), buf = (PH + h + 1) % NB;
        make_bf(1 - h, buf, i);
        load_w(2 * kt + h + 1 + NB, 1 - h, buf, i, fast_tag);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (nk > 0) {
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      fetch_ids(h, h & 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) load_w(h, h & 1, h, i, std::false_type{});
    }
    fetch_ids(NB, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) make_bf(0, 0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_w(NB, 0, 0, i, std::false_type{});
    fetch_ids(NB + 1, 1);
    asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int n = 0; n < D; ++n) frag(0, n);
    __builtin_amdgcn_sched_barrier(0);
    const int nfast = min((Kb - kofs) / (64 * KG), nk / KG);
    constexpr std::integral_constant<int, 0> ph0{};
    constexpr std::integral_constant<int, 2> ph1{};
    int kt = 0;
    if (NB == 2) {
      for (; kt + 2 < nfast; ++kt) step(kt, ph0, std::true_type{});
      for (; kt < rounds; ++kt) step(kt, ph0, std::false_type{});
    } else {
      for (; kt + 4 < nfast; kt += 2) {
        step(kt, ph0, std::true_type{});
        step(kt + 1, ph1, std::true_type{});
      }
      while (kt < rounds) {
        step(kt, ph0, std::false_type{});
        if (++kt >= rounds) break;
        step(kt, ph1, std::false_type{});
        ++kt;
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies requested past the end
  }

  if (KG > 1) {
    // group g keeps token tiles i with i % 2 == g and hands the others over through LDS
    static_assert(KG == 1 || (KG == 2 && MT % 2 == 0 && S * KG * STAGE >= NW * MT / 2 * 4 * 1024), "ring too small for the hand-over");
    __syncthreads();                                       // everyone is done with the ring
    f32x4_t *red = reinterpret_cast<f32x4_t *>(smem);
    const int mine = wave * (MT / 2 * 4) * 64 + lane, other = (wave + (kgrp ? -WN : WN)) * (MT / 2 * 4) * 64 + lane;
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if ((i & 1) != kgrp) {
#pragma unroll
        for (int f = 0; f < 4; ++f) red[mine + (i / 2 * 4 + f) * 64] = acc[i][f];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if ((i & 1) == kgrp) {
#pragma unroll
        for (int f = 0; f < 4; ++f) acc[i][f] += red[other + (i / 2 * 4 + f) * 64];
      }
  }
  const int col = colw + col4;
  if (colw >= p.d_model) return;
#pragma unroll
  for (int i = 0; i < MT; ++i)
    if (KG == 1 || (i & 1) == kgrp)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rowl = i * 16 + 4 * q + e;
      if (rowl < tl.rows_valid)
        gemm2_store<BM>(p, tl, rowl, col, make_float4(acc[i][0][e], acc[i][1][e], acc[i][2][e], acc[i][3][e]));
    }
}

// The same product for calls with few tokens or columns: 64 x 64 tiles, whose eight wavefronts take the list's groups of 32
// positions in turn and wait for nobody until they add up at the end (in wavefront order).  Each copies H of its group into LDS of
// its own and loads its rows into registers as above, the next group's while this one's products are formed; two workgroups on a
// CU, so that four wavefronts of a SIMD wait in turn.  The tiles above pass a barrier every 64 positions, and cut into pieces that
// fill the chip they write and read partial sums for as long as the products take.  What binds this one is the latency of
// each group's loads, and, with many tiles, that a row is fetched once for every 64 tokens.
// Whole calls of ff_sparse_ffn, half of the neurons, us, without this tile and with it: 256 tokens of 256/688 17.0 -> 14.1; 2048/8192,
// 9 tokens 25.9 -> 22.7, 64 28.9 -> 26.3, 256 in one block 44.4 -> 41.7; 4096/14336, 9 tokens 51.7 -> 45.6, 30 51.6 -> 48.0, 64 60.6
// -> 55.9.  Forced, 100 tokens of 4096/14336 86.5 -> 88.4 and 700 of 2048/8192 93.6 -> 104.
// RM 0: the identity list; 1: the tile's list in an LDS table of 16-bit ids.
constexpr int kSplitWaves = 8;
template <int RM>
__global__ __launch_bounds__(kSplitWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
void ff_gemm2_ksplit_kernel(Gemm2Params p, int V, int mt, int N, int xs) {
  constexpr int NW = kSplitWaves, MT = 4, BM = MT * 16, BN = 64, STAGE = BM * 64;
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4;
  const Gemm2Tile tl = gemm2_tile<BM, BN, 64>(p, V, mt, N, xs);
  if (!tl.valid) return;
  const int Kb = tl.Kb, ntot = tl.ntot, kofs = tl.kofs, nh = 2 * tl.nk;
  uint16_t *tab = reinterpret_cast<uint16_t *>(smem + 2 * NW * STAGE);
  if (RM == 1) {
    // eight list entries per thread in flight at a time (left to itself the loop waits for every load)
    const int32_t *gl = p.idx + (size_t)tl.b * p.k_stride;
    constexpr int U = 8;
    for (int i0 = tid; i0 < nh * 32; i0 += U * NW * 64) {
      int raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = gl[min(kofs + i0 + u * NW * 64, Kb - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * NW * 64, pos = kofs + i;
        if (i < nh * 32) tab[i] = (uint16_t)(pos < Kb ? min(max(raw[u], 0), p.d_ffn - 1) : (pos < ntot ? p.d_ffn + (pos - Kb) : 0));
      }
    }
    __syncthreads();
  }
  // H: copy i of a group covers rows 16 i .. + 15, 64 bytes of each
  const uint64_t a_base = (uint64_t)(uintptr_t)(p.h + (size_t)tl.t0 * p.hs + kofs);
  uint32_t a_off[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int row = 16 * i + lane / 4;
    a_off[i] = (uint32_t)(min(row, tl.rows_valid - 1) * p.hs + ((lane & 3) ^ swz<32>(row)) * 8) * 2u;
  }
  const uint32_t lds0 = lds_addr_of(smem) + (uint32_t)wave * (2 * STAGE);
  const uint8_t *mine = smem + wave * (2 * STAGE) + c * 64 + ((q ^ swz<32>(c)) << 4);   // (row 16 m + c: the same swizzle)
  const int hi = c >> 3;                                                  // which of a pair of rows this lane loads
  const uint32_t row_bytes = (uint32_t)p.d_model * 2u;
  const uint32_t col_bytes = (uint32_t)(min(tl.n0, p.d_model - BN) + 8 * (c & 7)) * 2u;
  typedef const __attribute__((address_space(1))) u32x4_t *gptr_t;
  typedef const __attribute__((address_space(1))) uint8_t *gbyte_t;
  const uint32_t lane_off = (8u * (uint32_t)q + (uint32_t)hi) * row_bytes + col_bytes;
  u32x4_t wb[4];
  // group h's copies and rows (FAST: all of its positions are W_down rows; the launcher has checked that their offsets fit 32 bits)
  auto request = [&](int h, uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MT; ++i) gload_lds16_off(a_base + (uint64_t)(uint32_t)h * 64u, a_off[i], lds0 + slot * STAGE + (uint32_t)i * 1024u);
    u32x4_t ids = {0, 0, 0, 0};
    if (RM == 1) ids = *reinterpret_cast<const u32x4_t *>(tab + h * 32 + 8 * q);
    const int pos0 = kofs + h * 32;
    if (pos0 + 32 <= Kb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (RM == 1) wb[i] = *(gptr_t)((uintptr_t)p.wd + (__umul24((ids[i] >> (16 * hi)) & 0xffffu, row_bytes) + col_bytes));
        else {
          const gbyte_t row0 = (gbyte_t)(uintptr_t)p.wd + (size_t)(uint32_t)(pos0 + 2 * i) * row_bytes;   // scalar
          wb[i] = *(gptr_t)(row0 + lane_off);
        }
      }
    } else {
      int pos8 = pos0 + 8 * q + hi;
      asm volatile("" : "+v"(pos8));                                      // (nothing of this ahead of the loop: no registers for it)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int pos = pos8 + 2 * i;
        const uint32_t r = RM == 1 ? (ids[i] >> (16 * hi)) & 0xffffu : (uint32_t)(pos < Kb ? min(pos, p.d_ffn - 1) : (pos < ntot ? p.d_ffn + (pos - Kb) : 0));
        const uintptr_t base = r < (uint32_t)p.d_ffn ? (uintptr_t)p.wd : (uintptr_t)p.wc2 - (size_t)p.d_ffn * row_bytes;
        wb[i] = *(gptr_t)(base + (size_t)r * row_bytes + col_bytes);
      }
    }
  };
  f32x4_t acc[MT][4];                         // [token tile][f]
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < 4; ++f) acc[i][f] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t slot = 0;
  if (wave < nh) request(wave, 0);
  for (int h = wave; h < nh; h += NW) {
    // everything of group h has landed (a wavefront reads what it copied itself: no barrier)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    u32x4_t bf[4];
    // rows 2 i and 2 i + 1 lie in lanes c and c ^ 8, as in ff_gemm2_direct_kernel
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      constexpr int ROR8 = 0x128;
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const uint32_t lo = wb[i][d], up = wb[i][2 + d];
        const uint32_t ev = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)up, ROR8, 0xf, 0xc, false);
        const uint32_t od = (uint32_t)__builtin_amdgcn_update_dpp((int)up, (int)lo, ROR8, 0xf, 0x3, false);
        bf[2 * d][i] = __builtin_amdgcn_perm(od, ev, 0x05040100u);
        bf[2 * d + 1][i] = __builtin_amdgcn_perm(od, ev, 0x07060302u);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (the other place's last reader was the group before, whose products are out)
    if (h + NW < nh) request(h + NW, slot ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    u32x4_t af[2];
    af[0] = *reinterpret_cast<const u32x4_t *>(mine + slot * STAGE);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m + 1 < MT) af[(m + 1) & 1] = *reinterpret_cast<const u32x4_t *>(mine + slot * STAGE + (m + 1) * 1024);
#pragma unroll
      for (int f = 0; f < 4; ++f) acc[m][f] = mfma16(af[m & 1], bf[f], acc[m][f]);
      __builtin_amdgcn_sched_barrier(0);
    }
    slot ^= 1;
  }
  // the wavefronts' sums, in order, 16 rows at a time: lane (c, q) holds columns 8 (c mod 8) + 4 (c / 8) + f of rows 4 q + e
  float4 *red = reinterpret_cast<float4 *>(smem);                        // [wave][16 rows][16 columns of four]
  const int col4 = 2 * (c & 7) + hi;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    __syncthreads();                                                     // the copies' LDS, or the last rows, are free
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(wave * 16 + 4 * q + e) * 16 + col4] = make_float4(acc[m][0][e], acc[m][1][e], acc[m][2][e], acc[m][3][e]);
    __syncthreads();
    const int rowl = 16 * m + (tid >> 4);
    if (tid < 256 && rowl < tl.rows_valid && tl.n0 < p.d_model) {
      float4 v = red[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float4 o = red[w * 256 + tid];
        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
      }
      gemm2_store<BM>(p, tl, rowl, tl.n0 + 4 * (tid & 15), v);
    }
  }
}

// ---- variant tables --------------------------------------------------------
struct Variant {
  const void *fn;
  int bm, bn, threads, lds;
  const void *fn_rm[3];  // gemm2 only: the kernels for row-id modes 1, 2 and (or nullptr) 3 (fn is mode 0)
};
int g_lds_limit = 65536;

template <int WM, int WN, int TM, int TN, int BK, int S, int KG = 1>
Variant g1() {
  return Variant{reinterpret_cast<const void *>(&ff_gemm1_kernel<WM, WN, TM, TN, BK, S, KG>), WM * TM * 32,
                 WN * TN * 32, WM * WN * KG * 64, S * (WM * TM * 32 + 2 * WN * TN * 32) * BK * 2, {nullptr, nullptr, nullptr}};
}
template <int WM, int WN, int TM, int BK, int S, int KG = 1>
Variant g2() {
  return Variant{reinterpret_cast<const void *>(&ff_gemm2_kernel<WM, WN, TM, BK, S, 0, KG>), WM * TM * 32,
                 WN * 128, WM * WN * KG * 64, S * (WM * TM * 32 * BK * 2 + BK * WN * 128 * 2),
                 {reinterpret_cast<const void *>(&ff_gemm2_kernel<WM, WN, TM, BK, S, 1, KG>),
                  reinterpret_cast<const void *>(&ff_gemm2_kernel<WM, WN, TM, BK, S, 2, KG>),
                  // the streamed list only where the table may not fit and scalar loads cost too much
                  KG > 1 ? reinterpret_cast<const void *>(&ff_gemm2_kernel<WM, WN, TM, BK, S, (KG > 1 ? 3 : 2), KG>) : nullptr}};
}
template <int MT, int WN, int NBUF>
Variant g1d() {
  return Variant{reinterpret_cast<const void *>(&ff_gemm1_direct_kernel<MT, WN, NBUF>), MT * 32, WN * 32, WN * 64,
                 kDirectStages * MT * 32 * 128, {nullptr, nullptr, nullptr}};
}
template <int MT, int KG = 1>
Variant g2d() {
  return Variant{reinterpret_cast<const void *>(&ff_gemm2_direct_kernel<MT, 0, KG>), MT * 16, kDirectWaves / KG * 64, kDirectWaves * 64,
                 kDirectStages * KG * MT * 16 * 128, {reinterpret_cast<const void *>(&ff_gemm2_direct_kernel<MT, 1, KG>), nullptr, nullptr}};
}
Variant g2k() {
  return Variant{reinterpret_cast<const void *>(&ff_gemm2_ksplit_kernel<0>), 64, 64, kSplitWaves * 64, 2 * kSplitWaves * 64 * 64,
                 {reinterpret_cast<const void *>(&ff_gemm2_ksplit_kernel<1>), nullptr, nullptr}};
}
constexpr int kIdRingBytes = 8 * 256;   // row-id mode 3: eight stages of 64 raw list entries

// tokens x list positions of the tile, wavefronts, BK, ring stages (LDS).  1, 2 and 4 run only where an option names them: at
// none of twelve shapes from 60 to 8192 tokens were they faster than the choice below (222 us against 225, 264 and 342 at the
// closest, 700 tokens of 4096/14336).  They keep their numbers, and add the same sums in another order for comparisons.
const Variant kGemm1[] = {
    g1<2, 2, 2, 2, 64, 3, 2>(),  // 0: 128 x 128, 8 waves in 2 k-groups, BK 64, 3 stages (144 KB)
    g1<2, 4, 2, 2, 32, 3>(),     // 1: 128 x 256, 8 waves, BK 32, 3 stages (120 KB)
    g1<2, 2, 2, 2, 32, 3>(),     // 2: 128 x 128, 4 waves, BK 32, 3 stages (72 KB, two workgroups per CU)
    g1<4, 2, 2, 2, 64, 2>(),     // 3: 256 x 128, 8 waves, BK 64, 2 stages (128 KB)
    g1<1, 4, 2, 2, 32, 4>(),     // 4: 64 x 256, 4 waves, BK 32, 4 stages (144 KB)
    g1<1, 4, 2, 2, 64, 2, 2>(),  // 5: 64 x 256, 8 waves in 2 k-groups, BK 64, 2 stages (144 KB)
    g1<2, 4, 2, 2, 64, 2>(),     // 6: 128 x 256, 8 waves, BK 64, 2 stages (160 KB)
    g1<2, 2, 1, 1, 64, 6>(),     // 7: 64 x 64, 4 waves, BK 64, 6 stages (144 KB): remainder tile, latency-bound, deep ring
    g1<2, 2, 2, 1, 64, 4>(),     // 8: 128 x 64, 4 waves, BK 64, 4 stages (128 KB; 2 stages: 67 against 48 us on 224 tiles): the heavy blocks' surplus
    g1<2, 1, 2, 1, 64, 6, 2>(),  // 9: 128 x 32, 4 waves in 2 k-groups, BK 64, 6 stages (144 KB): a single block over the whole chip
    g1<1, 1, 2, 1, 64, 8, 2>(),  // 10: 64 x 32, 2 waves in 2 k-groups, BK 64, 8 stages (128 KB): the same for a short block
    g1d<4, 8, 2>(),                 // 11: 128 x 256, 8 waves, weights in registers (64 KB)
    g1d<2, 8, 3>(),              // 12: 64 x 256, the same, weights of three steps on their way (32 KB)
    // (5 and 6 serve matrices of 4 GiB and more, whose rows' offsets have more than 32 bits)
    // (tiles whose wavefronts need 256 accumulator registers -- 128 x 256 or 256 x 128 on 4 waves -- were measured
    //  10-25% slower: one wavefront per SIMD cannot keep the matrix pipe issuing back to back)
};
// tokens x output columns of the tile (1 likewise only where an option names it)
const Variant kGemm2[] = {
    g2<2, 4, 2, 32, 3>(),  // 0: 128 x 512, 8 waves, 3 stages (120 KB)
    g2<2, 2, 2, 32, 3>(),  // 1: 128 x 256, 4 waves, 3 stages (72 KB)
    g2<4, 2, 2, 32, 3>(),  // 2: 256 x 256, 8 waves, 3 stages (96 KB)
    g2<1, 4, 2, 32, 3>(),  // 3: 64 x 512, 4 waves, 3 stages (108 KB)
    g2<2, 2, 2, 64, 3, 2>(),  // 4: 128 x 256, 8 waves in 2 k-groups, BK 64, 3 stages (144 KB)
    g2d<8>(),                 // 5: 128 x 512, 8 waves, weights in registers (64 KB)
    g2d<4>(),                 // 6: 64 x 512, weights in registers
    g2d<8, 2>(),              // 7: 128 x 256, weights in registers, 2 k-groups (128 KB)
    g2d<4, 2>(),              // 8: 64 x 256, the same (64 KB)
    g2k(),                    // 9: 64 x 64, weights in registers, 8 wavefronts that take groups of 32 positions in turn (64 KB)
};
constexpr int kNumGemm1 = sizeof(kGemm1) / sizeof(Variant);
constexpr int kNumGemm2 = sizeof(kGemm2) / sizeof(Variant);

}  // namespace

int ff_gemm1_num_variants() { return kNumGemm1; }
int ff_gemm2_num_variants() { return kNumGemm2; }

hipError_t ff_gemm_init(int lds_limit) {
  g_lds_limit = lds_limit;
  for (int i = 0; i < kNumGemm1; ++i) {
    if (kGemm1[i].lds > lds_limit) continue;  // not launchable on this device
    hipError_t e = hipFuncSetAttribute(kGemm1[i].fn, hipFuncAttributeMaxDynamicSharedMemorySize, kGemm1[i].lds);
    if (e != hipSuccess) return e;
  }
  for (int i = 0; i < kNumGemm2; ++i) {  // the ring plus, when there is room, the row-id table
    const void *fns[4] = {kGemm2[i].fn, kGemm2[i].fn_rm[0], kGemm2[i].fn_rm[1], kGemm2[i].fn_rm[2]};
    for (const void *fn : fns) {
      if (fn == nullptr) continue;
      hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

constexpr int kNumCU = 256;

// How the 8 XCDs share V virtual blocks x N n-tiles (see map_tile): log2 of the groups of virtual blocks.
// Eight groups give every XCD its own blocks, whose tokens then stay in one L2, but with V no multiple of 8
// some XCDs get one block more than others, and below 8 some get none at all.  So: fewest rounds of workgroups
// on the busiest XCD (32 CUs; below one round its tiles count), but eight groups unless that saves a thirtieth.
// (Gate/up launch, always eight groups against this rule: 4096/14336, K 7168, 128-token blocks: 1 block 130 -> 69 us,
// 4 blocks 141 -> 79, 12 blocks 241 -> 192; 65 blocks of 77: 938 -> 894; 64 blocks unchanged; 3584/18944 dense, 300
// tokens: 459 -> 185, 9001 tokens 2264 -> 2038, and the down launch 1715 -> 1260.)
// Among grids of no more rounds, or all of one round, the one that fetches less from beyond an XCD's L2: an XCD holds 32 tiles at a time, as many
// of its blocks as it has and the rest tiles of the same block.  A weight line is fetched once for those of its resident
// blocks that keep the neuron, a line of X once for the resident tiles of its block, so more blocks and fewer tiles pay where
// blocks are short and lists sparse.  Fewer groups of blocks have to save a sixth of it.  (4096/14336, eight groups against
// this: 64 blocks of 64, K 3584: gate/up 343 -> 333 us, down 147 -> 138; 64 blocks of 128, K 7168: down 397 -> 389; 2048/8192,
// 32 blocks of 128, K 4096: both 1% less; eight blocks of 128, K 7168, one round of 128 x 256: the call 230 -> 203, 15 of K 3584
// 189 -> 175.)  Two blocks in one round stay apart: they would share too little (256 tokens of 4096/14336 79.6 -> 83.5).
struct Share {
  int w_rows, x_rows;   // a tile's rows (or their pieces) of weights and of X or H, in proportion to the bytes
  double keep;          // share of the neurons on a list; 0: tiles that share nothing to speak of
  int mt;               // token tiles of a block, which share its list
};
static int xcd_groups(long V, long N, const Share &sh) {
  int best = 3;
  double best_cost = 0.0, cost[4];
  for (int xs = 3; xs >= 0; --xs) {
    const long tiles = ((V + (1 << xs) - 1) >> xs) * ((N + (8 >> xs) - 1) / (8 >> xs));
    const long rounds = (tiles + kNumCU / 8 - 1) / (kNumCU / 8);
    cost[xs] = rounds > 1 ? (double)rounds : (double)tiles / (kNumCU / 8);
    if (xs == 3) best_cost = cost[xs] * 31.0 / 32.0;
    else if (cost[xs] < best_cost) { best = xs; best_cost = cost[xs]; }
  }
  if (sh.keep <= 0.0 || (cost[best] <= 1.0 && V <= 2)) return best;
  auto fetch = [&](int xs) {
    const long blocks = std::min<long>((V + (1 << xs) - 1) >> xs, kNumCU / 8);
    const long tiles = std::min<long>((N + (8 >> xs) - 1) / (8 >> xs), std::max<long>(1, kNumCU / 8 / blocks));
    double none = 1.0;
    for (long l = 0; l < std::max<long>(1, blocks / sh.mt); ++l) none *= 1.0 - sh.keep;
    return sh.w_rows * (1.0 - none) / ((double)blocks * sh.keep) + (double)sh.x_rows / (double)tiles;
  };
  const double rounds_best = std::max(1.0, cost[best]);
  for (int xs = best - 1; xs >= 0; --xs)
    if (cost[xs] <= rounds_best && fetch(xs) < fetch(best) * 5.0 / 6.0) best = xs;
  return best;
}
// what the tiles of variant v share in a launch of these parameters
template <class Params>
static Share share_of(const Variant &v, const Params &p, bool gemm1) {
  // (a few much longer lists: their tiles are everywhere; 16 blocks, two of them dense, lose 20 us of 260 in four groups)
  const double keep = p.k.n_heavy > 0 ? 0.0 : (p.idx == nullptr ? 1.0 : std::min(1.0, (double)p.k.k_max / p.d_ffn));
  return Share{gemm1 ? 2 * v.bn : v.bn, v.bm, keep, p.idx == nullptr ? 1 : (p.block + v.bm - 1) / v.bm};
}

// V virtual blocks (each block cut into M tiles of v.bm tokens) x N tiles, preceded by the
// heavy blocks' n_first_per_vb tiles each
static hipError_t launch_variant(const Variant &v, const void *fn, const void *params, int block, int n_blocks,
                                 int N, int n_heavy, int n_first_per_vb, bool gemm1, const Share &share, hipStream_t s) {
  int mt = (block + v.bm - 1) / v.bm;
  int V = n_blocks * mt;
  int NX = n_first_per_vb;
  int xs = xcd_groups(V, N, share);
  int grid = n_heavy * mt * n_first_per_vb + 8 * ((V + (1 << xs) - 1) >> xs) * ((N + (8 >> xs) - 1) / (8 >> xs));
  if (grid <= 0) return hipSuccess;
  void *args1[] = {const_cast<void *>(params), &V, &mt, &N, &xs, &NX};
  void *args2[] = {const_cast<void *>(params), &V, &mt, &N, &xs};
  return hipLaunchKernel(fn, dim3(grid), dim3(v.threads), gemm1 ? args1 : args2, v.lds, s);
}

// Rounds of workgroups (one per CU) that V x N tiles take on the busiest XCD under the mapping that
// launch_variant will use, behind `first` tiles that all XCDs share.
static long xcd_rounds(long V, long N, long first = 0) {
  const int xs = xcd_groups(V, N, Share{});   // (what is shared takes no grid of more rounds)
  const long tiles = ((V + (1 << xs) - 1) >> xs) * ((N + (8 >> xs) - 1) / (8 >> xs)) + (first + 7) / 8;
  return (tiles + kNumCU / 8 - 1) / (kNumCU / 8);
}

static int up64(int v) { return (v + 63) / 64 * 64; }   // (tiles narrower than 64 positions also zero H up to there)

constexpr int kRemainderVariant = 7;
constexpr int kHeavySurplusVariant = 8;
constexpr int kWide128 = 6;
constexpr int kGemm1Direct128 = 11, kGemm1Direct64 = 12;   // the gate/up tiles with the weights in registers
constexpr int kDirect128 = 5, kDirect64 = 6, kDirect128Narrow = 7, kDirect64Narrow = 8, kSplit64 = 9;   // the down-GEMM tiles
constexpr int kHalf128Wide = 4;     // the 128 x 256 down-GEMM tile with eight wavefronts (144 KB)

static bool gemm1_direct(int variant) { return variant >= kGemm1Direct128; }
// whether the offsets of a row and of a token of a tile have 32 bits, which the tiles with the weights in registers need
static bool gemm1_direct_addresses(const Gemm1Params &p) {
  const uint64_t row_bytes = (uint64_t)p.d_model * 2u;
  return (uint64_t)std::max({p.d_ffn, p.rc, 256}) * row_bytes >> 32 == 0;   // (256: the highest tile)
}

// Gate/up tiles by the cost of one round of 256 of them, relative to a round of the 128 x 256 tile (117 us at
// d_model 4096 with the chip full, 4096/14336).  Tiles with fewer positions move more bytes per FLOP, hence cost
// more than their share (0.52, 0.33 and 0.24 for a half, a quarter and an eighth), but fill the chip where a call has
// too few big tiles or would start a last round with a few of them.
struct Gemm1Cost { int variant; double round; };
// One block of up to 64 tokens shares its rows with nobody: a round of 128 x 128 tiles whose lower half is empty waits for fewer
// bytes than two of 64 x 64 (3584/18944, list of all neurons, 61 tokens 74.5 -> 65.5 us, 30 tokens 69.8 -> 60.9; where one round
// of the smaller tiles is enough they win by far: K 14208 59.0 against 40.9; of merged lists only the likely length says so).
constexpr Gemm1Cost kGemm1Short[] = {{kGemm1Direct64, 0.74}, {5, 0.90}, {0, 0.52}, {kRemainderVariant, 0.27}, {10, 0.22}};   // blocks up to 64 tokens
constexpr Gemm1Cost kGemm1Mid[] = {{0, 0.52}, {kHeavySurplusVariant, 0.33}, {9, 0.24}};                      // up to 255
constexpr Gemm1Cost kGemm1Long[] = {{3, 1.0}, {0, 0.52}, {kHeavySurplusVariant, 0.33}, {9, 0.24}};           // 256 and more, and without a list

// The 128 x 256 tile's round where it competes with 128 x 128 for lists of equal length: two of those take 1.10 of it (fitted to 46 calls,
// then to 330.  At 1.08 3584/18944, K 9472, 8200 to 9500 tokens ran 22 rounds of 128 x 128 for 12: 9312 tokens 1872 -> 1755 us, 8401 1604 ->
// 1515; of 20000 calls 79 choose another tile, in the mean 1% faster, the worst 3.5% slower, 3169 tokens in blocks of 177 821 -> 850).
constexpr double kWideRound = 0.945;

hipError_t ff_launch_gemm1(const Gemm1Params &p_in, int variant, int split, int heavy_tiles, int k_likely, hipStream_t s) {
  Gemm1Params p = p_in;
  if (p.idx != nullptr) p.block = std::min(p.block, p.T);   // (one short block: tiles for the tokens that there are)
  p.off32 = gemm1_direct_addresses(p);
  const int n_extent = p.k.k_max + p.rc;                  // longest list
  const bool ragged = p.k.per_block != nullptr;           // lists of unequal length
  const int base_extent = (p.k.n_heavy > 0 ? p.k.k_base : p.k.k_max) + p.rc;   // what all but the heavy blocks have
  const bool chosen = variant < 0;
  if (variant < 0) {
    // Fewest rounds x cost of a round; a smaller tile has to save a thirtieth.  (Measured, us, the larger tile that
    // used to be taken against this choice: 4096/14336, K 7168: 100 tokens, 128 x 128 51 -> 128 x 32 29; 30 tokens in
    // one block, 64 x 256 92 -> 64 x 32 26; K 3584, ten blocks of 64, 64 x 256 114 -> 64 x 64 100; 1100 tokens in blocks
    // of 256, 256 x 128 216 -> 128 x 128 178; dense 3584/18944, 300 tokens, 256 x 128 190 -> 128 x 128 110.)
    const Gemm1Cost *tab = p.block > 64 ? (p.block >= 256 ? kGemm1Long : kGemm1Mid) : kGemm1Short;
    const int n_tab = p.block >= 256 ? 4 : p.block > 64 ? 3 : 5;
    double best = 0.0;
    for (int i = 0; i < n_tab; ++i) {
      const Variant &v = kGemm1[tab[i].variant];
      if (tab == kGemm1Short && tab[i].variant == 0 && (p.n_blocks > 1 || (k_likely > 0 && k_likely + p.rc <= kNumCU * kGemm1[kRemainderVariant].bn))) continue;
      if (v.lds > g_lds_limit || (gemm1_direct(tab[i].variant) && !gemm1_direct_addresses(p))) continue;
      // without a list the blocks mean nothing: token tiles of this variant's height
      const long V = p.idx == nullptr ? (p.T + v.bm - 1) / v.bm : (long)p.n_blocks * ((p.block + v.bm - 1) / v.bm);
      const long first = (long)p.k.n_heavy * ((p.block + v.bm - 1) / v.bm) * ((up64(n_extent) + v.bn - 1) / v.bn - (up64(base_extent) + v.bn - 1) / v.bn);
      const long N = (up64(base_extent) + v.bn - 1) / v.bn;
      const long rounds = first == 0 ? xcd_rounds(V, N) : (V * N + first + kNumCU - 1) / kNumCU;
      const double cost = rounds * tab[i].round;
      if (variant < 0 || cost < best * (30.0 / 31.0)) { variant = tab[i].variant; best = cost; }
    }
    if (variant < 0) return hipErrorInvalidValue;
    if (p.block > 64 && p.block < 256) {
      // The 128 x 256 tile (with the weights in registers where it can address them) moves fewer bytes per FLOP.  It takes lists whole, or
      // leaves its part-filled last tile to the remainder launch (with lists of unequal length every block's own): 0.03 rounds and 0.15 per 8192
      // tokens if that is compensator units alone, nothing if half a tile of them (they cost the main launch as much), else 0.22 per round
      // of remainder tiles.  Rounds are those of the busiest XCD: a whole chip's count took 252 tiles of 18 blocks for one round, and no XCD split
      // of them is.  (ff_sparse_ffn, us, lists cut and rounds of the whole chip -> this: 4096/14336: 700 tokens, K 7168 182 -> 173, 2000 356 ->
      // 338; 2200, K 3584 311 -> 232; 1400, K 5734 315 -> 257; 2900 478 -> 431; 2000, K 10752 515 -> 500; 3584/18944: 480 tokens, K
      // 9472 170 -> 156, 4000 771 -> 740; 1600, K 4736 282 -> 227; 2048/8192: 900 tokens, K 4096 92 -> 91; 2050, K 2048 107 -> 89.  Of
      // 70 calls from 200 to 11000 tokens 3 chose a tile more than 2% slower than the fastest: 5, 6 and 7%.)
      // A few much longer lists: the launch of their ends besides (half a round of tiles at most, 0.4; else further wide tiles).
      // (Measured, wide against 128 x 128: 4096/14336, 16 blocks of 7168 with the first and last dense 0.332 / 0.267 ms.)
      const int wide = gemm1_direct_addresses(p) ? kGemm1Direct128 : kWide128;
      const Variant &w = kGemm1[wide];
      const int n_full = base_extent / w.bn, rem_w = base_extent % w.bn;
      const bool fits = w.lds <= g_lds_limit;
      if (fits && !ragged) {
        const long V = (long)p.n_blocks * ((p.block + w.bm - 1) / w.bm);
        const bool behind = n_full * w.bn >= p.k.k_max;      // nothing but compensator units is left
        const double rest = rem_w == 0 || (behind && rem_w <= 32) ? 0.0 : behind ? 0.03 + 0.15 * p.T / 8192.0 :
                            0.22 * (double)((2 * V * ((rem_w + 63) / 64) + kNumCU - 1) / kNumCU);
        const double whole = (double)xcd_rounds(V, (up64(base_extent) + w.bn - 1) / w.bn);
        const double cut = n_full == 0 ? 1e30 : (double)xcd_rounds(V, n_full) + rest;
        if (kWideRound * (split == 0 ? whole : split > 0 ? cut : std::min(whole, cut)) <= best) {
          variant = wide;
          if (split < 0) split = rem_w > 0 && cut <= whole;
        }
      } else if (fits) {
        const long wide_full = (long)p.n_blocks * n_full;
        const long rem_wgs = (long)p.n_blocks * 2 * ((rem_w + 63) / 64);
        const long surplus = (long)p.k.n_heavy * (n_extent / w.bn - n_full);
        const bool surplus_own = surplus > 0 && 2 * surplus <= kNumCU;
        const double cost_wide = (double)((wide_full + (surplus_own ? 0 : surplus) + kNumCU - 1) / kNumCU) + (surplus_own ? 0.4 : 0.0) +
                                 0.22 * (double)((rem_wgs + kNumCU - 1) / kNumCU);
        // (merged lists: only a bound of their lengths is known here)
        const bool unknown = p.k.n_heavy == 0;
        if (split != 0 && n_full > 0 && (unknown || cost_wide <= best) && wide_full >= 224) {
          variant = wide;
          split = 1;
        }
      }
    }
  }
  if (variant >= kNumGemm1 || kGemm1[variant].lds > g_lds_limit) return hipErrorInvalidValue;
  if (gemm1_direct(variant) && !gemm1_direct_addresses(p)) return hipErrorInvalidValue;   // forced
  const Variant &v = kGemm1[variant];
  if (p.idx == nullptr) {
    p.block = v.bm;
    p.n_blocks = (p.T + v.bm - 1) / v.bm;
  }
  // One or two blocks with rows a multiple of 4 KB apart: tiles in step ask for the same channels of all their rows at once, and
  // how much that costs depends on where the matrices lie in memory.  From different places on, 4096/14336, list of 14193, 30
  // tokens: 57.6 -> 47.4 us in one process, 45.5 -> 46.0 in another; 256 tokens in two blocks, K 10752, 80.0 -> 74.8 and 74.8 ->
  // 74.6.  Other rows gain nothing, and two blocks lose where they share most rows (two merged lists of 3584/18944 139 -> 145); more
  // blocks lose anyhow: three of 3584/18944, K 9472, 66.9 -> 84.9, four of 4096/14336, K 10752, 124 -> 155, five 121 -> 169.
  // (A start by the tile's position, the same for all blocks, is as good with one block, gains nothing with two and still loses
  // from three on.  The tiles with the weights in registers do not have it.)
  p.spread = p.idx != nullptr && p.block <= v.bm && p.n_blocks <= 2 && p.d_model % 2048 == 0;
  Gemm1Params q = p;
  q.full_only = 0;
  q.rem_bn = 0;
  // The positions beyond a block's last full N tile (the compensator's units, typically) would
  // cost the block a whole extra tile.  When that extra tile starts a new round of workgroups
  // over the CUs, they go to a second launch with 64 x 64 tiles instead, which spreads that
  // little work over the whole chip.
  const int rem = n_extent % v.bn;
  bool do_split = false;
  // (Never with a tile of less than 64 positions, forced or not: H is zero up to the next multiple of 64 behind a list, and
  // a remainder that may start on any multiple of 32 would leave that to nobody where a list ends on one.)
  if ((chosen ? split != 0 : split > 0) && (rem > 0 || ragged) && n_extent >= v.bn && v.bn >= (chosen ? 128 : 64) && variant != kRemainderVariant) {
    const int n_full = base_extent / v.bn;
    // One workgroup per CU, whatever its LDS would allow: every tile chosen here has eight wavefronts of more than 128
    // registers.  Rounds are those of the busiest XCD.  (With two workgroups per CU where LDS has room for two, which the tiles
    // with the weights in registers leave, and rounds over the whole chip, gate/up us -> this: 64-token blocks of 4096/14336, 4096
    // tokens, K 7168 626 -> 595, K 5120 478 -> 452, 2103 tokens, K 3584 238 -> 208; 2048/8192, 2785 tokens, K 4096 160 -> 139;
    // 128-token blocks of 4096/14336, 2795 tokens, K 7168 339 -> 324.  Of 90 calls that it changes the least favoured: 423 -> 430.)
    // With a few longer lists the ends of those are tiles in front of the others (4096/14336, both ends dense, 1907 tokens in blocks
    // of 64, K 10752, split without counting them 490 -> 505), or, with tiles of 128 tokens, a third launch that a split has to
    // pay for too, so there the whole chip's count has to fall (2048/8192, 1845 tokens in blocks of 128, K 4096: 96 -> 112).
    const long mt = (p.block + v.bm - 1) / v.bm, vb = (long)p.n_blocks * mt;
    const bool third = ragged && v.bm >= kGemm1[kHeavySurplusVariant].bm;
    const long ends = (long)p.k.n_heavy * mt * (n_extent / v.bn - n_full);
    auto rounds = [&](long n) { return third ? (vb * n + kNumCU - 1) / kNumCU : xcd_rounds(vb, n, ends); };
    const long rounds_all = rounds(n_full + 1), rounds_full = rounds(n_full);
    do_split = split > 0 || (rounds_full < rounds_all && 2 * (base_extent % v.bn) <= v.bn);
  }
  const int heavy = p.k.n_heavy;
  if (!do_split) {
    const int N = (up64(base_extent) + v.bn - 1) / v.bn, N_all = (up64(n_extent) + v.bn - 1) / v.bn;
    return launch_variant(v, v.fn, &q, p.block, p.n_blocks, N, heavy, N_all - N, true, share_of(v, p, true), s);
  }
  q.full_only = 1;
  const int N = base_extent / v.bn, N_all = n_extent / v.bn;
  // The heavy blocks' positions beyond the common length.  As tiles of the main launch (with the first ids)
  // they start one more round of workgroups on a mostly idle chip; up to half a round of them run instead
  // as a launch of their own with 128 x 64 tiles, which spreads them over all of it
  // (first and last block dense on 4096/14336, 64 blocks: 0.952 -> 0.920 ms for the three launches).
  const Variant &hv = kGemm1[kHeavySurplusVariant];
  // the remainder's tile: 64 x 64 with a deep ring while that is what it takes to give every CU a workgroup,
  // 128 x 64 (fewer bytes per FLOP) once those fill the chip as well
  const int rem_est = ragged ? (heavy > 0 ? base_extent % v.bn : v.bn / 2) : rem;
  const bool rem_wide = hv.bm <= v.bm && variant != kHeavySurplusVariant &&
                        (long)p.n_blocks * ((p.block + hv.bm - 1) / hv.bm) * ((rem_est + hv.bn - 1) / hv.bn) >= kNumCU;
  const Variant &r = kGemm1[rem_wide ? kHeavySurplusVariant : kRemainderVariant];
  const long surplus_tiles = (long)heavy * ((p.block + v.bm - 1) / v.bm) * (N_all - N);
  const bool heavy_small = heavy > 0 && surplus_tiles > 0 && hv.bm <= v.bm && variant != kHeavySurplusVariant &&
                           (heavy_tiles > 0 || (heavy_tiles < 0 && 2 * surplus_tiles <= kNumCU));
  {
    hipError_t e = launch_variant(v, v.fn, &q, p.block, p.n_blocks, N, heavy, heavy_small ? 0 : N_all - N, true, share_of(v, p, true), s);
    if (e != hipSuccess) return e;
  }
  q.full_only = 0;
  q.rem_bn = v.bn;
  const int rem0 = n_extent - rem;
  const bool only_comp = !ragged && rem0 >= p.k.k_max && rem0 % 64 == 0 && (uint64_t)p.rc * (uint64_t)p.d_model * 2u >> 32 == 0;
  if (only_comp) {
    // Nothing but compensator units is left, the same columns for every token.  64 tokens to a workgroup where 32 would be more
    // workgroups than CUs.
    int K = p.k.k_max, u0 = rem0 - K;
    const bool narrow = rem <= 32, tall = p.T > 32 * kNumCU;
    const void *fn = narrow ? (tall ? reinterpret_cast<const void *>(&ff_comp_kernel<2, 32>) : reinterpret_cast<const void *>(&ff_comp_kernel<1, 32>))
                            : (tall ? reinterpret_cast<const void *>(&ff_comp_kernel<2, 64>) : reinterpret_cast<const void *>(&ff_comp_kernel<1, 64>));
    const int bm = tall ? 64 : 32;
    void *args[] = {&q, &K, &u0};
    return hipLaunchKernel(fn, dim3((p.T + bm - 1) / bm, narrow ? 1 : up64(rem) / 64), dim3(512), args, 0, s);
  }
  if (heavy_small) {
    // everything of a heavy block from where the main launch stopped, its part-filled last tile included
    Gemm1Params qh = q;
    qh.rem_cap = N * v.bn;
    hipError_t e = launch_variant(hv, hv.fn, &qh, p.block, p.n_blocks, 0, heavy, (n_extent - qh.rem_cap + hv.bn - 1) / hv.bn, true, Share{}, s);
    if (e != hipSuccess) return e;
    q.skip_heavy = 1;
  }
  q.k.n_heavy = heavy_small ? q.k.n_heavy : 0;   // every block has at most one part-filled tile: no heavy region
  const int rem_max = ragged ? v.bn - 1 : rem;
  return launch_variant(r, r.fn, &q, p.block, p.n_blocks, (rem_max + r.bn - 1) / r.bn, 0, 0, true, Share{}, s);
}



// The tile with its source of gathered row ids: computed for the identity list; else an LDS table of 16-bit ids
// behind the ring when it fits (ids run up to d_ffn + rc - 1), the streamed list where the tile has it, scalar loads.
// row_mode > 0 forces one of them where the tile has it and it fits (else fn = nullptr).
static Variant with_rows(Variant v, const Gemm2Params &p, int row_mode, int tab_bytes) {
  if (p.idx == nullptr) return v;
  const bool table_fits = p.d_ffn + p.rc <= 65536 && v.lds + tab_bytes <= g_lds_limit;
  const bool ring_fits = v.fn_rm[2] != nullptr && v.lds + kIdRingBytes <= g_lds_limit;
  const int mode = row_mode > 0 ? row_mode : (table_fits ? 1 : (ring_fits ? 3 : 2));
  if (mode == 1 && table_fits && v.fn_rm[0] != nullptr) {
    v.lds += tab_bytes;
    v.fn = v.fn_rm[0];
  } else if (mode == 3 && ring_fits) {
    v.lds += kIdRingBytes;
    v.fn = v.fn_rm[2];
  } else {
    v.fn = mode == 2 ? v.fn_rm[1] : nullptr;
  }
  return v;
}

// What a round of 256 tiles costs, in us, with the weights coming from HBM: fixed + 64-position steps x (idle .. full:
// a few workgroups on the chip, or all of it busy).  The tiles with the weights in registers run a step of 128 x 512 in 1.6 us
// with the chip full (1.32 PFLOP/s dense), one of 64 x 512 in 1.1 to 1.24; alone on the chip they wait for their loads.  The
// tiles of 256 columns serve calls with few columns and blocks (2048/8192, K 4096, 32 blocks of 128, one round: 75.9 us with both
// operands in LDS, 66.5 with the weights in registers).  The 64 x 64 tiles: see their kernel; with one or two tiles of tokens, one
// on each CU, a step takes 0.25 to 0.3, with four 0.35 to 0.45 (200 tokens of 4096/14336, K 3584: at 0.33 throughout they would be
// taken, 65.8 -> 68.3; at 0.41 the gains of 3 to 8% on 9 to 100 tokens of 4096/14336 would be lost; at 0.37 478 tokens of 2048/8192, both
// ends dense, 77.0 -> 78.7).
// (The figures of the tiles in registers of 512, 256 and, below 128 tokens, 256 columns are fitted to every tile and cut of 127 calls of the
// three larger layers.  Calls, us, by the figures before, 1.25 .. 1.6, 0.8 .. 0.95 and 0.45 .. 1.1 a step, and by these: 2048/8192, 1350 tokens
// 117 -> 111, first and last block dense 520 122 -> 110, 850 138 -> 127, 4096 298 -> 285, dense 850 105 -> 98; 4096/14336, 2300 in blocks of 64
// 602 -> 574; 3584/18944, both ends dense 520 349 -> 323.  Every tile and cut of 836 calls of these layers measured, from 9 to 16000 tokens:
// the two sets of figures choose differently in 119, geometric mean 0.966, of which 8 lost more than 1%, 2% but for one of 4% and one of 7%.)
// The last three, slower at the same tile, are what matrices of 4 GiB and more and lists too long for the row-id table get.
struct Gemm2Cost { int variant; double idle, full, fixed; };
constexpr Gemm2Cost kGemm2Cost[] = {{kDirect128, 1.15, 1.7, 9.0}, {kDirect64, 1.15, 1.24, 6.0}, {kHalf128Wide, 0.75, 1.1, 6.0},
                                     {kDirect128Narrow, 0.61, 0.95, 9.0}, {kDirect64Narrow, 0.53, 0.69, 8.7}, {kSplit64, 0.25, 0.33, 5.0},
                                     {0, 1.4, 2.05, 9.0}, {2, 1.25, 2.07, 9.0}, {3, 1.25, 1.45, 8.0}};
// A W_down of at most 4 MiB, an XCD's L2, is fetched once and waited for little after that, and its lists are few steps long: what it costs
// to start a tile decides.  These figures are fitted to every tile and cut of 554 calls of 256/688, 256/1024, 256/4096, 512/1024, 512/2048,
// 512/4096, 640/3072 and 768/2048, 100 to 16384 tokens: dense, lists of equal length, first and last block dense.  Geometric mean over each
// call's fastest tile 1.005, by the figures above 1.033; 6 more than 1% slower than by those, the most 4% (256/688, K 516, 9000 tokens).  (256/688,
// us, by the figures above and by these: dense 5000 tokens 26.3 -> 23.5, 7000 33.8 -> 27.5, 9566 38.4 -> 35.2; K 344, 5000 24.5 -> 20.4, 7000
// 31 -> 23.5; K 172, 14000 26.1 -> 24.1; both ends dense, 9000 31.1 -> 29.5.  With 5.5 MiB and more the figures above choose well enough, 1.010
// of the fastest for 1024/2816, 1.016 for 1024/4096.)
constexpr uint64_t kXcdL2Bytes = 4 << 20;
constexpr Gemm2Cost kGemm2CostL2[] = {{kHalf128Wide, 0.75, 1.1, 6.5}, {kDirect64Narrow, 0.55, 0.65, 6.5}, {kSplit64, 0.2, 0.2, 3.0}};
// g for V tiles of tokens, with lists of equal length and with a few longer ones alike (two blocks of 45 tokens, one dense,
// 4096/14336, K 3584: 64 x 256 tiles by figures that did not know V, 123.8 us, 64 x 64 ones 118.8)
static Gemm2Cost gemm2_price(Gemm2Cost g, const Gemm2Params &p, long V, bool heavy_cut) {
  if ((uint64_t)p.d_ffn * (uint64_t)p.d_model * 2u <= kXcdL2Bytes) {
    for (const Gemm2Cost &c : kGemm2CostL2)
      if (c.variant == g.variant) g = c;
    // With one tile of 256 columns a longer call is many tiles of tokens, and the H of 64 tokens is mostly in the L2 of the XCD that the
    // gate/up tile of their 128 ran on: another one.  (256/688, 64 x 256 against 128 x 256: K 344, 14000 tokens 34.0 / 32.5, 8200 25.1 / 24.9;
    // K 172, three steps, 14000 24.1 / 26.1.  Blocks of 16 merged, 10956 tokens, 64 x 64 against 128 x 256: 64.5 / 61.0.)
    if (p.d_model <= kGemm2[kDirect64Narrow].bn && p.idx != nullptr && p.block > 64 && !heavy_cut) {
      if (g.variant == kDirect64Narrow) g.full = 1.0;
      if (g.variant == kSplit64) g.full = 0.25;
    }
    return g;
  }
  // 64 x 64 tiles fetch every row once for each 64 tokens: more than two such tiles of tokens make each other wait
  if (g.variant == kSplit64 && V > 2) g.full = 0.365;
  // one or two tiles of 64 tokens share no rows between the 64 x 256 ones of a column: a full chip of those runs at HBM's rate
  if (g.variant == kDirect64Narrow && V <= 2) return {g.variant, 0.45, 1.1, 6.0};
  return g;
}
static bool gemm2_direct(int variant) { return variant >= kDirect128; }
// Whether the tiles with the weights in registers can address these matrices: a listed row's offset into W_down is the
// product of two 24-bit numbers in 32 bits, a token's offset into a tile of H has 32 bits too.
static bool gemm2_direct_addresses(const Gemm2Params &p) {
  const uint64_t row_bytes = (uint64_t)p.d_model * 2u;
  if (row_bytes >> 24 || (uint64_t)kGemm2[kDirect128].bm * (uint64_t)p.hs * 2u >> 32) return false;
  return p.idx == nullptr || (uint64_t)p.d_ffn * row_bytes >> 32 == 0;
}
// whether the launcher takes the tile for these lists of ntot positions: it has the source of row ids that was asked for, if
// any; weights in registers need W_down below 4 GiB and the row ids in LDS
static bool gemm2_takes(int variant, const Gemm2Params &p, int row_mode, int ntot) {
  const Variant &v = kGemm2[variant];
  if (gemm2_direct(variant) && (!gemm2_direct_addresses(p) || (uint64_t)p.d_ffn * (uint64_t)p.d_model * 2u >> 32)) return false;
  if (v.lds + (gemm2_direct(variant) ? 0 : kIdRingBytes) > g_lds_limit) return false;
  return with_rows(v, p, row_mode, 2 * up64(ntot)).fn != nullptr;
}

// every list cut into n pieces (n >= 2, p.split_part has room for them)
static hipError_t launch_gemm2_cut(Gemm2Params p, int variant, int n, int row_mode, hipStream_t s) {
  const int len = ((p.k.k_max + p.rc + n - 1) / n + 63) / 64 * 64;
  const Variant v = with_rows(kGemm2[variant], p, row_mode, 2 * len);
  if (v.fn == nullptr) return hipErrorInvalidValue;
  if (p.idx == nullptr) {
    p.block = v.bm;
    p.n_blocks = (p.T + v.bm - 1) / v.bm;
  }
  p.n_split = n;
  p.n_cols = (p.d_model + v.bn - 1) / v.bn;
  p.part = p.split_part;
  p.k.n_heavy = 0;
  hipError_t e = launch_variant(v, v.fn, &p, p.block, p.n_blocks, p.n_cols * n, 0, 0, false, Share{}, s);
  if (e != hipSuccess) return e;
  void *args[] = {&p};
  return hipLaunchKernel(reinterpret_cast<const void *>(&ff_gemm2_reduce_kernel), dim3(p.T, (p.d_model + 1023) / 1024), dim3(256), args, 0, s);
}

constexpr int kMaxShortPieces = kMaxPieces - 1;
constexpr int kMaxFreePieces = 4;   // what the launcher takes by itself: more partial sums cost more than shorter pieces gain
constexpr size_t kPartCapBytes = (size_t)48 << 20;

constexpr size_t kSplitCapBytes = (size_t)96 << 20;
size_t ff_gemm2_split_bytes(int n_tokens, int d_model) {
  const size_t per_piece = (size_t)n_tokens * d_model * sizeof(float);
  // (cuts are tried up to two rounds of tiles; blocks only make the tiles more)
  long tiles = 2 * kNumCU;
  for (const Gemm2Cost &g : kGemm2Cost) {
    const Variant &v = kGemm2[g.variant];
    tiles = std::min<long>(tiles, ((long)n_tokens + v.bm - 1) / v.bm * (((long)d_model + v.bn - 1) / v.bn));
  }
  const size_t n = std::min<size_t>({kSplitCapBytes / per_piece, (size_t)(kMaxPieces - 1), (size_t)(2 * kNumCU / tiles)});
  return n >= 2 ? n * per_piece : 0;
}

size_t ff_gemm2_part_bytes(int n_tokens, int block, int d_model) {
  if (n_tokens <= block) return 0;   // one block: nothing is longer than the rest
  const size_t want = (size_t)2 * kMaxPieces * block * d_model * sizeof(float);
  return want < kPartCapBytes ? want : kPartCapBytes;
}

hipError_t ff_launch_gemm2(const Gemm2Params &p_in, int variant, int split, int row_mode, int ksplit, int nsplit, hipStream_t s) {
  Gemm2Params p = p_in;
  p.block = std::min(p.block, p.T);
  const bool chosen = variant < 0;
  const size_t per_piece = (size_t)p.T * p.d_model * sizeof(float);
  const long room = p.split_part != nullptr ? std::min<long>((long)(p.split_bytes / per_piece), kMaxPieces - 1) : 1;
  int pieces = nsplit > 1 ? (int)std::min<long>(nsplit, room) : 1;
  if (chosen) {
    // The tile, and into how many pieces every list is cut: the cheapest by the measured times above.  A cut adds one
    // more launch and its partial sums written and read once (3 us + 0.3 per MB).  (A few much longer lists have a cut
    // of their own, below, that leaves the other blocks' sums alone.)  In us, whole lists on the tiles with both operands in
    // LDS against this choice: 4096/14336, K 7168: 64 blocks of 128 456 -> 378, one of 100 tokens 91 -> 28; K 3584, 64
    // blocks of 64 172 -> 145; 2048/8192, K 4096, 700 tokens 58 -> 32; 3584/18944, K 10419, 128 blocks 1220 -> 1005; dense
    // 4096/14336, 4096 tokens 474 -> 364; dense 3584/18944, 300 tokens 275 -> 75.
    const bool may_cut = nsplit < 0 && split < 0 && ksplit < 0 && p.k.n_heavy == 0;
    const int base = (p.k.n_heavy > 0 ? p.k.k_base : p.k.k_max) + p.rc, ntot = p.k.k_max + p.rc;
    const int n0 = pieces;
    double best = 0.0;
    // A few much longer lists that will be cut (below): their pieces start first, on CUs that the common tiles leave idle
    // where there are such, else ahead of everybody.  That favours the tiles with the weights in registers, the large ones, which
    // leave the most, ahead of the 64 x 64 ones; the others only where none of those applies.  (First and last block dense, us per call at 4096/14336,
    // priced without the pieces against this: 2000 tokens 502 / 471, 500 327 / 303, 2000 in blocks of 256 565 / 537, 1500 in
    // blocks of 64, K 3584 361 / 336; 64 x 512 tiles must save a tenth, since they take twice the pieces, those
    // after them 7%.)  Not asked: ksplit, which is to
    // change the long lists' sums and no others, hence no tile.
    const int surplus = up64(ntot) - up64(base);
    const bool heavy_cut = split != 1 && p.part != nullptr && p.k.n_heavy > 0 && 8L * surplus >= up64(base);
    const bool narrow = gemm2_takes(kDirect64Narrow, p, row_mode, ntot);
    for (const Gemm2Cost &g : kGemm2Cost) {
      if (heavy_cut && (narrow || (variant >= 0 && gemm2_direct(variant))) && !gemm2_direct(g.variant)) continue;
      const Variant &v = kGemm2[g.variant];
      if (narrow && v.bn > kGemm2[kDirect64Narrow].bn && p.d_model <= kGemm2[kDirect64Narrow].bn) continue;   // (half of its columns would not exist)
      const long V = p.idx == nullptr ? (p.T + v.bm - 1) / v.bm : (long)p.n_blocks * ((p.block + v.bm - 1) / v.bm);
      const long N = (p.d_model + v.bn - 1) / v.bn;
      for (int n = n0; n == n0 || (may_cut && n <= room && V * N * n <= 2 * kNumCU && ntot >= n * 64); ++n) {
        if (!gemm2_takes(g.variant, p, row_mode, (ntot + n - 1) / n)) continue;
        const int xs = xcd_groups(V, N * n, n > 1 ? Share{} : share_of(v, p, false));
        const long tiles = ((V + (1 << xs) - 1) >> xs) * ((N * n + (8 >> xs) - 1) / (8 >> xs));   // of the busiest XCD
        const double steps = ((base + n - 1) / n + 63) / 64, busy = (double)(tiles % (kNumCU / 8)) / (kNumCU / 8);
        const Gemm2Cost c = gemm2_price(g, p, V, heavy_cut);
        double cost = (double)(tiles / (kNumCU / 8)) * (c.fixed + steps * c.full);
        if (busy > 0.0) cost += c.fixed + steps * (c.idle + (c.full - c.idle) * busy);
        if (n > 1) cost += 3.0 + (double)n * (double)per_piece / 3.3e6;
        if (heavy_cut) {
          const long heavy = (long)p.k.n_heavy * ((p.block + v.bm - 1) / v.bm) * N;
          const long free_pieces = std::max<long>(1, std::min<long>(kNumCU / heavy, kMaxFreePieces));
          const double piece_steps = (double)((surplus + free_pieces - 1) / free_pieces) / 64;
          // With more than a round of common tiles the CUs that no piece is on go on with those, which the large tiles, of few and long pieces, gain by
          // most: 128 x 512 ones, in blocks of up to 64 tokens 64 x 512 ones, cost their share of a round, the others' pieces a round, as they do
          // beside fewer common tiles.  (First and last block dense, us, a round for all of them against this: 4096/14336, K 3584, 2600 tokens in
          // blocks of 64 459 -> 434, 3000 483 -> 461; 3584/18944, K 4736, 2909 549 -> 515; 2048/8192, K 2048, blocks of 128, 11609 366 -> 338.  Of every
          // tile of 404 calls, 64 to 320 tokens a block: 1.003 of the fastest, a round for all of them 1.005; filling up the last round with all tiles' pieces
          // as so many tiles more, 1.005 too, lost 6% and more on 4096/14336, K 3584, 1600 tokens in blocks of 192 (361 -> 385) and 3584/18944, K
          // 9472, 2909 in blocks of 160 (1031 -> 1099).  What this loses against a round for all: 2048/8192, K 4096, 5713 in blocks of 160 493 -> 525,
          // 4096/14336, K 7168, 3300 in blocks of 96 818 -> 845, 4951 in blocks of 128 922 -> 944.)
          const bool shares = g.variant == (p.block > 64 ? kDirect128 : kDirect64);
          const double rounds = (double)(heavy * free_pieces) / kNumCU;
          if (V * N + heavy * free_pieces <= kNumCU)
            cost = c.fixed + steps * (c.idle + (c.full - c.idle) * (double)(V * N + heavy * free_pieces) / kNumCU);
          else
            cost += (V * N > kNumCU && shares ? rounds : std::ceil(rounds)) * (c.fixed + piece_steps * c.full);
        }
        if (variant < 0 || cost < best * (!heavy_cut ? 0.98 : g.variant == kDirect64 ? 0.9 : 0.93)) { variant = g.variant; pieces = n; best = cost; }
      }
    }
  }
  if (variant < 0 || variant >= kNumGemm2) return hipErrorInvalidValue;
  if (gemm2_direct(variant) && !gemm2_direct_addresses(p)) return hipErrorInvalidValue;   // forced
  if (pieces > 1) return launch_gemm2_cut(p, variant, pieces, row_mode, s);
  const int n_pad = (p.k.k_max + p.rc + 63) / 64 * 64;   // whole k-steps of the longest BK
  const int tab_bytes = ((2 * n_pad + 15) / 16) * 16;
  // the eight-wavefront 128 x 256 tile leaves 16 KB for that table; a longer list streams through
  // a small LDS ring instead (row-id mode 3)
  const int half128 = kHalf128Wide;
  if (p.idx == nullptr) {   // without a list the blocks mean nothing: token tiles of this variant's height
    p.block = kGemm2[variant].bm;
    p.n_blocks = (p.T + p.block - 1) / p.block;
  }
  Gemm2Params q = p;
  auto with_row_mode = [&](const Variant &v) { return with_rows(v, p, row_mode, tab_bytes); };
  const Variant v = with_row_mode(kGemm2[variant]);
  if (v.fn == nullptr) return hipErrorInvalidValue;
  const int N = (p.d_model + v.bn - 1) / v.bn;
  // Heavy blocks first only when their k loops are much longer (a dense block among half-sparse
  // ones): moving their tiles off their own XCD costs that XCD's even share of tiles, which
  // for a slightly longer list is all loss (measured 0.48 -> 0.63 ms for one list one longer).
  // Cut along k instead, the long lists cost their XCD nothing, which is worth it from an eighth longer on:
  // the surplus over the common length becomes short pieces, as many as give every CU one (they start at
  // once and take a fraction of a tile time), no shorter than 256 positions, no more than p.part has room for.
  const int cut0 = (p.k.k_base + p.rc + 63) / 64 * 64;
  const int surplus = n_pad - cut0;
  if (ksplit != 0 && split != 1 && p.part != nullptr && p.k.n_heavy > 0 && 8L * surplus >= cut0) {
    const long heavy_tiles = (long)p.k.n_heavy * ((p.block + v.bm - 1) / v.bm) * N;
    const size_t per_piece = (size_t)p.k.n_heavy * p.block * p.d_model * sizeof(float);
    long want = std::min<long>(ksplit > 0 ? ksplit : kNumCU / heavy_tiles, ksplit > 0 ? kMaxShortPieces : kMaxFreePieces);
    want = std::min<long>(want, (long)(p.part_bytes / per_piece) - 1);
    if (want >= (ksplit > 0 ? 1 : 2)) {
      const int len = std::max(256, (int)((surplus + want - 1) / want + 63) / 64 * 64);
      q.piece_len = len;
      q.cut0 = cut0;
      q.n_pieces = 1 + (surplus + len - 1) / len;
    }
  }
  if (q.n_pieces == 0 && 2L * (p.k.k_max + p.rc) < 3L * (p.k.k_base + p.rc)) q.k.n_heavy = 0;
  // Equal tiles in whole rounds: V x N tiles on kNumCU CUs take ceil(V N / kNumCU) tile times, and a last
  // round that is at most half full wastes the rest of the chip (3584 columns, 128 blocks: 896 tiles,
  // 3.5 rounds).  Then the last nq column tiles of every block leave the main launch, which
  // becomes whole rounds, and run as tiles of half the size in a second launch of one round that
  // takes little more than half a tile time.  (Tiles with both operands in LDS only; those with the weights in registers
  // are priced with their part-filled last round.)
  Variant h = with_row_mode(kGemm2[half128]);
  if (h.fn == nullptr) { row_mode = -1; h = with_row_mode(kGemm2[half128]); }   // the second launch's tile picks its own
  const int V = p.n_blocks * ((p.block + v.bm - 1) / v.bm);
  int nq = 0;
  const bool bigger = v.bm * v.bn > h.bm * h.bn;   // the main tile is larger than the second launch's
  if (split == 1 && N >= 2 && bigger) {
    nq = 1;
  } else if (split < 0 && chosen && !gemm2_direct(variant) && p.k.per_block == nullptr && bigger && v.lds * 2 > g_lds_limit) {
    const long tiles = (long)V * N;
    const long full = tiles / kNumCU, rem = tiles % kNumCU;
    if (full >= 2 && rem > 0 && 2 * rem <= kNumCU) {
      const int cand = (int)((rem + V - 1) / V);
      const long main_tiles = (long)V * (N - cand);
      const long half_tiles = (long)p.n_blocks * ((p.block + h.bm - 1) / h.bm) * ((p.d_model - (N - cand) * v.bn + h.bn - 1) / h.bn);
      if (cand < N && (main_tiles + kNumCU - 1) / kNumCU == full && half_tiles <= kNumCU) nq = cand;
    }
  }
  if (q.n_pieces > 0) {   // (then nq == 0: the column split is for lists of equal length, or forced)
    hipError_t e = launch_variant(v, v.fn, &q, p.block, p.n_blocks, N, q.k.n_heavy, N * (q.n_pieces - 1), false, share_of(v, p, false), s);
    if (e != hipSuccess) return e;
    void *args[] = {&q};
    return hipLaunchKernel(reinterpret_cast<const void *>(&ff_gemm2_reduce_kernel), dim3(q.k.n_heavy * p.block, (p.d_model + 1023) / 1024), dim3(256),
                           args, 0, s);
  }
  if (nq == 0) return launch_variant(v, v.fn, &q, p.block, p.n_blocks, N, q.k.n_heavy, N, false, share_of(v, p, false), s);
  hipError_t e = launch_variant(v, v.fn, &q, p.block, p.n_blocks, N - nq, q.k.n_heavy, N - nq, false, share_of(v, p, false), s);
  if (e != hipSuccess) return e;
  q.col0 = (N - nq) * v.bn;
  const int N2 = (p.d_model - q.col0 + h.bn - 1) / h.bn;
  return launch_variant(h, h.fn, &q, p.block, p.n_blocks, N2, q.k.n_heavy, N2, false, share_of(h, p, false), s);
}
