// Expert-neuron predictor (Sec. 3.2): pooling (Eq. 12), two-layer MLP (Eq. 13)
// and top-K selection (Eq. 14), all in float64 so that the selected set is the
// one the real-number scores define.  Every reduction has a fixed order, so
// results are bitwise reproducible from run to run.
#include "ff_internal.h"

#include <algorithm>
#include <utility>

namespace {

__device__ __forceinline__ void unpack8(const uint4 &v, double *o) {
  o[0] = (double)__uint_as_float(v.x << 16); o[1] = (double)__uint_as_float(v.x & 0xffff0000u);
  o[2] = (double)__uint_as_float(v.y << 16); o[3] = (double)__uint_as_float(v.y & 0xffff0000u);
  o[4] = (double)__uint_as_float(v.z << 16); o[5] = (double)__uint_as_float(v.z & 0xffff0000u);
  o[6] = (double)__uint_as_float(v.w << 16); o[7] = (double)__uint_as_float(v.w & 0xffff0000u);
}

// ---- Eq. 12, logits z_t = q . x_t / sqrt(d_model): one wavefront per token ----
__global__ __launch_bounds__(256) void ff_logits_kernel(const bf16_t *__restrict__ x,
                                                        const bf16_t *__restrict__ q,
                                                        double *__restrict__ z, int T, int d_model) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + wave;
  if (t >= T) return;
  const bf16_t *row = x + (size_t)t * d_model;
  double acc = 0.0;
  for (int c = lane * 8; c < d_model; c += 512) {
    double xv[8], qv[8];
    unpack8(*reinterpret_cast<const uint4 *>(row + c), xv);
    unpack8(*reinterpret_cast<const uint4 *>(q + c), qv);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc = fma(xv[j], qv[j], acc);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) z[t] = acc / sqrt((double)d_model);
}

// ---- Eq. 12, a_b = sum_t p_t x_t over one block, and its share of Eq. 13's first layer ----
// grid (ceil(d_model/512), n_blocks, shares of the r outputs), 256 threads: each lane owns 8 channels,
// the four wavefronts take every fourth token and are summed in wave order.  The workgroup
// then multiplies its 512 pooled channels into the first predictor layer, hpart[b][slice][j] =
// sum_{c in slice} a_b[c] W1[c][j]; the next kernel adds the slices in slice order.
template <bool SOFTMAX>
__global__ __launch_bounds__(256) void ff_pool_kernel(const bf16_t *__restrict__ x,
                                                      const double *__restrict__ z,
                                                      const bf16_t *__restrict__ w1,
                                                      double *__restrict__ hpart, int T,
                                                      int d_model, int Nb, int r) {
  extern __shared__ double p_s[];          // SOFTMAX: Nb weights
  __shared__ double red[4][512];
  __shared__ double red1[8];
  __shared__ double a_s[512];              // this workgroup's pooled channels
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b = blockIdx.y;
  const int t0 = b * Nb;
  const int n = min(T, t0 + Nb) - t0;
  const int c = blockIdx.x * 512 + lane * 8;
  const bf16_t *xc = x + (size_t)t0 * d_model + min(c, d_model - 8);   // (channels past d_model: not used)
  uint4 v[8];
  auto load_rows = [&](int i) __attribute__((always_inline)) {     // past the end: the last row again, not added
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint4 *>(xc + (size_t)min(i + 4 * u, n - 1) * d_model);
  };
  if (SOFTMAX) {
    // the first rows are on their way while the weights are formed
    const double z0 = z[t0 + min(tid, n - 1)];
    if (wave < n) load_rows(wave);
    __builtin_amdgcn_sched_barrier(0);
    // every wavefront reduces by lane exchanges, the four results go through LDS once (a tree over the workgroup had sixteen
    // barriers: 700 tokens in blocks of 128, logits and pooling 18.2 us,
    // this way, with the first rows requested above, 16.7)
    double m = -INFINITY;
    for (int i = tid; i < n; i += 256) m = fmax(m, i == tid ? z0 : z[t0 + i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if (lane == 0) red1[wave] = m;
    __syncthreads();
    m = fmax(fmax(red1[0], red1[1]), fmax(red1[2], red1[3]));
    double part = 0.0;
    for (int i = tid; i < n; i += 256) {
      const double e = exp((i == tid ? z0 : z[t0 + i]) - m);
      p_s[i] = e;
      part += e;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    if (lane == 0) red1[4 + wave] = part;
    __syncthreads();
    const double s = (red1[4] + red1[5]) + (red1[6] + red1[7]);
    for (int i = tid; i < n; i += 256) p_s[i] = p_s[i] / s;
    __syncthreads();
  }
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (SOFTMAX) {
    for (int i = wave; i < n; i += 32) {     // 8 token rows in flight, added in token order
      if (i > wave) load_rows(i);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i + 4 * u < n) {
          double xv[8];
          unpack8(v[u], xv);
          const double w = p_s[i + 4 * u];
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[j] = fma(w, xv[j], acc[j]);
        }
    }
  } else if (c < d_model) {
    // (the mean: with the loop above, its conditions cost 1.2 us of 13.3 for 32 blocks)
    int i = wave;
    for (; i + 28 < n; i += 32) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint4 *>(xc + (size_t)(i + 4 * u) * d_model);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        double xv[8];
        unpack8(v[u], xv);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += xv[j];
      }
    }
    for (; i < n; i += 4) {
      double xv[8];
      unpack8(*reinterpret_cast<const uint4 *>(xc + (size_t)i * d_model), xv);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += xv[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[wave][lane * 8 + j] = acc[j];
  __syncthreads();
  for (int ch = tid; ch < 512; ch += 256) {
    const int cc = blockIdx.x * 512 + ch;
    double tot = 0.0;
    if (cc < d_model) {
      tot = ((red[0][ch] + red[1][ch]) + red[2][ch]) + red[3][ch];
      if (!SOFTMAX) tot = tot / (double)n;
    }
    a_s[ch] = tot;                       // channels past d_model count as zero
  }
  __syncthreads();
  // First layer over this slice: hpart[b][slice][j] = sum_c a_s[c] W1[c_base + c][j].
  const int c_base = blockIdx.x * 512;
  const int n_ch = min(512, d_model - c_base);
  const int n_slices = gridDim.x;
  double *dst = hpart + ((size_t)b * n_slices + blockIdx.x) * r;
  if ((r & 7) == 0) {
    // Thread (cl, o) takes the 8 outputs 8 o .. 8 o + 7 (one 16-byte load per channel) over the channels
    // cl, cl + CL, ... in ascending order, eight loads in flight; the CL partial sums of an output are then
    // added in cl order.
    const int o_per = ((r >> 3) + gridDim.z - 1) / gridDim.z, o0 = blockIdx.z * o_per;
    const int n_oct = min(o_per, (r >> 3) - o0);                // <= 128
    if (n_oct <= 0) return;
    int o_ceil = 1;
    while (o_ceil < n_oct) o_ceil <<= 1;
    const int CL = 256 / o_ceil;                                // 2 .. 256 channel lanes
    const int o = tid % o_ceil, cl = tid / o_ceil;
    double acc8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (o < n_oct) {
      const bf16_t *wp = w1 + (size_t)c_base * r + 8 * (o0 + o);
      int cq = cl;
      for (; cq + 7 * CL < n_ch; cq += 8 * CL) {
        uint4 wv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wv[u] = *reinterpret_cast<const uint4 *>(wp + (size_t)(cq + u * CL) * r);
        __builtin_amdgcn_sched_barrier(0);                      // all eight loads go out before the first use
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          double wd[8];
          unpack8(wv[u], wd);
          const double av = a_s[cq + u * CL];
#pragma unroll
          for (int q = 0; q < 8; ++q) acc8[q] = fma(av, wd[q], acc8[q]);
        }
      }
      for (; cq < n_ch; cq += CL) {
        double wd[8];
        unpack8(*reinterpret_cast<const uint4 *>(wp + (size_t)cq * r), wd);
        const double av = a_s[cq];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc8[q] = fma(av, wd[q], acc8[q]);
      }
    }
    double *ps = &red[0][0];                                    // [CL][8 o_ceil] = 2048 doubles: red is free by now
#pragma unroll
    for (int q = 0; q < 8; ++q) ps[(cl * o_ceil + o) * 8 + q] = acc8[q];
    __syncthreads();
    for (int j = tid; j < 8 * n_oct; j += 256) {
      double tot = 0.0;
#pragma unroll 8
      for (int q = 0; q < CL; ++q) tot += ps[q * o_ceil * 8 + j];
      dst[8 * o0 + j] = tot;
    }
  } else {
    // any r: a thread per output, channels in ascending order
    for (int j = tid + 256 * blockIdx.z; j < r; j += 256 * gridDim.z) {
      const bf16_t *col = w1 + (size_t)c_base * r + j;
      double acc = 0.0;
      for (int cq = 0; cq < n_ch; ++cq) acc = fma(a_s[cq], (double)bf16_to_f32(col[(size_t)cq * r]), acc);
      dst[j] = acc;
    }
  }
}

// Pooling for calls whose blocks are few but not short.  Above, every workgroup of 512 channels, several of which share a slice's
// outputs, converts and adds all rows in fp64, a wavefront every fourth of them, waits for two rounds of W1 behind that, and then one
// thread adds up to 128 partial sums of an output.  Here a workgroup has 8 LW channels, LW lanes to a row, all rows of
// a block of 128 on their way at once and W1's with them; the rows' sums go through lanes, then wavefronts, in fixed order, the
// outputs' in eights.  Bound by latency: (the logits, the weights' exponentials,) one round of loads, five to eight barriers.  The price is
// paid by the scores kernel, which adds up four or two times as many slices.  (ff_predict alone, us, the kernel above -> this:
// softmax: 100 tokens of 4096/14336 23.2 -> 21.4, 2000 30.8 -> 29.3, 700 of 2048/8192 23.1 -> 19.6, 4096 27.0 -> 23.9, one block of 300
// 27.4 -> 19.0, one of 4096 tokens of 4096/14336 165 -> 57; the mean: 700 of 2048/8192 17.1 -> 15.4, 250 of 4096/14336 17.7 ->
// 16.6, blocks of 256 tokens of 3584/18944 28.9 -> 25.0, one block of 4096 of 4096/14336 107 -> 45.)
// SERIAL: a workgroup takes all of its block's slices and adds them up, in the order in which the scores kernels would.
// grid (slices of 8 LW channels, or 1, n_blocks)
constexpr int kPoolFineThreads = 512;
template <bool SOFTMAX, int LW, bool SERIAL>
__global__ __launch_bounds__(kPoolFineThreads) void ff_pool_fine_kernel(const bf16_t *__restrict__ x,
                                                                       const double *__restrict__ z,
                                                                       const bf16_t *__restrict__ w1,
                                                                      double *__restrict__ hpart, int T,
                                                                      int d_model, int Nb, int r) {
  constexpr int NT = kPoolFineThreads, NW = NT / 64, CH = 8 * LW, RPW = 64 / LW, STEP = NW * RPW, U = LW / 4, WU = LW / 4;
  __shared__ double red1[2 * NW];
  // Nb <= 4096 weights; rows' sums [wavefront][channel]; the outputs' [8][thread] and [group][output]
  __shared__ __align__(16) double ps[8 * NT];
  double *p_s = ps;
  __shared__ double a_s[CH];               // this workgroup's pooled channels
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b = blockIdx.y, t0 = b * Nb, n = min(T, t0 + Nb) - t0;
  auto one = [&](int slice) __attribute__((always_inline)) {
    const int c_base = slice * CH, n_ch = min(CH, d_model - c_base);
    const int sub = lane / LW, c8 = 8 * (lane % LW);
    const bf16_t *xc = x + (size_t)t0 * d_model + c_base + min(c8, n_ch - 8);   // (channels past d_model: not used)
    const int row0 = wave * RPW + sub;
    uint4 v[U];
    auto load_rows = [&](int i) __attribute__((always_inline)) {     // past the end: the last row again, not added
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const uint4 *>(xc + (size_t)min(i + u * STEP, n - 1) * d_model);
    };
    const double z0 = SOFTMAX ? z[t0 + min(tid, n - 1)] : 0.0;
    load_rows(row0);
    // thread (cl, o) takes the outputs 8 o .. 8 o + 7 over the channels cl, cl + CL, ...
    const int n_oct = r >> 3;                                     // <= 128
    const int o_bits = n_oct > 1 ? 32 - __builtin_clz(n_oct - 1) : 0, o_ceil = 1 << o_bits, CL = NT >> o_bits;
    const int o = tid & (o_ceil - 1), cl = tid >> o_bits;
    const bf16_t *wp = w1 + (size_t)c_base * r + 8 * min(o, n_oct - 1);
    uint4 wv[WU];
    auto load_w1 = [&](int cq) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < WU; ++u) wv[u] = *reinterpret_cast<const uint4 *>(wp + (size_t)min(cq + u * CL, n_ch - 1) * r);
    };
    load_w1(cl);
    __builtin_amdgcn_sched_barrier(0);
    if (SOFTMAX) {
      double m = -INFINITY;
      for (int i = tid; i < n; i += NT) m = fmax(m, i == tid ? z0 : z[t0 + i]);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
      if (lane == 0) red1[wave] = m;
      __syncthreads();
      m = red1[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) m = fmax(m, red1[w]);
      double part = 0.0;
      for (int i = tid; i < n; i += NT) {
        const double e = exp((i == tid ? z0 : z[t0 + i]) - m);
        p_s[i] = e;
        part += e;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
      if (lane == 0) red1[NW + wave] = part;
      __syncthreads();
      double s = red1[NW];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += red1[NW + w];
      for (int i = tid; i < n; i += NT) p_s[i] = p_s[i] / s;
      __syncthreads();
    }
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = row0; i < n; i += U * STEP) {
      if (i > row0) load_rows(i);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i + u * STEP < n) {
          double xv[8];
          unpack8(v[u], xv);
          const double w = SOFTMAX ? p_s[i + u * STEP] : 1.0;
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[j] = SOFTMAX ? fma(w, xv[j], acc[j]) : acc[j] + xv[j];
        }
    }
#pragma unroll
    for (int off = LW; off < 64; off <<= 1)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += __shfl_xor(acc[j], off);
    if (SOFTMAX) __syncthreads();            // (the weights have been read)
    if (sub == 0) {
#pragma unroll
      for (int j = 0; j < 8; j += 2) *reinterpret_cast<double2 *>(&ps[wave * CH + c8 + j]) = make_double2(acc[j], acc[j + 1]);
    }
    __syncthreads();
    if (tid < CH) {
      double tot = ps[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) tot += ps[w * CH + tid];
      a_s[tid] = SOFTMAX ? tot : tot / (double)n;
    }
    __syncthreads();
    double acc8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int cq = cl; cq < n_ch; cq += WU * CL) {
      if (cq > cl) {
        load_w1(cq);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int u = 0; u < WU; ++u)
        if (cq + u * CL < n_ch) {
          double wd[8];
          unpack8(wv[u], wd);
          const double av = a_s[cq + u * CL];
#pragma unroll
          for (int q = 0; q < 8; ++q) acc8[q] = fma(av, wd[q], acc8[q]);
        }
    }
    // ps[q][cl][o]; an output's CL sums are added in eights, then those
#pragma unroll
    for (int q = 0; q < 8; ++q) ps[q * NT + tid] = acc8[q];
    __syncthreads();
    double *dst = hpart + ((size_t)b * gridDim.x + blockIdx.x) * r;
    const int cols = 8 << o_bits, per = min(8, CL), G = CL / per;     // cols * G = 8 NT / per
    double sum[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {                                    // (cols = 1024: two outputs a thread)
      const int e = tid + h * NT, j = e & (cols - 1), g = e / cols;
      sum[h] = 0.0;
      if (g < G) {
        const double *src = &ps[(j >> o_bits) * NT + g * per * o_ceil + (j & (o_ceil - 1))];
        for (int q = 0; q < per; ++q) sum[h] += src[q * o_ceil];
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = tid + h * NT;
      if (e < cols * G) ps[e] = sum[h];
    }
    __syncthreads();
    for (int j = tid; j < cols; j += NT) {
      const int oo = j & (o_ceil - 1);
      if (oo < n_oct) {
        double tot = 0.0;
        for (int g = 0; g < G; ++g) tot += ps[g * cols + j];
        dst[8 * oo + (j >> o_bits)] = SERIAL && slice > 0 ? dst[8 * oo + (j >> o_bits)] + tot : tot;
      }
    }
  };
  if (SERIAL) {
    for (int slice = 0; slice * CH < d_model; ++slice) {
      one(slice);
      __syncthreads();                       // (the next slice uses the same LDS)
    }
  } else {
    one(blockIdx.x);
  }
}

// A workspace may have no room for the narrow slices' partial sums.  A call's scores have the same bits without it: the sums go where the
// scores will be, and this kernel adds a block's in slice order, as the scores kernels would; where that place is too small as well (many
// outputs, few neurons) the pooling kernel does so itself (SERIAL).  (ff_predict alone, us, with the room,
// without it, without it by 512-channel slices and so with other bits: 100 tokens of 4096/14336 16.0, 17.2, 16.2, softmax 21.4, 22.2, 22.4; 700
// of 2048/8192, softmax 18.8, 21.0, 22.6; 100 of 256/688 12.7, 15.7, 13.9.)
// hid[b][j] = sum_s part[b][s][j]; grid (ceil(r / 64), n_blocks)
__global__ __launch_bounds__(64) void ff_pool_sum_kernel(const double *__restrict__ part, double *__restrict__ hid, int n_slices, int r) {
  const int j = blockIdx.x * 64 + threadIdx.x, b = blockIdx.y;
  if (j >= r) return;
  const double *src = part + (size_t)b * n_slices * r + j;
  double acc = 0.0;
  for (int s0 = 0; s0 < n_slices; s0 += 16) {    // sixteen loads in flight (past the end: the last again, not added)
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = src[(size_t)min(s0 + u, n_slices - 1) * r];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (s0 + u < n_slices) acc += v[u];
  }
  hid[(size_t)b * r + j] = acc;
}

// ---- Eq. 13 in float64 ---------------------------------------------------------------------
// The first layer (long contraction over d_model, few outputs) is cut into slices of 512 channels that
// ride along with the pooling kernel above; the second (short contraction, d_ffn outputs) takes MLP_BB
// blocks per workgroup so that every weight is loaded once per MLP_BB blocks, each thread keeping
// MLP_LD weight loads in flight.
constexpr int MLP_BB = 4;    // blocks per workgroup: 8 halves the weight loads but leaves too few wavefronts to hide the scalar loads
constexpr int MLP_LD = 16;   // rows of W2 a thread has in flight

// ---- Eq. 13, second layer with the hidden units formed on the way in -------------------------
// scores[b][n] = sum_j h_b[j] W2[j][n], h_b[j] = ReLU(sum_s hpart[b][s][j]) (slices added in slice order).
// grid (ceil(d_ffn / 1024), ceil(n_blocks / MLP_BB)), 256 threads: a workgroup first forms the r hidden units of its
// MLP_BB blocks in LDS (every workgroup of a block group repeats these few sums rather than wait for a launch of
// their own), then every thread owns four adjacent score columns and reads the hidden units as LDS broadcasts.
__global__ __launch_bounds__(256) void ff_scores_kernel(const double *__restrict__ hpart,
                                                        const bf16_t *__restrict__ w2,
                                                        double *__restrict__ scores, int n_blocks, int r,
                                                        int n_slices, int d_ffn) {
  extern __shared__ double hid[];          // [MLP_BB][r]
  const int tid = threadIdx.x;
  const int b0 = blockIdx.y * MLP_BB;
  const int nb = min(MLP_BB, n_blocks - b0);
  for (int e = tid; e < MLP_BB * r; e += 256) {
    const int i = e / r, j = e - i * r;
    double acc = 0.0;
    if (i < nb) {
      const double *src = hpart + (size_t)(b0 + i) * n_slices * r + j;
      int s = 0;
      for (; s + 8 <= n_slices; s += 8) {      // eight loads in flight, added in slice order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(s + u) * r];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
      }
      for (; s < n_slices; ++s) acc += src[(size_t)s * r];
    }
    hid[e] = fmax(acc, 0.0);
  }
  __syncthreads();
  // A hidden unit read from LDS (the same address in every lane) costs a full-width LDS access, and a
  // load instruction costs the same whether a lane asks for 2 bytes or 8: every thread takes four
  // adjacent score columns, one 8-byte load per row of W2 (d_ffn is a multiple of 8, so a group of
  // four columns is whole and aligned), and each hidden unit read feeds 4 x MLP_BB multiply-adds.
  const int n_quads = d_ffn >> 2;
  const int quad = (int)(blockIdx.x * 256) + tid;
  const int n0 = 4 * min(quad, n_quads - 1);               // past the end: the last group again, not stored
  double acc[4][MLP_BB];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < MLP_BB; ++i) acc[q][i] = 0.0;
  const bf16_t *wp = w2 + n0;
  auto mac_row = [&](const uint2 &wv, int jrow) __attribute__((always_inline)) {
    const double wd[4] = {(double)__uint_as_float(wv.x << 16), (double)__uint_as_float(wv.x & 0xffff0000u),
                          (double)__uint_as_float(wv.y << 16), (double)__uint_as_float(wv.y & 0xffff0000u)};
    double hv[MLP_BB];
#pragma unroll
    for (int i = 0; i < MLP_BB; ++i) hv[i] = hid[i * r + jrow];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < MLP_BB; ++i) acc[q][i] = fma(hv[i], wd[q], acc[q][i]);
  };
  int j = 0;
  for (; j + MLP_LD <= r; j += MLP_LD) {   // MLP_LD rows of W2 in flight
    uint2 wv[MLP_LD];
#pragma unroll
    for (int u = 0; u < MLP_LD; ++u) wv[u] = *reinterpret_cast<const uint2 *>(wp + (size_t)(j + u) * d_ffn);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < MLP_LD; ++u) mac_row(wv[u], j + u);
  }
  for (; j < r; ++j) mac_row(*reinterpret_cast<const uint2 *>(wp + (size_t)j * d_ffn), j);
  if (quad < n_quads) {
#pragma unroll
    for (int i = 0; i < MLP_BB; ++i)
      if (i < nb) {
        double *dst = scores + (size_t)(b0 + i) * d_ffn + n0;
        *reinterpret_cast<double2 *>(dst) = make_double2(acc[0][i], acc[1][i]);
        *reinterpret_cast<double2 *>(dst + 2) = make_double2(acc[2][i], acc[3][i]);
      }
  }
}

// The same layer for calls with too few blocks to fill the chip above (a workgroup there walks all r rows of its
// 1024 columns: one block is 14 workgroups at d_ffn 14336).  Here a workgroup has 4 * QUADS columns and its THREADS / QUADS row
// groups take every so-many-th row of W2, so that few rounds of loads are all a thread waits for; the groups' sums are
// added through LDS in group order.  Bound by the latency of its two dependent rounds of loads.
template <int BB, int QUADS, int THREADS>
__global__ __launch_bounds__(THREADS) void ff_scores_split_kernel(const double *__restrict__ hpart,
                                                                  const bf16_t *__restrict__ w2,
                                                                  double *__restrict__ scores, int n_blocks, int r,
                                                                  int n_slices, int d_ffn) {
  constexpr int JG = THREADS / QUADS, LD = 8;
  extern __shared__ double hid[];          // [BB][r]
  __shared__ __align__(16) double red[JG][4 * QUADS];
  const int tid = threadIdx.x, g = tid / QUADS;
  const int b0 = blockIdx.y * BB;
  const int nb = min(BB, n_blocks - b0);
  const int n_quads = d_ffn >> 2;
  const int quad = (int)(blockIdx.x * QUADS) + tid % QUADS;
  const bf16_t *wp = w2 + 4 * min(quad, n_quads - 1);       // past the end: the last group again, not stored
  // the first rows are on their way while the hidden units are formed
  uint2 wv[LD];
#pragma unroll
  for (int u = 0; u < LD; ++u) wv[u] = *reinterpret_cast<const uint2 *>(wp + (size_t)min(g + u * JG, r - 1) * d_ffn);
  __builtin_amdgcn_sched_barrier(0);
  for (int e = tid; e < BB * r; e += THREADS) {
    const int i = e / r, j = e - i * r;
    double acc = 0.0;
    if (i < nb) {
      const double *src = hpart + (size_t)(b0 + i) * n_slices * r + j;
      int s = 0;
      for (; s + 16 <= n_slices; s += 16) {    // (finer slices) sixteen, then eight loads in flight, added in slice order
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = src[(size_t)(s + u) * r];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
      }
      for (; s + 8 <= n_slices; s += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(s + u) * r];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
      }
      for (; s < n_slices; ++s) acc += src[(size_t)s * r];
    }
    hid[e] = fmax(acc, 0.0);
  }
  __syncthreads();
  double acc[BB][4];
#pragma unroll
  for (int i = 0; i < BB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = 0.0;
  for (int j = g; j < r; j += LD * JG) {
    uint2 nx[LD];
    const int jn = j + LD * JG;
    if (jn < r) {
#pragma unroll
      for (int u = 0; u < LD; ++u) nx[u] = *reinterpret_cast<const uint2 *>(wp + (size_t)min(jn + u * JG, r - 1) * d_ffn);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < LD; ++u)
      if (j + u * JG < r) {
        const double wd[4] = {(double)__uint_as_float(wv[u].x << 16), (double)__uint_as_float(wv[u].x & 0xffff0000u),
                              (double)__uint_as_float(wv[u].y << 16), (double)__uint_as_float(wv[u].y & 0xffff0000u)};
#pragma unroll
        for (int i = 0; i < BB; ++i) {
          const double hv = hid[i * r + j + u * JG];
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[i][q] = fma(hv, wd[q], acc[i][q]);
        }
      }
    if (jn < r) {
#pragma unroll
      for (int u = 0; u < LD; ++u) wv[u] = nx[u];
    }
  }
#pragma unroll
  for (int i = 0; i < BB; ++i) {
    if (i >= nb) break;
    double *mine = &red[g][4 * (tid % QUADS)];
    *reinterpret_cast<double2 *>(mine) = make_double2(acc[i][0], acc[i][1]);
    *reinterpret_cast<double2 *>(mine + 2) = make_double2(acc[i][2], acc[i][3]);
    __syncthreads();
    const int col = (int)(blockIdx.x * QUADS) * 4 + tid;
    if (tid < 4 * QUADS && col < d_ffn) {
      double tot = 0.0;
#pragma unroll 8
      for (int q = 0; q < JG; ++q) tot += red[q][tid];
      scores[(size_t)(b0 + i) * d_ffn + col] = tot;
    }
    __syncthreads();
  }
}

// ---- Eq. 14: top-K, one workgroup of 1024 threads per block -----------------------
// Scores become 64-bit keys whose unsigned order is the score order (-0 == +0).  The
// selected set is {key > theta} plus the lowest-index (K - count) keys equal to theta,
// where theta is the key of the K-th largest score; it is written in ascending index
// order through two prefix sums.  theta is found exactly in two steps: a histogram over
// 4096 buckets of a monotone map of the score range locates the bucket holding the K-th
// largest, then the few keys of that bucket are ranked against each other.  When that
// bucket holds too many keys (heavy ties) an 8-pass MSB-first radix select on the keys
// finds theta instead.
__device__ __forceinline__ unsigned long long score_key(double s) {
  s = s + 0.0;  // -0.0 -> +0.0
  unsigned long long u = (unsigned long long)__double_as_longlong(s);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_score(unsigned long long k) {
  const unsigned long long u = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double((long long)u);
}

// inclusive prefix sum over the wavefront by data-parallel-primitive lane exchanges (six lane exchanges through LDS, each
// waiting for the one before, take several times as long): shifts inside the rows of 16 lanes, then each row's last lane
// into the rows above
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add_step(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
  v = dpp_add_step<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
  v = dpp_add_step<0x112, 0xf>(v);
  v = dpp_add_step<0x114, 0xf>(v);
  v = dpp_add_step<0x118, 0xf>(v);
  v = dpp_add_step<0x142, 0xa>(v);   // lane 15 into row 1, lane 47 into row 3
  return dpp_add_step<0x143, 0xc>(v);   // lane 31 into rows 2 and 3
}

constexpr int TOPK_FEW = 16;   // candidates that are ranked by fours of lanes

// LDS of the threshold search, shared by both top-K kernels
struct TopkShared {
  __align__(16) unsigned int bins[64 + TOPK_BUCKETS];   // in front of the histogram: what buckets -1 .. -64 count
  double cand[TOPK_CAND + TOPK_FEW];
  int wsum[16];
  unsigned int wtot[4];
  unsigned int sel_bin, sel_rem, n_cand;
  double theta;
  int ties, n_ties;
  __device__ __forceinline__ unsigned int *hist() { return bins + 64; }   // (also the 256-bin histogram of the radix path)
};

// The bucket that holds the K-th largest score, and which of its scores that is (sh.sel_bin, sh.sel_rem), from a full histogram.
__device__ __forceinline__ void topk_find_bucket(TopkShared &sh, int K) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // thread t owns buckets 4095-4t .. 4092-4t (descending); prefix over threads = scores in higher buckets
  const uint4 h4 = *reinterpret_cast<const uint4 *>(&sh.hist()[TOPK_BUCKETS - 4 - 4 * tid]);
  const int h[4] = {(int)h4.w, (int)h4.z, (int)h4.y, (int)h4.x};
  const int local = (h[0] + h[1]) + (h[2] + h[3]);
  const int inc = wave_incl_scan(local);
  if (lane == 63) sh.wsum[wave] = inc;
  __syncthreads();
  const int w = lane < 16 ? sh.wsum[lane] : 0;                // every wavefront scans the 16 totals itself
  int above = __builtin_amdgcn_readlane(wave_incl_scan(w) - w, wave) + inc - local;
  if (above < K && K <= above + local) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (above < K && K <= above + h[q]) { sh.sel_bin = (unsigned int)(TOPK_BUCKETS - 1 - (4 * tid + q)); sh.sel_rem = (unsigned int)(K - above); }
      above += h[q];
    }
  }
  __syncthreads();
}

// The need-th largest of the c candidates, how many of its equals are kept, and how many there are.  (sh.cand has NaN, which
// compares with nothing, behind the last one: topk_pad, before the barrier that everybody's candidates need anyway.)
__device__ __forceinline__ void topk_pad(TopkShared &sh, int c) {
  if (threadIdx.x < TOPK_FEW) sh.cand[c + (int)threadIdx.x] = __longlong_as_double(0x7ff8000000000000ll);
}
__device__ __forceinline__ void topk_rank(TopkShared &sh, int c, int need, double &theta, int &ties_taken, int &n_ties) {
  const int tid = threadIdx.x, lane = tid & 63;
  // rank of candidate i among the c; the need-th largest has n_gt < need <= n_gt + n_eq (all holders of its value agree)
  auto rank = [&](double mine, int &n_gt, int &n_eq) __attribute__((always_inline)) {
    n_gt = n_eq = 0;
#pragma unroll 1
    for (int j0 = 0; j0 < c; j0 += 8) {          // eight reads in flight (more than that spill)
      double o[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) o[u] = sh.cand[j0 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        n_gt += o[u] > mine;
        n_eq += o[u] == mine;
      }
    }
  };
  int n_gt, n_eq;
  if (c <= 64) {                                 // every wavefront finds it itself
    double mine;
    if (c <= TOPK_FEW) {                         // lanes 4 i .. 4 i + 3 hold candidate i against four of the others each
      mine = sh.cand[lane >> 2];
      int both = 0;
#pragma unroll
      for (int u = 0; u < TOPK_FEW / 4; ++u) {
        const double o = sh.cand[(lane & 3) * (TOPK_FEW / 4) + u];
        both += (o > mine ? 1 : 0) + (o == mine ? 65536 : 0);
      }
      both += __builtin_amdgcn_update_dpp(0, both, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
      both += __builtin_amdgcn_update_dpp(0, both, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
      n_gt = both & 0xffff;
      n_eq = both >> 16;
    } else {
      mine = lane < c ? sh.cand[lane] : sh.cand[c];
      rank(mine, n_gt, n_eq);
    }
    const int src = __ffsll((unsigned long long)__ballot(n_gt < need && need <= n_gt + n_eq)) - 1;
    const unsigned long long bits = (unsigned long long)__double_as_longlong(mine);
    const unsigned int b0 = __builtin_amdgcn_readlane((unsigned int)bits, src), b1 = __builtin_amdgcn_readlane((unsigned int)(bits >> 32), src);
    theta = __longlong_as_double((long long)(((unsigned long long)b1 << 32) | b0));
    ties_taken = need - __builtin_amdgcn_readlane(n_gt, src);
    n_ties = __builtin_amdgcn_readlane(n_eq, src);
  } else {
    if (tid < c) {
      const double mine = sh.cand[tid];
      rank(mine, n_gt, n_eq);
      if (n_gt < need && need <= n_gt + n_eq) { sh.theta = mine; sh.ties = need - n_gt; sh.n_ties = n_eq; }
    }
    __syncthreads();
    theta = sh.theta;
    ties_taken = sh.ties;
    n_ties = sh.n_ties;
  }
}

// The K-th largest score theta and the number of scores equal to theta that are kept, found exactly by the 1024 threads of a
// workgroup.  each(fn) calls fn(score, score rounded to fp32) once for every score the calling thread owns; gather(bucket_of,
// tb, append) calls append(score) for those of bucket tb.  [lo_v, hi_v]
// encloses the scores (it only shapes the bucket map); need_radix skips the buckets.  Scores are compared as numbers (-0 ==
// +0), except where the radix path had to order them: it returns true, and theta as a key.  A chain of latencies, so: a
// prefix sum whose 16 totals every wavefront scans itself, candidates that every wavefront ranks itself, no 64-bit keys.
// (Buckets of the fp32 roundings, against fp64 arithmetic on every score: one block of 14336 1.8 us less; scores whose range is
// 2^-14 of their size, which fp32 has no steps for: 12.6 us in fp64 buckets, 30.2 on the radix path.)
// On entry sh.hist is zero, sh.n_cand is 0 and a barrier has been passed.
template <class Each, class Gather>
__device__ __forceinline__ bool topk_threshold(TopkShared &sh, int K, double lo_v, double hi_v, bool need_radix,
                                               Each each, Gather gather, double &theta, unsigned long long &theta_key, int &ties_taken) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TopkMap map = topk_map(lo_v, hi_v);
  const bool fine = __builtin_amdgcn_readfirstlane(map.fine);   // the same for all threads, as everything about the range
  need_radix = need_radix || map.none;
  // bucket_of(score, rounding): the bucket map.  False: the threshold's bucket holds too many scores.
  auto by_buckets = [&](auto bucket_of) __attribute__((always_inline)) -> bool {
    each([&](double v, float s) { atomicAdd(&sh.hist()[bucket_of(v, s)], 1u); });
    __syncthreads();
    topk_find_bucket(sh, K);
    const int tb = __builtin_amdgcn_readfirstlane((int)sh.sel_bin);
    const int need = __builtin_amdgcn_readfirstlane((int)sh.sel_rem);   // rank of theta inside bucket tb (1 = largest)
    const int c = __builtin_amdgcn_readfirstlane((int)sh.hist()[tb]);
    if (c > TOPK_CAND) return false;              // uniform: every thread reads the same hist[tb]
    topk_pad(sh, c);
    gather(bucket_of, tb, [&](double v) { sh.cand[atomicAdd(&sh.n_cand, 1u)] = v; });
    __syncthreads();
    int n_ties;
    topk_rank(sh, c, need, theta, ties_taken, n_ties);
    return true;
  };
  // (the rare map's code out of the way: between the other's passes it made every call 0.5 to 1.4 us longer)
  if (!need_radix) {
    if (__builtin_expect(fine, 0)) need_radix = !by_buckets([&](double v, float) { return map.bucket64(v); });
    else need_radix = !by_buckets([&](double, float s) { return map.bucket(s); });
  }
  if (__builtin_expect(!need_radix, 1)) return false;
  // 8-pass MSB-first radix select on the keys (heavy ties, or no ordered range)
  unsigned long long prefix = 0;  // digits decided so far (high part of theta)
  unsigned int rem = (unsigned int)K;
  for (int pass = 7; pass >= 0; --pass) {
    const int shift = pass * 8;
    __syncthreads();
    if (tid < 256) sh.hist()[tid] = 0;
    __syncthreads();
    each([&](double v, float) {
      const unsigned long long k = score_key(v);
      const bool match = (pass == 7) || ((k >> (shift + 8)) == prefix);
      if (match) atomicAdd(&sh.hist()[(unsigned int)(k >> shift) & 255u], 1u);
    });
    __syncthreads();
    // suffix sums S[d] = sum_{d' >= d} hist[d'] over the 256 digits
    unsigned int hv = 0, suf = 0;
    if (tid < 256) {
      hv = sh.hist()[tid];
      suf = hv;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned int t = __shfl_down(suf, off);
        if (lane + off < 64) suf += t;
      }
      if (lane == 0) sh.wtot[wave] = suf;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = wave + 1; w < 4; ++w) suf += sh.wtot[w];
      // the digit of the K-th largest: S[d] >= rem > S[d+1]
      if (suf >= rem && suf - hv < rem) {
        sh.sel_bin = (unsigned int)tid;
        sh.sel_rem = rem - (suf - hv);
      }
    }
    __syncthreads();
    prefix = (prefix << 8) | (unsigned long long)sh.sel_bin;
    rem = sh.sel_rem;
  }
  theta_key = prefix;      // key of the K-th largest score
  ties_taken = (int)rem;   // keys equal to it that are kept
  return true;
}

// The general kernel, for d_ffn beyond what ff_topk_reg_kernel keeps in registers: every pass
// re-reads the scores (coalesced, from L2).  LDS_MODE 1: a byte per key (above / equal to / below
// theta) is kept in LDS for the two passes of the ordered compaction.  0: not even that fits.
template <int LDS_MODE>
__global__ __launch_bounds__(1024) void ff_topk_kernel(const double *__restrict__ scores,
                                                       int32_t *__restrict__ indices, int d_ffn,
                                                       int k_stride, KSpec ks) {
  extern __shared__ unsigned long long dyn[];
  __shared__ TopkShared sh;
  __shared__ double red_lo[16], red_hi[16];
  __shared__ int wsum[17], wcnt_eq[16];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  const double *sc = scores + (size_t)b * d_ffn;
  int32_t *out = indices + (size_t)b * k_stride;
  int K = ks.per_block ? ks.per_block[b] : ks.uniform;
  K = max(1, min(K, min(d_ffn, k_stride)));

  unsigned char *cls = reinterpret_cast<unsigned char *>(dyn);

  // keys, and the score range
  double lo_v = INFINITY, hi_v = -INFINITY;
  int not_finite = 0;
  for (int base = 0; base < d_ffn; base += 8 * 1024) {   // 8 loads in flight per thread
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = sc[min(base + u * 1024 + tid, d_ffn - 1)] + 0.0;   // past the end: the last score again
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      lo_v = fmin(lo_v, v[u]);
      hi_v = fmax(hi_v, v[u]);
      not_finite |= !(fabs(v[u]) <= 1.7976931348623157e308);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo_v = fmin(lo_v, __shfl_xor(lo_v, off));
    hi_v = fmax(hi_v, __shfl_xor(hi_v, off));
  }
  if (lane == 0) { red_lo[wave] = lo_v; red_hi[wave] = hi_v; }
  for (int i = tid; i < TOPK_BUCKETS; i += 1024) sh.hist()[i] = 0;
  if (tid == 0) sh.n_cand = 0;
  // fmin/fmax skip a NaN, whose key nevertheless ranks above (or below) every number: the bucket map
  // would not be monotone over the keys.  The radix path orders the keys themselves, whatever they are.
  not_finite = __syncthreads_or(not_finite);
  lo_v = red_lo[0]; hi_v = red_hi[0];
#pragma unroll
  for (int w = 1; w < 16; ++w) { lo_v = fmin(lo_v, red_lo[w]); hi_v = fmax(hi_v, red_hi[w]); }
  const bool need_radix = not_finite || !(hi_v > lo_v);   // all scores equal (or not ordered): no range to cut into buckets
  double theta_v = 0.0;
  unsigned long long theta = 0;
  int ties_taken;
  if (!topk_threshold(sh, K, lo_v, hi_v, need_radix,
                      [&](auto fn) __attribute__((always_inline)) { for (int i = tid; i < d_ffn; i += 1024) fn(sc[i], (float)sc[i]); },
                      [&](auto bucket_of, int tb, auto append) __attribute__((always_inline)) {
                        for (int i = tid; i < d_ffn; i += 1024)
                          if (bucket_of(sc[i], (float)sc[i]) == tb) append(sc[i]);
                      },
                      theta_v, theta, ties_taken))
    theta = score_key(theta_v);

  if (LDS_MODE == 1) {
    for (int i = tid; i < d_ffn; i += 1024) {
      const unsigned long long key = score_key(sc[i]);
      cls[i] = key > theta ? 2 : (key == theta ? 1 : 0);
    }
    __syncthreads();
  }
  // 2 = above theta, 1 = equal, 0 = below
  auto class_at = [&](int i) -> int {
    if (LDS_MODE == 1) return cls[i];
    const unsigned long long key = score_key(sc[i]);
    return key > theta ? 2 : (key == theta ? 1 : 0);
  };
  // Ordered compaction.  Wavefront w owns the index range [w * span, (w + 1) * span) and walks it 64
  // consecutive indices at a time, so the rank of a kept index among the kept ones is the count over
  // lower wavefronts (one scan over 16 totals) plus the count over earlier rows and lower lanes
  // (ballots).  Ties keep exactly the ties_taken lowest indices.
  const int span = ((d_ffn + 15) / 16 + 63) / 64 * 64;
  const int w0 = wave * span;
  int n_gt = 0, n_eq = 0;
  for (int j = 0; j < span; j += 64) {
    const int i = w0 + j + lane;
    const int c = i < d_ffn ? class_at(i) : 0;
    n_gt += __popcll(__ballot(c == 2));
    n_eq += __popcll(__ballot(c == 1));
  }
  if (lane == 0) { wsum[wave] = n_gt; wcnt_eq[wave] = n_eq; }
  __syncthreads();
  // every wavefront scans the 16 pairs itself: lane l < 16 holds wavefront l's totals
  const int e_l = lane < 16 ? wcnt_eq[lane] : 0;
  const int e_incl = wave_incl_scan(e_l);
  const int quota_l = max(0, min(e_l, ties_taken - (e_incl - e_l)));
  const int kept_l = (lane < 16 ? wsum[lane] : 0) + quota_l;
  const int kept_incl = wave_incl_scan(kept_l);
  int eq_seen = __shfl(e_incl - e_l, wave);          // ties at lower indices than this wavefront's range
  int pos = __shfl(kept_incl - kept_l, wave);        // kept indices below this wavefront's range
  const unsigned long long lower = (1ull << lane) - 1ull;
  for (int j = 0; j < span; j += 64) {
    const int i = w0 + j + lane;
    const int c = i < d_ffn ? class_at(i) : 0;
    const unsigned long long m_eq = __ballot(c == 1);
    const bool take = c == 2 || (c == 1 && eq_seen + (int)__popcll(m_eq & lower) < ties_taken);
    const unsigned long long m_take = __ballot(take);
    const int at = pos + __popcll(m_take & lower);
    if (take && at < K) out[at] = i;               // never past the list, whatever the scores were
    pos += __popcll(m_take);
    eq_seen += __popcll(m_eq);
  }
  for (int i = K + tid; i < k_stride; i += 1024) out[i] = -1;
}

// min over each row of 16 lanes, by data-parallel-primitive lane exchanges
template <int CTRL>
__device__ __forceinline__ unsigned int dpp_min_step(unsigned int v) {
  return min(v, (unsigned int)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ unsigned int row_min_u32(unsigned int v) {
  v = dpp_min_step<0xB1>(v);    // quad_perm [1,0,3,2]
  v = dpp_min_step<0x4E>(v);    // quad_perm [2,3,0,1]
  v = dpp_min_step<0x141>(v);   // row_half_mirror
  return dpp_min_step<0x140>(v);   // row_mirror
}

// The same selection for d_ffn <= 1024 * ROWS with every score in a register.  Wavefront w owns the consecutive indices
// [64 w ROWS, 64 (w + 1) ROWS), read with all loads in flight, no pass reads them back, and the rank of a kept index among the
// kept ones is a scan over 16 per-wavefront totals plus counts over earlier rows and lower lanes (ballots).
// What binds it is the issue of vector instructions: with 16 wavefronts on four SIMDs one instruction per row of 64 scores costs
// 16 cycles.  So: the range from the fp32 roundings, minimum and maximum of two rows an instruction; the bucket of a score is
// kept beside it, for two compares per row in each later pass; an index past the end has a bucket below all others, where no
// pass looks (slots in front of the histogram count them), so no pass asks whether an index is valid; scores are looked at
// again only in rows that hold a candidate of the threshold's bucket.  (Kernel alone, back to back, us, with keys, valid
// indices and buckets formed again in every pass -> this: one block of 688 5.8 -> 3.4, 4096 6.7 -> 4.0, 8192 7.8 -> 5.1, 14336
// 11.6 -> 6.9, 18944 16.8 -> 9.0; 64 blocks of 14336 11.9 -> 7.7.  Of one block of 14336 a third is the scores' way to the CU.)
// Whatever the roundings cannot order (a range too narrow or too wide for fp32, NaN or infinite scores, a bucket with too many
// ties) goes through topk_threshold, as in the kernel above.
template <int ROWS>
__global__ __launch_bounds__(1024) void ff_topk_reg_kernel(const double *__restrict__ scores,
                                                           int32_t *__restrict__ indices, int d_ffn,
                                                           int k_stride, KSpec ks) {
  __shared__ TopkShared sh;
  __shared__ unsigned int red[32];      // every wavefront's ends of the score range
  __shared__ int2 cnt[16];              // scores above theta and equal to it, per wavefront

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x;
  const double *sc = scores + (size_t)b * d_ffn;
  int32_t *out = indices + (size_t)b * k_stride;
  int i0 = wave * ROWS * 64 + lane;         // this thread's index in row 0

  // An index past the end repeats the last score, which leaves the range as it is.
  double v[ROWS];
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    v[u] = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(sc) + (uint32_t)min(i0 + u * 64, d_ffn - 1) * 8u);
    if (u % 8 == 7) __builtin_amdgcn_sched_barrier(0);
  }
  int K = ks.per_block ? ks.per_block[b] : ks.uniform;
  K = max(1, min(K, min(d_ffn, k_stride)));
  static_assert(TOPK_BUCKETS == 4 * 1024, "a thread clears and scans four buckets");
  *reinterpret_cast<uint4 *>(&sh.hist()[4 * tid]) = make_uint4(0, 0, 0, 0);
  if (tid == 0) sh.n_cand = 0;
  int bk[ROWS];                          // roundings, then buckets
  float lo = (float)v[0], hi = lo;
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const float r = (float)v[u];
    bk[u] = __float_as_int(r);
    if (u % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    lo = __builtin_elementwise_minimum(lo, r);     // (these keep a NaN)
    hi = __builtin_elementwise_maximum(hi, r);
  }
  asm("" : "+v"(i0));                   // (the rows' indices are formed again where they are used: no registers for them in between)
  auto order = [](float x) __attribute__((always_inline)) -> unsigned int {     // unsigned order = score order, NaN at either end
    const unsigned int u = __float_as_uint(x);
    return u ^ ((unsigned int)((int)u >> 31) | 0x80000000u);
  };
  auto value = [](unsigned int u) __attribute__((always_inline)) -> float { return __uint_as_float((u >> 31) ? (u & 0x7fffffffu) : ~u); };
  // both ends as minima, of the order and of its complement: the halves of the wavefront take one each
  auto ends = [&](unsigned int of_lo, unsigned int of_hi, unsigned int &l, unsigned int &h) __attribute__((always_inline)) {
    const auto sw = __builtin_amdgcn_permlane32_swap(of_lo, ~of_hi, false, false);
    unsigned int m = min(sw[0], sw[1]);
    m = row_min_u32(m);
    l = min(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16));
    h = min(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48));
    if (lane == 0) { red[wave] = l; red[16 + wave] = h; }
    __syncthreads();
    m = row_min_u32(red[lane & 31]);
    l = __builtin_amdgcn_readlane(m, 0);
    h = ~__builtin_amdgcn_readlane(m, 16);
  };
  unsigned int lo_w, hi_w;
  ends(order(lo), order(hi), lo_w, hi_w);
  lo = value(lo_w);
  hi = value(hi_w);
  auto below = [&](unsigned long long m, int from) __attribute__((always_inline)) -> int {   // from + set bits in lower lanes
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, (unsigned int)from));
  };
  // kept scores and ties of lower wavefronts, from every wavefront's totals (every wavefront scans the 16 pairs itself)
  auto before = [&](int n_gt, int n_eq, int ties_taken, int &pos, int &eq_seen) __attribute__((always_inline)) {
    if (lane == 0) cnt[wave] = make_int2(n_gt, n_eq);
    __syncthreads();
    const int2 mine = lane < 16 ? cnt[lane] : make_int2(0, 0);
    const int e_before = wave_incl_scan(mine.y) - mine.y;
    const int kept = mine.x + max(0, min(mine.y, ties_taken - e_before));
    eq_seen = __builtin_amdgcn_readlane(e_before, wave);
    pos = __builtin_amdgcn_readlane(wave_incl_scan(kept) - kept, wave);
  };

  bool done = false, found = false;
  double theta = 0.0;
  int ties_taken = 0, pos, eq_seen;
  if (__builtin_expect(topk_fp32_range(lo, hi), 1)) {
    const float scale = topk_fp32_scale(lo, hi);
#pragma unroll
    for (int u = 0; u < ROWS; ++u) bk[u] = TopkMap::bucket(__int_as_float(bk[u]), lo, scale);
    if ((wave + 1) * ROWS * 64 > d_ffn) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) bk[u] = i0 + u * 64 < d_ffn ? bk[u] : ~lane;
    }
    unsigned int *hist = sh.hist();
#pragma unroll
    for (int u = 0; u < ROWS; ++u) atomicAdd(hist + bk[u], 1u);
    __syncthreads();
    topk_find_bucket(sh, K);
    int tb = __builtin_amdgcn_readfirstlane((int)sh.sel_bin);
    const int need = __builtin_amdgcn_readfirstlane((int)sh.sel_rem);   // rank of theta inside bucket tb (1 = largest)
    const int c = __builtin_amdgcn_readfirstlane((int)sh.hist()[tb]);
    if (c <= TOPK_CAND) {                       // (uniform: every thread reads the same)
      topk_pad(sh, c);
      unsigned int open_rows = 0;               // rows that hold a candidate
      int n_gt = 0;
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        n_gt += __popcll(__ballot(bk[u] > tb));
        if (__ballot(bk[u] == tb)) {
          open_rows |= 1u << u;
          if (bk[u] == tb) sh.cand[atomicAdd(&sh.n_cand, 1u)] = v[u];
        }
      }
      __syncthreads();
      // (the compiler would keep these passes' conditions for the next ones, in more scalar registers than there are)
      open_rows = __builtin_amdgcn_readfirstlane(open_rows);
      asm volatile("" : "+s"(tb));
      int n_ties;
      topk_rank(sh, c, need, theta, ties_taken, n_ties);
      if (__builtin_expect(ties_taken == n_ties, 1)) {       // all that equal theta are kept (else: by their order, below)
        // candidates that are kept move to the bucket above
        if (open_rows) {
#pragma unroll
          for (int u = 0; u < ROWS; ++u)
            if ((open_rows >> u) & 1u) {
              const bool kept = bk[u] == tb && v[u] >= theta;
              n_gt += __popcll(__ballot(kept));
              bk[u] += kept;
            }
        }
        before(n_gt, 0, 0, pos, eq_seen);
        asm volatile("" : "+s"(tb));
        // (K of them together, so nothing is written past the list)
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          const unsigned long long m = __ballot(bk[u] > tb);
          const uint32_t at = (uint32_t)below(m, pos) * 4u;
          if (bk[u] > tb) *reinterpret_cast<int32_t *>(reinterpret_cast<char *>(out) + at) = i0 + u * 64;
          pos += __popcll(m);
        }
        done = true;
      }
      found = true;
    }
    if (!done) __syncthreads();                 // (the histogram has been read)
  }
  if (__builtin_expect(!done, 0)) {
    // (what the compiler cannot follow: it would keep conditions, roundings and keys of earlier passes, in scratch memory)
    auto valid = [&](int u) __attribute__((always_inline)) -> bool {
      int i = i0;
      asm volatile("" : "+v"(i));
      return i + u * 64 < d_ffn;
    };
    auto score = [&](int u) __attribute__((always_inline)) -> double {
      double x = v[u];
      asm volatile("" : "+v"(x));
      return x;
    };
    unsigned long long theta_key = 0;
    if (!found) {
      // as in the general kernel: buckets of the fp64 scores where they have an ordered range, else keys
      unsigned int lo64 = 0xffffffffu, hi64 = 0u;      // the high words of the smallest and the largest key enclose the scores
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const unsigned int hw = (unsigned int)((unsigned long long)__double_as_longlong(v[u]) >> 32);
        const unsigned int key = hw ^ ((unsigned int)((int)hw >> 31) | 0x80000000u);
        lo64 = min(lo64, key);
        hi64 = max(hi64, key);
      }
      __syncthreads();                                 // (red has been read)
      ends(lo64, hi64, lo64, hi64);
      const double lo_v = key_score((unsigned long long)lo64 << 32), hi_v = key_score(((unsigned long long)hi64 << 32) | 0xffffffffull);
      const bool need_radix = topk_fp32_range(lo, hi) || !(hi_v > lo_v);   // too many ties for the buckets, or no ordered range
      if (!topk_threshold(sh, K, lo_v, hi_v, need_radix,
                          [&](auto fn) __attribute__((always_inline)) {
#pragma unroll
                            for (int u = 0; u < ROWS; ++u) {
                              const double x = score(u);
                              if (valid(u)) fn(x, (float)x);
                            }
                          },
                          [&](auto bucket_of, int tb, auto append) __attribute__((always_inline)) {
#pragma unroll
                            for (int u = 0; u < ROWS; ++u) {
                              const double x = score(u);
                              if (valid(u) && bucket_of(x, (float)x) == tb) append(x);
                            }
                          },
                          theta, theta_key, ties_taken))
        found = true;
    }
    if (found) theta_key = score_key(theta);
    int n_gt = 0, n_eq = 0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const unsigned long long key = score_key(score(u));
      n_gt += __popcll(__ballot(valid(u) && key > theta_key));
      n_eq += __popcll(__ballot(valid(u) && key == theta_key));
    }
    before(n_gt, n_eq, ties_taken, pos, eq_seen);
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const unsigned long long key = score_key(score(u));
      const bool eq = valid(u) && key == theta_key;
      const unsigned long long m_eq = __ballot(eq);
      const bool take = (valid(u) && key > theta_key) || (eq && below(m_eq, eq_seen) < ties_taken);
      const unsigned long long m = __ballot(take);
      const int at = below(m, pos);
      if (take && at < K) out[at] = i0 + u * 64;     // never past the list, whatever the scores were
      eq_seen += __popcll(m_eq);
      pos += __popcll(m);
    }
  }
  for (int i = K + tid; i < k_stride; i += 1024) out[i] = -1;
}

}  // namespace

static int g_topk_lds_raised = 0;

// the top-K kernel with 2 * half rows, 1 <= half <= 16: as few as hold the block (a row that none of its indices is in still
// costs its share of every pass)
typedef void (*topk_reg_t)(const double *, int32_t *, int, int, KSpec);
template <int... H>
static topk_reg_t topk_reg_pick(int half, std::integer_sequence<int, H...>) {
  constexpr topk_reg_t fn[] = {ff_topk_reg_kernel<2 * H + 2>...};
  return fn[half - 1];
}
static topk_reg_t topk_reg_kernel(int half) { return topk_reg_pick(half, std::make_integer_sequence<int, 16>{}); }

// Lanes to a row of ff_pool_fine_kernel (0: it does not apply).  128 channels to a workgroup as long as a workgroup of the scores kernel
// then has at most 4096 partial sums to add, else 256 (1200 tokens of 3584/18944 in blocks of 256 favour 128, 29.6 against 30.5 us,
// 2000 of 4096/14336 256, 21.4 against 23.2).  Short blocks' rows are few loads anyhow, and the scores kernel's further slices cost 0.5 to
// 1 us (softmax: 160 tokens of 3584/18944 in blocks of 32 27.1 -> 27.6, 256 of 256/688 in blocks of 64 16.5 -> 16.2; the mean: 64 tokens of
// 4096/14336 16.7 -> 17.1, 100 16.7 -> 16.4).
static int pool_fine_lanes(int n_tokens, int block, int d_model, int r, bool softmax) {
  const int64_t n_blocks = ((int64_t)n_tokens + block - 1) / block, dm = d_model;   // (where room is asked for nobody has looked at r)
  if (std::min(n_tokens, block) < (softmax ? 64 : 96) || (dm + 511) / 512 * n_blocks > 128 || r <= 0 || r > 1024 || r % 8 != 0) return 0;
  return (n_blocks <= 2 ? 1 : MLP_BB) * r * ((dm + 127) / 128) <= 4096 ? 16 : 32;
}
size_t ff_pool_fine_bytes(int n_tokens, int block, int d_model, int r, bool softmax) {
  const size_t ch = 8 * (size_t)pool_fine_lanes(n_tokens, block, d_model, r, softmax);
  return ch == 0 ? 0 : ((size_t)n_tokens + block - 1) / block * (((size_t)d_model + ch - 1) / ch) * r * sizeof(double);
}

static decltype(&ff_pool_fine_kernel<true, 16, true>) pool_fine_kernel(bool softmax, int lanes, bool serial) {
  if (lanes == 16)
    return softmax ? (serial ? ff_pool_fine_kernel<true, 16, true> : ff_pool_fine_kernel<true, 16, false>)
                   : (serial ? ff_pool_fine_kernel<false, 16, true> : ff_pool_fine_kernel<false, 16, false>);
  return softmax ? (serial ? ff_pool_fine_kernel<true, 32, true> : ff_pool_fine_kernel<true, 32, false>)
                 : (serial ? ff_pool_fine_kernel<false, 32, true> : ff_pool_fine_kernel<false, 32, false>);
}

hipError_t ff_launch_predict(const PredictParams &p, int lds_limit, hipStream_t s, Profiler *prof) {
  int n_slices = (p.d_model + 511) / 512;
  double *hpart = p.hpart;
  // Few blocks: the first layer's outputs are shared out over up to 8 workgroups per slice (each pools the slice again),
  // at least 32 outputs each, until there is one for every CU (d_model 4096, r 128: one token 7.5 -> 5.3 us, a block of
  // 100 9.0 -> 7.5, 16 blocks 12.8 -> 11.6).  How many share them decides which channels are summed together first, so the
  // last bits of fp64 scores depend on the number of blocks, here and below.
  int oz = 256 / (n_slices * p.n_blocks);
  oz = std::max(1, std::min({oz, 8, p.r / 32}));
  prof_begin(prof, FF_STAGE_POOL, s);
  const size_t fine_bytes = ff_pool_fine_bytes(p.T, p.block, p.d_model, p.r, p.q_pred != nullptr);
  if (p.q_pred) hipLaunchKernelGGL(ff_logits_kernel, dim3((p.T + 3) / 4), dim3(256), 0, s, p.x, p.q_pred, p.z, p.T, p.d_model);
  if (fine_bytes > 0) {
    const int lw = pool_fine_lanes(p.T, p.block, p.d_model, p.r, p.q_pred != nullptr);
    const double *z = p.q_pred ? p.z : nullptr;
    n_slices = (p.d_model + 8 * lw - 1) / (8 * lw);
    const bool room = p.hpart_fine_bytes >= fine_bytes, at_scores = !room && (int64_t)n_slices * p.r <= p.d_ffn;
    double *part = room ? p.hpart_fine : at_scores ? p.scores : p.hpart;
    const auto fn = pool_fine_kernel(p.q_pred != nullptr, lw, !room && !at_scores);
    hipLaunchKernelGGL(fn, dim3(room || at_scores ? n_slices : 1, p.n_blocks), dim3(kPoolFineThreads), 0, s,
                       p.x, z, p.w1, part, p.T, p.d_model, p.block, p.r);
    if (at_scores) hipLaunchKernelGGL(ff_pool_sum_kernel, dim3((p.r + 63) / 64, p.n_blocks), dim3(64), 0, s, part, p.hpart, n_slices, p.r);
    if (room) hpart = part;
    else n_slices = 1;
  } else if (p.q_pred) {
    hipLaunchKernelGGL(ff_pool_kernel<true>, dim3(n_slices, p.n_blocks, oz), dim3(256),
                       (size_t)p.block * sizeof(double), s, p.x, p.z, p.w1, hpart, p.T, p.d_model,
                       p.block, p.r);
  } else {
    hipLaunchKernelGGL(ff_pool_kernel<false>, dim3(n_slices, p.n_blocks, oz), dim3(256),
                       0, s, p.x, (const double *)nullptr, p.w1, hpart, p.T, p.d_model, p.block, p.r);
  }
  prof_end(prof, s);
  prof_begin(prof, FF_STAGE_MLP, s);
  const int n_groups = (p.n_blocks + MLP_BB - 1) / MLP_BB;
  // One or two blocks: 128 columns per workgroup and 32 row groups, else 256 columns and 8 row groups with every weight
  // shared by four blocks, as long as 1024 columns per workgroup would leave half of the CUs without one.  (d_ffn 14336,
  // r 128: one block 14.1 -> 4.5 us, 16 blocks 18.2 -> 8.2; d_ffn 8192, r 64: 6 blocks 9.1 -> 5.4, 32 blocks 9.2 -> 5.6.
  // 64 blocks at d_ffn 14336 take 21.4 us as they are, 23.0 this way: every workgroup forms the hidden units again.)
  if (p.n_blocks <= 2) {
    hipLaunchKernelGGL((ff_scores_split_kernel<1, 32, 1024>), dim3((p.d_ffn + 127) / 128, p.n_blocks), dim3(1024),
                       (size_t)p.r * sizeof(double), s, hpart, p.w2, p.scores, p.n_blocks, p.r, n_slices, p.d_ffn);
  } else if (n_groups * ((p.d_ffn + 1023) / 1024) <= 128) {
    hipLaunchKernelGGL((ff_scores_split_kernel<MLP_BB, 64, 512>), dim3((p.d_ffn + 255) / 256, n_groups), dim3(512),
                       (size_t)MLP_BB * p.r * sizeof(double), s, hpart, p.w2, p.scores, p.n_blocks, p.r, n_slices, p.d_ffn);
  } else {
    hipLaunchKernelGGL(ff_scores_kernel, dim3((p.d_ffn + 1023) / 1024, n_groups), dim3(256),
                       (size_t)MLP_BB * p.r * sizeof(double), s, hpart, p.w2, p.scores, p.n_blocks, p.r,
                       n_slices, p.d_ffn);
  }
  prof_end(prof, s);
  prof_begin(prof, FF_STAGE_TOPK, s);
  if (p.d_ffn <= 32 * 1024) {
    hipLaunchKernelGGL(topk_reg_kernel((p.d_ffn + 2047) / 2048), dim3(p.n_blocks), dim3(1024), 0, s, p.scores, p.indices, p.d_ffn, p.k_stride, p.k);
  } else {
    // the kernel's own static arrays (bucket histogram, candidates, scan scratch) take under 26 KiB
    const size_t dyn_limit = (size_t)lds_limit - 26 * 1024;
    if (!g_topk_lds_raised) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(ff_topk_kernel<1>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_limit);
      if (e != hipSuccess) return e;
      g_topk_lds_raised = 1;
    }
    const size_t cls_bytes = ((size_t)p.d_ffn + 15) / 16 * 16;
    if (cls_bytes <= dyn_limit) {
      hipLaunchKernelGGL(ff_topk_kernel<1>, dim3(p.n_blocks), dim3(1024), cls_bytes, s, p.scores,
                         p.indices, p.d_ffn, p.k_stride, p.k);
    } else {
      hipLaunchKernelGGL(ff_topk_kernel<0>, dim3(p.n_blocks), dim3(1024), 0, s, p.scores,
                         p.indices, p.d_ffn, p.k_stride, p.k);
    }
  }
  prof_end(prof, s);
  return hipGetLastError();
}
