// The pool and the queries for few tokens (bf16, head dims 64 and 96, N <= kFewRows): decode
// steps, where the work is reading each weight once and the rest is latency.
//
// The GEMM path prepares for many tokens: a pass over the weights to fold the gains in, a
// table of angles, the rows' norms, then tiles of 64 tokens or more whose K loop is a chain of
// short loads (one sequence, one layer of 6 heads of 96, D = 512: 17 us in four launches; at
// L = 24, D = 1024, 16 tokens 34 us per projection, 13-20 of them the folding). Here one
// workgroup makes one head of one projection in one launch: four waves take a quarter of K
// each, straight from memory into MFMA operands with a batch of eight k16 steps in flight,
// and the norm of the tokens' rows, the gain, the angles, the head norm and the store are in
// the same kernel. Weights are used as given; the gain multiplies the activations (one
// rounding to bf16 per product, as folding it into the weights has).
#include <algorithm>
#include <cmath>

#include "wm_device.hpp"
#include "wm_internal.hpp"

namespace wm {

constexpr int kFewWaves = 4, kFewBatch = 8;
static_assert(kFewRows == 32, "one tile of tokens");

// A wave's share of a product of 32 NDT weight rows with 32 tokens. Its rows' next 128
// columns (weights, then tokens; 256-byte pieces, four rows per instruction) are copied into
// an LDS area of its own, all of them in flight at once, and read back as MFMA operands;
// loaded into operand registers directly, each instruction would touch 32 rows, and the
// cache's one row per cycle made that 9 us for one head at D = 512. 16-byte chunk c of row
// t sits at chunk c ^ (t mod 16), so 16 rows' reads of one chunk hit 16 bank groups.
template <int NDT> struct FewTile {
  static constexpr int ROWS = 32 * NDT + 32, BYTES = ROWS * 256, NI = ROWS / 4;
  static_assert(NI <= 63, "one vmcnt covers a batch");
};

// acc[dt] += W (x g)^T over the columns [k0, k1) (k0 a multiple of 16), and the sum of
// squares of the tokens over them. Lane (h, r) of the operands: weight row 32 dt + r, token
// r. wv, xv: views whose row t starts at byte t wrow / xoff(t); gain: the D gains; sq: this
// lane's token's sums of squares of every eight columns, or null (then taken from x).
template <int NDT, class XOff>
__device__ __forceinline__ float few_product(__amdgpu_buffer_rsrc_t wv, uint32_t wrow, int wlast,
                                             __amdgpu_buffer_rsrc_t xv, XOff xoff,
                                             const bf16* __restrict__ gain,
                                             const float* __restrict__ sq, int k0, int k1,
                                             f32x16 (&acc)[NDT], char* area, int lane) {
  using F = FewTile<NDT>;
  const int h = lane >> 5, r = lane & 31;
  // eight sums of D / 64 terms at most: one of all of them is off by 4e-7 at D = 512 and more
  // past it, these by 1e-7, as a row's norm in a kernel of its own
  float ss[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, sg = 0.f;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)area);
  for (int kb = k0; kb < k1; kb += 16 * kFewBatch) {
#pragma unroll
    for (int i = 0; i < F::NI; ++i) {
      const int row = 4 * i + (lane >> 4), c = (lane & 15) ^ (row & 15);
      const uint32_t base = 4 * i < 32 * NDT ? (uint32_t)min(row, wlast) * wrow
                                             : xoff(row - 32 * NDT);
      const uint32_t off = kb + 8 * c < k1 ? base + 2u * (uint32_t)(kb + 8 * c) : kOffOob;
      lds_dma16(lds + 1024 * i, off, 4 * i < 32 * NDT ? wv : xv);
    }
    bf16x8 gf[kFewBatch];
#pragma unroll
    for (int i = 0; i < kFewBatch; ++i)  // past the range: read again, times zeros
      gf[i] = ld_frag<bf16>(gain + min(kb + 16 * i, k1 - 16) + 8 * h);
    if (sq) {
      f32x2 v[kFewBatch / 2];  // half h: its half of the batch's k16 steps, two sums each
#pragma unroll
      for (int i = 0; i < kFewBatch / 2; ++i)
        v[i] = *(const f32x2*)(sq + min(kb + 16 * (kFewBatch / 2 * h + i), k1 - 16) / 8);
#pragma unroll
      for (int i = 0; i < kFewBatch / 2; ++i)
        sg += kb + 16 * (kFewBatch / 2 * h + i) < k1 ? v[i][0] + v[i][1] : 0.f;
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
    for (int i = 0; i < kFewBatch; ++i) {
      const int c = 16 * ((2 * i + h) ^ (r & 15));
      const bf16x8 xf = *(const bf16x8*)(area + (32 * NDT + r) * 256 + c);
      bf16x8 xg;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float v = (float)xf[t];
        ss[t] = fmaf(v, v, ss[t]);
        xg[t] = (bf16)(v * (float)gf[i][t]);
      }
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
        acc[dt] = mma32(acc[dt], *(const bf16x8*)(area + (32 * dt + r) * 256 + c), xg);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the area takes the next batch
  }
  const float sx = ((ss[0] + ss[1]) + (ss[2] + ss[3])) + ((ss[4] + ss[5]) + (ss[6] + ss[7]));
  return halves_sum(sq ? sg : sx);
}

struct FewProj {
  const bf16* X;         // token n of group g at X + g xg + n xn
  long xg, xn;
  const bf16 *W0, *W1;   // groups [0, split) from W0, the rest from W1, [H DH][D] each
  int split;
  const bf16* gain;      // [groups][D] the gain of the tokens' RMSNorm
  const float* sq;       // [groups][M][D / 8] the tokens' sums of squares, or null
  const bf16* hgain;     // [split][DH] the head norm's gain (groups below split)
  int M, D, H, T_new, B, gs, gq;
  const int32_t* ctx_len;
  int ctx_hi;
  float eps;
  double freq[kMaxHeadDim / 2];  // theta^(-2m/d)
  // queries: out0[g][b][head][i][DH]; keys, values: the caches [split][B][H][S_cap][DH]
  bf16 *out0, *out1;
  int S_cap;
};

// One head of one projection for the call's tokens: grid (heads, groups). KV: keys
// (norm, rotation) and values (neither) into the caches; else queries.
template <int DH, bool KV>
__global__ __launch_bounds__(64 * kFewWaves) void few_proj_kernel(FewProj a) {
  constexpr int NDT = DH / 32, LD = DH + 4, PP = DH / 16;
  using F = FewTile<NDT>;
  static_assert(32 * LD * 4 <= F::BYTES, "a wave's result fits its copy area");
  __shared__ __align__(16) char area[kFewWaves][F::BYTES];
  __shared__ float ssq[kFewWaves][32];
  __shared__ double freq[DH / 2];
  const int head = blockIdx.x, g = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool rotate = !KV || g < a.split;
  // the epilogue's thread: token n, rotation pairs m0 .. m0 + PP - 1 (m and m + DH / 2)
  const int n = tid >> 3, m0 = (tid & 7) * PP;
  const int nn = min(n, a.M - 1), b = nn / a.T_new, ti = nn - b * a.T_new;
  const long pos = (long)ctx_at(a.ctx_len, b, a.ctx_hi) + a.gq + (long)a.gs * ti;
  bf16 hg[2][PP];
  if (rotate) {
#pragma unroll
    for (int i = 0; i < PP; i += 2) {
      const bf16* hp = a.hgain + (long)g * DH + m0 + i;
      const bf16x2 p0 = *(const bf16x2*)hp, p1 = *(const bf16x2*)(hp + DH / 2);
      hg[0][i] = p0[0], hg[0][i + 1] = p0[1], hg[1][i] = p1[0], hg[1][i + 1] = p1[1];
    }
  }
  const long wper = (long)a.H * DH * a.D;
  const bf16* W = (g < a.split ? a.W0 + g * wper : a.W1 + (g - a.split) * wper) +
                  (long)head * DH * a.D;
  const auto wv = make_view(W, (uint32_t)(DH * a.D * 2));
  const auto xv = make_view(a.X + g * a.xg, (uint32_t)(((a.M - 1) * a.xn + a.D) * 2));
  if (tid < DH / 2) freq[tid] = a.freq[tid];
  const int per = 16 * ((a.D / 16 + kFewWaves - 1) / kFewWaves);
  f32x16 acc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) acc[dt] = zero16();
  const float ss = few_product<NDT>(
      wv, (uint32_t)a.D * 2, DH - 1, xv,
      [&](int x) { return (uint32_t)(min(x, a.M - 1) * a.xn * 2); },
      a.gain + (long)g * a.D,
      KV && a.sq ? a.sq + ((long)g * a.M + min(r, a.M - 1)) * (a.D / 8) : nullptr, w * per,
      min(a.D, (w + 1) * per), acc, area[w], lane);
  float* red = (float*)area[w];  // [32 tokens][LD]
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = acc[dt][4 * q4 + i];
      *(f32x4*)(red + r * LD + 32 * dt + 8 * q4 + 4 * h) = v;
    }
  if (h == 0) ssq[w][r] = ss;
  __syncthreads();
  float v1[PP], v2[PP], sq = 0.f;
#pragma unroll
  for (int ww = 0; ww < kFewWaves; ++ww) sq += ssq[ww][n];
  const float rinv = 1.0f / sqrtf(sq / (float)a.D + a.eps);
  float hs = 0.f;
#pragma unroll
  for (int i = 0; i < PP; ++i) {
    v1[i] = v2[i] = 0.f;
#pragma unroll
    for (int ww = 0; ww < kFewWaves; ++ww) {
      const float* rw = (const float*)area[ww] + n * LD + m0 + i;
      v1[i] += rw[0];
      v2[i] += rw[DH / 2];
    }
    v1[i] *= rinv;
    v2[i] *= rinv;
    hs += v1[i] * v1[i] + v2[i] * v2[i];
  }
  if (rotate) {
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) hs += __shfl_xor(hs, o, 64);
    const float rs = 1.0f / sqrtf(hs / (float)DH + a.eps);
    constexpr double kTwoPi = 6.283185307179586476925286766559;
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      const float x1 = v1[i] * (rs * (float)hg[0][i]);
      const float x2 = v2[i] * (rs * (float)hg[1][i]);
      // the angle in double, reduced modulo 2 pi (as rope_table_kernel)
      const double ang = (double)pos * freq[m0 + i];
      float sn, cs;
      sincosf((float)(ang - kTwoPi * rint(ang / kTwoPi)), &sn, &cs);
      v1[i] = x1 * cs - x2 * sn;
      v2[i] = x2 * cs + x1 * sn;
    }
  }
  if (n >= a.M) return;
  bf16* dst;
  if constexpr (KV) {
    if (pos < 0 || pos >= a.S_cap) return;
    const int j = g < a.split ? g : g - a.split;
    dst = (g < a.split ? a.out0 : a.out1) +
          ((((long)j * a.B + b) * a.H + head) * a.S_cap + pos) * DH;
  } else {
    dst = a.out0 + ((((long)g * a.B + b) * a.H + head) * a.T_new + ti) * DH;
  }
#pragma unroll
  for (int i = 0; i < PP; i += 2) {
    *(bf16x2*)(dst + m0 + i) = bf16x2{(bf16)v1[i], (bf16)v1[i + 1]};
    *(bf16x2*)(dst + m0 + i + DH / 2) = bf16x2{(bf16)v2[i], (bf16)v2[i + 1]};
  }
}

bool few_tokens(const Shape& sh) {
  return sh.N() > 0 && sh.N() <= kFewRows && (sh.d == 64 || sh.d == 96);
}

template <bool KV> static void few_proj(FewProj& a, const Shape& sh, int groups, hipStream_t s) {
  const int d = sh.d;
  // the rotation's frequencies of this theta and head dim, kept by the calling thread (48
  // powers in double cost the host as much as a launch, and the kernel 2 us before its store)
  thread_local float theta = 0.f;
  thread_local int dim = 0;
  thread_local double freq[kMaxHeadDim / 2];
  if (theta != sh.rope_theta || dim != d) {
    for (int m = 0; m < d / 2; ++m) freq[m] = std::pow((double)sh.rope_theta, -2.0 * m / d);
    theta = sh.rope_theta;
    dim = d;
  }
  std::copy(freq, freq + d / 2, a.freq);
  const dim3 grid(a.H, groups), blk(64 * kFewWaves);
  if (d == 96) hipLaunchKernelGGL((few_proj_kernel<96, KV>), grid, blk, 0, s, a);
  else hipLaunchKernelGGL((few_proj_kernel<64, KV>), grid, blk, 0, s, a);
}

void launch_few_queries(const Shape& sh, const bf16* H, const bf16* g_in, const bf16* Wq,
                        const bf16* g_qnorm, const int32_t* ctx_len, bf16* Q, int l0, int nl,
                        hipStream_t s) {
  const long D = sh.D, per = (long)sh.Hq * sh.d * D;
  FewProj a{H + l0 * D, D, (long)sh.L * D, Wq + l0 * per, nullptr, nl, g_in + l0 * D,
            nullptr, g_qnorm + (long)l0 * sh.d, sh.N(), sh.D, sh.Hq, sh.T_new, sh.B, sh.gs, sh.gq,
            ctx_len, sh.ctx_hi, sh.eps, {}, Q, nullptr, 0};
  few_proj<false>(a, sh, nl, s);
}

// ------------------------------------------------------------------- router
// part[m][n][br kL + o] = (W_alpha[br][o][m] . (g_pre x)) / RMS(x) for stacked source m (layer
// s0 + p m): grid (row tiles of 32 per branch, sources, branches).
__global__ __launch_bounds__(64 * kFewWaves) void few_router_kernel(
    const bf16* H, const bf16* W, const bf16* g_pre, int M, int L, int Lp, int D, int kL, int s0,
    int p, int nofb, float eps, float* part) {
  using F = FewTile<1>;
  constexpr int LD = 36;
  __shared__ __align__(16) char area[kFewWaves][F::BYTES];
  __shared__ float ssq[kFewWaves][32];
  const int o0 = 32 * blockIdx.x, m = blockIdx.y, br = blockIdx.z, lay = s0 + p * m;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long K = (long)Lp * D;
  const int rows = min(32, kL - o0), per = 16 * ((D / 16 + kFewWaves - 1) / kFewWaves);
  const auto wv = make_view(W + ((long)br * kL + o0) * K + (long)m * D,
                            (uint32_t)(((rows - 1) * K + D) * 2));
  const auto xv = make_view(H + (long)lay * D, (uint32_t)((((long)M - 1) * L * D + D) * 2));
  f32x16 acc[1] = {zero16()};
  const float ss = few_product<1>(
      wv, (uint32_t)(K * 2), rows - 1, xv,
      [&](int x) { return (uint32_t)min(x, M - 1) * (uint32_t)(L * D * 2); },
      g_pre + ((long)br * L + lay) * D, nullptr, w * per, min(D, (w + 1) * per), acc, area[w],
      lane);
  float* red = (float*)area[w];  // [32 tokens][LD]
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = acc[0][4 * q4 + i];
    *(f32x4*)(red + r * LD + 8 * q4 + 4 * h) = v;
  }
  if (h == 0) ssq[w][r] = ss;
  __syncthreads();
  const int n = tid >> 3, c = 4 * (tid & 7);
  if (n >= M) return;
  float sq = 0.f;
#pragma unroll
  for (int ww = 0; ww < kFewWaves; ++ww) sq += ssq[ww][n];
  const float rinv = 1.0f / sqrtf(sq / (float)D + eps);
  float* dst = part + ((long)m * M + n) * 2 * kL + (long)br * kL;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = o0 + c + i;
    float v = 0.f;
#pragma unroll
    for (int ww = 0; ww < kFewWaves; ++ww) v += ((const float*)area[ww])[n * LD + c + i];
    // without feedback channel o / L reads only the sources of layers <= o / L
    if (o < kL) dst[o] = nofb && lay > o / L ? 0.f : v * rinv;
  }
}

// ---------------------------------------------------------------------- mix
// One token and a slice of the columns: the logits (the sources' partial sums in order, plus
// the bias), the weights (mask, softmax), their products with 1 / RMS of the states, and the
// mixed channels of both branches, all in fp32, and for the mid norm the sums of squares of
// every eight columns before their rounding to bf16 (as the many-token mix takes them; 0.3 to
// 1.2 us a pool more than the sums of the rounded ones, mostly at 32 tokens). A thread makes
// kFewJc channels of 8 columns.
constexpr int kFewJc = 4;

__global__ __launch_bounds__(256) void few_mix_kernel(const bf16* H, const bf16* g_pre,
                                                      const float* part, const bf16* bias, int M,
                                                      int L, int k, int D, int sources,
                                                      int softmax, int nofb, float eps,
                                                      int cols, bf16* mixed, float* sq) {
  extern __shared__ __align__(16) float sm[];
  const int kL = k * L, n = blockIdx.x, c0 = blockIdx.y * cols;
  float* coef = sm;           // [2][k][L]
  float* rinv = sm + 2 * kL;  // [L]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bf16* x = H + (long)n * L * D;
  // logits: kE entries per thread and kS sources at a time, all their loads in flight
  constexpr int kE = 3, kS = 8;
  for (int e0 = tid; e0 < 2 * kL; e0 += 256 * kE) {
    float v[kE];
#pragma unroll
    for (int i = 0; i < kE; ++i) v[i] = (float)bias[min(e0 + 256 * i, 2 * kL - 1)];
    for (int m0 = 0; m0 < sources; m0 += kS) {
      float pv[kE][kS];
#pragma unroll
      for (int i = 0; i < kE; ++i)
#pragma unroll
        for (int q = 0; q < kS; ++q)
          pv[i][q] = part[((long)min(m0 + q, sources - 1) * M + n) * 2 * kL +
                          min(e0 + 256 * i, 2 * kL - 1)];
#pragma unroll
      for (int i = 0; i < kE; ++i)
#pragma unroll
        for (int q = 0; q < kS; ++q) v[i] += m0 + q < sources ? pv[i][q] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kE; ++i)
      if (e0 + 256 * i < 2 * kL) coef[e0 + 256 * i] = v[i];
  }
  // 1 / RMS of the states: kR rows of a wave at a time
  constexpr int kR = 4;
  for (int l0 = w; l0 < L; l0 += 4 * kR) {
    float ss[kR];
#pragma unroll
    for (int i = 0; i < kR; ++i) ss[i] = 0.f;
    for (int e = 8 * lane; e < D; e += 512) {
      bf16x8 v[kR];
#pragma unroll
      for (int i = 0; i < kR; ++i) v[i] = ld_frag<bf16>(x + (long)min(l0 + 4 * i, L - 1) * D + e);
#pragma unroll
      for (int i = 0; i < kR; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) ss[i] += (float)v[i][t] * (float)v[i][t];
    }
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      const float v = wave_sum(ss[i]);
      if (lane == 0 && l0 + 4 * i < L) rinv[l0 + 4 * i] = 1.0f / sqrtf(v / (float)D + eps);
    }
  }
  __syncthreads();
  for (int row = tid; row < 2 * k; row += 256) {  // (see alpha_rows_kernel)
    float* a = coef + row * L;
    const int nl = nofb ? row % k + 1 : L;
    if (softmax) {
      float mx = a[0];
      for (int l = 1; l < nl; ++l) mx = fmaxf(mx, a[l]);
      float z = 0.f;
      for (int l = 0; l < nl; ++l) z += expf(a[l] - mx);
      const float iz = 1.0f / z;
      for (int l = 0; l < nl; ++l) a[l] = expf(a[l] - mx) * iz;
    }
    for (int l = 0; l < L; ++l) a[l] = l < nl ? a[l] * rinv[l] : 0.f;
  }
  __syncthreads();
  const int nch = min(cols, D - c0) / 8, ngrp = (k + kFewJc - 1) / kFewJc;
  for (int it = tid; it < 2 * nch * ngrp; it += 256) {
    const int ch = it % nch, jg = it / nch % ngrp, br = it / (nch * ngrp);
    const int e = c0 + 8 * ch, j0 = jg * kFewJc;
    const bf16* xp = x + e;
    const bf16* gp = g_pre + (long)br * L * D + e;
    const float* cf = coef + ((long)br * k + j0) * L;
    float acc[kFewJc][8];
#pragma unroll
    for (int jj = 0; jj < kFewJc; ++jj)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[jj][i] = 0.f;
    constexpr int kL8 = 8;  // layers in flight
    for (int l0 = 0; l0 < L; l0 += kL8) {
      bf16x8 xf[kL8], gf[kL8];
#pragma unroll
      for (int q = 0; q < kL8; ++q) {
        xf[q] = ld_frag<bf16>(xp + (long)min(l0 + q, L - 1) * D);
        gf[q] = ld_frag<bf16>(gp + (long)min(l0 + q, L - 1) * D);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < kL8; ++q) {
        if (l0 + q >= L) break;
        float xv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) xv[i] = (float)xf[q][i] * (float)gf[q][i];
#pragma unroll
        for (int jj = 0; jj < kFewJc; ++jj) {
          const float cj = cf[(j0 + jj < k ? jj : 0) * L + l0 + q];
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[jj][i] += cj * xv[i];
        }
      }
    }
#pragma unroll
    for (int jj = 0; jj < kFewJc; ++jj) {
      if (j0 + jj >= k) break;
      const long row = ((long)br * k + j0 + jj) * M + n;
      store8(mixed + row * D + e, acc[jj]);
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += acc[jj][i] * acc[jj][i];
      sq[row * (D / 8) + e / 8] = ss;
    }
  }
}

size_t few_router_bytes(const Shape& sh) {
  return few_tokens(sh) && sh.router_mode != 1
             ? (size_t)sh.Lp * sh.N() * 2 * sh.k * sh.L * sizeof(float) : 0;
}

void launch_few_router(const Shape& sh, int s0, const bf16* H, const bf16* g_pre,
                       const bf16* W_alpha, float* part, hipStream_t s) {
  if (sh.router_mode == 1) return;  // static weights: no router
  const int kL = sh.k * sh.L, M = sh.N();
  hipLaunchKernelGGL(few_router_kernel, dim3((kL + 31) / 32, sh.Lp, 2),
                     dim3(64 * kFewWaves), 0, s, H, W_alpha, g_pre, M, sh.L, sh.Lp, sh.D, kL, s0,
                     sh.p, sh.router_mode == 2 ? 1 : 0, sh.eps, part);
}

void launch_few_mix(const Shape& sh, const bf16* H, const bf16* g_pre, const bf16* b_alpha,
                    const float* part, bf16* mixed, float* sq, hipStream_t s) {
  // columns per workgroup: 128 or more, fewer workgroups per token as the tokens grow (each
  // sums the logits and the norms of its token again)
  const int parts = std::max(1, std::min(sh.D / 128, 128 / sh.N()));
  const int cols = (sh.D / 8 + parts - 1) / parts * 8;
  const size_t lds = (2ul * sh.k * sh.L + sh.L) * sizeof(float);
  hipLaunchKernelGGL(few_mix_kernel, dim3(sh.N(), (sh.D + cols - 1) / cols), dim3(256), lds, s, H,
                     g_pre, part, b_alpha, sh.N(), sh.L, sh.k, sh.D,
                     sh.router_mode == 1 ? 0 : sh.Lp, sh.mix_softmax,
                     sh.router_mode == 2 ? 1 : 0, sh.eps, cols, mixed, sq);
}

void launch_few_kv(const Shape& sh, const bf16* mixed, const float* sq, const bf16* g_mid,
                   const bf16* Wk, const bf16* Wv, const bf16* g_knorm, const int32_t* ctx_len,
                   bf16* Kc, bf16* Vc, hipStream_t s) {
  const long D = sh.D;
  FewProj a{mixed, (long)sh.N() * D, D, Wk, Wv, sh.k, g_mid, sq, g_knorm, sh.N(), sh.D, sh.Hkv,
            sh.T_new, sh.B, sh.gs, sh.gq, ctx_len, sh.ctx_hi, sh.eps, {}, Kc, Vc, sh.S_cap};
  few_proj<true>(a, sh, 2 * sh.k, s);
}

}  // namespace wm
