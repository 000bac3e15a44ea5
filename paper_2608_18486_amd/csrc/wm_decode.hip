// Decode form of the channel attention (paper Section 3.1 Step 3, Section 3.2): few new
// tokens per sequence (T_new <= 4) against a long cache.
//
// Split-S over the cache, one workgroup per (split, channel with a reader, sequence, KV head)
// serving every query row that reads that channel and head (all its consumer layers, grouped
// query heads and new tokens), so each channel slice is streamed from HBM once.
#include <algorithm>

#include "wm_device.hpp"
#include "wm_frag.hpp"
#include "wm_internal.hpp"

namespace wm {

// ------------------------------------------------------------------ decode
// Cache slots per split workgroup: long splits amortise a workgroup's set-up and its
// partial-state write; they are halved (down to 256) while the grid of splits x
// (channel, sequence, KV head) would hold fewer than kDecodeMinBlocks workgroups.
constexpr int kSplitMax = 4096, kSplitMin = 256;
constexpr long kDecodeMinBlocks = 4096;

int decode_split_len(const Shape& sh) {
  const long kend = (long)sh.ctx_max + sh.span();  // upper bound on visible slots
  const long slices = (long)sh.k * sh.B * sh.Hkv;
  int len = kSplitMax;
  while (len > kSplitMin && slices * ((kend + len - 1) / len) < kDecodeMinBlocks) len /= 2;
  return len;
}

int decode_splits(const Shape& sh) {
  const long kend = (long)sh.ctx_max + sh.span();
  const int len = decode_split_len(sh);
  int n = (int)((kend + len - 1) / len);
  return n < 1 ? 1 : n;
}

size_t decode_partials_bytes(const Shape& sh) {
  size_t rows = (size_t)sh.L * sh.B * sh.Hq * sh.T_new;
  return rows * decode_splits(sh) * (sh.d + 2) * sizeof(float);
}

template <typename T> struct DecodeArgs {
  const T *Q, *Kc, *Vc, *Kd, *Vd;
  const int32_t* ctx_len;
  const int32_t* doc;  // [B][T_new] first position of each token's document, or null
  float* part;  // [L][B][Hq][T_new][nsplit][d + 2]: unnormalised o, m, l
  T* O;
  int B, T_new, L, Hq, Hkv, S_cap, mask_paper, nsplit, split_len;
  int gs, gq, ctx_hi;  // query i of sequence b sits at position ctx_len[b] + gq + gs i
  float scale_log2;
  LayerTable chan;
  // the grid's channels, those with a reader: live[i], its consumers offsets[i] .. offsets[i + 1]
  LayerTable live;
  ChannelGroups cg;
};

// Merge online-softmax state (m2, l2, o2) into (m, l, o).
__device__ __forceinline__ void merge_state(float& m, float& l, float* o, float m2, float l2,
                                            const float* o2, int n, float c) {
  float M = fmaxf(m, m2);
  float a1 = fast_exp2((m - M) * c), a2 = fast_exp2((m2 - M) * c);
  l = l * a1 + l2 * a2;
  for (int i = 0; i < n; ++i) o[i] = o[i] * a1 + o2[i] * a2;
  m = M;
}

// ---------------------------------------------- decode on the matrix cores (bf16)
// bf16, head dims 64 and 96. The rows of one (channel, sequence, KV head) -- consumers x
// grouped heads x new tokens -- are the columns of S^T = K Q^T and O^T = V^T P^T on 32x32x16
// MFMAs, as in the full-sequence kernel, so a slot costs the same for 1 row and for 32.
// (The VALU kernel below spends 16 fused multiply-adds and a butterfly per slot, lane and
// row: at 16 rows, B = 8, ctx 4001, k = 8, 6/3 heads of 96 it ran 383 us on 221 MB of
// cache; this one 47 us. At 2 rows and head dim 64 both run at the rate of the cache
// stream at B = 16, ctx 8191, k = 12; at one consumer over 709 slots this one
// takes 7 us and the VALU kernel 10.6.) What is left is the stream: each of NW waves walks
// every NW-th 32-slot block through a ring of two blocks of its own in LDS (LDS-DMA, no
// barrier: a wave waits only for its own copies). Measured at the two shapes above:
// waves on a CU count for more than copies in flight per wave (three or four blocks per
// ring, with half the waves, 4-30% slower). The weights are the VALU kernel's: scores from the
// unscaled bf16 queries, weights in fp32, cut into three bf16 parts (8 + 8 + 8 bits, exact)
// for three PV products, the normaliser summed from the fp32 ones. (Two rounded parts, 16
// bits, left 2.7e-6 of the terms' sum where two values cancel, three 5e-8; a step at 12 heads
// of 64, k = 12, ctx 8000 99.2 us with two, 100.8 with three; at B = 8, T_new = 4, ctx 4001,
// 6/3 heads of 96 80.7 and 80.8. The parts are truncated: rounding them takes longer, 107.7.)
template <int DH, int NW_> struct DecMfma {
  static constexpr int NW = NW_, NT = 64 * NW, NS = 2, BKV = 32;
  static constexpr int NKS = DH / 16, NDT = DH / 32;
  static constexpr int ROW_BYTES = 2 * DH, CPR = ROW_BYTES / 16;
  static constexpr int BLK = BKV * ROW_BYTES;      // one K (or V) block of 32 slots
  static constexpr int NI = BLK / 1024;            // copy instructions per block
  static constexpr int STAGE = 2 * BLK;            // K then V
  static constexpr int RING = NS * STAGE;          // per wave
  static constexpr int OLD = DH + 4;               // row stride of the merge staging (floats)
  static_assert(32 * OLD * 4 + 256 <= RING, "the merge staging fits a wave's ring");
  static_assert(2 * NI * (NS - 1) <= 63, "the copies in flight behind one vmcnt");
};

// Sum of 16 values as a balanced tree.
__device__ __forceinline__ float sum16(const f32x16& v) {
  float t[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = v[i] + v[8 + i];
  return ((t[0] + t[4]) + (t[1] + t[5])) + ((t[2] + t[6]) + (t[3] + t[7]));
}

// lds_dma16 (wm_device.hpp) for bytes that are read once: non-temporal, so the stream does
// not fill L2 and the Infinity Cache with lines nobody reads again (B = 16, ctx 8191, k = 12,
// 16 heads of 64: the step 1004 -> 902 us, its attention 5.6 -> 6.2 TB/s, the rate of a plain
// read of HBM; at B = 8, ctx 4001, whose 221 MB could stay in that cache, 133 -> 124 us).
__device__ __forceinline__ void lds_dma16_stream(uint32_t lds_addr, uint32_t voff,
                                                 __amdgpu_buffer_rsrc_t rsrc) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}

template <int DH, int NW, bool DOC, bool ONCE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3)))
void attend_decode_mfma_kernel(DecodeArgs<bf16> a) {
  using C = DecMfma<DH, NW>;
  __shared__ __align__(16) char smem[C::NW * C::RING];
  const int split = blockIdx.x;
  int y = blockIdx.y;
  const int kvh = y % a.Hkv;
  y /= a.Hkv;
  const int b = y % a.B, ci = y / a.B, c = a.live.v[ci];
  const int off = a.cg.offsets[ci], nmem = a.cg.offsets[ci + 1] - off;
  const int grp = a.Hq / a.Hkv;
  const int G = nmem * grp * a.T_new, g0 = 32 * blockIdx.z;
  if (g0 >= G) return;
  const int pos0 = __builtin_amdgcn_readfirstlane(ctx_at(a.ctx_len, b, a.ctx_hi)) + a.gq;
  const int gs = a.gs, incl = a.mask_paper ? 0 : 1;
  const int kend = min(pos0 + gs * (a.T_new - 1) + incl, a.S_cap);
  const int s0 = split * a.split_len, s1 = min(s0 + a.split_len, kend);
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float cl2 = a.scale_log2;

  // this lane's row (both halves of the wave share it) and the slots it reads
  auto row_of = [&](int g, int& i) {
    i = g % a.T_new;
    const int gq = (g / a.T_new) % grp, mi = g / (a.T_new * grp);
    const int l = a.cg.members[off + mi], hq = kvh * grp + gq;
    return (((long)l * a.B + b) * a.Hq + hq) * a.T_new + i;
  };
  int vis = 0, lov = 0;
  bf16x8 qf[C::NKS];
  {
    const bool ok = g0 + r < G;
    int i = 0;
    const long rowid = ok ? row_of(g0 + r, i) : 0;
    if (ok) {
      vis = min(pos0 + gs * i + incl, s1);
      if (DOC) lov = doc_first(a.doc, b, a.T_new, i, pos0 + gs * i);
    }
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks)
      qf[ks] = ok ? ld_frag<bf16>(a.Q + rowid * DH + 16 * ks + 8 * h) : zero_frag<bf16>();
  }

  const int nblk = s1 > s0 ? (s1 - s0 + C::BKV - 1) / C::BKV : 0;
  const int nw = (nblk - w + C::NW - 1) / C::NW;  // this wave's blocks: w, w + NW, ...
  const long cbase = (((long)c * a.B + b) * a.Hkv + kvh) * (long)a.S_cap * DH;
  // views end at the last visible slot: rows past it arrive as zeros
  const auto kview = make_view(a.Kc + cbase, (uint32_t)max(kend, 0) * C::ROW_BYTES);
  const auto vview = make_view(a.Vc + cbase, (uint32_t)max(kend, 0) * C::ROW_BYTES);
  uint32_t coff[C::NI];
#pragma unroll
  for (int n = 0; n < C::NI; ++n) {
    const int ch = 64 * n + lane, row = ch / C::CPR;
    coff[n] = (uint32_t)row * C::ROW_BYTES + 16u * (uint32_t)((ch % C::CPR) ^ pf_swz<DH>(row));
  }
  char* ring = smem + w * C::RING;
  const uint32_t ring_at = (uint32_t)(uintptr_t)ring;
  // block j of this wave into ring stage st (blocks past the wave's last are copied as
  // zeros, so the count of copies in flight is the same at every wait)
  auto issue = [&](int j, int st) {
    const uint32_t base =
        j < nw ? (uint32_t)(s0 + C::BKV * (w + C::NW * j)) * C::ROW_BYTES : kOffOob;
#pragma unroll
    for (int n = 0; n < 2 * C::NI; ++n) {
      const uint32_t o = base + coff[n % C::NI];
      const uint32_t lds =
          __builtin_amdgcn_readfirstlane(ring_at + st * C::STAGE + 1024 * n);
      if constexpr (ONCE) lds_dma16_stream(lds, o, n < C::NI ? kview : vview);
      else lds_dma16(lds, o, n < C::NI ? kview : vview);
    }
  };

  const int all_vis = min(pos0 + incl, s1);  // slots below it are visible to every row
  float m = kNegBig, lsum = 0.f;
  f32x16 o[C::NDT];
#pragma unroll
  for (int dt = 0; dt < C::NDT; ++dt) o[dt] = zero16();
  // (a wave without a block of the split walks one of zeros, every slot of it hidden)
  const PfLane<DH> lo = pf_lane<DH>(lane);
#pragma unroll
  for (int u = 0; u + 1 < C::NS; ++u) issue(u, u);
  int j = 0, st = 0;
  do {
    // the stage block j-1 was read from (its reads have returned) takes block j+NS-1
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    issue(j + C::NS - 1, st == 0 ? C::NS - 1 : st - 1);
    wait_copies<2 * C::NI * (C::NS - 1)>();
    const uint32_t kh = st * C::STAGE, vh = kh + C::BLK;
    f32x16 sc = zero16();
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) sc = mma32(sc, pf_ldk<DH>(ring, lo, kh, ks), qf[ks]);
    const int at = s0 + C::BKV * (w + C::NW * j);  // the block's first slot
    if (DOC || __builtin_expect(at + C::BKV > all_vis, 0)) {
      // some row may not read some of the block's slots
      asm volatile("" : "+v"(vis));  // (keeps the comparisons out of the common path)
      const int base = at + 4 * h;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int s = base + 8 * (q >> 2) + (q & 3);
        sc[q] = s >= vis || (DOC && s < lov) ? kNegBig : sc[q];
      }
    }
    float mx = sc[0];
#pragma unroll
    for (int q = 1; q < 16; ++q) mx = fmaxf(mx, sc[q]);
    mx = halves_max(mx);
    if (__builtin_expect(__any(mx > m), 0)) {
      const float mn = fmaxf(m, mx), al = fast_exp2((m - mn) * cl2);
      lsum *= al;
#pragma unroll
      for (int dt = 0; dt < C::NDT; ++dt) {
        asm volatile("" : "+v"(o[dt]));  // (keeps the products out of the common path)
        o[dt] *= al;
      }
      m = mn;
    }
    // hidden slots (-1e30) get weight 0, also while the row has seen none (m = -1e30)
    const float mc = m > 0.5f * kNegBig ? m * cl2 : 0.f;
    f32x16 p;
#pragma unroll
    for (int q = 0; q < 16; ++q) p[q] = fast_exp2(fmaf(sc[q], cl2, -mc));
    float ps = sum16(p);
    if (__builtin_expect(__any(!(ps <= 3.0e38f)), 0)) {  // a NaN score weighs nothing
#pragma unroll
      for (int q = 0; q < 16; ++q) p[q] = sc[q] > 0.5f * kNegBig ? p[q] : 0.f;
      ps = sum16(p);
    }
    lsum += ps;
    // a weight's upper 16 bits are its first part; twice more from what is left: 24 bits
    bf16x8 pw[3][2];
#pragma unroll
    for (int q = 0; q < 16; q += 2) {
      uint32_t r0 = __float_as_uint(p[q]), r1 = __float_as_uint(p[q + 1]);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const bf16x2 w2 = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(r1, r0, 0x07060302u));
        pw[u][q >> 3][q & 7] = w2[0];
        pw[u][q >> 3][(q & 7) + 1] = w2[1];
        r0 = __float_as_uint(__uint_as_float(r0) - __uint_as_float(r0 & 0xffff0000u));
        r1 = __float_as_uint(__uint_as_float(r1) - __uint_as_float(r1 & 0xffff0000u));
      }
    }
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      bf16x8 vf[C::NDT];
#pragma unroll
      for (int dt = 0; dt < C::NDT; ++dt) vf[dt] = pf_ldv<DH>(ring, lo, vh, hf, dt);
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int dt = 0; dt < C::NDT; ++dt) o[dt] = mma32(o[dt], vf[dt], pw[u][hf]);
    }
    st = st + 1 == C::NS ? 0 : st + 1;
  } while (++j < nw);
  wait_copies<0>();  // no copy may land in the staging below, or after the block ends
  // merge the waves' states: each writes its rows [r][DH] and (m, l) to its own ring
  const float lt = halves_sum(lsum);
  float* so = (float*)ring;
#pragma unroll
  for (int dt = 0; dt < C::NDT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = o[dt][4 * g + i];
      *(f32x4*)(so + r * C::OLD + 32 * dt + 8 * g + 4 * h) = v;
    }
  if (h == 0) {
    so[32 * C::OLD + 2 * r] = m;
    so[32 * C::OLD + 2 * r + 1] = lt;
  }
  __syncthreads();
  const int ng = min(32, G - g0);
  for (int e = tid; e < ng * DH; e += C::NT) {
    const int gi = e / DH, dd = e - gi * DH;
    float M = kNegBig;
#pragma unroll
    for (int ww = 0; ww < C::NW; ++ww)
      M = fmaxf(M, ((const float*)(smem + ww * C::RING))[32 * C::OLD + 2 * gi]);
    float lw = 0.f, ow = 0.f;
#pragma unroll
    for (int ww = 0; ww < C::NW; ++ww) {
      const float* sw = (const float*)(smem + ww * C::RING);
      const float al = fast_exp2((sw[32 * C::OLD + 2 * gi] - M) * cl2);
      lw += sw[32 * C::OLD + 2 * gi + 1] * al;
      ow += sw[gi * C::OLD + dd] * al;
    }
    int i;
    float* dst = a.part + (row_of(g0 + gi, i) * a.nsplit + split) * (DH + 2);
    dst[dd] = ow;
    if (dd == 0) {
      dst[DH] = M;
      dst[DH + 1] = lw;
    }
  }
}

// ---------------------------------------------- decode on the VALU (fp32, head dim 32)
template <typename T, int DH, int NG>
__global__ __launch_bounds__(256) void attend_decode_kernel(DecodeArgs<T> a) {
  // A cache slot is read by LPS lanes of 8 elements each.
  constexpr int LPS = DH / 8;
  static_assert(DH == 32 || DH == 64, "the lanes of a slot sum by butterflies");
  constexpr int SPW = 64 / LPS;  // slots per wave per sweep step
  constexpr int U = NG <= 2 ? 2 : 1;  // sweep steps per batch (U slots per lane)
  constexpr int SPB = 4 * SPW * U;  // slots per batch of the 4 waves
  __shared__ float red[4][NG][DH + 2];

  const int split = blockIdx.x;
  int y = blockIdx.y;
  const int kvh = y % a.Hkv;
  y /= a.Hkv;
  const int b = y % a.B, ci = y / a.B, c = a.live.v[ci];
  const int off = a.cg.offsets[ci], nmem = a.cg.offsets[ci + 1] - off;
  const int grp = a.Hq / a.Hkv;
  const int G = nmem * grp * a.T_new;
  // position of query i: pos0 + gs i (wave-uniform)
  const int pos0 = __builtin_amdgcn_readfirstlane(ctx_at(a.ctx_len, b, a.ctx_hi)) + a.gq;
  const int gs = a.gs;
  const int incl = a.mask_paper ? 0 : 1;
  const int kend = min(pos0 + gs * (a.T_new - 1) + incl, a.S_cap);
  const int s0 = split * a.split_len, s1 = min(s0 + a.split_len, kend);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int sg = lane / LPS, c8 = lane % LPS;
  const float cl2 = a.scale_log2;
  const float thresh = 8.0f / cl2;  // log2 headroom before a rescale

  const long cbase = (((long)c * a.B + b) * a.Hkv + kvh) * (long)a.S_cap * DH;
  // the slice through buffer views: slots at or past s1 read zeros without a branch
  const __amdgpu_buffer_rsrc_t kview = make_view(a.Kc + cbase, (uint32_t)a.S_cap * DH * sizeof(T));
  const __amdgpu_buffer_rsrc_t vview = make_view(a.Vc + cbase, (uint32_t)a.S_cap * DH * sizeof(T));
  auto slot_off = [&](int s) {
    return s < s1 ? (uint32_t)(s * DH + 8 * c8) * (uint32_t)sizeof(T) : kOffOob;
  };

  for (int g0 = 0; g0 < G; g0 += NG) {
    const int ng = min(NG, G - g0);
    float q[NG][8], m[NG], ls[NG], o[NG][8];
    int vis[NG], lov[NG];  // the row reads slots lov <= s < vis
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      m[gi] = kNegBig;
      ls[gi] = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[gi][i] = 0.f;
      if (gi < ng) {
        int g = g0 + gi;
        int i = g % a.T_new, gq = (g / a.T_new) % grp, mi = g / (a.T_new * grp);
        int l = a.cg.members[off + mi], hq = kvh * grp + gq;
        long rowid = (((long)l * a.B + b) * a.Hq + hq) * a.T_new + i;
        vis[gi] = pos0 + gs * i + incl;
        lov[gi] = doc_first(a.doc, b, a.T_new, i, pos0 + gs * i);
        load8(a.Q + rowid * DH + 8 * c8, q[gi]);
      } else {
        vis[gi] = 0;
        lov[gi] = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) q[gi][i] = 0.f;
      }
    }

    // raw K/V fragments of a batch (U slots per lane), double-buffered across batches
    // (two batches per loop trip keep the buffer indices static)
    frag_t<T> kr0[U], vr0[U], kr1[U], vr1[U];
    auto fetch = [&](int sb, frag_t<T>* kr, frag_t<T>* vr) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t so = slot_off(sb + w * SPW * U + u * SPW + sg);
        kr[u] = buf_frag<T>(kview, so);
        vr[u] = buf_frag<T>(vview, so);
      }
    };
    auto consume = [&](int sb, const frag_t<T>* kr, const frag_t<T>* vr) {
      float p[U][NG];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = sb + w * SPW * U + u * SPW + sg;
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
          float d = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i) d += q[gi][i] * to_f32(kr[u][i]);
#pragma unroll
          for (int x = 1; x < LPS; x <<= 1) d += __shfl_xor(d, x, 64);
          p[u][gi] = s < s1 && s < vis[gi] && s >= lov[gi] ? d : kNegBig;
        }
      }
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        float mx = p[0][gi];
#pragma unroll
        for (int u = 1; u < U; ++u) mx = fmaxf(mx, p[u][gi]);
        if (mx > m[gi] + thresh) {  // lazy rescale (per lane; merged exactly below)
          const float al = fast_exp2((m[gi] - mx) * cl2);
          ls[gi] *= al;
#pragma unroll
          for (int i = 0; i < 8; ++i) o[gi][i] *= al;
          m[gi] = mx;
        }
        const float mc = m[gi] * cl2;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float pe = p[u][gi] > 0.5f * kNegBig ? fast_exp2(p[u][gi] * cl2 - mc) : 0.f;
          ls[gi] += pe;
#pragma unroll
          for (int i = 0; i < 8; ++i) o[gi][i] += pe * to_f32(vr[u][i]);
        }
      }
    };
    // batches past the split read zeros (and are masked), so the loop runs in pairs
    fetch(s0, kr0, vr0);
    for (int sb = s0; sb < s1; sb += 2 * SPB) {
      fetch(sb + SPB, kr1, vr1);
      consume(sb, kr0, vr0);
      fetch(sb + 2 * SPB, kr0, vr0);
      consume(sb + SPB, kr1, vr1);
    }
    // merge the slot groups of the wave (lanes that share c8)
#pragma unroll
    for (int msk = LPS; msk < 64; msk <<= 1)
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        float m2 = __shfl_xor(m[gi], msk, 64), l2 = __shfl_xor(ls[gi], msk, 64), o2[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) o2[i] = __shfl_xor(o[gi][i], msk, 64);
        merge_state(m[gi], ls[gi], o[gi], m2, l2, o2, 8, cl2);
      }
    if (sg == 0) {
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
#pragma unroll
        for (int i = 0; i < 8; ++i) red[w][gi][8 * c8 + i] = o[gi][i];
        if (c8 == 0) {
          red[w][gi][DH] = m[gi];
          red[w][gi][DH + 1] = ls[gi];
        }
      }
    }
    __syncthreads();
    for (int e = tid; e < ng * DH; e += 256) {
      int gi = e / DH, dd = e % DH;
      float M = kNegBig;
      for (int ww = 0; ww < 4; ++ww) M = fmaxf(M, red[ww][gi][DH]);
      float Lsum = 0.f, Osum = 0.f;
      for (int ww = 0; ww < 4; ++ww) {
        float sc = fast_exp2((red[ww][gi][DH] - M) * cl2);
        Lsum += red[ww][gi][DH + 1] * sc;
        Osum += red[ww][gi][dd] * sc;
      }
      // recompute the row id for gi (registers are per-lane; rows are uniform)
      int g = g0 + gi;
      int i = g % a.T_new, gq = (g / a.T_new) % grp, mi = g / (a.T_new * grp);
      int l = a.cg.members[off + mi], hq = kvh * grp + gq;
      long rid = (((long)l * a.B + b) * a.Hq + hq) * a.T_new + i;
      float* dst = a.part + (rid * a.nsplit + split) * (DH + 2);
      dst[dd] = Osum;
      if (dd == 0) {
        dst[DH] = M;
        dst[DH + 1] = Lsum;
      }
    }
    __syncthreads();
  }
}

// One wave per query row: fold the dummy slot and all split partials.
template <typename T, int DH>
__global__ __launch_bounds__(256) void attend_combine_kernel(DecodeArgs<T> a) {
  constexpr int EPL = (DH + 63) / 64;  // elements per lane: channel 64 e + lane
  const long rows = (long)a.L * a.B * a.Hq * a.T_new;
  const long rid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (rid >= rows) return;
  long t = rid;
  const int i = (int)(t % a.T_new);
  t /= a.T_new;
  const int hq = (int)(t % a.Hq);
  t /= a.Hq;
  const int b = (int)(t % a.B), l = (int)(t / a.B);
  const int c = a.chan.v[l], kvh = hq / (a.Hq / a.Hkv);
  const float cl2 = a.scale_log2;

  float M, Lsum, o[EPL];
  auto active = [&](int e) { return 64 * e + lane < DH; };
  if (a.mask_paper) {
    const T* q = a.Q + rid * DH;
    const T* kd = a.Kd + ((long)c * a.Hkv + kvh) * DH;
    const T* vd = a.Vd + ((long)c * a.Hkv + kvh) * DH;
    float part = 0.f;
    for (int e = 0; e < EPL; ++e)
      if (active(e)) part += to_f32(q[64 * e + lane]) * to_f32(kd[64 * e + lane]);
    M = wave_sum(part);
    Lsum = 1.f;
    for (int e = 0; e < EPL; ++e) o[e] = active(e) ? to_f32(vd[64 * e + lane]) : 0.f;
  } else {
    M = kNegBig;
    Lsum = 0.f;
    for (int e = 0; e < EPL; ++e) o[e] = 0.f;
  }
  const float* src = a.part + rid * a.nsplit * (DH + 2);
  for (int sidx = 0; sidx < a.nsplit; ++sidx) {
    const float* ps = src + (long)sidx * (DH + 2);
    float o2[EPL];
    for (int e = 0; e < EPL; ++e) o2[e] = active(e) ? ps[64 * e + lane] : 0.f;
    merge_state(M, Lsum, o, ps[DH], ps[DH + 1], o2, EPL, cl2);
  }
  T* dst = a.O + ((((long)l * a.B + b) * a.T_new + i) * a.Hq + hq) * DH;
  for (int e = 0; e < EPL; ++e)
    if (active(e)) dst[64 * e + lane] = from_f32<T>(o[e] / Lsum);
}

template <typename T, int DH>
static void decode_dispatch(const DecodeArgs<T>& a, int G, dim3 grid, hipStream_t s) {
  if (G <= 1)
    hipLaunchKernelGGL((attend_decode_kernel<T, DH, 1>), grid, dim3(256), 0, s, a);
  else if (G <= 2)
    hipLaunchKernelGGL((attend_decode_kernel<T, DH, 2>), grid, dim3(256), 0, s, a);
  else if (G <= 4)
    hipLaunchKernelGGL((attend_decode_kernel<T, DH, 4>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((attend_decode_kernel<T, DH, 8>), grid, dim3(256), 0, s, a);
  long rows = (long)a.L * a.B * a.Hq * a.T_new;
  hipLaunchKernelGGL((attend_combine_kernel<T, DH>), dim3((unsigned)((rows + 3) / 4)), dim3(256),
                     0, s, a);
}

// Splits of the matrix-core kernel: slots per workgroup halved (down to decode_split_len,
// which sizes the partials' workspace) only until the grid holds this many workgroups, 2 per
// CU: a workgroup's set-up and merge cost about as much as 300 slots (B = 8, ctx 4001:
// 512 workgroups or more 132 us a step, 1024 or more 147, 2048 or more 167). Only channels
// with a reader count: layer by layer one of the k has one, and with all of them counted
// (us a layer, query and attention) k = 12, 16 heads of 64, B 2, ctx 8191 took 89 and takes
// 34; k = 12, 12 heads of 64, B 4, ctx 4000 86 and 30; k = 16, 6/3 heads of 96, B 8, ctx 4000
// 54 and 30.
constexpr long kDecodeMfmaBlocks = 512;
// Cache bytes from which a call's slots are taken to be read from HBM. Attention alone, us,
// plain copies / non-temporal ones: 221 MB 133 / 124 a step; at 13 MB that the next call
// reads again (B 1, ctx 709, L 16, layer by layer) 475 / 490 a token, so what the Infinity
// Cache (256 MB) can keep next to the rest of a step stays plain.
constexpr long kDecodeStreamBytes = 128L << 20;

template <int DH>
static void decode_mfma(DecodeArgs<bf16> a, int G, int nlive, const Shape& sh, hipStream_t s) {
  const int z = std::max(1, (G + 31) / 32);
  const long slices = (long)nlive * sh.B * sh.Hkv * z, kend = (long)sh.ctx_max + sh.span();
  int len = kSplitMax;
  while (len > a.split_len && slices * ((kend + len - 1) / len) < kDecodeMfmaBlocks) len /= 2;
  a.split_len = len;  // at least decode_split_len, so the partials fit their workspace
  a.nsplit = std::max(1, (int)((kend + len - 1) / len));
  const dim3 grid(a.nsplit, sh.Hkv * sh.B * nlive, z);
  // a cache read once by one row tile, and larger (all channels: layer by layer, the other
  // layers' calls read theirs in between) than the caches keep from call to call
  const bool once = z == 1 && 4L * sh.k * sh.B * sh.Hkv * kend * DH >= kDecodeStreamBytes;
  // Waves per workgroup: 2, which leaves a CU's LDS to five workgroups (three at head dim
  // 96); 1 where a workgroup's walk is at most 128 slots (four blocks); 4 where the workgroups
  // fit the CUs all at once with four (one per CU at head dim 96, two at 64), and at head dim
  // 64 for long walks in several rounds of workgroups. Attention alone with 1 / 2 / 4 waves, us:
  // ctx 100, B 64, L 24, k 12, heads of 64: 77 / 87 / 111; ctx 4000, B 4: 172 / 126 / 133; ctx
  // 1500, B 16, L 12: 144 / 156 / 144; ctx 3000, B 24: 426 / 424 / 400; heads of 96, k = 8: ctx
  // 1000, B 4: 19 / 16.7 / 18.7; ctx 8000, B 1, k = 2: 31 / 26 / 23.6. One layer of 16 heads of
  // 64 with its query, 2 / 4 waves: ctx 700, B 1 19.6 / 19.1; ctx 3000, B 8 38.9 / 33.5; ctx 7948,
  // B 8 62.5 / 57.7; of 12 heads 60.1 / 48.2.
  const long wgs = a.nsplit * slices, per = std::min<long>(kend, len), cus = device_cus();
  const bool four = DH == 96 ? wgs <= cus : wgs <= 2 * cus || (wgs > 5 * cus && per >= 1024);
  const int waves = per <= 128 ? 1 : four ? 4 : 2;
#define WM_DEC_GO(NW, DOC, ONCE)                                                              \
  hipLaunchKernelGGL((attend_decode_mfma_kernel<DH, NW, DOC, ONCE>), grid, dim3(64 * (NW)), 0, \
                     s, a)
#define WM_DEC_NW(DOC, ONCE)                                                                   \
  do {                                                                                         \
    if (waves == 1) WM_DEC_GO(1, DOC, ONCE);                                                   \
    else if (waves == 2) WM_DEC_GO(2, DOC, ONCE);                                              \
    else WM_DEC_GO(4, DOC, ONCE);                                                              \
  } while (0)
  if (a.doc) {
    if (once) WM_DEC_NW(true, true);
    else WM_DEC_NW(true, false);
  } else {
    if (once) WM_DEC_NW(false, true);
    else WM_DEC_NW(false, false);
  }
#undef WM_DEC_NW
#undef WM_DEC_GO
  const long rows = (long)a.L * a.B * a.Hq * a.T_new;
  hipLaunchKernelGGL((attend_combine_kernel<bf16, DH>), dim3((unsigned)((rows + 3) / 4)),
                     dim3(256), 0, s, a);
}

template <typename T>
void launch_attend_decode(const Shape& sh, const LayerTable& chan_map, const ChannelGroups& cg,
                          const T* Q, const T* Kc, const T* Vc, const T* Kd, const T* Vd,
                          const int32_t* ctx_len, const int32_t* doc, float* partials, T* O,
                          hipStream_t s) {
  if (sh.N() <= 0) return;
  DecodeArgs<T> a{Q, Kc, Vc, Kd, Vd, ctx_len, doc, partials, O, sh.B, sh.T_new, sh.L, sh.Hq, sh.Hkv,
                  sh.S_cap, sh.mask_paper, decode_splits(sh), decode_split_len(sh), sh.gs, sh.gq,
                  sh.ctx_hi, kLog2e / sqrtf((float)sh.d), chan_map, {}, cg};
  int maxmem = 0, nlive = 0;
  for (int c = 0; c < sh.k; ++c) {
    int n = cg.offsets[c + 1] - cg.offsets[c];
    if (n == 0) continue;
    a.cg.offsets[nlive] = cg.offsets[c];
    a.live.v[nlive++] = c;
    if (n > maxmem) maxmem = n;
  }
  a.cg.offsets[nlive] = cg.offsets[sh.k];
  int G = maxmem * (sh.Hq / sh.Hkv) * sh.T_new;
  dim3 grid(a.nsplit, sh.Hkv * sh.B * nlive);
  if constexpr (sizeof(T) == 2) {  // fp32 at d = 96 is rejected by validation
    if (sh.d == 96) decode_mfma<96>(a, G, nlive, sh, s);
    else if (sh.d == 64) decode_mfma<64>(a, G, nlive, sh, s);
    else decode_dispatch<T, 32>(a, G, grid, s);
  } else if (sh.d == 64)
    decode_dispatch<T, 64>(a, G, grid, s);
  else
    decode_dispatch<T, 32>(a, G, grid, s);
}

#define WM_INST(T)                                                                              \
  template void launch_attend_decode<T>(const Shape&, const LayerTable&, const ChannelGroups&,  \
                                        const T*, const T*, const T*, const T*, const T*,       \
                                        const int32_t*, const int32_t*, float*, T*, hipStream_t);
WM_INST(float)
WM_INST(bf16)
#undef WM_INST

}  // namespace wm
