// Full-sequence attention for few rows (bf16, head dims 64 and 96, no documents): the calls
// whose 32-row tiles find a CU each, above all one layer of one strided group of the pass
// driver at a small batch.
//
// A workgroup takes 32 query rows of one head, and its four waves cut the slots between them:
// wave w walks the 32-slot blocks w, w + 4, ... through a ring of two blocks of its own in
// LDS (LDS-DMA, no barrier: a wave waits only for its own copies), and the waves' softmax
// states meet in LDS once, at the end. What bounds such a call is the longest walk, a chain
// of dependent steps (scores, maximum, weights, values) of one wave per SIMD: it is four
// times shorter here than in the 128-query tile, whose waves own rows and read every block of
// the longest row's range, and no partial state goes through memory, as with that tile's
// split ranges. K and V are read once per 32 rows, which is why larger grids keep the 128-query
// tiles. 4 sequences x 256 queries of a group of 8 over 2048 slots,
// 6/3 heads of 96 (192 workgroups): split ranges and their merge 23.7 + 4.8 us, this kernel
// 16.2 us (a third block per ring 16.5, with the next block's scores started ahead 16.6, two
// waves 26, two row tiles per wave 24.8).
#include "wm_device.hpp"
#include "wm_frag.hpp"
#include "wm_internal.hpp"

namespace wm {

struct TileArgs {
  const bf16 *Q, *Kc, *Vc, *Kd, *Vd;
  const int32_t* ctx_len;
  bf16* O;
  int B, T, L, Hq, Hkv, S_cap, mask_paper;
  int gs, gq, ctx_hi;  // query i of sequence b sits at position ctx_len[b] + gq + gs i
  int n_qtiles;        // grid: n_qtiles for each head of each (layer, sequence)
  float scale_log2;
  LayerTable chan, lord;  // lord: consumers sorted by channel
};

template <int DH> struct TileCfg {
  static constexpr int NW = 4, NT = 64 * NW, NS = 2, BKV = 32;
  static constexpr int NKS = DH / 16, NDT = DH / 32;
  static constexpr int ROW_BYTES = 2 * DH, CPR = ROW_BYTES / 16;
  static constexpr int BLK = BKV * ROW_BYTES;  // one K (or V) block of 32 slots
  static constexpr int NI = BLK / 1024;        // copy instructions per block
  static constexpr int STAGE = 2 * BLK;        // K then V
  static constexpr int RING = NS * STAGE;      // per wave
  static constexpr int OLD = DH + 4;           // row stride of the merge staging (floats)
  static_assert(32 * OLD * 4 + 256 <= RING, "the merge staging fits a wave's ring");
};

template <int DH>
__global__ __launch_bounds__(TileCfg<DH>::NT) void attend_tile_kernel(TileArgs a) {
  using C = TileCfg<DH>;
  constexpr int NW = C::NW;
  __shared__ __align__(16) char smem[NW * C::RING];
  // consecutive tiles read one K/V slice (query tiles, then grouped heads, then the channel's
  // other consumers), so an XCD's contiguous share of them keeps it in its L2
  const int tile = xcd_tile(blockIdx.x, (int)gridDim.x);
  const int qtile = a.n_qtiles - 1 - tile % a.n_qtiles;
  const int G = a.Hq / a.Hkv;
  int y = tile / a.n_qtiles;
  const int hg = y % G;
  y /= G;
  const int li = y % a.L;
  y /= a.L;
  const int kvh = y % a.Hkv, b = y / a.Hkv;
  const int hq = kvh * G + hg, l = a.lord.v[li], c = a.chan.v[l];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos0 = __builtin_amdgcn_readfirstlane(ctx_at(a.ctx_len, b, a.ctx_hi)) + a.gq;
  const int gs = a.gs, incl = a.mask_paper ? 0 : 1;
  const float cl2 = a.scale_log2;
  const int q0 = qtile * 32, qi = q0 + r, qlast = min(q0 + 32, a.T) - 1;
  const int kend = max(min(pos0 + gs * qlast + incl, a.S_cap), 0);  // slots the tile may see
  const int vis = qi < a.T ? min(pos0 + gs * qi + incl, kend) : 0;  // ... this lane's row
  const int all_vis = min(pos0 + gs * q0 + incl, kend);             // ... every row

  const int nblk = (kend + C::BKV - 1) / C::BKV;
  const int nw = (nblk - w + NW - 1) / NW;  // this wave's blocks: w, w + NW, ...
  const long cbase = (((long)c * a.B + b) * a.Hkv + kvh) * (long)a.S_cap * DH;
  // views end at the last visible slot: rows past it arrive as zeros
  const auto kview = make_view(a.Kc + cbase, (uint32_t)kend * C::ROW_BYTES);
  const auto vview = make_view(a.Vc + cbase, (uint32_t)kend * C::ROW_BYTES);
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
    const uint32_t base = j < nw ? (uint32_t)(C::BKV * (w + NW * j)) * C::ROW_BYTES : kOffOob;
#pragma unroll
    for (int n = 0; n < 2 * C::NI; ++n)
      lds_dma16(__builtin_amdgcn_readfirstlane(ring_at + st * C::STAGE + 1024 * n),
                base + coff[n % C::NI], n < C::NI ? kview : vview);
  };

  // the rows (buffer loads: rows past T are zeros), and the dummy slot, which starts the
  // first wave's state
  bf16x8 qf[C::NKS];
  const auto qv = make_view(a.Q + (((long)l * a.B + b) * a.Hq + hq) * (long)a.T * DH,
                            (uint32_t)a.T * C::ROW_BYTES);
  const bool dummy = a.mask_paper && w == 0;
  const long dof = ((long)c * a.Hkv + kvh) * DH;
  const auto kdv = make_view(dummy ? a.Kd + dof : nullptr, dummy ? C::ROW_BYTES : 0u);
  const auto vdv = make_view(dummy ? a.Vd + dof : nullptr, dummy ? C::ROW_BYTES : 0u);
  float part = 0.f;
#pragma unroll
  for (int ks = 0; ks < C::NKS; ++ks) {
    const uint32_t col = (uint32_t)(16 * ks + 8 * h) * 2u;
    qf[ks] = buf_frag<bf16>(qv, qi < a.T ? (uint32_t)qi * C::ROW_BYTES + col : kOffOob);
    const bf16x8 kd = buf_frag<bf16>(kdv, col);
#pragma unroll
    for (int i = 0; i < 8; ++i) part += (float)qf[ks][i] * (float)kd[i];
  }
  f32x16 o[C::NDT];
#pragma unroll
  for (int dt = 0; dt < C::NDT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const bf16x4 vd = __builtin_bit_cast(
          bf16x4, __builtin_amdgcn_raw_buffer_load_b64(vdv, (32 * dt + 8 * g + 4 * h) * 2u, 0, 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) o[dt][4 * g + i] = (float)vd[i];
    }
  float m = dummy ? halves_sum(part) : kNegBig, lsum = dummy && h == 0 ? 1.f : 0.f;

  const PfLane<DH> lo = pf_lane<DH>(lane);
  issue(0, 0);
  int j = 0;
  do {  // (a wave without a block walks one of zeros, every slot of it hidden)
    const int st = j & 1;
    // the stage block j-1 was read from (its reads have returned) takes block j+1
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    issue(j + 1, st ^ 1);
    wait_copies<2 * C::NI>();
    f32x16 sc = zero16();  // S^T: 32 slots by this lane's row
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks)
      sc = mma32(sc, pf_ldk<DH>(ring, lo, st * C::STAGE, ks), qf[ks]);
    const uint32_t vh = st * C::STAGE + C::BLK;
    const int at = C::BKV * (w + NW * j);  // the block's first slot
    if (at + C::BKV > all_vis) {  // some row may not read some of the block's slots
      const int base = at + 4 * h;
#pragma unroll
      for (int q = 0; q < 16; ++q)
        sc[q] = base + 8 * (q >> 2) + (q & 3) >= vis ? kNegBig : sc[q];
    }
    float mx = sc[0];
#pragma unroll
    for (int q = 1; q < 16; ++q) mx = fmaxf(mx, sc[q]);
    mx = halves_max(mx);
    if (__builtin_expect(__any(mx > m), 0)) {
      const float mn = fmaxf(m, mx), al = fast_exp2((m - mn) * cl2);
      lsum *= al;
#pragma unroll
      for (int dt = 0; dt < C::NDT; ++dt) o[dt] *= al;
      m = mn;
    }
    // hidden slots (-1e30) get weight 0, also while the row has seen none (m = -1e30)
    const float mc = m > 0.5f * kNegBig ? m * cl2 : 0.f;
    bf16x8 pf[2];
#pragma unroll
    for (int q = 0; q < 16; ++q) pf[q >> 3][q & 7] = (bf16)fast_exp2(fmaf(sc[q], cl2, -mc));
    lsum += pf_wsum(pf[0], pf[1]);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int dt = 0; dt < C::NDT; ++dt)
        o[dt] = mma32(o[dt], pf_ldv<DH>(ring, lo, vh, hf, dt), pf[hf]);
  } while (++j < nw);
  wait_copies<0>();  // no copy may land in the staging below, or after the block ends

  // merge the waves' states: each writes its rows [r][DH] and (m, l) to its own ring
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
  const float lt = halves_sum(lsum);
  if (h == 0) {
    so[32 * C::OLD + 2 * r] = m;
    so[32 * C::OLD + 2 * r + 1] = lt;
  }
  __syncthreads();
  constexpr int C4 = DH / 4;
  for (int e = tid; e < 32 * C4; e += C::NT) {
    const int row = e / C4, d4 = 4 * (e - row * C4);
    if (q0 + row >= a.T) break;  // rows only grow
    float M = kNegBig;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww)
      M = fmaxf(M, ((const float*)(smem + ww * C::RING))[32 * C::OLD + 2 * row]);
    float lw = 0.f, ow[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const float* sw = (const float*)(smem + ww * C::RING);
      const float al = fast_exp2((sw[32 * C::OLD + 2 * row] - M) * cl2);
      lw += sw[32 * C::OLD + 2 * row + 1] * al;
      const f32x4 ov = *(const f32x4*)(sw + row * C::OLD + d4);
#pragma unroll
      for (int i = 0; i < 4; ++i) ow[i] += ov[i] * al;
    }
    const float inv = 1.0f / lw;
#pragma unroll
    for (int i = 0; i < 4; ++i) ow[i] *= inv;
    store4(a.O + ((((long)l * a.B + b) * a.T + q0 + row) * a.Hq + hq) * DH + d4, ow);
  }
}

void launch_attend_tiles(const Shape& sh, const LayerTable& chan, const LayerTable& lord,
                         const bf16* Q, const bf16* Kc, const bf16* Vc, const bf16* Kd,
                         const bf16* Vd, const int32_t* ctx_len, bf16* O, hipStream_t s) {
  const TileArgs a{Q, Kc, Vc, Kd, Vd, ctx_len, O, sh.B, sh.T_new, sh.L, sh.Hq, sh.Hkv, sh.S_cap,
                   sh.mask_paper, sh.gs, sh.gq, sh.ctx_hi, (sh.T_new + 31) / 32,
                   kLog2e / sqrtf((float)sh.d), chan, lord};
  const dim3 grid((unsigned)(a.n_qtiles * sh.B * sh.L * sh.Hq));
  if (sh.d == 64)
    hipLaunchKernelGGL(attend_tile_kernel<64>, grid, dim3(TileCfg<64>::NT), 0, s, a);
  else
    hipLaunchKernelGGL(attend_tile_kernel<96>, grid, dim3(TileCfg<96>::NT), 0, s, a);
}

}  // namespace wm
