// bf16 implicit-GEMM convolution on CDNA4 MFMA, operands copied from memory
// straight into LDS (forward and data gradient, 16-byte chunk path).
//
// What it computes is ConvArgs' definition (xp_kernels.h); the general kernel
// in k_gemm.hip takes what this one does not, or does faster (see launch_conv_lds).
#include "xp_device.h"
#include "xp_lds.h"
#include "xp_kernels.h"

#include <cstdio>

namespace xp {

namespace {

// One workgroup per BM x BN output tile, WM x WN waves of 32x32x16 MFMA tiles.
//
// A reduction step is BK channels of one filter tap (RAG: BK consecutive
// (tap, channel) positions, a tap per 16-byte chunk).  The A tile (BM pixels'
// im2col rows) and the B tile (BN filters) of a step sit in LDS as BK-element
// rows without padding; the 16-byte chunk c of row r is stored at position
// c ^ swz(r), so that the rows one fragment read touches lie in different
// banks.  A copy instruction writes 64 consecutive chunks; the swizzle is in
// which chunk each lane asks for, and is the same for all of a lane's rows.
// NS buffers: NS - 1 steps are in flight while one is multiplied, and a wave
// waits only for its own copies of the step it needs (vmcnt), then for the
// others' at the barrier.
//
// GM 0: same grid; 1: strided or unpadded forward (rows = Ho x Wo grid);
// 2: strided data gradient.  There the rows are taken by the residue of their
// row and column modulo the stride: the pixels of one residue class meet the
// same taps, every tap that is multiplied reaches an output pixel, and a class
// that no tap reaches (1x1 stride 2) is written without a product.
//
// FEW (few tiles, a long reduction): a 32 x 32 tile whose four waves hold 16 x 16
// results each (16x16x32 MFMA), with more steps in flight; one wave finishes
// the tile.  Every element is still one chain of sums in channel order.
template <int BM, int BN, int WM, int WN, int BK, int NS, bool RAG, int GM, bool DG, bool FEW>
__global__ __launch_bounds__(FEW ? 256 : WM * WN * 64) void k_conv_gemm_lds(ConvArgs a, int tiles_m) {
  constexpr int NW = FEW ? 4 : WM * WN;
  static_assert(!FEW || (WM * WN == 1 && BM == 32 && BN == 32 && BK == 64), "four 16 x 16 waves");
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  static_assert(WTM % 32 == 0 && (WTN == 32 || WTN == 64), "wave tile");
  static_assert(BK == 32 || BK == 64, "step");
  constexpr int CPR = BK / 8;    // chunks per row
  constexpr int RPI = 64 / CPR;  // rows per copy instruction
  constexpr int A_T = BM / RPI, B_T = BN / RPI;  // copy instructions per step
  constexpr int A_I = (A_T + NW - 1) / NW, B_I = (B_T + NW - 1) / NW;  // per wave (some twice)
  constexpr int LOADS = A_I + B_I;
  constexpr int SZ = (BM + BN) * BK;
  constexpr int SZ0 = SZ > WM * WN * WTN * 32 ? SZ : WM * WN * WTN * 32;  // the epilogue's strips: 16 rows at least
  __shared__ __align__(16) bf16_t st0[SZ0];
  __shared__ __align__(16) bf16_t st1[SZ];
  __shared__ __align__(16) bf16_t st2[NS > 2 ? SZ : 8];
  __shared__ __align__(16) bf16_t st3[NS > 3 ? SZ : 8];
  __shared__ __align__(16) bf16_t st4[NS > 4 ? SZ : 8];
  __shared__ __align__(16) bf16_t st5[NS > 5 ? SZ : 8];
  __shared__ __align__(16) bf16_t st6[NS > 6 ? SZ : 8];
  __shared__ __align__(16) bf16_t st7[NS > 7 ? SZ : 8];
  __shared__ double sred[WM][2][BN];
  static_assert(NS >= 2 && NS <= 8, "stages");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool finish = !FEW || wave == 0;  // the waves of the epilogue
  // separate arrays: the compiler then knows which copies a read can meet
  auto stage = [&](auto I) __attribute__((always_inline)) -> bf16_t* {
    constexpr int i = decltype(I)::value;
    if constexpr (i == 0) return st0;
    else if constexpr (i == 1) return st1;
    else if constexpr (i == 2) return st2;
    else if constexpr (i == 3) return st3;
    else if constexpr (i == 4) return st4;
    else if constexpr (i == 5) return st5;
    else if constexpr (i == 6) return st6;
    else return st7;
  };

  const int wm = FEW ? 0 : wave / WN, wn = FEW ? 0 : wave % WN;
  const int H = a.H, W = a.W, C = a.C, S = a.S;
  const int Ho = GM ? a.Ho : H, Wo = GM ? a.Wo : W;
  const int sd = GM ? a.stride : 1;
  const int tlin = xcd_tile(blockIdx.x, gridDim.x);
  const int ntn = gridDim.x / tiles_m;
  const int tm = tlin / ntn, tn = tlin - tm * ntn;
  const int n0 = tn * BN;

  // the rows of this tile: pixel (img, h, w) of a gh x gw grid, output pixel
  // (img, oy + h * od, ox + w * od), and the taps r0 + i * rs, s0 + j * rs
  int m0 = tm * BM, gh = Ho, gw = Wo, oy = 0, ox = 0, od = 1;
  int nR = a.R, nS = S, r0 = 0, s0 = 0, rs = 1;
  if constexpr (GM == 2) {
    od = rs = sd;
    int t = tm;
    for (int p = 0; p < sd * sd; ++p) {
      oy = p / sd;
      ox = p - oy * sd;
      gh = (Ho - oy + sd - 1) / sd;
      gw = (Wo - ox + sd - 1) / sd;
      const int tiles = (a.nb * gh * gw + BM - 1) / BM;
      if (t < tiles || p == sd * sd - 1) break;
      t -= tiles;
    }
    m0 = t * BM;
    r0 = (oy + a.pad) % sd;
    s0 = (ox + a.padw) % sd;
    nR = r0 < a.R ? (a.R - r0 + sd - 1) / sd : 0;
    nS = s0 < S ? (S - s0 + sd - 1) / sd : 0;
  }
  const int M = a.nb * gh * gw;
  const int K = a.R * S * C;

  // resources: the input view, from (as many pixels before it as a tap's
  // offset is made non-negative by), and the weights
  const int back = GM == 2 ? (nR > 0 && nS > 0 ? (nR - 1) * W + nS - 1 : 0) : a.pad * W + a.padw;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const bf16_t*)a.x - (size_t)back * a.ldx), (short)0,
      (int)((((size_t)a.nb * H * W - 1 + back) * a.ldx + C) * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.w, (short)0, (int)((size_t)a.N * K * 2), 0x00020000);

  // the chunk of a row this lane copies, and per copy the row's byte offset
  // and one bit per tap row (column) that does not land in the image
  const int lrow = lane / CPR, lpos = lane % CPR;
  const int kc = BK == 64 ? lpos ^ lrow : lpos ^ ((lrow >> 1) & 3);
  uint32_t a_off[A_I], a_hb[A_I], a_wb[A_I], b_off[B_I];
#pragma unroll
  for (int i = 0; i < A_I; ++i) {
    const int m = m0 + min(wave * A_I + i, A_T - 1) * RPI + lrow;
    const int mm = m < M ? m : 0;
    const int img = mm / (gh * gw), rem = mm - img * gh * gw, h = rem / gw, w = rem - h * gw;
    uint32_t hb = ~0u, wb = ~0u;
    int bh, bw;  // first source row and column (GM 2: last)
    if constexpr (GM == 2) {
      bh = h + (oy + a.pad - r0) / sd;
      bw = w + (ox + a.padw - s0) / sd;
      for (int r = 0; r < nR; ++r) hb ^= (uint32_t)((unsigned)(bh - r) < (unsigned)H) << r;
      for (int q = 0; q < nS; ++q) wb ^= (uint32_t)((unsigned)(bw - q) < (unsigned)W) << q;
    } else {
      bh = h * sd;
      bw = w * sd;
      for (int r = 0; r < nR; ++r) hb ^= (uint32_t)((unsigned)(bh + r - a.pad) < (unsigned)H) << r;
      for (int q = 0; q < nS; ++q) wb ^= (uint32_t)((unsigned)(bw + q - a.padw) < (unsigned)W) << q;
    }
    a_off[i] = (uint32_t)((((size_t)(img * H + bh) * W + bw) * a.ldx + (RAG ? 0 : kc * 8)) * 2);
    a_hb[i] = m < M ? hb : ~0u;
    a_wb[i] = wb;
  }
#pragma unroll
  for (int i = 0; i < B_I; ++i) {
    const int n = n0 + min(wave * B_I + i, B_T - 1) * RPI + lrow;
    b_off[i] = n < a.N ? (uint32_t)(((size_t)n * K + (RAG ? 0 : kc * 8)) * 2) : ~0u;
  }

  // cursor of the next step to copy: tap (ci, cj), channel cc (RAG: of this
  // lane's chunk), held at the last step
  const int nk = RAG ? (nR * nS * C + BK - 1) / BK : nR * nS * (C / BK);
  int ci = 0, cj = 0, cc = 0, copied = 0;
  int av_r = 0, av_s = 0, av_c = 0;  // RAG: one step's advance
  if constexpr (RAG) {
    const int k0 = kc * 8, t0 = k0 / C;
    cc = k0 - t0 * C;
    ci = nS > 0 ? t0 / nS : 0;
    cj = t0 - ci * nS;
    const int t = BK / C;
    av_c = BK - t * C;
    av_r = nS > 0 ? t / nS : 0;
    av_s = t - av_r * nS;
  }
  auto copy = [&](auto I) __attribute__((always_inline)) {
    bf16_t* sa = stage(I);
    bf16_t* sb = stage(I) + BM * BK;
    const int pix = GM == 2 ? (nR - 1 - ci) * W + (nS - 1 - cj) : ci * W + cj;
    const int ka = (pix * a.ldx + cc) * 2;
    const int kb = (((r0 + ci * rs) * S + s0 + cj * rs) * C + cc) * 2;
    const int past = RAG ? (ci < nR ? 0 : -1) : 0;
#pragma unroll
    for (int i = 0; i < A_I; ++i) {
      const int bad = bit_mask(a_hb[i], ci) | bit_mask(a_wb[i], cj);
      if constexpr (RAG) load_lds16(xr, sa + min(wave * A_I + i, A_T - 1) * 512, (int)(a_off[i] + (uint32_t)ka) | bad, 0);
      else load_lds16(xr, sa + min(wave * A_I + i, A_T - 1) * 512, (int)a_off[i] | bad, ka);
    }
#pragma unroll
    for (int i = 0; i < B_I; ++i) {
      if constexpr (RAG)
        load_lds16(wr, sb + min(wave * B_I + i, B_T - 1) * 512, b_off[i] == ~0u ? -1 : (int)(b_off[i] + (uint32_t)kb) | past, 0);
      else load_lds16(wr, sb + min(wave * B_I + i, B_T - 1) * 512, (int)b_off[i], kb);
    }
    const bool adv = ++copied < nk;
    if constexpr (RAG) {
      if (adv) {
        cc += av_c;
        cj += av_s;
        ci += av_r;
        if (cc >= C) {
          cc -= C;
          ++cj;
        }
        if (cj >= nS) {
          cj -= nS;
          ++ci;
        }
      }
    } else {
      const bool wc = adv && cc + BK >= C;
      const bool wq = wc && cj + 1 == nS;
      cc = wc ? 0 : cc + (adv ? BK : 0);
      cj = wq ? 0 : cj + (int)wc;
      ci += (int)wq;
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

  f32x4_t acc4 = {0.f, 0.f, 0.f, 0.f};  // FEW

  // fragment of a 32-row, 16-deep slice: lane l holds row l % 32, elements 8 (l / 32) .. + 8
  const int frow = lane & 31, fsw = BK == 64 ? frow & 7 : (frow >> 1) & 3;
  auto multiply = [&](auto I) __attribute__((always_inline)) {
    if constexpr (FEW) {
      // 16 rows, 32 deep: lane l holds row l % 16, elements 8 (l / 16) .. + 8
      const bf16_t* sa = stage(I) + ((wave >> 1) * 16 + (lane & 15)) * BK;
      const bf16_t* sb = stage(I) + (BM + (wave & 1) * 16 + (lane & 15)) * BK;
#pragma unroll
      for (int kk = 0; kk < BK / 32; ++kk) {
        const int p = ((kk * 4 + (lane >> 4)) ^ (lane & 7)) * 8;
        const bf16x8_t af = *reinterpret_cast<const bf16x8_t*>(sa + p), bf = *reinterpret_cast<const bf16x8_t*>(sb + p);
        acc4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc4, 0, 0, 0);
      }
      return;
    }
    const bf16_t* sa = stage(I) + (wm * WTM + frow) * BK;
    const bf16_t* sb = stage(I) + (BM + wn * WTN + frow) * BK;
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int p = ((kk * 2 + (lane >> 5)) ^ fsw) * 8;
      bf16x8_t af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(sa + i * 32 * BK + p);
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = *reinterpret_cast<const bf16x8_t*>(sb + j * 32 * BK + p);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
  };

  if (nk > 0) {
    // steps are copied and multiplied U at a time, one barrier each
    constexpr int U = FEW ? 2 : 1;
    static_assert(NS % U == 0 && NS >= 2 * U, "whole groups of buffers");
    static_for<0, NS - U>([&](auto I) __attribute__((always_inline)) { copy(I); });
    int k = 0;
    while (true) {
      bool done = false;
      static_for<0, NS / U>([&](auto G) __attribute__((always_inline)) {
        constexpr int g = decltype(G)::value * U;
        if (!done) {
          // this wave's copies of these steps have landed; past the barrier so
          // have the others', and all waves have read the buffers that are refilled
          wait_step<(NS - 2 * U) * LOADS>();
          static_for<0, U>([&](auto J) __attribute__((always_inline)) {
            copy(std::integral_constant<int, (g + NS - U + decltype(J)::value) % NS>{});
          });
          __builtin_amdgcn_sched_barrier(0);  // (left to itself the compiler issues the copies last)
          static_for<0, U>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            if (j == 0 || k + j < nk) multiply(std::integral_constant<int, g + j>{});
          });
          k += U;
          done = k >= nk;
        }
      });
      if (done) break;
    }
  }
  wait_step<0>();
  if constexpr (FEW) {
    // the four results to the finishing wave, as its 32x32 result
    float* red = reinterpret_cast<float*>(st1);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      red[((wave >> 1) * 16 + 4 * (lane >> 4) + q) * 32 + (wave & 1) * 16 + (lane & 15)] = acc4[q];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = red[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)];
  }

  // ------------------------------------------------------------- epilogue
  // Each wave finishes its tile in strips of rows through its own part of LDS
  // (no barrier), with 16-byte global accesses.  Column sums (batch-norm
  // statistics of the stored values, or backward partials) are fp64, added in
  // registers over the wave's rows and then across lanes and waves in a fixed
  // order.
  constexpr int CW = WTN / 8;                         // 8-column chunks per strip row
  constexpr int SR = SZ0 >= WM * WN * WTN * 64 ? 32 : 16;  // strip rows
  constexpr int PASS = SR * CW / 64;                  // chunks per lane and strip
  constexpr int LPR = 64 / CW;                        // rows per pass
  constexpr int STRIPS = TM * 32 / SR;
  const int ch = lane % CW, n = n0 + wn * WTN + ch * 8;
  const bool live_n = n < a.N;
  bf16_t* y = (bf16_t*)a.y;
  const bf16_t* mask = (const bf16_t*)a.mask;
  // of the batch norm that column tid belongs to: 1 / deviation (0 for a bias's columns,
  // which have the first sum only, and for columns of neither, which have no sums)
  double col_rstd = 0.0;
  bool col_sum = false;
  if (DG && a.bn_part && tid < BN && n0 + tid < a.N) {
    const int c = n0 + tid;
#pragma unroll
    for (int q = 0; q < CONV_BN_SEGS; ++q)
      if (q < a.bn_nseg && c >= a.bn_c0[q] && c < a.bn_c1[q]) {
        col_sum = true;
        if (a.bn_z[q]) col_rstd = a.bn_rstd[q][c - a.bn_c0[q]];
      }
  }
  // output pixel of the lane's chunk of pass p in strip t, or -1
  auto out_row = [&](int t, int p) __attribute__((always_inline)) -> int {
    const int m = m0 + wm * WTM + t * SR + p * LPR + lane / CW;
    if (!live_n || m >= M) return -1;
    if constexpr (GM == 2) {
      const int img = m / (gh * gw), rem = m - img * gh * gw, h = rem / gw, w = rem - h * gw;
      return (img * Ho + oy + h * od) * Wo + ox + w * od;
    }
    return m;
  };
  const int n_in = live_n ? n : 0;
  // input and means of the batch norm whose output gradient these columns are (else
  // any readable chunk, whose sums are not kept)
  const bf16_t* z = (const bf16_t*)a.x;
  int ldz = 0;
  double mean[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (DG && a.bn_part && live_n) {
#pragma unroll
    for (int q = 0; q < CONV_BN_SEGS; ++q)
      if (q < a.bn_nseg && n >= a.bn_c0[q] && n < a.bn_c1[q] && a.bn_z[q]) {
        z = (const bf16_t*)a.bn_z[q] + (n - a.bn_c0[q]);
        ldz = a.ld_bnz[q];
#pragma unroll
        for (int e = 0; e < 8; ++e) mean[e] = a.bn_mean[q][n - a.bn_c0[q] + e];
      }
  }
  // a data gradient's operands in 16-byte chunks: mask, earlier contribution,
  // batch-norm input
  u32x4_t c_mask[PASS], c_old[PASS], c_z[PASS];
  int c_m[PASS];
  // loads of strip t (rows and columns past the end read the first ones: guarded
  // per lane the compiler waits for each before the next)
  auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < PASS; ++p) {
      c_m[p] = out_row(t, p);
      c_mask[p] = (u32x4_t){0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // no mask: all positive
      c_old[p] = c_z[p] = (u32x4_t){0u, 0u, 0u, 0u};
    }
    if (mask)
#pragma unroll
      for (int p = 0; p < PASS; ++p)
        c_mask[p] = *reinterpret_cast<const u32x4_t*>(mask + (size_t)max(c_m[p], 0) * a.ldm + n_in);
    if (a.accumulate)
#pragma unroll
      for (int p = 0; p < PASS; ++p)
        c_old[p] = *reinterpret_cast<const u32x4_t*>(y + (size_t)max(c_m[p], 0) * a.ldy + n_in);
    if (a.bn_part)
#pragma unroll
      for (int p = 0; p < PASS; ++p)
        c_z[p] = *reinterpret_cast<const u32x4_t*>(z + (size_t)max(c_m[p], 0) * ldz);
  };
  if constexpr (!DG) {
    // Forward: a lane holds a column of each 32x32 result (16 rows of it), so
    // bias, ReLU, the rounding and the column sums are taken there, and the
    // strip goes through LDS as bf16.
    bf16_t* ot = st0 + (FEW ? 0 : wave) * (SR * WTN);
    float bias[TN];
    double s0[TN], s1[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * WTN + j * 32 + (lane & 31);
      bias[j] = a.bias && col < a.N ? a.bias[col] : 0.f;
      s0[j] = s1[j] = 0.0;
    }
    const int rows = M - m0 - wm * WTM;  // rows of this wave's tile that exist
    const bool cut = a.bias && rows < WTM;
#pragma unroll
    for (int t = 0; t < (finish ? STRIPS : 0); ++t) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < SR / 2; r += 2) {
          // register r of the 32x32 result: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
          const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          const int q = (t * SR % 32) / 2 + r;
          float f0 = acc[t * SR / 32][j][q] + bias[j], f1 = acc[t * SR / 32][j][q + 1] + bias[j];
          if (a.relu) {
            f0 = f0 > 0.f ? f0 : 0.f;
            f1 = f1 > 0.f ? f1 : 0.f;
          }
          if (cut) {  // rows past the last hold the bias alone
            f0 = t * SR + row < rows ? f0 : 0.f;
            f1 = t * SR + row + 1 < rows ? f1 : 0.f;
          }
          const uint32_t pr = f32x2_to_bf16x2(f0, f1);
          int col = j * 32 + (lane & 31);
          if constexpr (WTN == 64) col ^= 32 * (lane >> 5);  // (row & 4): the halves' rows in different banks
          ot[row * WTN + col] = (bf16_t)pr;
          ot[(row + 1) * WTN + col] = (bf16_t)(pr >> 16);
          if (a.stat_part) {
            const double v0 = (double)__uint_as_float(pr << 16), v1 = (double)__uint_as_float(pr & 0xffff0000u);
            s0[j] += v0;
            s1[j] += v0 * v0;
            s0[j] += v1;
            s1[j] += v1 * v1;
          }
        }
#pragma unroll
      for (int p = 0; p < PASS; ++p) {
        const int row = p * LPR + lane / CW;
        int col = ch * 8;
        if constexpr (WTN == 64) col ^= (row & 4) << 3;
        const u32x4_t pr = *reinterpret_cast<const u32x4_t*>(ot + row * WTN + col);
        const int m = out_row(t, p);
        if (m >= 0) *reinterpret_cast<u32x4_t*>(y + (size_t)m * a.ldy + n) = pr;
      }
    }
    if (!a.stat_part) return;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      s0[j] += __shfl_xor(s0[j], 32, 64);
      s1[j] += __shfl_xor(s1[j], 32, 64);
      if (finish && lane < 32) {
        sred[wm][0][wn * WTN + j * 32 + lane] = s0[j];
        sred[wm][1][wn * WTN + j * 32 + lane] = s1[j];
      }
    }
  } else {
    // Data gradient: mask, earlier contribution and batch-norm input come in
    // 16-byte chunks, so the fp32 strip goes through LDS and a lane finishes
    // chunks of one chunk column.
    float* ot = reinterpret_cast<float*>(st0) + (FEW ? 0 : wave) * (SR * WTN);
    double v[16];  // column sums: of g, then of g (z - mean)
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = 0.0;
#pragma unroll
    for (int t = 0; t < (finish ? STRIPS : 0); ++t) {
      fetch(t);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < SR / 2; ++r) {
          const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          int col = j * 32 + (lane & 31);
          if constexpr (WTN == 64) col ^= 32 * (lane >> 5);
          ot[row * WTN + col] = acc[t * SR / 32][j][(t * SR % 32) / 2 + r];
        }
#pragma unroll
      for (int p = 0; p < PASS; ++p) {
        const int row = p * LPR + lane / CW;
        int col = ch * 8;
        if constexpr (WTN == 64) col ^= (row & 4) << 3;
        const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(ot + row * WTN + col);
        const f32x4_t hi = *reinterpret_cast<const f32x4_t*>(ot + row * WTN + col + 4);
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t mw = c_mask[p][e >> 1];
          const float x = e < 4 ? lo[e] : hi[e - 4];
          f[e] = __uint_as_float((e & 1) ? (mw & 0xffff0000u) : (mw << 16)) > 0.0f ? x : 0.f;
        }
        if (a.accumulate) {
          // one fp32 rounding of acc + y equals the rounding of their exact
          // double sum (53 >= 2 * 24 + 2)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t ow = c_old[p][e >> 1];
            f[e] += __uint_as_float((e & 1) ? (ow & 0xffff0000u) : (ow << 16));
          }
        }
        u32x4_t pr;
#pragma unroll
        for (int q = 0; q < 4; ++q) pr[q] = f32x2_to_bf16x2(f[2 * q], f[2 * q + 1]);
        const int m = c_m[p];
        if (m >= 0) {
          *reinterpret_cast<u32x4_t*>(y + (size_t)m * a.ldy + n) = pr;
          if (a.bn_part) {
            // the stored gradient, as what reads it sees it
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const uint32_t w = pr[e >> 1], zw = c_z[p][e >> 1];
              const double g = (double)__uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
              v[e] += g;
              v[8 + e] += g * ((double)__uint_as_float((e & 1) ? (zw & 0xffff0000u) : (zw << 16)) - mean[e]);
            }
          }
        }
      }
    }
    if (!a.bn_part) return;
    // add across the lanes of one chunk column, halving the values a lane keeps
    int idx = 0, nv = 16;
#pragma unroll
    for (int st = 32; st >= CW; st >>= 1) {
      const bool hi = (lane & st) != 0;
      nv >>= 1;
      double got[8];  // (all of a level's exchanges before its sums: one wait)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e < nv) got[e] = __shfl_xor(hi ? v[e] : v[e + nv], st, 64);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e < nv) v[e] = (hi ? v[e + nv] : v[e]) + got[e];
      idx += hi ? nv : 0;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (e < nv && finish) sred[wm][(idx + e) >> 3][wn * WTN + ch * 8 + ((idx + e) & 7)] = v[e];
  }
  __syncthreads();
  double* part = DG ? a.bn_part : a.stat_part;
  static_assert(BN <= NW * 64, "a column per thread");
  if (tid < BN && n0 + tid < a.N) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int w = 0; w < WM; ++w) {
      s0 += sred[w][0][tid];
      s1 += sred[w][1][tid];
    }
    if (DG) {
      s0 = col_sum ? s0 : 0.0;
      s1 = col_rstd != 0.0 ? s1 * col_rstd : 0.0;
    }
    part[((size_t)(n0 + tid) * 2 + 0) * tiles_m + tm] = s0;
    part[((size_t)(n0 + tid) * 2 + 1) * tiles_m + tm] = s1;
  }
}

template <int BM, int BN, int WM, int WN, int BK, int NS, bool RAG, int GM, bool DG = GM == 2, bool FEW = false>
hipError_t go(const ConvArgs& a, hipStream_t s, int* row_tiles) {
  int tiles = 0;
  if (GM == 2) {
    for (int p = 0; p < a.stride * a.stride; ++p)
      tiles += (a.nb * ((a.Ho - p / a.stride + a.stride - 1) / a.stride) *
                    ((a.Wo - p % a.stride + a.stride - 1) / a.stride) + BM - 1) / BM;
  } else {
    tiles = (a.nb * (GM ? a.Ho * a.Wo : a.H * a.W) + BM - 1) / BM;
  }
  if (row_tiles) *row_tiles = tiles;
  const double rows = GM == 1 ? (double)a.Ho * a.Wo : (double)a.H * a.W;  // (GM 2: each dy pixel meets each tap)
  const double flops = 2.0 * a.nb * rows * a.N * a.R * a.S * a.C;
  static const struct Name {
    char s[80];
    Name() {
      snprintf(s, sizeof s, "k_conv_gemm_lds<%d,%d,%d,%d,%d,%d,%s,%d,%s,%s>", BM, BN, WM, WN, BK, NS,
               RAG ? "true" : "false", GM, DG ? "true" : "false", FEW ? "true" : "false");
    }
  } name;
  XP_LAUNCH(name.s, flops, (k_conv_gemm_lds<BM, BN, WM, WN, BK, NS, RAG, GM, DG, FEW>),
            dim3(tiles * ((a.N + BN - 1) / BN)), dim3(FEW ? 256 : WM * WN * 64), 0, s, a, tiles);
  return hipGetLastError();
}

bool chunks16(const void* p, int ld) { return (reinterpret_cast<uintptr_t>(p) % 16) == 0 && ld % 8 == 0; }

int64_t tiles(int64_t rows, int bm, int cols, int bn) { return ((rows + bm - 1) / bm) * ((cols + bn - 1) / bn); }

// 128-column tiles pad N by at most an eighth more than 64-column ones
bool fits128(int N) { return 8 * ((N + 127) / 128 * 128) <= 9 * ((N + 63) / 64 * 64); }

// Tile by size, from a sweep of the stages' shapes (us per launch, MI355X):
//  - up to 32 columns 128x32 (same-grid data gradients of those do not come here), up
//    to 64 128x64 (3x3 64->64 at 56x56x100: 46.5, 64x64 tiles 52.5), 65..96 96x96
//    (3x3 64->96 at 35x35x32: 14.6; 64x128 15.5, 128x64 16.0);
//  - wider: 128x128 on eight waves while it gives 400 tiles (1x1 256->1024 at
//    14x14x100: 27.4, 64x128 30.6; below that, 3x3 256->256 there, 306 tiles:
//    41.3 against 38.1), then 64x128, then 64x64 (3x3 512->512 at 7x7x100:
//    43.8 / 39.5); 64 columns where 128 would pad by more than an eighth
//    (1x1 256->176: 15.4 against 16.8; 7x1 32->320 at 11x11x102: 10.5 / 11.5);
//  - a data gradient's epilogue (up to four tensors, fp64 sums) costs most per
//    workgroup, so it keeps the larger tiles for longer (1x1 256->1024 at
//    14x14x32, accumulated: 128x128 15.2, 64x64 31; 3x3 256->256 at 14x14x100:
//    41.4, 64x128 45.6), and over very many rows takes 256 columns in one
//    workgroup (1x1 64->256 at 56x56x100: 131, 128x128 150).
// Two buffers: a third or fourth lost more workgroups per CU than it hid.
template <bool RAG, int GM, bool DG>
hipError_t pick_tile(const ConvArgs& a, int64_t rows, hipStream_t s, int* row_tiles) {
  if constexpr (!DG || GM == 2)
    if (a.N <= 32) return go<128, 32, 4, 1, 64, 2, RAG, GM, DG>(a, s, row_tiles);
  if (a.N > 96 && fits128(a.N)) {
    if constexpr (DG && GM == 0)
      if (a.N % 256 == 0 && tiles(rows, 256, a.N, 256) >= 1024)
        return go<256, 256, 2, 4, 64, 2, RAG, GM, DG>(a, s, row_tiles);
    if (tiles(rows, 128, a.N, 128) >= (DG ? 192 : 400))
      return go<128, 128, 4, 2, 64, 2, RAG, GM, DG>(a, s, row_tiles);
    if (tiles(rows, 64, a.N, 128) >= (DG ? 192 : 400))
      return go<64, 128, 2, 2, 64, 2, RAG, GM, DG>(a, s, row_tiles);
  } else if (tiles(rows, 128, a.N, 64) >= (DG ? 256 : 512)) {
    if (a.N > 64 && a.N <= 96) return go<96, 96, 1, 3, 32, 3, RAG, GM, DG>(a, s, row_tiles);
    return go<128, 64, 4, 2, 64, 2, RAG, GM, DG>(a, s, row_tiles);
  }
  return go<64, 64, 2, 2, 64, 2, RAG, GM, DG>(a, s, row_tiles);
}

template <int GM, bool DG>
hipError_t pick_step(const ConvArgs& a, int64_t rows, hipStream_t s, int* row_tiles) {
  // (the 96x96 tile steps by 32 channels)
  const int bk = a.N > 64 && a.N <= 96 && tiles(rows, 128, a.N, 64) >= (DG ? 256 : 512) ? 32 : 64;
  return a.C % bk == 0 ? pick_tile<false, GM, DG>(a, rows, s, row_tiles)
                       : pick_tile<true, GM, DG>(a, rows, s, row_tiles);
}

// Few tiles: 32x32, four buffers, or eight where the reduction is so long that
// its operands' path is the limit (us per launch, general kernel's 32x64 tiles
// before: 3x3 512->512 at 4x4x32 16.1 with eight and 20.5 with four, 20.6; 3x3 128->128
// at 8x8x32 6.8, 8.0; 7x1 160->192 at 12x12x4 7.3, 13.1; 1x1 352->128 at 14x14x12
// 5.6, 7.2; linear 2048->200 over 100 rows 8.7, 10.8; 3x3 stride 2 256->256 at
// 28x28x8 12.0, 22.0).  One chain of sums per element keeps the stored bits of
// the other tiles; the reduction split over eight waves took 12.1 us on the
// first of these, but other bits flip ReLU and pool decisions downstream.
template <int GM, bool DG>
hipError_t few(const ConvArgs& a, hipStream_t s, int* row_tiles) {
  if (a.C % 64 != 0) return go<32, 32, 1, 1, 64, 4, true, GM, DG, true>(a, s, row_tiles);
  if constexpr (!DG)  // (a data gradient comes here from 4096 products on)
    if ((int64_t)a.R * a.S * a.C < 4096) return go<32, 32, 1, 1, 64, 4, false, GM, DG, true>(a, s, row_tiles);
  return go<32, 32, 1, 1, 64, 8, false, GM, DG, true>(a, s, row_tiles);
}

}  // namespace

bool launch_conv_lds(const ConvArgs& a, hipStream_t s, int* row_tiles, hipError_t* e) {
  const int stride = a.stride < 1 ? 1 : a.stride;
  const bool dg = a.tr || a.mask || a.accumulate || a.bn_part;
  const bool grid = a.Ho > 0;
  const int64_t rows = (int64_t)a.nb * (grid ? a.Ho * a.Wo : a.H * a.W);
  // what the kernel is written for: 16-byte chunks of every view, byte offsets
  // of 31 bits from the first tap on, whole chunks of columns per batch norm,
  // bias and ReLU forward, mask and accumulation backward
  bool fits = a.C % 8 == 0 && a.N % 8 == 0 && chunks16(a.x, a.ldx) && chunks16(a.y, a.ldy) && chunks16(a.w, 8) &&
              (!a.mask || chunks16(a.mask, a.ldm)) && !(dg && (a.bias || a.relu || a.stat_part)) &&
              (grid || (!a.tr && stride == 1));
  const int64_t pixels = (int64_t)a.nb * a.H * a.W + (int64_t)a.R * a.W + a.S;
  fits = fits && pixels * a.ldx * 2 < ((int64_t)1 << 31) && (int64_t)a.N * a.R * a.S * a.C * 2 < ((int64_t)1 << 31);
  if (a.bn_part)
    for (int k = 0; k < a.bn_nseg; ++k)
      fits = fits && a.bn_c0[k] % 8 == 0 && a.bn_c1[k] % 8 == 0 && (!a.bn_z[k] || chunks16(a.bn_z[k], a.ld_bnz[k]));
  // the residue classes' last tiles stay within conv_max_row_tiles
  fits = fits && (!a.tr || rows >= 256);
  if (!fits || (grid && dg && !a.tr)) return false;
  ConvArgs b = a;
  b.stride = stride;
  // Which calls the general kernel does faster, from a sweep of 1x1 to 5x5, strided and
  // unpadded layers over 8 to 512 columns, reductions of 8 to 12800 and 512 to 100 352
  // rows (us per launch, general kernel / here; a data gradient with mask and
  // batch-norm partials).  Both form the same sums.
  const int64_t K = (int64_t)a.R * a.S * a.C;
  const int cols = a.N <= 32 ? 32 : 64;
  const bool w96 = a.N > 64 && a.N <= 96, tile128 = a.N > 96 && fits128(a.N) && tiles(rows, 128, a.N, 128) >= 192;
  const int64_t t64 = tiles(rows, 64, a.N, cols);
  if (a.tr) {
    // The residue classes leave a product a quarter of the steps, so a short one is all
    // epilogue: 1x1 stride 2, 32 columns of 16 at 12 544 rows 7.8 / 11.2, 64 of 128 10.5 /
    // 11.5, 128 of 64 at 19 600 rows 13.3 / 16.0; from 512 on 0.6 to 0.9 of its time, 32
    // columns from 1025 on 0.5 to 0.8.
    if (a.N <= 32 ? K <= 1024 : K <= 256 && (!tile128 || K <= 32)) return false;
  } else if (dg) {
    // A data gradient's epilogue counts for more than the loop where the reduction is
    // short, or 32-row tiles spread it better: 32 columns of 64 at 50 176 rows 10.1 / 13.7,
    // of 4608 at 12 544 rows 26.5 / 40.8; 96 of 32 at 25 088 rows 12.3 / 16.3.  Its 64x96
    // tile takes 3x3 filters (96 of 576 at 25 088 rows 19.3 / 22.0), not 1x1 or 5x5 ones
    // (96 of 512 0.55 to 0.87 of its time here, 96 of 2400 0.7).
    if (K < 64 || (K < 128 && a.C % 64 != 0) || a.N <= 32) return false;
    const int taps = a.R * a.S;
    if (a.N > 96 ? tiles(rows, 128, a.N, 128) >= 192 : tiles(rows, 128, a.N, 64) >= 256) {
      if (w96 && K < (taps == 1 || taps >= 25 ? 256 : 1024)) return false;
    } else if (a.N > 96 && K >= 1024 && tiles(rows, 64, a.N, 128) >= 192) {
      // (1x1 1024->256 at 14x14x32: 20.0 / 15.0)
    } else if (K >= 2048 && t64 >= (w96 ? 192 : 256)) {
      // (64 of 2304, 196 tiles 20.8 / 25.7; 307 tiles 0.96, 452 0.78 of its time)
    } else if (K >= 4096 && t64 <= (w96 ? 192 : 64)) {
      // (3x3 512->512 at 4x4x32: 21.5 / 19.4; 128 of 4608, 154 tiles 30 / 40)
      *e = few<0, true>(b, s, row_tiles);
      return true;
    } else {
      return false;  // (1x1 256->512 at 14x14x16: 9.2 / 9.8; 3x3 64->64 at 28x28x16: 8.4 / 10.1)
    }
  } else if (t64 < 192 && (K > 256 || t64 < 96)) {
    // fewer 64x64 tiles than CUs (two or four steps: not far fewer, 1x1 128->512
    // over 1000 rows, 128 tiles: 4.5 against 4.8 us)
    if (grid) *e = few<1, false>(b, s, row_tiles);
    else *e = few<0, false>(b, s, row_tiles);
    return true;
  } else if (a.N <= 32) {
    // one column tile, so rows / 128 workgroups: below one per CU the smaller tiles are
    // better (3x3 256->32 at 14 700 rows 15.6 / 21.5, few's 14.2); a short reduction hides
    // less (1x1 32->32 at 100 352 rows 9.1 / 11.1); and where the input exceeds the L2s'
    // 32 MB its rows come from further away for every filter tap (3x3 256->32 there 54 /
    // 77, 128->32 0.85 of its time)
    if (K <= 288 || (!grid && a.C > 128 && rows * a.C > 18000000)) return false;
    if (!grid && rows < 24576) {
      *e = few<0, false>(b, s, row_tiles);
      return true;
    }
  } else if ((K <= 32 && !(w96 && tiles(rows, 128, a.N, 64) >= 512)) || (K >= 3584 && !grid && t64 < 256)) {
    // a step of mostly zeros (1x1 32->256 at 12 544 rows 7.8 / 9.0); 192 to 255 tiles of
    // long chains (3x3 512->64 at 12 544 rows 30 / 36)
    return false;
  }
  if (a.tr) *e = pick_step<2, true>(b, rows, s, row_tiles);
  else if (grid) *e = pick_step<1, false>(b, rows, s, row_tiles);
  else if (dg) *e = pick_step<0, true>(b, rows, s, row_tiles);
  else *e = pick_step<0, false>(b, rows, s, row_tiles);
  return true;
}

}  // namespace xp
