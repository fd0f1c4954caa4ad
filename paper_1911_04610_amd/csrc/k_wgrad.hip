// bf16 weight gradient on CDNA4 MFMA, operands copied from memory straight into
// LDS (16-byte chunk path).  WgradArgs (xp_kernels.h) defines what it computes;
// the general kernels in k_gemm.hip take what this one does not (see
// launch_wgrad), and add the splits' partials.
#include "xp_device.h"
#include "xp_lds.h"
#include "xp_kernels.h"

#include <cstdio>

namespace xp {

namespace {

// LDS tiles hold one row per pixel, WID (64 or 128) elements wide, without padding:
// the 16-byte chunk c of row p sits at position c ^ swz(p), which moves four
// consecutive rows (what 16 lanes of a transposing read touch) to different 64-byte
// bank groups.  swz is the same for all rows that a lane copies, and for all that it
// reads.
template <int WID>
XP_DEV int swz(int row) {
  static_assert(WID == 64 || WID == 128, "tile width");
  return WID == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2;
}

// One workgroup per BM x BN tile (output channels x reduction chunks) and pixel
// split, WM x WN waves of 32x32x16 MFMA tiles, BP pixels per step, two buffers.
// The reduction runs over pixels, which are the rows of both operands in
// memory, so the fragments (8 consecutive pixels of one column per lane) are
// read with the transposing LDS read.  GRID: strided or unpadded convolutions
// (dz lives on the Ho x Wo grid).
template <int BM, int BN, int WM, int WN, int BP, bool GRID>
__global__ __launch_bounds__(WM * WN * 64) void k_wgrad_lds(WgradArgs a, int tiles_n, int tiles_k) {
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BP % 16 == 0, "wave tile");
  constexpr int ACPR = BM / 8, ARPI = 64 / ACPR, BCPR = BN / 8, BRPI = 64 / BCPR;
  constexpr int A_T = BP / ARPI, B_T = BP / BRPI;  // copy instructions per step
  constexpr int A_I = (A_T + NW - 1) / NW, B_I = (B_T + NW - 1) / NW;
  constexpr int SZ = BP * (BM + BN);
  __shared__ __align__(16) bf16_t st0[SZ];
  __shared__ __align__(16) bf16_t st1[SZ];
  auto stage = [&](auto I) __attribute__((always_inline)) -> bf16_t* {
    if constexpr (decltype(I)::value == 0) return st0;
    else return st1;
  };

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int H = a.H, W = a.W, C = a.C, S = a.S, N = a.N;
  const int sd = GRID && a.stride > 1 ? a.stride : 1;
  const int Ho = GRID && a.Ho > 0 ? a.Ho : H, Wo = GRID && a.Ho > 0 ? a.Wo : W;
  const int M = a.nb * Ho * Wo;
  const int K = a.R * S * C;
  // the tiles of one split are neighbours on one XCD: they read the same pixels
  const int tlin = xcd_tile(blockIdx.x, gridDim.x);
  const int split = tlin / (tiles_n * tiles_k), tile = tlin - split * tiles_n * tiles_k;
  const int n0 = (tile / tiles_k) * BM, k0 = (tile % tiles_k) * BN;
  const int mps = ((M + a.splits - 1) / a.splits + BP - 1) / BP * BP;
  const int mbeg = min(split * mps, M), mend = min(M, mbeg + mps);
  const int cnt = mend - mbeg, nk = (cnt + BP - 1) / BP;

  // dz rows from the split's end on are past the resource's end and read zeros
  const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)a.dz, (short)0, mend > 0 ? (int)((((size_t)mend - 1) * a.lddz + N) * 2) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)a.x, (short)0, (int)((((size_t)a.nb * H * W - 1) * a.ldx + C) * 2), 0x00020000);

  uint32_t a_off[A_I];
#pragma unroll
  for (int i = 0; i < A_I; ++i) {
    const int row = min(wave * A_I + i, A_T - 1) * ARPI + lane / ACPR;
    const int n = n0 + ((lane % ACPR) ^ swz<BM>(row)) * 8;
    a_off[i] = n < N ? (uint32_t)((((size_t)mbeg + row) * a.lddz + n) * 2) : ~0u;
  }
  // this lane's reduction chunk: filter position and channel, the same for all
  // of its rows
  const int kk = k0 + ((lane % BCPR) ^ swz<BN>(lane / BCPR)) * 8;
  const bool kok = kk < K;
  const int krs = kok ? kk / C : 0, kch = kok ? kk - krs * C : 0;
  const int kr = krs / S - a.pad, kq = krs % S - (GRID ? a.padw : a.pad);
  // and per copy its pixel of the step: row, column, the pixel of x it starts at
  int b_row[B_I], b_h[B_I], b_w[B_I], b_pix[B_I];
#pragma unroll
  for (int i = 0; i < B_I; ++i) {
    b_row[i] = min(wave * B_I + i, B_T - 1) * BRPI + lane / BCPR;
    const int m = mbeg + b_row[i];
    const int img = m / (Ho * Wo), rem = m - img * Ho * Wo;
    b_h[i] = rem / Wo;
    b_w[i] = rem - b_h[i] * Wo;
    b_pix[i] = (img * H + b_h[i] * sd) * W + b_w[i] * sd;
  }
  const int tap = kr * W + kq;  // pixels from there to the filter position
  // one step's advance in images, rows, columns (and in pixels of x)
  const int st_i = BP / (Ho * Wo), st_r = BP - st_i * Ho * Wo, st_h = st_r / Wo, st_w = st_r - st_h * Wo;
  const int st_pix = (st_i * H + st_h * sd) * W + st_w * sd;

  int copied = 0;
  auto copy = [&](auto I) __attribute__((always_inline)) {
    bf16_t* sa = stage(I);
    bf16_t* sb = stage(I) + BP * BM;
    const int m = copied * BP;
#pragma unroll
    for (int i = 0; i < A_I; ++i)
      load_lds16(dr, sa + min(wave * A_I + i, A_T - 1) * 512, (int)a_off[i], m * a.lddz * 2);
    const bool adv = copied + 1 < nk;  // held at the last step
#pragma unroll
    for (int i = 0; i < B_I; ++i) {
      const int hh = b_h[i] * sd + kr, ww = b_w[i] * sd + kq;
      const bool ok = kok && m + b_row[i] < cnt && (unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W;
      const int off = ok ? (int)(((uint32_t)(b_pix[i] + tap) * a.ldx + kch) * 2) : -1;
      load_lds16(xr, sb + min(wave * B_I + i, B_T - 1) * 512, off, 0);
      if (adv) {
        int h = b_h[i] + st_h, w = b_w[i] + st_w, p = b_pix[i] + st_pix;
        const bool cw = w >= Wo;
        w -= cw ? Wo : 0;
        h += (int)cw;
        p += cw ? (W - Wo) * sd : 0;
        const bool ch = h >= Ho;
        h -= ch ? Ho : 0;
        p += ch ? (H - Ho * sd) * W : 0;
        b_h[i] = h;
        b_w[i] = w;
        b_pix[i] = p;
      }
    }
    copied += (int)adv;
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

  // Transposing LDS read: in each group of 16 lanes, output e (0..3) of lane i
  // is element i % 4 of the 8 bytes that lane 4 e + i / 4 of the group
  // addressed.  A 32x32x16 fragment (lane l: column l % 32, pixels 8 (l / 32) ..
  // + 8) is two such reads: lane j of a group addresses pixel 8 (l / 32) + j / 4
  // (+ 4 for the second read), columns 16 ((l % 32) / 16) + 4 (j % 4) .. + 4.
  const int px = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int cl = 16 * ((lane & 31) >> 4) + 4 * (lane & 3);
  auto frag_off = [&](int col, auto WIDTH) __attribute__((always_inline)) -> int {
    constexpr int wid = decltype(WIDTH)::value;
    const int c = col + cl;
    return px * wid + (((c >> 3) ^ swz<wid>(px)) << 3) + (c & 7);
  };
  int a_fo[TM], b_fo[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_fo[i] = frag_off(wm * WTM + i * 32, std::integral_constant<int, BM>{});
#pragma unroll
  for (int j = 0; j < TN; ++j) b_fo[j] = frag_off(wn * WTN + j * 32, std::integral_constant<int, BN>{});
  auto frag = [&](const bf16_t* p, int pitch) __attribute__((always_inline)) {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef short v8i16 __attribute__((ext_vector_type(8)));
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p));
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p + 4 * pitch));
    const v8i16 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  };
  auto multiply = [&](auto I) __attribute__((always_inline)) {
    const bf16_t* sa = stage(I);
    const bf16_t* sb = stage(I) + BP * BM;
#pragma unroll
    for (int p = 0; p < BP / 16; ++p) {
      bf16x8_t af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = frag(sa + a_fo[i] + p * 16 * BM, BM);
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = frag(sb + b_fo[j] + p * 16 * BN, BN);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
  };

  if (nk > 0) {
    copy(std::integral_constant<int, 0>{});
    int k = 0;
    while (true) {
      bool done = false;
      static_for<0, 2>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        if (!done) {
          // this wave's copies of step k have landed; past the barrier so have
          // the others', and all waves have read the buffer that is refilled
          wait_step<0>();
          copy(std::integral_constant<int, 1 - i>{});
          __builtin_amdgcn_sched_barrier(0);
          multiply(I);
          done = ++k == nk;
        }
      });
      if (done) break;
    }
    wait_step<0>();
  }

  // 32x32 result: lane l, register r holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
  float* part = (float*)a.part + (size_t)split * N * K;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int n = n0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      if (n >= N) continue;
      float* row = part + (size_t)n * K;
      if (a.direct) {
        // one split: added straight into the accumulator, as the split
        // reduction would; row n of the sibling that holds it
        float* g = a.grad;
        int q = n;
        for (int j = 0; j < a.nseg; ++j)
          if (n >= a.seg_row0[j] && n < a.seg_row0[j + 1]) {
            g = a.seg_grad[j];
            q = n - a.seg_row0[j];
          }
        row = g + (size_t)q * K;
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int k = k0 + wn * WTN + j * 32 + (lane & 31);
        if (k < K) row[k] = a.direct ? (float)((double)row[k] + (double)acc[i][j][r]) : acc[i][j][r];
      }
    }
}

template <int BM, int BN, int WM, int WN, int BP, bool GRID>
hipError_t go(const WgradArgs& a, hipStream_t s) {
  const int K = a.R * a.S * a.C;
  const int tn = (a.N + BM - 1) / BM, tk = (K + BN - 1) / BN;
  const double flops = 2.0 * a.nb * (a.Ho > 0 ? a.Ho * a.Wo : a.H * a.W) * (double)a.N * K;
  static const struct Name {
    char s[64];
    Name() { snprintf(s, sizeof s, "k_wgrad_lds<%d,%d,%d,%d,%d,%s>", BM, BN, WM, WN, BP, GRID ? "true" : "false"); }
  } name;
  WgradArgs b = a;
  b.direct = a.splits == 1;
  XP_LAUNCH(name.s, flops, (k_wgrad_lds<BM, BN, WM, WN, BP, GRID>), dim3(tn * tk * a.splits), dim3(WM * WN * 64), 0,
            s, b, tn, tk);
  return hipGetLastError();
}

// Rows of the tile, from a sweep of the stages' shapes over the same splits (us per
// launch with the split reduction, MI355X; the register-staged 64x64, 96x128 and
// 192x64 tiles before): 128x64 on eight waves for more than 64 channels from 2048
// pixels on (3x3 256->256 at 14x14x100 49.4, 64x64 60.4, 91.6 before; 3x3 512->512 at
// 7x7x100 52.3, 60.2, 123; 3x3 256->512 at 8x8x32 28.0, 30.9, 41.0; 3x3 96->96 at
// 35x35x32 32.8, 38.9, 34.3; strided 3x3 256->256 at 28x28x100 52.7, 64.9, 95.3; 1x1
// 1024->512 at 8x8x32 20.9, 21.2, 24.6), else 64x64 (3x3 64->64 at 56x56x100 68, 121;
// 3x3 512->512 at 4x4x32 17.5, 128x64 17.7, 28.8; 3x3 256->256 there 19.3, 19.8, 22.5;
// linear 2048->200 over 100 rows 8.7, 9.1, 21.5).
// 128x128 and 256x128 tiles were 2 to 20% behind, three buffers within 3%.
int tile_rows(int N, int64_t M) { return N > 64 && M >= 2048 ? 128 : 64; }

}  // namespace

// Splits of the plan's that hold pixels: their lengths are whole steps, so the last
// ones can be empty.  Where that takes a launch below a whole number of workgroups
// per CU it saves a round (us with the reduction: 3x3 96->96 at 35x35x32, 74 -> 69
// splits, 34.0 -> 32.2; 3x3 64->96, 57 -> 56, 28.0 -> 26.2; 3x3 128->128 at 28x28x32 31.0 -> 27.9).
int wgrad_lds_splits(int M, int splits) {
  const auto chain = [M](int n) { return ((M + n - 1) / n + 63) / 64 * 64; };
  const int n = (M + chain(splits) - 1) / chain(splits);
  return chain(n) == chain(splits) ? n : splits;
}

hipError_t launch_wgrad_lds(const WgradArgs& a, hipStream_t s) {
  const bool grid = a.Ho > 0 || a.pad != a.padw;
  if (tile_rows(a.N, (int64_t)a.nb * (a.Ho > 0 ? a.Ho * a.Wo : a.H * a.W)) == 128)
    return grid ? go<128, 64, 4, 2, 64, true>(a, s) : go<128, 64, 4, 2, 64, false>(a, s);
  return grid ? go<64, 64, 2, 2, 64, true>(a, s) : go<64, 64, 2, 2, 64, false>(a, s);
}

}  // namespace xp
