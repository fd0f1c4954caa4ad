// bf16 convolutions of images (three channels: the networks' first layers), and
// weight gradients of small filters over channel counts that are no multiple of 8,
// on CDNA4 MFMA.
//
// A filter row's S x C values are one run of the NHWC row, so a workgroup stages
// the input rows of several output rows in LDS (zeros around the image) and takes
// its operands from there value by value: no index arithmetic and no 2-byte load
// from memory per value, which bound the general kernels.  Bound now: one 2-byte
// LDS read per operand value and the epilogue's fp64 sums, at two waves per SIMD (7x7
// stride 2 on 224x224x3, 64 channels, micro-batch 100, before / after: forward 409 /
// 88 us, weight gradient with its reduction 560 / 85 us; the memory floor of either is
// about 35 us).  The weight gradient's sums differ from the general kernel's in order:
// eight waves' chains per workgroup, each a fraction as long (there 3.7e-7 / 1.5e-7 of
// the gradient off 64-bit sums, over smaller maps 6.5e-8 / 5.5e-8).
#include "xp_device.h"
#include "xp_lds.h"
#include "xp_kernels.h"

#include <algorithm>
#include <atomic>
#include <cstdio>

namespace xp {

namespace {

constexpr int CONV_LDS = 80 * 1024;           // bytes: two workgroups per CU
constexpr int WGRAD_ROWS = 80 * 1024 / 2;     // values of input rows (one workgroup per CU)

// Copies rows r0 .. r0 + rows of an image (its first value at x; WC values per row)
// to LDS, row i at sx[i * pitch + lead]; rows outside the image become zeros.
// Rows of whole 16-byte chunks are copied straight into LDS and have landed after
// the caller's vmcnt(0) and barrier; others go through registers.
XP_DEV void stage_rows(const bf16_t* x, int H, int WC, int r0, int rows, int lead, int pitch, bf16_t* sx, int tid,
                       int nt) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (WC % 8 == 0 && (reinterpret_cast<uintptr_t>(x) % 16) == 0) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)x, (short)0, H * WC * 2, 0x00020000);
    for (int i = wave; i < rows; i += nt / 64) {
      const int h = r0 + i;
      for (int c = 0; c < WC; c += 512)
        if (c + lane * 8 < WC)
          load_lds16(r, sx + i * pitch + lead + c, (unsigned)h < (unsigned)H ? (h * WC + c + lane * 8) * 2 : -1, 0);
    }
    return;
  }
  for (int i = wave; i < rows; i += nt / 64) {
    const int h = r0 + i;
    const bool in = (unsigned)h < (unsigned)H;
    const bf16_t* row = x + (in ? (size_t)h * WC : 0);
    for (int c = lane; c < WC; c += 8 * 64) {
      bf16_t v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = row[min(c + e * 64, WC - 1)];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (c + e * 64 < WC) sx[i * pitch + lead + c + e * 64] = in ? v[e] : (bf16_t)0;
    }
  }
}

// this wave's vector memory operations and LDS accesses are done; then the workgroup's
XP_DEV void wait_all() { wait_step<0>(); }

// Forward.  R x R filter over three channels.  A workgroup keeps the weights of 64
// channels in registers and walks units of rb output rows of one image; its four
// waves take 32-pixel pieces of the rows in turn.  The reduction runs over
// k = (r, s, c) in steps of 16 without padding, as in the general kernel, so the
// sums are the same bit for bit.
template <int R>
__global__ __launch_bounds__(256, 2) void k_conv_gemm_image(ConvArgs a, int rb, int lead, int pitch, int row_blocks) {
  constexpr int C = 3, RUN = C * R, K = R * RUN, SL = (K + 15) / 16;  // a filter row's values; all; 16-deep slices
  constexpr int BP = (SL | 1) * 16 + 8;                               // weight row pitch: an odd number of 16-byte chunks
  extern __shared__ __align__(16) bf16_t smem[];
  bf16_t* so = smem;                // per wave a [32][64] strip
  bf16_t* sx = smem + 4 * 32 * 64;  // input rows; first the weights
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, n0 = blockIdx.y * 64;
  const int Ho = a.Ho > 0 ? a.Ho : a.H, Wo = a.Ho > 0 ? a.Wo : a.W, sd = a.Ho > 0 ? a.stride : 1;
  const bf16_t* w = (const bf16_t*)a.w;
#pragma unroll
  for (int i = 0; i < 64 * SL * 16 / 256; ++i) {
    const int q = i * 256 + tid, n = q / (SL * 16), k = q - n * (SL * 16);
    const bool in = n0 + n < a.N && k < K;
    const bf16_t v = w[in ? (size_t)(n0 + n) * K + k : 0];
    sx[n * BP + k] = in ? v : (bf16_t)0;
  }
  __syncthreads();
  bf16x8_t wf[SL][2];
#pragma unroll
  for (int s = 0; s < SL; ++s)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wf[s][j] = *reinterpret_cast<const bf16x8_t*>(sx + (j * 32 + (lane & 31)) * BP + s * 16 + half * 8);
  __syncthreads();
  for (int q = tid; q < ((rb - 1) * sd + R) * pitch; q += 256) sx[q] = 0;  // (what lies around the rows stays so)

  float bias[2];
  double s0[2] = {0.0, 0.0}, s1[2] = {0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = n0 + j * 32 + (lane & 31);
    bias[j] = a.bias && col < a.N ? a.bias[col] : 0.f;
  }
  bf16_t* y = (bf16_t*)a.y;
  bf16_t* ot = so + wave * (32 * 64);
  const int pieces = (Wo + 31) / 32, step = sd * C, units = a.nb * row_blocks;
  // A fragment is read value by value: wider LDS reads stall where they are not
  // aligned to their size, and a filter row starts at any value.  The compiler may
  // not see that odd values follow even ones, or it joins their reads.
  int one = 1;
  asm("" : "+v"(one));
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const int img = u / row_blocks, ho0 = (u - img * row_blocks) * rb, nrow = min(rb, Ho - ho0);
    __syncthreads();
    stage_rows((const bf16_t*)a.x + (size_t)img * a.H * a.W * C, a.H, a.W * C, ho0 * sd - a.pad, (nrow - 1) * sd + R, lead,
               pitch, sx, tid, 256);
    wait_all();
    for (int pc = wave; pc < nrow * pieces; pc += 4) {
      const int ro = pc / pieces, p0 = (pc - ro * pieces) * 32;
      // lane l: pixel p0 + l % 32, values k + 8 (l / 32) .. + 8 of a slice.  Value k lies
      // in row k / RUN; k + 8 in that row (`same`) or the next one (`next`).
      const bf16_t* same = sx + ro * sd * pitch + lead - a.padw * C + (p0 + (lane & 31)) * step + 8 * half;
      const bf16_t* next = same + half * (pitch - RUN);
      const bf16_t *same1 = same + one, *next1 = next + one;
      f32x16_t acc[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
#pragma unroll
      for (int s = 0; s < SL; ++s) {
        typedef short v8i16 __attribute__((ext_vector_type(8)));
        v8i16 f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // (values past the last one are zeroed, also against infinities)
          const int k = s * 16 + e, row = k / RUN, col = k - row * RUN;
          const bool wraps = col + 8 >= RUN && k + 8 < K;
          const bf16_t* p = e & 1 ? (wraps ? next1 : same1) - 1 : wraps ? next : same;
          f[e] = k < K ? (short)p[row * pitch + col] : (short)0;
          if (k < K && k + 8 >= K) f[e] = half ? (short)0 : f[e];
        }
        const bf16x8_t af = __builtin_bit_cast(bf16x8_t, f);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, wf[s][j], acc[j], 0, 0, 0);
        }
      }
      // bias, ReLU, rounding and column sums in the result's layout (register r:
      // pixel 8 (r / 4) + 4 (l / 32) + r % 4, channel l % 32), then through LDS to
      // 16-byte stores
      const int live = Wo - p0;  // pixels of this piece that exist
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] += bias[j];
      if (a.relu) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[j][r] = acc[j][r] > 0.f ? acc[j][r] : 0.f;
      }
      if (live < 32) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[j][r] = 8 * (r >> 2) + 4 * half + (r & 3) < live ? acc[j][r] : 0.f;
      }
      uint32_t pr[2][8];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int row = 8 * (r >> 2) + 4 * half + (r & 3);
          const int col = (j * 32 + (lane & 31)) ^ (32 * half);  // (row & 4): the halves' rows in different banks
          pr[j][r >> 1] = f32x2_to_bf16x2(acc[j][r], acc[j][r + 1]);
          ot[row * 64 + col] = (bf16_t)pr[j][r >> 1];
          ot[(row + 1) * 64 + col] = (bf16_t)(pr[j][r >> 1] >> 16);
        }
      if (a.stat_part) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const double v0 = (double)__uint_as_float(pr[j][r] << 16), v1 = (double)__uint_as_float(pr[j][r] & 0xffff0000u);
            s0[j] += v0;
            s1[j] += v0 * v0;
            s0[j] += v1;
            s1[j] += v1 * v1;
          }
      }
      const size_t m0 = ((size_t)img * Ho + ho0 + ro) * Wo + p0;
      const int ch = lane & 7, n = n0 + ch * 8;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = p * 8 + (lane >> 3);
        const u32x4_t pr = *reinterpret_cast<const u32x4_t*>(ot + row * 64 + ((ch * 8) ^ ((row & 4) << 3)));
        if (row < live && n < a.N) *reinterpret_cast<u32x4_t*>(y + (m0 + row) * a.ldy + n) = pr;
      }
    }
  }
  if (!a.stat_part) return;
  __syncthreads();
  double* sred = reinterpret_cast<double*>(smem);  // [wave][sum][channel]
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    s0[j] += __shfl_xor(s0[j], 32, 64);
    s1[j] += __shfl_xor(s1[j], 32, 64);
    if (lane < 32) {
      sred[(wave * 2 + 0) * 64 + j * 32 + lane] = s0[j];
      sred[(wave * 2 + 1) * 64 + j * 32 + lane] = s1[j];
    }
  }
  __syncthreads();
  if (tid < 128) {
    const int which = tid >> 6, col = tid & 63;
    if (n0 + col < a.N)
      a.stat_part[((size_t)(n0 + col) * 2 + which) * gridDim.x + blockIdx.x] =
          ((sred[tid] + sred[128 + tid]) + sred[256 + tid]) + sred[384 + tid];
  }
}

// Weight gradient.  A workgroup (a split) walks units of rb output rows and
// keeps the whole 64-channel x R*S*C tile (KT 32-column MFMA tiles) in each of
// its eight waves' accumulators; a wave takes every eighth group of 16 pixels of
// a unit, whose dz rows are copied straight into LDS three groups ahead.  The
// waves' tiles are added in a fixed order at the end.
template <int KT>
__global__ __launch_bounds__(512) void k_wgrad_image(WgradArgs a, int rb, int lead, int pitch, int row_blocks) {
  // (arrays of their own, so that a read waits for no other buffer's copies)
  __shared__ __align__(16) bf16_t z0[8 * 16 * 64], z1[8 * 16 * 64], z2[8 * 16 * 64], z3[8 * 16 * 64];
  __shared__ __align__(16) bf16_t sx[WGRAD_ROWS];  // input rows; at the end two tiles (fp32)
  static_assert(sizeof sx >= 2 * (size_t)2 * KT * 16 * 64 * 4, "two tiles");
  const auto slot = [&](auto I) -> bf16_t* {
    constexpr int i = decltype(I)::value % 4;
    if constexpr (i == 0) return z0;
    else if constexpr (i == 1) return z1;
    else if constexpr (i == 2) return z2;
    else return z3;
  };
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = a.C, S = a.S, R = a.R, K = R * S * C, N = a.N;
  const int Ho = a.Ho > 0 ? a.Ho : a.H, Wo = a.Ho > 0 ? a.Wo : a.W, sd = a.Ho > 0 ? a.stride : 1;
  const int n0 = blockIdx.y * 64;
  const int units = a.nb * row_blocks, groups_w = (Wo + 15) / 16, step = sd * C;
  for (int q = tid; q < ((rb - 1) * sd + R) * pitch; q += 512) sx[q] = 0;  // (what lies around the rows stays so)

  // the copies of dz, three groups ahead of the products: a group's 16 pixels
  // (zeros past the row and past N) as rows of swizzled 16-byte chunks
  const int zr = lane >> 3, zn = n0 + ((lane & 7) ^ (((zr >> 1) & 1) << 2)) * 8;  // (the same in row zr + 8)
  int cu = blockIdx.x, cg = wave, cn = 0;
  __amdgpu_buffer_rsrc_t cr = __builtin_amdgcn_make_buffer_rsrc((void*)a.dz, (short)0, 0, 0x00020000);
  int cpix = 0;  // first pixel of the unit in its image
  const auto copy_unit = [&]() __attribute__((always_inline)) {
    const int img = cu / row_blocks, h = (cu - img * row_blocks) * rb;
    cn = min(rb, Ho - h) * groups_w;
    cpix = h * Wo;
    cr = __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16_t*)a.dz + (size_t)img * Ho * Wo * a.lddz), (short)0,
                                           ((Ho * Wo - 1) * a.lddz + N) * 2, 0x00020000);
  };
  if (cu < units) copy_unit();
  const auto copy = [&](auto I) __attribute__((always_inline)) {
    while (cu < units && cg >= cn) {
      cu += a.splits;
      cg = wave;
      if (cu < units) copy_unit();
    }
    const int ro = cg / groups_w, p0 = (cg - ro * groups_w) * 16;
    bf16_t* z = slot(I) + wave * (16 * 64);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int p = p0 + i * 8 + zr;
      load_lds16(cr, z + i * 512, cu < units && p < Wo && zn < N ? ((cpix + ro * Wo + p) * a.lddz + zn) * 2 : -1, 0);
    }
    cg += 8;
  };

  // lane's column of each tile: filter row and place in its run
  int koff[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const int k = min(t * 32 + (lane & 31), K - 1);  // (columns past the last are not stored)
    koff[t] = k / (S * C) * pitch + k % (S * C);
  }
  f32x16_t acc[2][KT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][t][q] = 0.f;
  // the transposing read: lane i of 16 addresses pixel i / 4, channels 4 (i % 4) .. + 4
  const int px = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int cl = 16 * ((lane & 31) >> 4) + 4 * (lane & 3);
  const int swz = ((px >> 1) & 1) << 2;  // of px + 4 too
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef short v8i16 __attribute__((ext_vector_type(8)));
  const auto multiply = [&](auto I, int g) __attribute__((always_inline)) {
    const bf16_t* z = slot(I) + wave * (16 * 64);
    const int ro = g / groups_w, p0 = (g - ro * groups_w) * 16;
    // x of pixels 8 (l / 32) .. + 8 at the lane's column
    const bf16_t* xp = sx + ro * sd * pitch + lead - a.padw * C + (p0 + 8 * (lane >> 5)) * step;
    v8i16 xv[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[t][e] = (short)xp[koff[t] + e * step];
    // (pixels past the row have dz = 0; their x is zeroed too, against infinities)
    if (p0 + 16 > Wo) {
      const int left = Wo - p0 - 8 * (lane >> 5);
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[t][e] = e < left ? xv[t][e] : (short)0;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = i * 32 + cl;
      const bf16_t* p = z + px * 64 + (((c >> 3) ^ swz) << 3) + (c & 7);
      const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p));
      const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p + 4 * 64));
      const bf16x8_t af = __builtin_bit_cast(bf16x8_t, (v8i16)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int t = 0; t < KT; ++t)
        acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, __builtin_bit_cast(bf16x8_t, xv[t]), acc[i][t], 0, 0, 0);
    }
  };

  int u = blockIdx.x, g = wave, n = 0;
  const auto unit = [&]() __attribute__((always_inline)) {
    const int img = u / row_blocks, h = (u - img * row_blocks) * rb, nrow = min(rb, Ho - h);
    n = nrow * groups_w;
    __syncthreads();  // every wave has read the last unit's rows
    stage_rows((const bf16_t*)a.x + (size_t)img * a.H * a.W * C, a.H, a.W * C, h * sd - a.pad, (nrow - 1) * sd + R, lead,
               pitch, sx, tid, 512);
    wait_all();
  };
  if (u < units) {
    static_for<0, 3>([&](auto I) __attribute__((always_inline)) { copy(I); });
    unit();
    bool done = false;
    while (!done)
      static_for<0, 4>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        while (!done && g >= n) {  // (every wave passes every unit's barriers)
          u += a.splits;
          g = wave;
          done = u >= units;
          if (!done) unit();
        }
        if (!done) {
          asm volatile("" ::: "memory");
          __builtin_amdgcn_s_waitcnt(0xc07f);  // the reads of the slot to be filled have returned
          asm volatile("" ::: "memory");
          copy(std::integral_constant<int, i + 3>{});
          asm volatile("" ::: "memory");
          __builtin_amdgcn_s_waitcnt(0x0f70 | 6);  // this group's copies have landed: the three later groups' are left
          asm volatile("" ::: "memory");
          multiply(I, g);
          g += 8;
        }
      });
  }
  // the waves' tiles: the even and the odd waves' in wave order, then both
  constexpr int TILE = 2 * KT * 16 * 64;
  float* red = reinterpret_cast<float*>(sx);
  wait_all();
  for (int w = 0; w < 4; ++w) {
    if (wave >> 1 == w) {
      float* p = red + (wave & 1) * TILE + lane;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            float* o = p + ((i * KT + t) * 16 + q) * 64;
            *o = w == 0 ? acc[i][t][q] : *o + acc[i][t][q];
          }
    }
    __syncthreads();
  }
  float* part = (float*)a.part + (size_t)blockIdx.x * N * K;
  for (int o = tid; o < TILE; o += 512) {
    const int l = o & 63, q = (o >> 6) & 15, it = o >> 10, i = it / KT, t = it - i * KT;
    const int nn = n0 + i * 32 + 8 * (q >> 2) + 4 * (l >> 5) + (q & 3), k = t * 32 + (l & 31);
    if (nn < N && k < K) part[(size_t)nn * K + k] = red[o] + red[TILE + o];
  }
}

// Where rows lie in LDS: the first value of row i at i * pitch + lead (lead: whole
// 16-byte chunks that hold the zeros before it); reads go up to `past` values from
// the last pixel of the last `piece`-pixel piece on
struct Rows {
  int lead, pitch;
  Rows(int Wo, int piece, int step, int past, int zeros, int WC) {
    lead = (zeros + 7) / 8 * 8;
    const int end = lead - zeros + ((Wo + piece - 1) / piece * piece - 1) * step + past;
    pitch = (std::max(end, lead + WC) + 7) / 8 * 8;
  }
};

// Output rows per unit: the count that a workgroup's share of the units takes the
// least time with (its rows, and `idle` rows' time while a unit's input arrives),
// of those whose `most` input rows' values fit
int unit_rows(int64_t images, int Ho, int groups, int idle, int sd, int R, int pitch, int most) {
  int best = 0;
  int64_t cost = 0;
  for (int rb = 1; rb <= Ho && (int64_t)((rb - 1) * sd + R) * pitch <= most; ++rb) {
    const int64_t c = (images * ((Ho + rb - 1) / rb) + groups - 1) / groups * (rb + idle);
    if (best == 0 || c < cost) {
      best = rb;
      cost = c;
    }
  }
  return best;
}

// Maps that the kernels are for: of `least` output pixels or more, in rows of 8 or
// more.  A workgroup stages each image by itself and waits for it, and computes whole
// 16- or 32-pixel pieces of rows.  us per launch, general kernels / these: forward 3x3
// 3->64, 64 images, of 2x2 10.3 / 31, 6x6 11.1 / 15.1, 10x10 11.0 / 11.9, 12x12 10.9 / 10.4,
// 16x16 11.2 / 8.5, 4 images of 200x4 11.1 / 12.3, and 3->32, whose general tile pads
// less, of 12x12 9.7 / 10.2, 15x16 10.1 / 8.8; weight gradients with their reduction, 32
// images, of 1x1 100->200 at 1x1 17 / 71, 4x4 27 / 30, 3x3 12->64 at 7x7 24.5 / 26.9, 3x3
// 3->64 at 8x8 22.2 / 16.0, and of more than 96 products, five tiles a wave, 5x5 6->64 at
// 11x11 24.3 / 27.1, at 16x16 25.5 / 21.4.
bool fits_map(int Ho, int Wo, int least) { return Wo >= 8 && (int64_t)Ho * Wo >= least; }
constexpr int CONV_MAP = 144, CONV_MAP_NARROW = 240, WGRAD_MAP = 64, WGRAD_MAP_WIDE = 144;

template <int R>
hipError_t conv_go(const ConvArgs& a, int groups, int rb, const Rows& l, int row_blocks, size_t lds, hipStream_t s) {
  static const struct Name {
    char s[64];
    Name() { snprintf(s, sizeof s, "k_conv_gemm_image<%d>", R); }
  } name;
  const double rows = a.Ho > 0 ? (double)a.Ho * a.Wo : (double)a.H * a.W;
  const auto kernel = k_conv_gemm_image<R>;
  // the LDS above the default limit, allowed once per device (two threads may both ask)
  static std::atomic<uint64_t> allowed{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (!(allowed.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, CONV_LDS);
    if (e != hipSuccess) return e;
    allowed.fetch_or(bit, std::memory_order_release);
  }
  XP_LAUNCH(name.s, 2.0 * a.nb * rows * a.N * a.R * a.S * a.C, kernel, dim3(groups, (a.N + 63) / 64), dim3(256), lds,
            s, a, rb, l.lead, l.pitch, row_blocks);
  return hipGetLastError();
}

}  // namespace

bool launch_conv_image(const ConvArgs& a, hipStream_t s, int* row_tiles, hipError_t* e) {
  const int Ho = a.Ho > 0 ? a.Ho : a.H, Wo = a.Ho > 0 ? a.Wo : a.W, sd = a.Ho > 0 ? a.stride : 1;
  // forward, square filters, images without row gaps, 16-byte chunks of the output
  if (!fits_map(Ho, Wo, a.N <= 32 ? CONV_MAP_NARROW : CONV_MAP)) return false;
  if (a.C != 3 || a.R != a.S || (a.R != 3 && a.R != 5 && a.R != 7) || a.ldx != 3 || a.tr || a.mask || a.accumulate ||
      a.bn_part || a.N % 8 != 0 || a.ldy % 8 != 0 || (reinterpret_cast<uintptr_t>(a.y) % 16) != 0)
    return false;
  const Rows l(Wo, 32, sd * 3, 3 * a.R + 8, a.padw * 3, a.W * 3);
  const int ny = (a.N + 63) / 64, strips = 4 * 32 * 64, weights = 64 * (((a.R * a.R * 3 + 15) / 16 | 1) * 16 + 8);
  const int rb = unit_rows(a.nb, Ho, std::max(1, 512 / ny), 1, sd, a.R, l.pitch, CONV_LDS / 2 - strips);
  if (rb == 0 || (int64_t)a.H * a.W * 3 >= (1 << 30)) return false;
  const int row_blocks = (Ho + rb - 1) / rb;
  const int64_t units = (int64_t)a.nb * row_blocks;
  const int groups = (int)std::min<int64_t>({units, std::max(1, 512 / ny), conv_max_row_tiles(a.nb * Ho * Wo)});
  if (units >= (1 << 30)) return false;
  const size_t lds = (size_t)(strips + std::max(((rb - 1) * sd + a.R) * l.pitch, weights)) * 2;
  if (row_tiles) *row_tiles = groups;
  *e = a.R == 3   ? conv_go<3>(a, groups, rb, l, row_blocks, lds, s)
       : a.R == 5 ? conv_go<5>(a, groups, rb, l, row_blocks, lds, s)
                  : conv_go<7>(a, groups, rb, l, row_blocks, lds, s);
  return true;
}

bool launch_wgrad_image(const WgradArgs& a0, hipStream_t s, int* splits, hipError_t* e) {
  WgradArgs a = a0;
  const int Ho = a.Ho > 0 ? a.Ho : a.H, Wo = a.Ho > 0 ? a.Wo : a.W, sd = a.Ho > 0 ? a.stride : 1;
  const int K = a.R * a.S * a.C;
  if (!fits_map(Ho, Wo, K > 96 ? WGRAD_MAP_WIDE : WGRAD_MAP)) return false;
  // strided 1x1 filters read a quarter of the staged values; with many channels, in rows
  // that go through registers, the staging is the time (stride 2, 32 images of 46x46,
  // general kernel / here: 150->128 42 / 76 us, 60->128, whose rows are copied, 25 / 21)
  if (a.R < sd && a.C > 48 && a.W * a.C % 8 != 0) return false;
  if (a.C % 8 == 0 || a.ldx != a.C || K > 160 || a.N % 8 != 0 || a.lddz % 8 != 0 || a.nseg > 0 ||
      (reinterpret_cast<uintptr_t>(a.dz) % 16) != 0)
    return false;
  // a workgroup fills a CU (7x7 stride 2, 224x224x3 x 100: 342 splits of half the
  // workgroup 122 us, 256 of the whole 73 us)
  a.splits = std::min(a.splits, std::max(1, 256 / ((a.N + 63) / 64)));
  const Rows l(Wo, 16, sd * a.C, a.S * a.C, a.padw * a.C, a.W * a.C);
  const int rb = unit_rows(a.nb, Ho, a.splits, 2, sd, a.R, l.pitch, WGRAD_ROWS);
  if (rb == 0 || (int64_t)a.H * a.W * a.C >= (1 << 30) || (int64_t)Ho * Wo * a.lddz >= (1 << 30)) return false;
  const int row_blocks = (Ho + rb - 1) / rb;
  if ((int64_t)a.nb * row_blocks >= (1 << 30)) return false;
  const double flops = 2.0 * a.nb * Ho * Wo * (double)a.N * K;
  const dim3 grid(a.splits, (a.N + 63) / 64);
  if (K <= 32)
    XP_LAUNCH("k_wgrad_image<1>", flops, k_wgrad_image<1>, grid, dim3(512), 0, s, a, rb, l.lead, l.pitch, row_blocks);
  else if (K <= 96)
    XP_LAUNCH("k_wgrad_image<3>", flops, k_wgrad_image<3>, grid, dim3(512), 0, s, a, rb, l.lead, l.pitch, row_blocks);
  else
    XP_LAUNCH("k_wgrad_image<5>", flops, k_wgrad_image<5>, grid, dim3(512), 0, s, a, rb, l.lead, l.pitch, row_blocks);
  *splits = a.splits;
  *e = hipGetLastError();
  return true;
}

}  // namespace xp
