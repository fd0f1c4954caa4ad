// Copies from memory straight into LDS, and the waits they need (gfx950).
#pragma once
#include "xp_device.h"
#include <type_traits>

namespace xp {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// calls f(integral_constant<int, I>) for I = B .. E-1
template <int B, int E, typename F>
XP_DEV void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// -1 where bit i of m is set, else 0
XP_DEV int bit_mask(uint32_t m, int i) { return __builtin_amdgcn_sbfe((int)m, i, 1); }

// 16 bytes per lane from the buffer to LDS at lds + 16 * lane (lds is the same
// in all lanes); zeros where the offset is past the buffer's end
XP_DEV void load_lds16(__amdgpu_buffer_rsrc_t r, bf16_t* lds, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, 0);
}

// Waits until at most N of the wave's vector memory operations are outstanding
// and its LDS reads have returned, then for the workgroup (a barrier that
// leaves later loads to LDS in flight).
template <int N>
XP_DEV void wait_step() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace xp
