// A 16-byte store per lane with a scalar offset (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace hcms {

typedef unsigned int store_u32x4 __attribute__((ext_vector_type(4)));

// x to byte voff + soff of the resource.  A store of more than 8 bytes per
// lane reads its data registers after it has issued; with a scalar offset the
// compiler puts no wait state before an instruction that writes them, and
// such stores of attention_dma_kernel have stored the next instruction's
// value.  The s_nop, which takes x, is that wait state: x stays in its
// registers until it has issued.
__device__ inline void store_b128(store_u32x4 x, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b128(x, r, voff, soff, 0);
    asm volatile("s_nop 0" :: "v"(x));
}

}  // namespace hcms
