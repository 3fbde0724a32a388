// A load from global memory straight to LDS that the compiler does not know of as one: it makes every LDS access that it knows of wait for all
// outstanding loads into LDS, and a wave that reads LDS under its loads is not to wait.  The wave waits for them itself, with s_waitcnt vmcnt.
#ifndef CACNN_LDS_LOAD_H
#define CACNN_LDS_LOAD_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cacnn {

typedef int i32x4 __attribute__((ext_vector_type(4)));

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 64 lanes x 16 bytes, lane L's from byte off of the descriptor d to LDS byte dst + 16 L (d and dst wave-uniform).  No register is written; m0 belongs to
// no one for longer than the instruction that it is set for.
__device__ __forceinline__ void load_to_lds_unseen(i32x4 d, uint32_t off, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(d) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace cacnn
#endif
