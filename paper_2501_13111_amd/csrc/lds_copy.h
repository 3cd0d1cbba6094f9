// Buffer-to-LDS copies written in asm, for loops that keep copies in flight across LDS reads
// with exact wait counts of their own (issued through the compiler's builtin, every LDS read
// after a copy would wait for it).
#pragma once
#include "fp_device.h"

namespace fpk {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// The four words of a raw buffer resource over [base, base + bytes): no stride, 32-bit data
// format (the resource __builtin_amdgcn_make_buffer_rsrc builds), for copies written in asm.
__device__ __forceinline__ i32x4 rsrc_words(const void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    return i32x4{(int32_t)(uint32_t)p, (int32_t)((uint32_t)(p >> 32) & 0xFFFFu), (int32_t)bytes, 0x00020000};
}

// Buffer-to-LDS copy: lane l's W bytes (16 or 4) at voff + soff of the resource land at LDS
// address lds + W l (past the resource's end: zeros).  M0 carries the LDS address and is
// restored afterwards; one wait state separates its write from the copy.
template <int W>
__device__ __forceinline__ void lds_copy(const i32x4& r, uint32_t voff, uint32_t soff, uint32_t lds) {
    uint32_t keep;
    if constexpr (W == 16)
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %2, %3, %4 offen lds\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "buffer_load_dword %2, %3, %4 offen lds\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory");
}

}  // namespace fpk
