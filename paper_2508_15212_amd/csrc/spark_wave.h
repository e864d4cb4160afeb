// Wave-level building blocks shared by the pruning kernels (gfx950, wave64): data-parallel-primitive scans and
// reductions over the wavefront and over its rows of sixteen lanes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spark {

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// Inclusive prefix sum over the 64 lanes (lane l gets x_0 + ... + x_l) with data-parallel-primitive
// moves: shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the last lane of row 0 / 2 is added
// to row 1 / 3 and the last lane of row 1 to rows 2 and 3.  Lanes with no source add 0.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr 1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr 2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr 4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast 15 -> rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast 31 -> rows 2, 3
    return v;
}

// ---- sixteen lanes (a data-parallel-primitive row) per key row, four key rows per wavefront

// x of another lane of the same sixteen: CTRL 0x121..0x12F rotates by 1..15; 0x111..0x11F shifts up by 1..15 (lanes
// without a source get 0); 0x150 + l hands out lane l
template <int CTRL>
__device__ __forceinline__ uint32_t row16_move(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t row16_max(uint32_t x)
{
    x = max(x, row16_move<0x128>(x));
    x = max(x, row16_move<0x124>(x));
    x = max(x, row16_move<0x122>(x));
    return max(x, row16_move<0x121>(x));
}
__device__ __forceinline__ uint32_t row16_min(uint32_t x)
{
    x = min(x, row16_move<0x128>(x));
    x = min(x, row16_move<0x124>(x));
    x = min(x, row16_move<0x122>(x));
    return min(x, row16_move<0x121>(x));
}
__device__ __forceinline__ uint32_t row16_sum(uint32_t x)
{
    x += row16_move<0x128>(x);
    x += row16_move<0x124>(x);
    x += row16_move<0x122>(x);
    return x + row16_move<0x121>(x);
}
__device__ __forceinline__ float row16_sum_f32(float x)
{
    x += __uint_as_float(row16_move<0x128>(__float_as_uint(x)));
    x += __uint_as_float(row16_move<0x124>(__float_as_uint(x)));
    x += __uint_as_float(row16_move<0x122>(__float_as_uint(x)));
    return x + __uint_as_float(row16_move<0x121>(__float_as_uint(x)));
}
// lane i of sixteen gets x_0 + ... + x_i
__device__ __forceinline__ uint32_t row16_inclusive_sum(uint32_t x)
{
    x += row16_move<0x111>(x);
    x += row16_move<0x112>(x);
    x += row16_move<0x114>(x);
    return x + row16_move<0x118>(x);
}
__device__ __forceinline__ uint32_t row16_last(uint32_t x) { return row16_move<0x15F>(x); }      // lane 15 of the sixteen

// The lane's bits of eight wave masks as one byte, bit c from kb[c].
__device__ __forceinline__ uint32_t byte_of_masks(const uint64_t (&kb)[8])
{
    uint32_t m = 0;
    // (wait states first: a mask that a vector compare has just written must not be read by a vector instruction at
    //  once; and last: the byte may be read by a lane move next)
    asm("s_nop 1\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %8\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %7\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %6\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %5\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %4\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
        "s_nop 1"
        : "+v"(m)
        : "s"(kb[0]), "s"(kb[1]), "s"(kb[2]), "s"(kb[3]), "s"(kb[4]), "s"(kb[5]), "s"(kb[6]), "s"(kb[7])
        : "vcc");
    return m;
}

__device__ __forceinline__ void prune_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
// LDS byte address of a pointer into shared memory, and back
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ lds_u32 *lds_word(uint32_t byte_address) { return (lds_u32 *)(uintptr_t)byte_address; }

__device__ __forceinline__ uint32_t min8(const uint32_t (&x)[8])
{
    return min(min(min(x[0], x[1]), min(x[2], x[3])), min(min(x[4], x[5]), min(x[6], x[7])));
}

}  // namespace spark
