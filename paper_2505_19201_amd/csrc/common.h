// Internal helpers of libdream (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include <atomic>
#include "dream.h"
#include "sizes.h"

namespace dream {

// Thread-local last-error text, returned by dream_last_error().
char *error_buffer();
int fail(int status, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int check_launch(const char *what);

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Raises the dynamic-LDS limit of `kernel` on the current device, once per device; `done` is the kernel's own mask of devices.  (dream_init does it
// for every kernel, a call that is first to one otherwise.  Two threads may both do it: harmless.)
int raise_lds_limit(std::atomic<uint64_t> &done, const void *kernel, size_t bytes, const char *who);

int kv_splits_override();
int q_tiles_override();
int tile_waves_override();
int accept_spin_limit();

// per-file parts of dream_init()
int attn_init();
int compress_init();
int project_init();

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// the same from and to any address of a 16-bit value in global memory
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// LDS traffic inside one wave needs no barrier, only program order.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-wide reductions in a fixed order, in every lane: rotations inside the rows of 16 lanes (register moves; a shuffle is a trip through
// LDS), then the four rows' values as scalars.
template <int ROT>
__device__ __forceinline__ float row_rotate(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + ROT, 0xf, 0xf, false));   // row_ror:ROT
}
__device__ __forceinline__ float of_row(float v, int row) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), row * 16)); }
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, row_rotate<8>(v));
    v = fmaxf(v, row_rotate<4>(v));
    v = fmaxf(v, row_rotate<2>(v));
    return fmaxf(v, row_rotate<1>(v));
}
__device__ __forceinline__ float wave_max(float v)
{
    v = row_max(v);
    return fmaxf(fmaxf(of_row(v, 0), of_row(v, 1)), fmaxf(of_row(v, 2), of_row(v, 3)));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    v += row_rotate<1>(v);
    return (of_row(v, 0) + of_row(v, 1)) + (of_row(v, 2) + of_row(v, 3));
}

// 16 bytes per lane from base + offset straight to LDS: lane i's land at lds + 16 * i.  Inline assembly, because the compiler
// makes every LDS read wait for all such loads in flight; the caller waits with s_waitcnt vmcnt.  (Loads that the compiler
// counts itself are only waited for longer than needed beside these.)  ONCE: with the nontemporal hint.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is reserved; naming it as clobbered is right all the same
template <bool ONCE = false>
__device__ __forceinline__ void lds_load16(const void *base, uint32_t offset, uint32_t lds)
{
    if (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
// 4 bytes per lane
__device__ __forceinline__ void lds_load4(const void *base, uint32_t offset, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace dream
