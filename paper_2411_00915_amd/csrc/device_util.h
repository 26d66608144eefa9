// Small device helpers shared by the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned short bf16_t;   // raw bfloat16 bits
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

__device__ __forceinline__ float bf16_to_f32(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// round to nearest, ties to even
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const __bf16 h = (__bf16)f;                       // the hardware conversion of gfx950 (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(unsigned short, h);
#endif
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)0x7fc0;   // NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename T> struct elem;
template <> struct elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct elem<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Loads straight to LDS: lane i's 16 bytes at base + off -> LDS byte address lds_base + 16 i (base and lds_base
// wavefront-uniform).  Issued from inline assembly, so the waits for them are written out.  M0 carries the LDS address;
// nothing else in the kernels that use this uses M0 (LDS instructions of gfx9 and later do not read it).
typedef __attribute__((address_space(3))) void* lds_void_ptr;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_void_ptr)p; }
__device__ __forceinline__ void load16_to_lds(const char* base, uint32_t off, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_base) : "memory");
}

// Workgroups are dealt round-robin to the 8 XCDs; every XCD gets a contiguous run of tiles (so its L2 sees
// neighbouring tiles).  Inside a run the tiles go in groups of GN feature tiles, token tile fastest over GN
// feature tiles, so the 32 tiles an XCD works on at a time form an 8 x 4 block and share 8 x panels and 4 W
// panels (instead of 32 x panels and one W panel) in its L2.
__device__ __forceinline__ void tile_of_workgroup(int id, int tiles_n, int tiles_t, int& tile_n, int& tile_t)
{
    const int n_wg = tiles_n * tiles_t;
    const int per = n_wg / 8, rem = n_wg % 8;
    const int xcd = id & 7, q = id >> 3;
    id = xcd * per + (xcd < rem ? xcd : rem) + q;       // XCD k owns per + (k < rem) tiles
    constexpr int GN = 4;
    const int group = id / (GN * tiles_t), first_n = group * GN;
    const int group_n = min(tiles_n - first_n, GN);
    const int in_group = id - group * (GN * tiles_t);
    tile_n = first_n + in_group % group_n;
    tile_t = in_group / group_n;
}
