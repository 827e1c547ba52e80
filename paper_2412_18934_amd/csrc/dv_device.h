// Device helpers shared by the kernel files: scalar conversions, the V cache
// layout and the split layout of activations (dv_internal.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// scalar helpers

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// fp32 -> bf16 bits, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float *p, size_t i) { return p[i]; }
    static __device__ __forceinline__ void store(float *p, size_t i, float v) { p[i] = v; }
};
template <> struct Elem<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t *p, size_t i) { return bf2f(p[i]); }
    static __device__ __forceinline__ void store(uint16_t *p, size_t i, float v) { p[i] = f2bf(v); }
};

// Buffer resource over a device allocation (byte offsets below 2 GiB) and the
// cache-policy bit of buffer instructions for data read once (non-temporal).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, 0x7fffffff, 0x00020000);
}
#define DV_NT 2

// ---------------------------------------------------------------------------
// V cache layout: per (layer, head), 32-slot tiles one after another, each
// tile dim-major ([hd][32]): entry (dim j, slot s) at element
// ((s / 32) hd + j) 32 + s % 32 of the head, so one tile of 32 keys is one
// contiguous hd x 64-byte block and 8 consecutive slots of a dim are 16
// contiguous bytes (the PV B-operand).

__device__ __forceinline__ size_t v_index(int j, int s, int hd)
{
    return ((size_t)(s >> 5) * hd + j) * 32 + (s & 31);
}

// ---------------------------------------------------------------------------
// split layout of activations (see dv_internal.h)

// MT = 0 selects the half layout (tokens 0-7 only; lo in columns 8-15).
__device__ __forceinline__ size_t split_index(int m, int k, int MT)
{
    const int s = k >> 5, g = (k >> 3) & 3, j = k & 7, mt = m >> 4, n = m & 15;
    const size_t blk = MT ? ((size_t)s * MT + mt) * 2 : (size_t)s;
    return (blk * 64 + g * 16 + n) * 8 + j;  // hi; lo is + split_lo(MT)
}

__device__ __forceinline__ int split_lo(int MT) { return MT ? 512 : 64; }

// token tiles of a split-layout operand (0: half layout) and the tokens it
// holds
__device__ __forceinline__ int split_mt(int Mpad, int half) { return half ? 0 : Mpad >> 4; }
__device__ __forceinline__ int split_rows(int Mpad, int half) { return half ? 8 : Mpad; }

__device__ __forceinline__ void store_split(uint16_t *xs, int m, int k, int MT, float v)
{
    const size_t i = split_index(m, k, MT);
    const float hi = __uint_as_float(__float_as_uint(v) & 0xffff0000u);
    xs[i] = (uint16_t)(__float_as_uint(v) >> 16);
    xs[i + split_lo(MT)] = f2bf(v - hi);
}

// fp32 -> bf16 hi (truncation) + lo (RNE of the remainder), 8 values
__device__ __forceinline__ void split_hi_lo(const float4 &a, const float4 &b, bf16x8 &hi, bf16x8 &lo)
{
    const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float h = __uint_as_float(__float_as_uint(v[i]) & 0xffff0000u);
        hi[i] = (__bf16)h;
        lo[i] = (__bf16)(v[i] - h);
    }
}

// four consecutive columns k..k+3 (k % 4 == 0) of one token
__device__ __forceinline__ void store_split4(uint16_t *xs, int m, int k, int MT, float4 v)
{
    const size_t i = split_index(m, k, MT);
    const float f[4] = {v.x, v.y, v.z, v.w};
    uint32_t hi[2], lo[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        uint32_t h2 = 0, l2 = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float x = f[2 * p + q];
            const float h = __uint_as_float(__float_as_uint(x) & 0xffff0000u);
            h2 |= (__float_as_uint(x) >> 16) << (16 * q);
            l2 |= (uint32_t)f2bf(x - h) << (16 * q);
        }
        hi[p] = h2;
        lo[p] = l2;
    }
    *reinterpret_cast<uint2 *>(xs + i) = make_uint2(hi[0], hi[1]);
    *reinterpret_cast<uint2 *>(xs + i + split_lo(MT)) = make_uint2(lo[0], lo[1]);
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

// Four int8 values -> four bf16 (exact: |q| <= 128 needs 8 significant bits),
// two per dword, low byte first.
__device__ __forceinline__ uint2 i8x4_to_bf16(uint32_t d)
{
    const uint32_t f0 = __float_as_uint((float)(int8_t)(d & 0xff));
    const uint32_t f1 = __float_as_uint((float)(int8_t)((d >> 8) & 0xff));
    const uint32_t f2 = __float_as_uint((float)(int8_t)((d >> 16) & 0xff));
    const uint32_t f3 = __float_as_uint((float)(int8_t)(d >> 24));
    return make_uint2(__builtin_amdgcn_perm(f1, f0, 0x07060302u), __builtin_amdgcn_perm(f3, f2, 0x07060302u));
}
