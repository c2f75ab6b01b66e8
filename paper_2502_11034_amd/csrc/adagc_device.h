// Device code shared by kernels.hip and muon.hip: how a workgroup reads its work record and its tensor's, and how it
// accesses the caller's arrays.
#pragma once

#include <type_traits>

#include "adagc_internal.h"

// Pointers that come out of a table say nothing about where they point: without these the compiler uses "flat" accesses,
// which count in two of its memory counters, so that every wait for one of them is a wait for all that are on their way.
#define ADAGC_GLOBAL __attribute__((address_space(1)))
#define ADAGC_CONST __attribute__((address_space(4)))

namespace adagc {

// Native clang vectors (the nontemporal builtins do not take HIP's struct vector types).
typedef float    f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
// The same in the caller's arrays, which need no more than their elements' alignment: tensors laid end to end in a flat
// buffer start anywhere.  A vector access takes any such address on this part, and costs a wave one cache line more when it
// does not start on one.
typedef float    f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

// Single elements, at any address at all: what the element-by-element path reads and writes.
typedef float    f32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));

typedef ADAGC_GLOBAL f32_any*       gfloat;
typedef const ADAGC_GLOBAL f32_any* gcfloat;
typedef ADAGC_GLOBAL u16_any*       gu16;
typedef const ADAGC_GLOBAL u16_any* gcu16;
typedef const ADAGC_GLOBAL char*    gcbytes;

// Something that is the same for the whole workgroup and does not change while the kernel runs, through the scalar unit.
// Loads of this kind that do not depend on each other are on their way together.
template <typename T>
__device__ __forceinline__ T uniform_load(const T* p)
{
    return *(const ADAGC_CONST T*)p;
}

__device__ __forceinline__ WorkRef load_work(const WorkRef* work, uint32_t k)
{
    const u32x4 w = uniform_load(reinterpret_cast<const u32x4*>(work + k));
    return WorkRef{w.x, w.y, w.z, w.w};
}

__device__ __forceinline__ int64_t first_element(const WorkRef& w) { return (int64_t)w.index * kChunkElems; }

// A tensor's record, its 64 bytes in one load.
__device__ __forceinline__ TensorArgs load_tensor(const TensorArgs* targs, uint32_t i)
{
    const u64x8 r = uniform_load(reinterpret_cast<const u64x8*>(targs + i));
    TensorArgs a;
    a.param = reinterpret_cast<void*>(r[0]);
    a.grad = reinterpret_cast<const void*>(r[1]);
    a.exp_avg = reinterpret_cast<void*>(r[2]);
    a.exp_avg_sq = reinterpret_cast<void*>(r[3]);
    a.param_copy = reinterpret_cast<void*>(r[4]);
    a.numel = (int64_t)r[5];
    a.chunk_begin = (uint32_t)r[6];
    a.chunk_count = (uint32_t)(r[6] >> 32);
    a.vec_ok = (uint32_t)r[7];
    a.line_offset = (uint32_t)(r[7] >> 32);
    return a;
}
static_assert(offsetof(TensorArgs, grad) == 8 && offsetof(TensorArgs, exp_avg) == 16 && offsetof(TensorArgs, exp_avg_sq) == 24 &&
                  offsetof(TensorArgs, param_copy) == 32 && offsetof(TensorArgs, numel) == 40 && offsetof(TensorArgs, chunk_begin) == 48 &&
                  offsetof(TensorArgs, chunk_count) == 52 && offsetof(TensorArgs, vec_ok) == 56 && offsetof(TensorArgs, line_offset) == 60,
              "load_tensor takes the record apart by hand");

// Not templates of the vector's type: a deduced type is the vector without its typedef's alignment, and the access would claim
// the full one.
template <bool NT>
__device__ __forceinline__ f32x4 ld(const ADAGC_GLOBAL f32x4_any* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ u32x2 ld(const ADAGC_GLOBAL u32x2_any* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ void st(ADAGC_GLOBAL f32x4_any* p, f32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <bool NT>
__device__ __forceinline__ void st(ADAGC_GLOBAL u32x2_any* p, u32x2 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// Four consecutive gradient elements, widened to fp32.  `vec` counts groups of four from `base`.
template <bool BF16, bool NT>
__device__ __forceinline__ f32x4 load_grad4(gcbytes base, int vec)
{
    if constexpr (BF16) {
        const u32x2 r = ld<NT>((const ADAGC_GLOBAL u32x2_any*)base + vec);
        f32x4 o;
        o.x = __uint_as_float(r.x << 16);
        o.y = __uint_as_float(r.x & 0xFFFF0000u);
        o.z = __uint_as_float(r.y << 16);
        o.w = __uint_as_float(r.y & 0xFFFF0000u);
        return o;
    } else {
        return ld<NT>((const ADAGC_GLOBAL f32x4_any*)base + vec);
    }
}

template <bool BF16>
__device__ __forceinline__ float load_grad1(gcbytes base, int j)
{
    if constexpr (BF16) return bf16_bits_to_float(((gcu16)base)[j]);
    else return ((gcfloat)base)[j];
}

// Gradient element `first` of a tensor.
template <bool BF16>
__device__ __forceinline__ gcbytes grad_at(const void* grad, int64_t first)
{
    return (gcbytes)grad + first * (BF16 ? 2 : 4);
}

// fp32 -> bf16, round to nearest even (add half an ulp of the kept part, plus the parity bit).
__device__ __forceinline__ uint32_t float_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    uint32_t rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    uint32_t quiet_nan = (u >> 16) | 0x40u;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? quiet_nan : rounded;
}

}  // namespace adagc
