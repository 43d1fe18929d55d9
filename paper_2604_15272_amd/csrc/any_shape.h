// Elements of the storage types and pieces of consecutive ones, for the kernels that take any shape: everything is
// widened to fp32 on load and rounded once, on the store of a result.
#pragma once
#include "device_utils.h"

namespace prism {

// Storage types: widening and narrowing of one element.
struct StoreF32 {
    typedef float elem;
    static __device__ __forceinline__ float widen(elem v) { return v; }
    static __device__ __forceinline__ elem narrow(float v) { return v; }
};
struct StoreBf16 {
    typedef uint16_t elem;
    static __device__ __forceinline__ float widen(elem v) { return __builtin_bit_cast(float, (u32)v << 16); }
    static __device__ __forceinline__ elem narrow(float v) { return (elem)(pack_bf16(v, 0.0f) & 0xFFFFu); }
};
struct StoreF16 {
    typedef _Float16 elem;
    static __device__ __forceinline__ float widen(elem v) { return (float)v; }
    static __device__ __forceinline__ elem narrow(float v) { return (elem)v; }
};

constexpr float kFloatMax = 3.402823466e38f;

// NaN if x is one or an infinity, else t.
__device__ __forceinline__ float not_finite(float x, float t) { return fmaf(x, 0.f, t); }

// V consecutive elements, loaded in one piece from an address that is only aligned to one of them.
template <typename E, int V> struct Piece {
    typedef E vec __attribute__((ext_vector_type(V)));
    typedef vec loose __attribute__((aligned(sizeof(E))));
    vec v;
    __device__ __forceinline__ void load(const E* p) { v = *(const loose*)p; }
    __device__ __forceinline__ void store(E* p) const { *(loose*)p = v; }
    __device__ __forceinline__ E at(int i) const { return v[i]; }
    __device__ __forceinline__ void set(int i, E e) { v[i] = e; }
};
template <typename E> struct Piece<E, 1> {
    E v;
    __device__ __forceinline__ void load(const E* p) { v = *p; }
    __device__ __forceinline__ void store(E* p) const { *p = v; }
    __device__ __forceinline__ E at(int) const { return v; }
    __device__ __forceinline__ void set(int, E e) { v = e; }
};

}  // namespace prism
