// Elements of the storage types and pieces of consecutive ones, for the kernels that take any shape: everything is
// widened to fp32 on load and rounded once, on the store of a result.
#pragma once
#include "device_utils.h"
#include "prism_internal.h"

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

// 16-bit storage: products of 32-bit operands with stored values on the 16-bit matrix cores.  The operand goes in as P parts of
// the storage format, the value rounded to it, what that leaves rounded again, and so on; the stored values are taken as they are.
//   bf16: two parts carry a product of two stored values (16 significant bits) without loss, three any fp32 value.
//   f16: two parts carry such a product (22 bits) without loss and a fp32 value to 2^-23, where it is 2^-14 or more; the second is 2^11 times as
//   large as it should be, so that it does not run out of exponents before the first does, and has accumulators of its own.  Below 2^-14 the
//   error is 2^-36, no more than the rounding of a fp32 sum that has products of 2^-11 among them; rows of x * g that have none of that size
//   (small_products) are worked out in fp32.  Weights of a softmax, at most 1 and relative to each other, are therefore taken kWeightScale
//   times as large, their sums too: 2^-23 of a weight down to 2^-29 of the largest, 2^-51 of the largest below.
// Infinities, NaNs and what rounds to an infinity have no parts: the sum is not finite then.
template <typename S> struct PartProduct;
template <> struct PartProduct<StoreBf16> {
    static constexpr int kProductParts = 2, kFloatParts = 3, kAccumulators = 1;
    static constexpr float kWeightScale = 1.f;
    template <int P> static __device__ __forceinline__ void split8(const float (&value)[8], u32x4 (&part)[P]) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = value[i];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const u32 u = pack_bf16(v[2 * d], v[2 * d + 1]);
                part[p][d] = u;
                if (p + 1 < P) {
                    v[2 * d] -= bf16_lo(u);
                    v[2 * d + 1] -= bf16_hi(u);
                }
            }
    }
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) { return Bf16::mfma_16x16x32(a, b, c); }
    static __device__ __forceinline__ float sum(const f32x4 (&acc)[1], int e) { return acc[0][e]; }
};
template <> struct PartProduct<StoreF16> {
    static constexpr int kProductParts = 2, kFloatParts = 2, kAccumulators = 2;
    static constexpr float kWeightScale = 32768.f;
    static constexpr float kLogWeight = 10.375f;  // the same by the exponent (e^10.375 = 32048), in few bits: differences from f16 values are exact
    template <int P> static __device__ __forceinline__ void split8(const float (&v)[8], u32x4 (&part)[P]) {
        static_assert(P == 2, "two parts");
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const u32 u = F16::pack(v[2 * d], v[2 * d + 1]);
            part[0][d] = u;
            part[1][d] = F16::pack((v[2 * d] - F16::lo(u)) * 2048.f, (v[2 * d + 1] - F16::hi(u)) * 2048.f);
        }
    }
    static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) { return F16::mfma_16x16x32(a, b, c); }
    static __device__ __forceinline__ float sum(const f32x4 (&acc)[2], int e) { return fmaf(acc[1][e], 1.f / 2048.f, acc[0][e]); }
};

// Whether the products of x and g whose first f16 parts were or-ed into both halves of `bits` are all below 2^-11.  (2^-11 is where the upper three
// bits of the exponent are first set, so the or of them tells.)
__device__ __forceinline__ bool small_products(u32 bits) { return (bits & 0x70007000u) == 0; }

// Column j of eight rows of V columns each, as a matrix operand: eight K values.
template <typename E, int V> __device__ __forceinline__ u32x4 column_operand(const Piece<E, V> (&w)[8], int j) {
    static_assert(sizeof(E) == 2, "16-bit storage");
    u32x4 b;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if constexpr (V == 1) {
            b[d] = (u32)__builtin_bit_cast(uint16_t, w[2 * d].at(0)) | (u32)__builtin_bit_cast(uint16_t, w[2 * d + 1].at(0)) << 16;
        } else {
            typedef u32 dwords __attribute__((ext_vector_type(V / 2)));
            const dwords lo = __builtin_bit_cast(dwords, w[2 * d].v), hi = __builtin_bit_cast(dwords, w[2 * d + 1].v);
            b[d] = __builtin_amdgcn_perm(hi[j / 2], lo[j / 2], (j & 1) ? 0x07060302u : 0x05040100u);
        }
    }
    return b;
}

// 16 rows x 16 C columns of a product call by one wavefront, with the fp32 matrix instructions over the whole of K: for wavefronts that met a sum
// in parts that is not finite.  Few registers and little code, so that a kernel that hardly ever gets here carries neither; the price
// is bounded by the latency of its loads, about a microsecond for every 16 K values.
// m0: first row; column(p), p < 16 C: the column, -1 if it has none; stored(r, p): whether row m0 + r, column(p) is this wavefront's;
// row_scale(r): 1/rms of row m0 + r.
template <typename S, bool GATED, int C, typename Column, typename Stored, typename RowScale>
__device__ __forceinline__ void products_in_f32(const typename S::elem* __restrict__ X, const typename S::elem* __restrict__ g,
                                                const typename S::elem* __restrict__ W1, const typename S::elem* __restrict__ W2,
                                                typename S::elem* __restrict__ Y, int M, int K, int N, int m0, int flags, Column column,
                                                Stored stored, RowScale row_scale) {
    typedef typename S::elem E;
    constexpr int G = GATED ? 2 : 1;
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const bool gain = (flags & kFlagGain) != 0;
    const E* x_lane = X + (size_t)min(m0 + c, M - 1) * K;
    f32x4 acc[G][C];
#pragma unroll
    for (int m = 0; m < G; ++m)
#pragma unroll
        for (int j = 0; j < C; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma clang loop unroll(disable)
    for (int k0 = 0; k0 < K; k0 += 16) {
        float a[4], w[G][C][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // lane q: K values 4 q .. of the sixteen; past the end zeros in both operands
            const int k = min(k0 + 4 * q + i, K - 1);
            const bool ok = k0 + 4 * q + i < K;
            const float x = S::widen(x_lane[k]) * (gain ? S::widen(g[k]) : 1.f);
            a[i] = ok ? x : 0.f;
#pragma unroll
            for (int m = 0; m < G; ++m)
#pragma unroll
                for (int j = 0; j < C; ++j) {
                    const float v = S::widen((m == 0 ? W1 : W2)[(size_t)k * N + max(column(16 * j + c), 0)]);
                    w[m][j][i] = ok ? v : 0.f;
                }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < G; ++m)
#pragma unroll
                for (int j = 0; j < C; ++j) acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], w[m][j][i], acc[m][j], 0, 0, 0);
    }
    wait_stores_acknowledged();  // (what is stored now comes last)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int m = m0 + 4 * q + e;
        if (m >= M) continue;
        const float rinv = row_scale(4 * q + e);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int n = column(16 * j + c);
            if (n < 0 || !stored(4 * q + e, 16 * j + c)) continue;
            float y = acc[0][j][e] * rinv;
            if (GATED) {
                const float s = y;
                y = ((flags & kFlagSilu) ? s / (1.0f + expf(-s)) : s) * (acc[G - 1][j][e] * rinv);
            }
            Y[(size_t)m * N + n] = S::narrow(y);
        }
    }
}

}  // namespace prism
