// Group-query attention at one query position in fp32 on the matrix cores: any storage type, any number of heads, head
// dimensions 64 and 128 (what the 16-bit kernel of attention_kernel.hip does not take; other head dimensions go to the plain
// kernel there).  Scores, probabilities and sums stay in fp32.
//
// A workgroup owns 16 heads of one batch entry; its wavefronts take the blocks of 16 keys round-robin.  The scores are
// computed with the keys as rows, K . Q^T (v_mfma_f32_16x16x4_f32): lane (q, c), q = lane / 16, c = lane % 16, then holds
// the scores of head c for the keys 4 q .. 4 q + 3, which is the operand that P . V needs when its product i takes the keys
// 4 q + i (the order of K within a block is free): nothing is rearranged in between.  The maximum over a block's keys is four
// values in a lane and two exchanges.  Each wavefront keeps a running maximum per head; the partials meet in LDS at the end.
//
// What bounds it: the compute units that have a batch entry, one per sixteen heads: their matrix cores are busy 52 to 58 % of
// their cycles (f16 32 x 8 x 5001 x 64, 11 % of the units at work: 66 us, its products alone 33 us), the rest is the chain of a
// block's maximum, exponentials and rescaling.  One thread per key and per column (the plain kernel) waited for its loads: on
// changing keys that case 506 -> 66 us, fp32 32 x 8 x 5000 x 128 622 -> 127 us, fp32 2 x 8 x 2048 x 128 174 -> 48 us, one entry of
// 16384 keys (16 heads, f16, D = 64) 1175 -> 198 us, fp32 64 x 1 x 2500 x 64 297 -> 35 us; errors against 64 bits of fp32 storage are less than half of what they were.
#include "any_shape.h"
#include "device_utils.h"
#include "prism_internal.h"

namespace prism {

namespace {

constexpr int GW = kGqaGeneralWaves;

}  // namespace

// LDS: [GW][16][D] partial outputs, [GW][16] maxima, [GW][16] sums, [GW] flags.
template <typename S, int D>
__global__ __launch_bounds__(GW * 64) void gqa_general_kernel(const typename S::elem* __restrict__ Q,
                                                              const typename S::elem* __restrict__ K,
                                                              const typename S::elem* __restrict__ V,
                                                              typename S::elem* __restrict__ O, int G, int H, float scale,
                                                              int qk_norm, float eps) {
    typedef typename S::elem E;
    constexpr int XV = 16 / (int)sizeof(E);  // head-dimension values per piece
    constexpr int NP = D / (4 * XV);         // pieces of a row per lane: piece p is values XV (4 p + q) ..
    constexpr int VW = D / 16;               // columns of V per lane
    struct Blk {
        Piece<E, XV> k[NP];
        Piece<E, VW> v[4];
    };
    extern __shared__ __align__(16) float lds[];
    float* red = lds;
    float* wave_max = lds + GW * 16 * D;
    float* wave_sum = wave_max + GW * 16;
    float* wave_bad = wave_sum + GW * 16;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c = lane & 15;
    const int g0 = blockIdx.x * 16, bi = blockIdx.y;

    // Q of head c (heads past G: head G - 1 again, not stored), normalised if asked, scaled.
    float qv[NP * XV];
    {
        const E* q_row = Q + ((size_t)bi * G + min(g0 + c, G - 1)) * D + XV * q;
        float ss = 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            Piece<E, XV> x;
            x.load(q_row + 4 * XV * p);
#pragma unroll
            for (int i = 0; i < XV; ++i) {
                const float v = S::widen(x.at(i));
                qv[p * XV + i] = v;
                ss = fmaf(v, v, ss);
            }
        }
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        const float f = qk_norm ? scale / sqrtf(ss / (float)D + eps) : scale;
#pragma unroll
        for (int i = 0; i < NP * XV; ++i) qv[i] *= f;
    }

    const E* k_lane = K + ((size_t)bi * H + c) * D + XV * q;
    const E* v_lane = V + ((size_t)bi * H + 4 * q) * D + VW * c;
    f32x4 acc[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -__builtin_inff(), l_run = 0.f;  // of head c; the sum over this lane's keys only

    auto load = [&](Blk& b, int jb) __attribute__((always_inline)) {
        const size_t at = (size_t)jb * 16 * D;
#pragma unroll
        for (int p = 0; p < NP; ++p) b.k[p].load(k_lane + at + 4 * XV * p);
#pragma unroll
        for (int i = 0; i < 4; ++i) b.v[i].load(v_lane + at + i * D);
    };
    // The block that crosses the end of the keys: zeros past it (in V too: a weight of 0 may not meet an infinity).
    auto load_masked = [&](Blk& b, int jb) __attribute__((always_inline)) {
        const size_t at = (size_t)jb * 16 * D;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int i = 0; i < XV; ++i) b.k[p].set(i, S::narrow(0.f));
            if (16 * jb + c < H) b.k[p].load(k_lane + at + 4 * XV * p);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < VW; ++j) b.v[i].set(j, S::narrow(0.f));
            if (16 * jb + 4 * q + i < H) b.v[i].load(v_lane + at + i * D);
        }
    };
    auto block = [&](const Blk& b, int keys) __attribute__((always_inline)) {
        f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;  // two sums: a product need not wait for the one before it
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < XV; i += 2) {
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(S::widen(b.k[p].at(i)), qv[p * XV + i], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(S::widen(b.k[p].at(i + 1)), qv[p * XV + i + 1], s1, 0, 0, 0);
            }
        float s[4], mx = -__builtin_inff();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = 4 * q + e < keys ? s0[e] + s1[e] : -__builtin_inff();
            mx = fmaxf(mx, s[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
            // Element e of an accumulator belongs to head 4 q + e, whose factor lives in the lanes of that head.
            const float f = (m_run == -__builtin_inff()) ? 1.0f : expf(m_run - m_new);
            l_run *= f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float fe = __shfl(f, 4 * q + e, 64);
#pragma unroll
                for (int j = 0; j < VW; ++j) acc[j][e] *= fe;
            }
            m_run = m_new;
        }
        const float shift = (m_run == -__builtin_inff()) ? 0.f : m_run;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float w = expf(s[i] - shift);
            l_run += w;
#pragma unroll
            for (int j = 0; j < VW; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, S::widen(b.v[i].at(j)), acc[j], 0, 0, 0);
        }
    };
    // Two named blocks in turn, without a condition between a load and its use (general_kernel.hip).
    const int nfull = H / 16;
    auto all_blocks = [&]() __attribute__((always_inline)) {
        if (wave < nfull) {
            const int last = nfull - 1;
            Blk even, odd;
            load(even, wave);
            for (int jb = wave;; jb += 2 * GW) {
                load(odd, min(jb + GW, last));
                __builtin_amdgcn_sched_barrier(0);
                block(even, 16);
                if (jb + GW > last) break;
                load(even, min(jb + 2 * GW, last));
                __builtin_amdgcn_sched_barrier(0);
                block(odd, 16);
                if (jb + 2 * GW > last) break;
            }
        }
        if (nfull * 16 < H && wave == nfull % GW) {
            Blk tail;
            load_masked(tail, nfull);
            block(tail, H - nfull * 16);
        }
    };

    // Across the wavefronts that had keys.  Their weights are worked out once, in the lanes of each wavefront, not by every output
    // element for itself: that took a quarter of a call of few keys (us, before -> now: f16 2 x 44 x 4 x 128 7.5 -> 5.6, fp32
    // 32 x 16 x 64 x 128 9.1 -> 7.9, bf16 25 x 28 x 121 x 64 6.0 -> 5.9).  One to three heads have little to share and pay 0.1 to 0.3
    // for the check of the sums: f16 11 x 2 x 164 x 64 5.7 -> 6.0, fp32 10 x 3 x 411 x 64 8.8 -> 9.0.
    const int active = min(GW, (H + 15) / 16);
    // Lane (q, c) of every wavefront: maxima, weights and sums of head c in wavefronts q and q + 4.
    static_assert(GW == 8 && D % 64 == 0, "four lanes a head, a wavefront's outputs are of one head");
    float mx[2], weight[2], sum[2], gmax;
    // Relative to a maximum that is still to rise, sums of very large values of V can pass the type's range although the result does
    // not.  Where any sum is not finite, the keys are gone through once more with the heads' maxima known.
    for (bool again = false;; again = true) {
        all_blocks();
        l_run += __shfl_xor(l_run, 16, 64);
        l_run += __shfl_xor(l_run, 32, 64);
        float bad[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < VW; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) bad[e] = not_finite(acc[j][e], bad[e]);
        const float all = (bad[0] + bad[1]) + (bad[2] + bad[3]);
        const bool any = __builtin_amdgcn_ballot_w64(all != all) != 0;
        if (lane == 0) wave_bad[wave] = any ? 1.f : 0.f;
        if (q == 0) {
            wave_max[wave * 16 + c] = m_run;
            wave_sum[wave * 16 + c] = l_run;
        }
        if (wave < active) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < VW; ++j) red[(wave * 16 + 4 * q + e) * D + VW * c + j] = acc[j][e];
        }
        __syncthreads();
        const float flag = wave_bad[lane % GW];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool had = q + 4 * i < active;
            mx[i] = had ? wave_max[(q + 4 * i) * 16 + c] : -__builtin_inff();
            sum[i] = had ? wave_sum[(q + 4 * i) * 16 + c] : 0.f;
        }
        gmax = fmaxf(mx[0], mx[1]);
        gmax = fmaxf(gmax, __shfl_xor(gmax, 16, 64));
        gmax = fmaxf(gmax, __shfl_xor(gmax, 32, 64));
        if (again || __builtin_amdgcn_ballot_w64(flag != 0.f) == 0) break;
        m_run = gmax;
        l_run = 0.f;
#pragma unroll
        for (int j = 0; j < VW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();  // everyone has read the maxima
    }
    // A wavefront with no key above -inf is relative to 0 and weighs nothing; a NaN in its sums stays one.
#pragma unroll
    for (int i = 0; i < 2; ++i) weight[i] = (mx[i] == -__builtin_inff()) ? 0.f : expf(mx[i] - gmax);
    auto of_head = [&](const float (&x)[2], int w, int head) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x[w >> 2]), (w & 3) * 16 + head));
    };
#pragma unroll
    for (int i = 0; i < 16 * D / (GW * 64); ++i) {
        const int head = (wave * 64 + i * (GW * 64)) / D;  // the same for all lanes
        if (g0 + head >= G) break;
        const int o = tid + i * (GW * 64);
        float v = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < GW; ++w) {
            if (w >= active) break;
            const float f = of_head(weight, w, head);
            v = fmaf(f, red[w * 16 * D + o], v);
            den = fmaf(f, of_head(sum, w, head), den);
        }
        O[((size_t)bi * G + g0) * D + o] = S::narrow(v / den);
    }
}

template <typename S, int D>
static hipError_t launch_gqa_general_as(const AttentionCall& c) {
    typedef typename S::elem E;
    dim3 grid((c.G + kGqaGeneralHeads - 1) / kGqaGeneralHeads, c.B), block(GW * 64);
    constexpr size_t lds = ((size_t)GW * 16 * (D + 2) + GW) * sizeof(float);
    auto kern = gqa_general_kernel<S, D>;
    static std::atomic<uint64_t> opted{0};
    if (hipError_t e = allow_large_lds((const void*)kern, lds, opted); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, c.stream, (const E*)c.Q, (const E*)c.K, (const E*)c.V, (E*)c.O, c.G, c.H, c.scale,
                       c.qk_norm, c.eps);
    return hipGetLastError();
}

template <typename S>
static hipError_t launch_gqa_general_of(const AttentionCall& c) {
    return c.D == 64 ? launch_gqa_general_as<S, 64>(c) : launch_gqa_general_as<S, 128>(c);
}

hipError_t launch_gqa_general(const AttentionCall& c, int dtype) {
    if (c.D != 64 && c.D != 128) return hipErrorInvalidValue;
    if (dtype == PRISM_F32) return launch_gqa_general_of<StoreF32>(c);
    if (dtype == PRISM_F16) return launch_gqa_general_of<StoreF16>(c);
    return launch_gqa_general_of<StoreBf16>(c);
}

}  // namespace prism
