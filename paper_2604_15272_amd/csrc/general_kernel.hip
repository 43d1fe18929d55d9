// Products for any M, K, N and every storage type, of 32-bit precision: fp32 storage on the matrix cores in fp32
// (v_mfma_f32_16x16x4_f32), 16-bit storage on the 16-bit ones (v_mfma_f32_16x16x32), x * g as two parts that carry it without loss
// (f16: products of 2^-14 or more; rows of smaller ones are worked out in fp32) and the stored w as it is (PartProduct in any_shape.h).
//
// A workgroup owns RG groups of 16 rows and 16 * VW columns; its wavefronts take the K-blocks (4 * XV deep, XV = the
// values of 16 bytes) round-robin and meet in LDS after the loop.  The order of K inside a block is free as long as
// both operands agree on it, and it is chosen so that neither operand needs rearranging: lane (q, c), q = lane / 16,
// c = lane % 16, holds the XV consecutive K values XV * q .. of row c and the rows XV * q .. of W at the VW columns from
// VW * c on.  In fp32, product i of the block takes element i of the first and row i of the second; in 16 bits a lane's eight K values
// are one operand, and a column of its eight rows of W the other (a byte permute per two rows).  The VW columns of a lane
// go to VW different accumulator tiles.  Sums of squares ride on the loads of X, the gain is applied in registers, and
// 1/rms goes on after the loop (paper Table 1, "matmul commutes with div denominator").
//
// Ragged sizes cost nothing in the loop: a column group that would cross the right edge starts at N - VW instead (its
// lanes repeat columns of their neighbour), rows past M repeat row M - 1 and are not stored, and the last K-block, if it
// is not full, runs through a masked copy of the loop body.  Rows of W start at any element: loads are of 16 bytes at
// the alignment of one element, which global loads take on this part.
//
// Measured against the plain FMA kernel that was here (8 rows x 256 columns per workgroup, one column per thread):
// bf16 8 x 4096 x 32003 1600 -> 54 us, fp32 8 x 256 x 512 31 us -> the launch.
// Of that, neighbouring column tiles on one XCD (xcd_run_tile): bf16 8 x 4096 x 32003 60.7 -> 54.0 us, fp32 1 x 4096 x 4096
// (stripes of 64 bytes, two to a cache line) 21.2 -> 13.5 us, fp32 16 x 4096 x 11000 38.3 -> 30.6 us.
//
// 16-bit storage in parts against the fp32 instructions, whose products took 27 us of it: bf16 8 x 4096 x 32003 54.9 -> 43.5 us, gated bf16 8 x
// 4096 x 14331 60.0 -> 48.8, f16 8 x 4096 x 32003 54.2 -> 45.2, bf16 40 x 4193 x 8041 51.8 -> 36.8, 169 x 500 x 3001 15.7 -> 9.2.  (fp32
// storage would need six products of three parts each, with w split anew for every 16 rows: no gain.)
// Values that have no parts (infinities, NaNs, x * g past the format's range) make sums that are not finite; a wavefront that met one works its
// outputs out once more with the fp32 instructions, at a bounded price (a NaN in the gain: bf16 8 x 4096 x 32003 40 -> 940 us).
//
// What bounds it: 16 rows of 16-bit storage: streaming W (262 MB at 6.0 TB/s); more rows: the operands' way from the caches; fp32
// storage: the fp32 matrix rate, 256 operations per clock and compute unit (157 TFLOP/s).
#include "any_shape.h"
#include "device_utils.h"
#include "prism_internal.h"

#include <type_traits>

namespace prism {

namespace {

// What a lane holds of one K-block.
template <typename E, int XV, int VW, int RG, int G> struct Block {
    Piece<E, XV> x[RG], g;
    Piece<E, VW> w[G][XV];
};

// K from which 16 x 16 tiles of one 16-bit matrix request a block ahead.  There are few wavefronts then, and each walks ten blocks or more with
// nothing but the others of its SIMD to hide the loads (us, ahead / one block at a time: f16 12 x 3501 x 41 13.1 / 15.0, 100 x 6001 x 500 23.0 /
// 25.7, bf16 189 x 3501 x 83 14.8 / 16.0, 16 x 2601 x 1287 11.1 / 11.3; shorter and no better on average: f16 189 x 2049 x 83 11.4 / 10.1, 16 x
// 1801 x 1287 8.5 / 9.1, bf16 100 x 601 x 500 5.2 / 5.0; two matrices: 0.82 of the time of two blocks with one, K 512 to 4096, 0.93 beyond).
constexpr int kNarrowAheadK = 2560;

}  // namespace

// AHEAD: the next K-block is requested before the present one is multiplied (see the loop).
// LDS: [G][waves][16][16 * VW] partial products of one row group, [waves][16 * RG] sums of squares.
template <typename S, bool GATED, int RG, int VW, bool AHEAD>
__global__ __launch_bounds__(general_max_waves(RG, VW) * 64) void general_kernel(
    const typename S::elem* __restrict__ X, const typename S::elem* __restrict__ g,
    const typename S::elem* __restrict__ W1, const typename S::elem* __restrict__ W2, typename S::elem* __restrict__ Y,
    int M, int K, int N, float eps, int flags) {
    typedef typename S::elem E;
    constexpr int G = GATED ? 2 : 1;
    constexpr int XV = 16 / (int)sizeof(E);
    constexpr int KB = 4 * XV;
    constexpr int TN = 16 * VW;
    typedef Block<E, XV, VW, RG, G> Blk;

    extern __shared__ __align__(16) float lds[];
    const int nw = blockDim.x >> 6;
    float* red = lds;
    float* ss_red = lds + G * nw * 16 * TN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c = lane & 15;
    const int tile = xcd_run_tile(blockIdx.x, (unsigned)((N + TN - 1) / TN));  // (gridDim.x would be one more load to wait for)
    const int n0 = tile * TN, m0 = blockIdx.y * (16 * RG);
    const bool gain = (flags & kFlagGain) != 0;

    const int nb = n0 + min(VW * c, N - VW - n0);  // this lane's first column (the host takes VW <= N)
    const E* w_lane[G];
    w_lane[0] = W1 + (size_t)(XV * q) * N + nb;
    if (GATED) w_lane[G - 1] = W2 + (size_t)(XV * q) * N + nb;
    const E* x_lane[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) x_lane[r] = X + (size_t)min(m0 + 16 * r + c, M - 1) * K + XV * q;
    const E* g_lane = (gain ? g : X) + XV * q;  // (without a gain the load is of no use, but it keeps the loop free of branches)

    constexpr bool PARTS = sizeof(E) == 2;  // 16-bit storage on the 16-bit matrix cores, in parts (PartProduct)
    constexpr int NA = PARTS && std::is_same<S, StoreF16>::value ? 2 : 1;
    f32x4 acc[G][RG][VW][NA];
    constexpr bool F16_PARTS = PARTS && std::is_same<S, StoreF16>::value;
    float ss[RG];
    u32 products[RG];  // f16 in parts: the bits of the first ones or-ed; one K-block's lane can see a single value, so the whole row decides
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        ss[r] = 0.f;
        products[r] = 0;
#pragma unroll
        for (int m = 0; m < G; ++m)
#pragma unroll
            for (int j = 0; j < VW; ++j)
#pragma unroll
                for (int a = 0; a < NA; ++a) acc[m][r][j][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    auto load = [&](Blk& b, int kb) __attribute__((always_inline)) {
        const size_t k = (size_t)kb * KB;
        b.g.load(g_lane + k);
#pragma unroll
        for (int r = 0; r < RG; ++r) b.x[r].load(x_lane[r] + k);
#pragma unroll
        for (int i = 0; i < XV; ++i)
#pragma unroll
            for (int m = 0; m < G; ++m) b.w[m][i].load(w_lane[m] + (k + i) * N);
    };
    // The block that crosses the end of K: element by element, zeros past the end (in W too: nothing may meet an infinity
    // there).
    auto load_masked = [&](Blk& b, int kb) __attribute__((always_inline)) {
        const size_t k = (size_t)kb * KB;
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            const bool ok = k + XV * q + i < (size_t)K;
            b.g.set(i, ok ? g_lane[k + i] : S::narrow(0.f));
#pragma unroll
            for (int r = 0; r < RG; ++r) b.x[r].set(i, ok ? x_lane[r][k + i] : S::narrow(0.f));
#pragma unroll
            for (int m = 0; m < G; ++m) {
#pragma unroll
                for (int j = 0; j < VW; ++j) b.w[m][i].set(j, S::narrow(0.f));
                if (ok) b.w[m][i].load(w_lane[m] + (k + i) * N);
            }
        }
    };
    auto multiply = [&](const Blk& b) __attribute__((always_inline)) {
        if constexpr (PARTS) {
            typedef PartProduct<S> PP;
            constexpr int P = PP::kProductParts;
            u32x4 a[RG][P];
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                float v[XV];
#pragma unroll
                for (int i = 0; i < XV; ++i) {
                    const float x = S::widen(b.x[r].at(i));
                    ss[r] = fmaf(x, x, ss[r]);
                    v[i] = x * (gain ? S::widen(b.g.at(i)) : 1.f);
                }
                PP::template split8<P>(v, a[r]);
                if (F16_PARTS) products[r] |= a[r][0][0] | a[r][0][1] | a[r][0][2] | a[r][0][3];
            }
#pragma unroll
            for (int m = 0; m < G; ++m)
#pragma unroll
                for (int j = 0; j < VW; ++j) {
                    const u32x4 w = column_operand(b.w[m], j);
#pragma unroll
                    for (int r = 0; r < RG; ++r)
#pragma unroll
                        for (int p = P - 1; p >= 0; --p) {
                            f32x4& t = acc[m][r][j][NA == 1 ? 0 : p];
                            t = PP::mfma(a[r][p], w, t);
                        }
                }
            return;
        } else {
#pragma unroll
            for (int i = 0; i < XV; ++i) {
                float a[RG];
                const float gk = gain ? S::widen(b.g.at(i)) : 1.f;
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    const float x = S::widen(b.x[r].at(i));
                    ss[r] = fmaf(x, x, ss[r]);
                    a[r] = x * gk;
                }
#pragma unroll
                for (int m = 0; m < G; ++m)
#pragma unroll
                    for (int j = 0; j < VW; ++j) {
                        const float w = S::widen(b.w[m][i].at(j));
#pragma unroll
                        for (int r = 0; r < RG; ++r)
                            acc[m][r][j][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], w, acc[m][r][j][0], 0, 0, 0);
                    }
            }
        }
    };

    // The next block is requested before the present one is multiplied: two named blocks in turn, and past the end the last
    // one is asked for again.  A condition or a copy between a load and its use makes the compiler wait for the load there
    // (fp32 64 x 4096 x 4096 30.2 -> 27.0 us without; three blocks: the same, bf16 8 x 4096 x 32003 8 % slower).
    // In parts, one block at a time: in half the registers (and half the code, of which a short call runs little) more wavefronts share a SIMD: gated
    // bf16 13 x 256 x 1920 4.5 -> 3.9 us, bf16 8 x 512 x 1024 4.6 -> 3.9, 8 x 4096 x 32003 45.3 -> 43.5, gated 8 x 4096 x 14331 51.6 -> 48.8; 27
    // x 704 x 2880 7.0 -> 7.2.  f16 and wide tiles: all loads of a block before its products, which the compiler else mixes (f16 8 x 4096 x
    // 32003 50.9 us mixed, 45.2 so; gated 8 x 4096 x 14331 56.0 / 50.6; narrow tiles lose 2 %).  (fp32 39 x 5568 x 960 would take 76 us instead
    // of 22.)
    const int nfull = K / KB;
    if constexpr (!AHEAD) {
        for (int kb = wave; kb < nfull; kb += nw) {
            Blk b;
            load(b, kb);
            if (F16_PARTS && VW >= 4) __builtin_amdgcn_sched_barrier(0);
            multiply(b);
        }
    } else if (wave < nfull) {
        const int last = nfull - 1;
        Blk even, odd;
        load(even, wave);
        for (int kb = wave;; kb += 2 * nw) {
            load(odd, min(kb + nw, last));
            __builtin_amdgcn_sched_barrier(0);
            multiply(even);
            if (kb + nw > last) break;
            load(even, min(kb + 2 * nw, last));
            __builtin_amdgcn_sched_barrier(0);
            multiply(odd);
            if (kb + 2 * nw > last) break;
        }
    }
    if (nfull * KB < K && wave == nfull % nw) {
        Blk tail;
        load_masked(tail, nfull);
        multiply(tail);
    }

#pragma unroll
    for (int r = 0; r < RG; ++r) {
        ss[r] += __shfl_xor(ss[r], 16, 64);
        ss[r] += __shfl_xor(ss[r], 32, 64);
        if constexpr (F16_PARTS) {
            // A row's products can be too small for their parts: a wavefront that saw only such ones says so by the sign.  (Without a gain the first
            // part is x itself.)
            const uint64_t lanes = __builtin_amdgcn_ballot_w64(gain && small_products(products[r]));
            const u32 both = (u32)lanes & (u32)(lanes >> 32), rows = both & both >> 16;
            if (rows >> c & 1) ss[r] = -ss[r];
        }
        if (q == 0) ss_red[wave * (16 * RG) + 16 * r + c] = ss[r];
    }
    bool bad = false;  // 16-bit storage: this thread met a sum that is not finite
    // Column of place p in the tile; none past the right edge, and where a group of VW columns has been moved in from it, its first ones are the
    // group's before it.
    auto column = [&](int p) __attribute__((always_inline)) {
        const int first = p / VW * VW, n = n0 + min(first, N - VW - n0) + p % VW;
        return first >= N - n0 || n < n0 + first ? -1 : n;
    };
    auto row_scale = [&](int r, int row) __attribute__((always_inline)) {
        float tot = 0.f;
        for (int w = 0; w < nw; ++w) tot += fabsf(ss_red[w * (16 * RG) + 16 * r + row]);
        return (flags & kFlagNorm) ? 1.0f / sqrtf(tot / (float)K + eps) : 1.0f;
    };
    // Across wavefronts, one row group at a time.  Element e of accumulator tile j in lane (q, c) is row 4 q + e,
    // column j of the lane's VW.
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        if (r > 0) __syncthreads();
#pragma unroll
        for (int m = 0; m < G; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < VW; ++j) {
                    float t = acc[m][r][j][0][e];
                    if constexpr (PARTS) t = PartProduct<S>::sum(acc[m][r][j], e);
                    red[((m * nw + wave) * 16 + 4 * q + e) * TN + VW * c + j] = t;
                }
        __syncthreads();
        for (int o = tid; o < 16 * TN; o += blockDim.x) {
            const int row = o / TN, col = o % TN;
            const int m = m0 + 16 * r + row, n = column(col);
            if (m >= M || n < 0) continue;
            float v = 0.f, u = 0.f, tot = 0.f;
            float seen = 0.f;  // f16: above 0 if some wavefront saw a product that is not too small
            for (int w = 0; w < nw; ++w) {
                v += red[(w * 16 + row) * TN + col];
                if (GATED) u += red[((nw + w) * 16 + row) * TN + col];
                const float squares = ss_red[w * (16 * RG) + 16 * r + row];
                tot += F16_PARTS ? fabsf(squares) : squares;
                if (F16_PARTS) seen = fmaxf(seen, squares);
            }
            const float rinv = (flags & kFlagNorm) ? 1.0f / sqrtf(tot / (float)K + eps) : 1.0f;
            // (A row whose 1/rms is a NaN is one anyway.)
            if (PARTS && !__builtin_isfinite(GATED ? fabsf(v) + fabsf(u) : v) && rinv == rinv) bad = true;
            if (F16_PARTS) bad = bad | ((seen == 0.f) & (tot > 0.f));  // (without a gain no sign is set)
            float y = v * rinv;
            if (GATED) {
                const float a = y;
                y = ((flags & kFlagSilu) ? a / (1.0f + expf(-a)) : a) * (u * rinv);
            }
            Y[(size_t)m * N + n] = S::narrow(y);
        }
    }
    if constexpr (PARTS) {
        // Values past the format's range and infinities have no parts: a wavefront that met one works its outputs out once more in fp32.
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {
            constexpr int C = VW < 2 ? VW : 2;  // (an output's wavefront is that of its place in the tile, 64 at a time)
#pragma clang loop unroll(disable)
            for (int t = 0; t < RG * (VW / C); ++t) {
                const int r = t / (VW / C), p0 = t % (VW / C) * (16 * C);
                if (TN == 128 && nw % 2 == 0 && ((p0 / 64 ^ wave) & 1) != 0) continue;  // none of its own
                products_in_f32<S, GATED, C>(
                    X, g, W1, W2, Y, M, K, N, m0 + 16 * r, flags, [&](int p) { return column(p0 + p); },
                    [&](int row, int p) { return (row * TN + p0 + p) / 64 % nw == wave; }, [&](int row) { return row_scale(r, row); });
            }
        }
    }
}

template <typename S, bool GATED, int RG, int VW, bool AHEAD = sizeof(typename S::elem) == 4>
static hipError_t launch_general_as(const Call& c) {
    const int waves = c.form.waves;
    typedef typename S::elem E;
    const int tn = 16 * VW;
    dim3 grid((c.N + tn - 1) / tn, (c.M + 16 * RG - 1) / (16 * RG)), block(waves * 64);
    const size_t lds = ((size_t)(GATED ? 2 : 1) * waves * 16 * tn + (size_t)waves * 16 * RG) * sizeof(float);
    auto kern = general_kernel<S, GATED, RG, VW, AHEAD>;
    static std::atomic<uint64_t> opted{0};
    if (hipError_t e = allow_large_lds((const void*)kern, lds, opted); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, c.stream, (const E*)c.X, (const E*)c.g, (const E*)c.W1,
                       (const E*)(GATED ? c.W2 : c.W1), (E*)c.Y, c.M, c.K, c.N, c.eps, c.flags);
    return hipGetLastError();
}

template <typename S, bool GATED>
static hipError_t launch_general_form(const Call& c) {
    constexpr bool wide = sizeof(typename S::elem) == 4;
    switch (c.form.row_groups * 10 + c.form.cols) {
        case 11:
            if constexpr (!wide && !GATED) {
                if (c.K >= kNarrowAheadK) return launch_general_as<S, GATED, 1, 1, true>(c);
            }
            return launch_general_as<S, GATED, 1, 1>(c);
        case 14: return launch_general_as<S, GATED, 1, 4>(c);
        case 18: if constexpr (!wide && !(GATED && std::is_same<S, StoreF16>::value)) return launch_general_as<S, GATED, 1, 8>(c); else break;
        case 21: if constexpr (wide || GATED) return launch_general_as<S, GATED, 2, 1>(c); else break;
        case 24: return launch_general_as<S, GATED, 2, 4>(c);
    }
    return hipErrorInvalidValue;
}

template <typename S>
static hipError_t launch_general(const Call& c, int dtype) {
    if (c.form.row_groups >= kTiledRowGroups) return launch_general_tiled(c, dtype);
    return c.gated ? launch_general_form<S, true>(c) : launch_general_form<S, false>(c);
}

hipError_t launch_simple_f32(const Call& c) { return launch_general<StoreF32>(c, PRISM_F32); }
hipError_t launch_simple_bf16(const Call& c) { return launch_general<StoreBf16>(c, PRISM_BF16); }
hipError_t launch_simple_f16(const Call& c) { return launch_general<StoreF16>(c, PRISM_F16); }

}  // namespace prism
