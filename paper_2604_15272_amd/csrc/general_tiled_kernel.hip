// Products for any M, K, N and every storage type where there are many rows: the fp32 matrix-core kernel with both
// operands through LDS.
//
// The kernel without LDS (general_kernel.hip) reads 32 rows of X and 64 columns of W per wavefront and K-block from the
// caches; with many rows that traffic, not the fp32 matrix rate, is what it waits for (fp32 gated 512 x 1024 x 4096:
// 94 us, 91 of 157 TFLOP/s).  Here a workgroup of eight wavefronts owns BM rows x 128 columns (gated: 64 of each
// matrix), two stages of 32 K values of both operands lie in LDS as fp32, and the next stage is on its way in registers
// while the present one is multiplied.  Two wavefronts per SIMD: the operand reads of one run under the products of the
// other.  Same case: 74 us, 115 TFLOP/s;
// 4096 x 1024 x 1024 94 -> 71 us; 512 x 1024 x 4096 53 -> 42 us with 64 rows.
// What bounds it: the fp32 matrix rate (65 us per 1024 K values of a 128-row tile, 84 % of the 54.6 us at 157 TFLOP/s;
// counted, the matrix cores are busy 76 to 81 % of the cycles in which a compute unit has a workgroup, without bank
// conflicts), and about 7 us of launch, first stage and last reduction per call.
// (With the next stage requested at the start of a trip and stored at its end the case took 86 us: every wavefront of the
// compute unit then waits for memory and stores at the same time.)
//
// Sums of squares and the gain are dealt with once per element, on the way into LDS.  A lane (q, c), q = lane / 16,
// c = lane % 16, reads the four K values 4 q .. of row c and the rows 4 q .. of W at its NC neighbouring columns; product i
// takes element i of the first and row i of the second (the order of K within a block is free).
//   X stage: [row][8 pieces of 4 K values], the pieces of row r rotated by XOR with r % 8.
//   W stage: [k][128 columns], blocks of 16 NC columns XORed with the low bits of k / 4, so that the four q of a read
//   fall into different banks.
// Ragged sizes: rows past M repeat row M - 1, a group of four columns that would cross the right edge starts at N - 4,
// K values past the end are zeros in both operands.
#include "any_shape.h"
#include "device_utils.h"
#include "prism_internal.h"

namespace prism {

namespace {

constexpr int TK = 32;     // K values per stage
constexpr int TC = 128;    // columns per workgroup, over all matrices
constexpr int NTH = 512;   // threads

}  // namespace

// LDS: [2][BM][8] pieces of X, [2][TK][TC / 4] pieces of W, [BM] sums of squares.
template <typename S, bool GATED, int BM>
__global__ __launch_bounds__(NTH, 4) void general_tiled_kernel(
    const typename S::elem* __restrict__ X, const typename S::elem* __restrict__ g,
    const typename S::elem* __restrict__ W1, const typename S::elem* __restrict__ W2, typename S::elem* __restrict__ Y,
    int M, int K, int N, float eps, int flags) {
    typedef typename S::elem E;
    constexpr int G = GATED ? 2 : 1;
    constexpr int CW = TC / G;          // output columns per workgroup
    constexpr int WM = BM / 32;         // wavefronts along the rows (32 rows each)
    constexpr int WN = 8 / WM;          // and along the columns
    constexpr int NC = TC / WN / 16 / G;  // neighbouring columns per lane and matrix
    constexpr int XP = BM * 8 / NTH;    // pieces of X per thread and stage
    constexpr int WP = TK * (TC / 4) / NTH;
    static_assert(NC == 1 || NC == 2 || NC == 4, "columns per lane");

    extern __shared__ __align__(16) float lds[];
    f32x4* xs = (f32x4*)lds;            // [2][BM * 8]
    f32x4* wst = xs + 2 * BM * 8;       // [2][TK * TC / 4]
    float* ss_red = (float*)(wst + 2 * TK * TC / 4);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int q = lane >> 4, c = lane & 15;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * CW;
    const bool gain = (flags & kFlagGain) != 0;

    // ---- staging maps: piece i of X is K values 4 xc .. of row xr + 64 i, piece i of W the columns 4 wc .. of row wr + 16 i
    const int xr = tid >> 3, xc = tid & 7;
    const int wr = tid >> 5, wc = tid & 31;
    const E* x_src[XP];
    int x_dst[XP];
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int r = xr + 64 * i;
        x_src[i] = X + (size_t)min(m0 + r, M - 1) * K + 4 * xc;
        x_dst[i] = r * 8 + (xc ^ (r & 7));
    }
    const int w_col = 4 * wc % CW;
    const E* w_src = (GATED && 4 * wc >= CW ? W2 : W1) + (size_t)wr * N + n0 + min(w_col, N - 4 - n0);
    int w_dst[WP];
#pragma unroll
    for (int i = 0; i < WP; ++i) {
        const int r = wr + 16 * i, col = 4 * wc;
        const int block = (col / (16 * NC)) ^ ((r >> 2) & (4 / NC - 1));
        w_dst[i] = r * (TC / 4) + (block * 16 * NC + col % (16 * NC)) / 4;
    }

    Piece<E, 4> px[XP], pg, pw[WP];
    float ss[XP];
#pragma unroll
    for (int i = 0; i < XP; ++i) ss[i] = 0.f;
    const E* g_src = (gain ? g : X) + 4 * xc;  // (without a gain the load is of no use, but it keeps the loop free of branches)
    auto load = [&](int kt) __attribute__((always_inline)) {
        const size_t k = (size_t)kt * TK;
        pg.load(g_src + k);
#pragma unroll
        for (int i = 0; i < XP; ++i) px[i].load(x_src[i] + k);
#pragma unroll
        for (int i = 0; i < WP; ++i) pw[i].load(w_src + (k + 16 * i) * N);
    };
    // The stage that crosses the end of K: element by element, zeros past the end (in W too).
    auto load_masked = [&](int kt) __attribute__((always_inline)) {
        const size_t k = (size_t)kt * TK;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool ok = k + 4 * xc + e < (size_t)K;
            pg.set(e, ok ? g_src[k + e] : S::narrow(0.f));
#pragma unroll
            for (int i = 0; i < XP; ++i) px[i].set(e, ok ? x_src[i][k + e] : S::narrow(0.f));
        }
#pragma unroll
        for (int i = 0; i < WP; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) pw[i].set(e, S::narrow(0.f));
            if (k + wr + 16 * i < (size_t)K) pw[i].load(w_src + (k + 16 * i) * N);
        }
    };
    auto store = [&](int stage) __attribute__((always_inline)) {
        f32x4 gk;
#pragma unroll
        for (int e = 0; e < 4; ++e) gk[e] = gain ? S::widen(pg.at(e)) : 1.f;
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = S::widen(px[i].at(e));
                ss[i] = fmaf(x, x, ss[i]);
                v[e] = x * gk[e];
            }
            xs[stage * BM * 8 + x_dst[i]] = v;
        }
#pragma unroll
        for (int i = 0; i < WP; ++i) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = S::widen(pw[i].at(e));
            wst[stage * (TK * TC / 4) + w_dst[i]] = v;
        }
    };

    f32x4 acc[G][2][NC];
#pragma unroll
    for (int m = 0; m < G; ++m)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[m][r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Operand addresses in a stage.
    const int a_row = (wm * 32 + c) * 8;                        // + 16 * 8 for the second row group
    int w_at[G];                                                // float index of the lane's columns in row 4 q
#pragma unroll
    for (int m = 0; m < G; ++m) {
        const int block = (m * (CW / (16 * NC)) + wn) ^ (q & (4 / NC - 1));
        w_at[m] = 4 * q * TC + block * 16 * NC + NC * c;
    }
    auto multiply = [&](int stage, int kb) __attribute__((always_inline)) {
        const f32x4* xa = xs + stage * BM * 8;
        const float* wa = (const float*)(wst + stage * (TK * TC / 4)) + 16 * kb * TC;
        f32x4 a[2];
        Piece<float, NC> b[4][G];
#pragma unroll
        for (int r = 0; r < 2; ++r) a[r] = xa[a_row + r * 128 + ((4 * kb + q) ^ (c & 7))];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < G; ++m)
                __builtin_memcpy(&b[i][m].v, __builtin_assume_aligned(wa + w_at[m] + i * TC, 4 * NC), 4 * NC);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < G; ++m)
#pragma unroll
                for (int j = 0; j < NC; ++j)
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        acc[m][r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r][i], b[i][m].at(j), acc[m][r][j], 0, 0, 0);
    };
    // Every wavefront's LDS accesses are complete; loads from memory stay in flight.
    auto stage_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Stage kt + 1 is stored from registers (into the stage that was last read before the barrier at the end of the previous
    // trip) and stage kt + 2 requested between the halves of the products of stage kt.
    const int nfull = K / TK;
    if (nfull > 0) {
        load(0);
        store(0);
        load(min(1, nfull - 1));
        stage_barrier();
        for (int kt = 0; kt < nfull - 1; ++kt) {
            multiply(kt & 1, 0);
            store((kt + 1) & 1);
            load(min(kt + 2, nfull - 1));
            multiply(kt & 1, 1);
            stage_barrier();
        }
        multiply((nfull - 1) & 1, 0);
        multiply((nfull - 1) & 1, 1);
    }
    if (nfull * TK < K) {  // into the stage that nobody reads any more
        load_masked(nfull);
        store(nfull & 1);
        stage_barrier();
        multiply(nfull & 1, 0);
        multiply(nfull & 1, 1);
    }

    // Eight neighbouring lanes hold the sums of squares of a row.
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        float v = ss[i];
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 4, 64);
        if (xc == 0) ss_red[xr + 64 * i] = v;
    }
    __syncthreads();

    // Element e of accumulator j in lane (q, c) is row 4 q + e, column j of the lane's NC.
    const int p = wn * 16 * NC + NC * c;     // column as laid out; those of a group of four stay together
    const int first = p & ~3;
    if (first >= N - n0) return;
    const int n = n0 + min(first, N - 4 - n0) + (p & 3);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int ml = wm * 32 + 16 * r + 4 * q + e;
            if (m0 + ml >= M) continue;
            const float rinv = (flags & kFlagNorm) ? 1.0f / sqrtf(ss_red[ml] / (float)K + eps) : 1.0f;
            Piece<E, NC> out;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                float y = acc[0][r][j][e] * rinv;
                if (GATED) {
                    const float a = y;
                    y = ((flags & kFlagSilu) ? a / (1.0f + expf(-a)) : a) * (acc[G - 1][r][j][e] * rinv);
                }
                out.set(j, S::narrow(y));
            }
            out.store(Y + (size_t)(m0 + ml) * N + n);
        }
}

template <typename S, bool GATED, int BM>
static hipError_t launch_general_tiled_as(const Call& c) {
    typedef typename S::elem E;
    constexpr int cw = GATED ? TC / 2 : TC;
    dim3 grid((c.N + cw - 1) / cw, (c.M + BM - 1) / BM), block(NTH);
    constexpr size_t lds = (size_t)2 * TK * (BM + TC) * 4 + BM * 4;
    auto kern = general_tiled_kernel<S, GATED, BM>;
    static std::atomic<uint64_t> opted{0};
    if (hipError_t e = allow_large_lds((const void*)kern, lds, opted); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, c.stream, (const E*)c.X, (const E*)c.g, (const E*)c.W1,
                       (const E*)(GATED ? c.W2 : c.W1), (E*)c.Y, c.M, c.K, c.N, c.eps, c.flags);
    return hipGetLastError();
}

template <typename S>
static hipError_t launch_general_tiled_of(const Call& c) {
    switch (c.form.row_groups) {
        case 4: return c.gated ? launch_general_tiled_as<S, true, 64>(c) : launch_general_tiled_as<S, false, 64>(c);
        case 8: return c.gated ? launch_general_tiled_as<S, true, 128>(c) : launch_general_tiled_as<S, false, 128>(c);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_general_tiled(const Call& c, int dtype) {
    if (dtype == PRISM_F32) return launch_general_tiled_of<StoreF32>(c);
    if (dtype == PRISM_F16) return launch_general_tiled_of<StoreF16>(c);
    return launch_general_tiled_of<StoreBf16>(c);
}

}  // namespace prism
