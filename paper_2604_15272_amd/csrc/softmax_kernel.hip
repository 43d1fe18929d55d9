// Softmax followed by a matrix product, Y = softmax(X over k) . W: the paper's running example
// (Figure 1).  The fused program of Figure 1(b) keeps two accumulators in its loop over k, the row
// sum of exp(X) and the product exp(X) . W, and divides after the loop; softmax(X) is never written
// to memory.  Both kernels here have that structure.  What the figure leaves out and a library
// needs is the row maximum: exp(x - max) instead of exp(x), which changes nothing in exact
// arithmetic and keeps every term in (0, 1].  The kernels keep a running maximum per wavefront and rescale their
// accumulators when it moves (so X is read once, streaming under the arithmetic).
//
// Matrix-core kernel (16-bit storage): a workgroup owns 16 rows (one MFMA row group) and 128 columns
// of W; its wavefronts take the 32-deep K-blocks round-robin.  X is K-contiguous, which is the
// layout of an MFMA A operand, so a lane loads its 8 K values of a row straight from memory,
// applies exp and rounds to the storage format; the row sums are a ninth MFMA against ones, so
// numerator and denominator weigh the same rounded values.  W is handled as in the decode kernel (8 x 8 sub-blocks per lane,
// permuted into B operands).  The partial products, sums and maxima of the wavefronts meet in LDS.
// X is the large operand here and the roofline is streaming it from HBM once; what the kernel is
// actually bound by at the paper's shape is the vector pipe (exponentials, conversions, the permutes
// of W, which every workgroup re-reads from the L2 for its 16 rows).
//
// Any shape and storage type: the same with 32-bit weights and sums (softmax_general_kernel).
#include <type_traits>

#include "any_shape.h"
#include "device_utils.h"
#include "prism_internal.h"
#include "w_block.h"

namespace prism {

namespace {

constexpr int TN = 128;  // columns of W per workgroup (matrix-core kernel)
constexpr int KB = 32;   // K depth of one MFMA

}  // namespace

// ---- matrix-core kernel --------------------------------------------------------------------------
// A wavefront walks its K-blocks in chunks of CH.  Per chunk: the chunk's row maxima (from the registers
// the loads landed in), the running maximum, a rescale of the accumulators by 2^((old - new) log2 e) if
// it moved, then exp, row sums and products of the chunk's K-blocks.  The next chunk's X is requested
// before the current one is worked on, so the stream from HBM runs under the arithmetic.
template <typename F, int NW>
__global__ __launch_bounds__(NW * 64) void softmax_rows_kernel(const uint16_t* __restrict__ X,
                                                               const uint16_t* __restrict__ W,
                                                               uint16_t* __restrict__ Y, int M, int K, int N) {
    constexpr int NT = NW * 64;
    constexpr int CPT = 16 * TN / NT;  // columns per thread in the epilogue
    constexpr int TPR = TN / CPT;      // threads per output row
    static_assert(CPT == 2 || CPT == 4 || CPT == 8, "epilogue mapping");
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr int CH = 4;  // K-blocks per wavefront and chunk (even: the W register sets alternate per block)

    extern __shared__ __align__(16) float lds[];  // 16-byte LDS accesses need the alignment said
    float* red = lds;                       // [NW][16][TN]
    float* wave_max = lds + NW * 16 * TN;   // [NW][16]
    float* wave_sum = wave_max + NW * 16;   // [NW][16]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane >> 4, c = lane & 15;
    const int n0 = blockIdx.x * TN, m0 = blockIdx.y * 16;
    const int kblocks = (K + KB - 1) / KB;

    // Descriptors: X from this workgroup's first row to the end of the matrix (rows past M are masked),
    // W from its first column to the end.
    const size_t x_left = ((size_t)(M - m0) * K) * 2;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + (size_t)m0 * K, (u32)(x_left < 0x7FFFFFFFull ? x_left : 0x7FFFFFFFull));
    const size_t w_left = ((size_t)K * N - n0) * 2;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(W + n0, (u32)(w_left < 0x7FFFFFFFull ? w_left : 0x7FFFFFFFull));
    const u32 row_bytes = (u32)N * 2u;
    const bool col_ok = (n0 + 8 * c) < N;
    const u32 w_lane = col_ok ? ((u32)(8 * q) * row_bytes + (u32)(16 * c)) : kOutOfRange;
    const bool row_ok = (m0 + c) < M;
    const u32 x_row = (u32)c * (u32)K * 2u;
    // Whether this lane's eight K values of block ib exist (implies ib < kblocks).  Everything in the loop below is
    // written with selects, not branches: loads whose values are used in a later conditional block get moved
    // into that block by the compiler, next to their use, and then nothing is in flight ahead of the arithmetic.
    auto k_valid = [&](int ib) { return ib * KB + 8 * q < K; };

    f32x4 acc[8], sum_acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -__builtin_inff();  // running maximum of row c over this wavefront's K-blocks so far

    auto load_chunk = [&](u32x4 (&xs)[CH], int i0) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int ib = i0 + u * NW;
            xs[u] = load16(rx, (k_valid(ib) & row_ok) ? x_row + (u32)(ib * KB + 8 * q) * 2u : kOutOfRange);
        }
    };
    auto load_w = [&](WRows& w, int ib) {
        load_w_block(w, rw, (ib < kblocks) ? w_lane + (u32)ib * KB * row_bytes : kOutOfRange, row_bytes);
    };
    WRows w[2];
    auto chunk = [&](const u32x4 (&xs)[CH], int i0) {
        float cm = -__builtin_inff();
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const float mx = F::max8(xs[u]);
            cm = fmaxf(cm, (k_valid(i0 + u * NW) & row_ok) ? mx : -__builtin_inff());
        }
        cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
        cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
        const float m_new = fmaxf(m_run, cm);
        if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
            // Accumulator element i of lane (q, c) belongs to row 4q + i; its factor lives in the lanes of row
            // 4q + i.  Rows that have seen nothing yet keep the factor 1 (their accumulators are zero).
            const float f = (m_run == -__builtin_inff()) ? 1.0f : __builtin_amdgcn_exp2f((m_run - m_new) * kLog2e);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float fi = __shfl(f, 4 * q + i, 64);
                sum_acc[i] *= fi;
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j][i] *= fi;
            }
            m_run = m_new;
        }
        const float shift = row_ok ? -m_run * kLog2e : 0.f;  // a row past M has no maximum: keep the arithmetic finite
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int ib = i0 + u * NW;                // a block past the end: its loads return zeros, a = 0
            load_w(w[(u + 1) & 1], ib + NW);           // the next block's W, into the other register set
            // The loads stay here, a whole block's arithmetic ahead of their use: without the fences the
            // scheduler pulls the next block's permutes up to just behind them.
            __builtin_amdgcn_sched_barrier(0);
            const bool v = k_valid(ib) & row_ok;
            u32x4 a;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const float e0 = __builtin_amdgcn_exp2f(fmaf(F::lo(xs[u][d]), kLog2e, shift));
                const float e1 = __builtin_amdgcn_exp2f(fmaf(F::hi(xs[u][d]), kLog2e, shift));
                a[d] = v ? F::pack(e0, e1) : 0u;
            }
            const WRows& wb = w[u & 1];
            acc[0] = F::mfma_16x16x32(a, b_operand<0>(wb), acc[0]);
            acc[1] = F::mfma_16x16x32(a, b_operand<1>(wb), acc[1]);
            acc[2] = F::mfma_16x16x32(a, b_operand<2>(wb), acc[2]);
            acc[3] = F::mfma_16x16x32(a, b_operand<3>(wb), acc[3]);
            acc[4] = F::mfma_16x16x32(a, b_operand<4>(wb), acc[4]);
            acc[5] = F::mfma_16x16x32(a, b_operand<5>(wb), acc[5]);
            acc[6] = F::mfma_16x16x32(a, b_operand<6>(wb), acc[6]);
            acc[7] = F::mfma_16x16x32(a, b_operand<7>(wb), acc[7]);
            // The row sums ride on the matrix cores too: a ninth product against a block of ones adds up
            // exactly the rounded values the other eight use (every column of the result is the row sum).
            sum_acc = F::mfma_16x16x32(a, ones8<F>(), sum_acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    {
        u32x4 xa[CH], xb[CH];
        load_chunk(xa, wave);
        load_w(w[0], wave);
        // Two chunks per trip of the loop, no exit between them (a chunk past the end adds zeros): see k_valid.
        for (int i0 = wave; i0 < kblocks; i0 += 2 * CH * NW) {
            load_chunk(xb, i0 + CH * NW);
            __builtin_amdgcn_sched_barrier(0);
            chunk(xa, i0);
            load_chunk(xa, i0 + 2 * CH * NW);
            __builtin_amdgcn_sched_barrier(0);
            chunk(xb, i0 + CH * NW);
        }
    }
    // Element i of the sum block in lane (q, c) is row 4q + i (any column c: they are all equal).
    if (c == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wave_sum[wave * 16 + 4 * q + i] = sum_acc[i];
    }
    if (q == 0) wave_max[wave * 16 + c] = m_run;

    // ---- across wavefronts through LDS: every wavefront's partials are relative to its own maximum, so they
    // are rescaled to the common one; then the division (Figure 1(b): Div after the loop).
    // Accumulator j, element i of lane (q, c) is row 4q + i, column 8c + j.
    const int m = tid / TPR;
    const int col = (tid % TPR) * CPT;
    const int n = n0 + col;
    store_acc_tile(red + wave * 16 * TN, TN, q, c, acc);
    __syncthreads();
    float gmax = -__builtin_inff();
#pragma unroll
    for (int w8 = 0; w8 < NW; ++w8) gmax = fmaxf(gmax, wave_max[w8 * 16 + m]);
    float v[CPT], den = 0.f;
#pragma unroll
    for (int e = 0; e < CPT; ++e) v[e] = 0.f;
#pragma unroll
    for (int w8 = 0; w8 < NW; ++w8) {
        const float mw = wave_max[w8 * 16 + m];
        // a wavefront without K-blocks (or a row past M) has maximum -inf and zero partials
        const float f = (mw == -__builtin_inff()) ? 0.f : __builtin_amdgcn_exp2f((mw - gmax) * kLog2e);
        const float* src = red + (w8 * 16 + m) * TN + col;
#pragma unroll
        for (int e = 0; e < CPT; ++e) v[e] = fmaf(f, src[e], v[e]);
        den = fmaf(f, wave_sum[w8 * 16 + m], den);
    }
    const int row = m0 + m;
    if (row < M && n < N) {  // N % 8 == 0 and CPT | 8: all CPT columns valid together
        const float inv = 1.0f / den;
        u32 packed[CPT / 2];
#pragma unroll
        for (int e = 0; e < CPT / 2; ++e) packed[e] = F::pack(v[2 * e] * inv, v[2 * e + 1] * inv);
        uint16_t* out = Y + (size_t)row * N + n;
        if (CPT == 2) *(u32*)out = packed[0];
        if (CPT == 4) *(u32x2*)out = u32x2{packed[0], packed[1]};
        if (CPT == 8) *(u32x4*)out = u32x4{packed[0], packed[1], packed[2 % (CPT / 2)], packed[3 % (CPT / 2)]};
    }
}

template <typename F>
static hipError_t launch_softmax_rows_fmt(const SoftmaxCall& c) {
    constexpr int NW = 8;
    dim3 grid((c.N + TN - 1) / TN, (c.M + 15) / 16), block(NW * 64);
    const size_t lds = (size_t)(NW * 16 * TN + 2 * NW * 16) * sizeof(float);
    auto kern = softmax_rows_kernel<F, NW>;
    static std::atomic<uint64_t> opted{0};
    if (hipError_t e = allow_large_lds((const void*)kern, lds, opted); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, c.stream, (const uint16_t*)c.X, (const uint16_t*)c.W, (uint16_t*)c.Y,
                       c.M, c.K, c.N);
    return hipGetLastError();
}

hipError_t launch_softmax_rows_16bit(const SoftmaxCall& c, bool f16) {
    return f16 ? launch_softmax_rows_fmt<F16>(c) : launch_softmax_rows_fmt<Bf16>(c);
}

// ---- any shape, any storage type --------------------------------------------------------------------
// The frame of the fp32 product kernel (general_kernel.hip): RG groups of 16 rows and 16 * VW columns per workgroup, the
// wavefronts take 32-deep K-blocks round-robin, lane (q, c) holds eight consecutive K values of row c and the same eight rows
// of W at its VW columns.  Products: fp32 storage on the matrix cores in fp32, 16-bit storage on the 16-bit ones, the weight as parts (three of
// bf16 carry it whole, two of f16 to 2^-23 from 2^-29 of the largest weight on and to 2^-51 of the largest below; PartProduct in any_shape.h).
// The softmax rides in the operand: a running maximum per row and wavefront (its accumulators are rescaled when it moves), the exponentials in
// registers, their row sums in fp32 beside the products; the wavefronts' partials meet in LDS relative to the common maximum.
// The kernel this replaces (8 rows x 256 columns, one thread per column, two passes over X) was bound by its serial loads:
// fp32 1624 x 3008 x 352 794 us, now 65 us.
// Bound now: nothing single.  fp32 4096 x 4096 x 128 takes 62 to 69 us, 62 to 69 of 157 TFLOP/s: the matrix cores are busy 46 % of the cycles
// in which a compute unit has a workgroup, beside 17e6 exponentials for every column tile and operands straight from the
// caches.  With few workgroups it is the chain of a wavefront's blocks.  16-bit storage, in parts against the fp32 instructions: f16
// 372 x 14151 x 393 112 -> 81 us, and with one block at a time bf16 2048 x 2049 x 513 96 -> 51, 4000 x 513 x 129 27.3 -> 13.1 (the
// exponentials and the weights' parts bound it).
template <typename S, int RG, int VW, bool AHEAD>
__global__ __launch_bounds__(general_max_waves(RG, VW) * 64) void softmax_general_kernel(const typename S::elem* __restrict__ X,
                                                                            const typename S::elem* __restrict__ W,
                                                                            typename S::elem* __restrict__ Y, int M, int K,
                                                                            int N) {
    typedef typename S::elem E;
    constexpr int XV = 8, KBG = 4 * XV, TNG = 16 * VW;
    struct Blk {
        Piece<E, XV> x[RG];
        Piece<E, VW> w[XV];
    };
    extern __shared__ __align__(16) float lds[];
    const int nw = blockDim.x >> 6;
    float* red = lds;                        // [waves][16][TNG], one row group at a time
    float* wave_max = lds + nw * 16 * TNG;   // [waves][16 * RG]
    float* wave_sum = wave_max + nw * 16 * RG;
    float* weight = wave_sum + nw * 16 * RG;    // [waves][16 * RG]
    float* total = weight + nw * 16 * RG;       // [16 * RG]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c = lane & 15;
    const int n0 = blockIdx.x * TNG, m0 = blockIdx.y * (16 * RG);
    // Columns past the right edge: the group starts at N - VW; rows past M: row M - 1 again (not stored).
    const E* w_lane = W + (size_t)(XV * q) * N + n0 + min(VW * c, N - VW - n0);
    const E* x_lane[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) x_lane[r] = X + (size_t)min(m0 + 16 * r + c, M - 1) * K + XV * q;

    constexpr bool PARTS = sizeof(E) == 2;
    constexpr int NA = std::is_same<S, StoreF16>::value ? 2 : 1;
    // Weights in f16 parts are relative to exp(BELOW) of the largest (PartProduct): all of them, and so their sums.
    constexpr float BELOW = std::is_same<S, StoreF16>::value ? PartProduct<StoreF16>::kLogWeight : 0.f;
    f32x4 acc[RG][VW][NA];
    float m_run[RG], l_run[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        m_run[r] = -__builtin_inff();
        l_run[r] = 0.f;
#pragma unroll
        for (int j = 0; j < VW; ++j)
#pragma unroll
            for (int a = 0; a < NA; ++a) acc[r][j][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto load = [&](Blk& b, int kb) __attribute__((always_inline)) {
        const size_t k = (size_t)kb * KBG;
#pragma unroll
        for (int r = 0; r < RG; ++r) b.x[r].load(x_lane[r] + k);
#pragma unroll
        for (int i = 0; i < XV; ++i) b.w[i].load(w_lane + (k + i) * N);
    };
    // The block that crosses the end of K: past it x = -inf (weight 0) and w = 0.
    auto load_masked = [&](Blk& b, int kb) __attribute__((always_inline)) {
        const size_t k = (size_t)kb * KBG;
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            const bool ok = k + XV * q + i < (size_t)K;
#pragma unroll
            for (int r = 0; r < RG; ++r) b.x[r].set(i, ok ? x_lane[r][k + i] : S::narrow(-__builtin_inff()));
#pragma unroll
            for (int j = 0; j < VW; ++j) b.w[i].set(j, S::narrow(0.f));
            if (ok) b.w[i].load(w_lane + (k + i) * N);
        }
    };
    auto multiply = [&](const Blk& b) __attribute__((always_inline)) {
        float shift[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            float cm = S::widen(b.x[r].at(0));
#pragma unroll
            for (int i = 1; i < XV; ++i) cm = fmaxf(cm, S::widen(b.x[r].at(i)));
            cm = fmaxf(cm, __shfl_xor(cm, 16, 64));
            cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
            const float m_new = fmaxf(m_run[r], cm - BELOW);
            if (__builtin_amdgcn_ballot_w64(m_new != m_run[r]) != 0) {
                // Element e of an accumulator in lane (q, c) belongs to row 4 q + e, whose factor lives in the lanes of that
                // row.  A row that has seen nothing yet keeps the factor 1.
                const float f = (m_run[r] == -__builtin_inff()) ? 1.0f : expf(m_run[r] - m_new);
                l_run[r] *= f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float fe = __shfl(f, 4 * q + e, 64);
#pragma unroll
                    for (int j = 0; j < VW; ++j)
#pragma unroll
                        for (int a = 0; a < NA; ++a) acc[r][j][a][e] *= fe;
                }
                m_run[r] = m_new;
            }
            // Nothing but -inf so far: those have weight 0 (a NaN among them stays one).
            shift[r] = (m_run[r] == -__builtin_inff()) ? 0.f : m_run[r];
        }
        if constexpr (PARTS) {
            typedef PartProduct<S> PP;
            constexpr int P = PP::kFloatParts;
            u32x4 a[RG][P];
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                float v[XV];
#pragma unroll
                for (int i = 0; i < XV; ++i) {
                    v[i] = expf(S::widen(b.x[r].at(i)) - shift[r]);
                    l_run[r] += v[i];
                }
                PP::template split8<P>(v, a[r]);
            }
#pragma unroll
            for (int j = 0; j < VW; ++j) {
                const u32x4 w = column_operand(b.w, j);
#pragma unroll
                for (int r = 0; r < RG; ++r)
#pragma unroll
                    for (int p = P - 1; p >= 0; --p) {
                        f32x4& t = acc[r][j][NA == 1 ? 0 : p];
                        t = PP::mfma(a[r][p], w, t);
                    }
            }
        } else {
#pragma unroll
            for (int i = 0; i < XV; ++i) {
                float a[RG];
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    a[r] = expf(S::widen(b.x[r].at(i)) - shift[r]);
                    l_run[r] += a[r];
                }
#pragma unroll
                for (int j = 0; j < VW; ++j) {
                    const float w = S::widen(b.w[i].at(j));
#pragma unroll
                    for (int r = 0; r < RG; ++r) acc[r][j][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], w, acc[r][j][0], 0, 0, 0);
                }
            }
        }
    };
    // AHEAD: two named blocks in turn, without a condition between a load and its use (general_kernel.hip), for one round of workgroups with a
    // deep K, which has nothing else to wait under (bf16 8 x 16383 x 67 53.2 us, 57.5 without; fp32 4096 x 4096 x 128 62.7 / 63.7).  Elsewhere
    // one block at a time: in half the registers more wavefronts share a SIMD (bf16 4000 x 513 x 129 20.6 -> 13.3, 2048 x 2049 x 513 65 -> 52, fp32
    // 1624 x 3008 x 352 74.6 -> 65.1, 45 x 512 x 192 5.9 -> 5.3).
    const int nfull = K / KBG;
    if constexpr (!AHEAD) {
        for (int kb = wave; kb < nfull; kb += nw) {
            Blk b;
            load(b, kb);
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
    if (nfull * KBG < K && wave == nfull % nw) {
        Blk tail;
        load_masked(tail, nfull);
        multiply(tail);
    }

    auto store_group = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < VW; ++j) {
                float t = acc[r][j][0][e];
                if constexpr (PARTS) t = PartProduct<S>::sum(acc[r][j], e);
                red[(wave * 16 + 4 * q + e) * TNG + VW * c + j] = t;
            }
    };
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        l_run[r] += __shfl_xor(l_run[r], 16, 64);
        l_run[r] += __shfl_xor(l_run[r], 32, 64);
        if (q == 0) {
            wave_max[wave * (16 * RG) + 16 * r + c] = m_run[r];
            wave_sum[wave * (16 * RG) + 16 * r + c] = l_run[r];
        }
    }
    store_group(0);
    __syncthreads();
    // The wavefronts' weights and the denominators: once per row where a thread has four outputs (bf16 4000 x 513 x 129
    // 28.7 -> 27.3 us), else by each output for itself (two: fp32 1624 x 3008 x 352 74.9 us, 75.8 us once per row; one: fp32 64 x
    // 256 x 128 4.7 / 6.3 us).
    constexpr bool PER_ROW = RG * VW >= 8;
    auto row_max = [&](int row) __attribute__((always_inline)) {
        float m = -__builtin_inff();
        for (int w = 0; w < nw; ++w) m = fmaxf(m, wave_max[w * (16 * RG) + row]);
        return m;
    };
    auto wave_weight = [&](int w, int row, float gmax) __attribute__((always_inline)) {
        const float mw = wave_max[w * (16 * RG) + row];
        return (mw == -__builtin_inff()) ? 0.f : expf(mw - gmax);  // 0: a wavefront that saw nothing
    };
    if (PER_ROW) {
        if (tid < nw * 16 * RG) {
            const int row = tid % (16 * RG), mine = tid / (16 * RG);
            const float gmax = row_max(row);
            float den = 0.f;
            for (int w = 0; w < nw; ++w) {
                const float f = wave_weight(w, row, gmax);
                den = fmaf(f, wave_sum[w * (16 * RG) + row], den);
                if (w == mine) weight[tid] = f;
            }
            if (mine == 0) total[row] = den;
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        if (r > 0) {
            __syncthreads();
            store_group(r);
            __syncthreads();
        }
        for (int o = tid; o < 16 * TNG; o += blockDim.x) {
            const int row = o / TNG, col = o % TNG;
            const int m = m0 + 16 * r + row;
            const int first = col / VW * VW;
            if (m >= M || first >= N - n0) continue;
            const int n = n0 + min(first, N - VW - n0) + col % VW;
            const float gmax = PER_ROW ? 0.f : row_max(16 * r + row);
            float v = 0.f, den = PER_ROW ? total[16 * r + row] : 0.f;
            for (int w = 0; w < nw; ++w) {
                const int at = w * (16 * RG) + 16 * r + row;
                const float f = PER_ROW ? weight[at] : wave_weight(w, 16 * r + row, gmax);
                v = fmaf(f, red[(w * 16 + row) * TNG + col], v);
                if (!PER_ROW) den = fmaf(f, wave_sum[at], den);
            }
            // Relative to a maximum that was still to rise, sums of very large values of W can pass the type's range although the
            // result does not: such an output is summed once more, one product after the other, with the maximum known.
            if (__builtin_expect(!(fabsf(v) <= kFloatMax), 0)) {
                const float shift = row_max(16 * r + row);
                if (den <= kFloatMax && shift > -__builtin_inff()) {  // (else a NaN or an infinity of X: the output is a NaN)
                    v = 0.f;
#pragma unroll 8
                    for (int k = 0; k < K; ++k)
                        v = fmaf(expf(S::widen(X[(size_t)m * K + k]) - shift), S::widen(W[(size_t)k * N + n]), v);
                }
            }
            Y[(size_t)m * N + n] = S::narrow(v / den);
        }
    }
}

template <typename S, int RG, int VW, bool AHEAD>
static hipError_t launch_softmax_general_as(const SoftmaxCall& c) {
    typedef typename S::elem E;
    constexpr int tn = 16 * VW;
    const int waves = c.form.waves;
    dim3 grid((c.N + tn - 1) / tn, (c.M + 16 * RG - 1) / (16 * RG)), block(waves * 64);
    const size_t lds = ((size_t)waves * (16 * tn + 3 * 16 * RG) + 16 * RG) * sizeof(float);
    auto kern = softmax_general_kernel<S, RG, VW, AHEAD>;
    static std::atomic<uint64_t> opted{0};
    if (hipError_t e = allow_large_lds((const void*)kern, lds, opted); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, block, lds, c.stream, (const E*)c.X, (const E*)c.W, (E*)c.Y, c.M, c.K, c.N);
    return hipGetLastError();
}

template <typename S, bool AHEAD>
static hipError_t launch_softmax_general_form(const SoftmaxCall& c) {
    constexpr bool wide = sizeof(typename S::elem) == 4;
    switch (c.form.row_groups * 10 + c.form.cols) {
        case 11: return launch_softmax_general_as<S, 1, 1, AHEAD>(c);
        case 14: return launch_softmax_general_as<S, 1, 4, AHEAD>(c);
        case 18: if constexpr (!wide) return launch_softmax_general_as<S, 1, 8, AHEAD>(c); else break;
        case 21: return launch_softmax_general_as<S, 2, 1, AHEAD>(c);
        case 24: return launch_softmax_general_as<S, 2, 4, AHEAD>(c);
    }
    return hipErrorInvalidValue;
}

template <typename S> static hipError_t launch_softmax_general(const SoftmaxCall& c) {
    return c.ahead ? launch_softmax_general_form<S, true>(c) : launch_softmax_general_form<S, false>(c);
}

hipError_t launch_softmax_simple(const SoftmaxCall& c, int dtype) {
    if (dtype == PRISM_F32) return launch_softmax_general<StoreF32>(c);
    if (dtype == PRISM_F16) return launch_softmax_general<StoreF16>(c);
    return launch_softmax_general<StoreBf16>(c);
}

}  // namespace prism
