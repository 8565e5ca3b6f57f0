// Hidden layers of the evaluation pass (the loss of the averaged model, Sec. 4.2): one dense product
// of all samples of the pass with one weight matrix, fp32 operands, on the bf16 matrix cores.
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate, and this pass is bound by them.
// An fp32 number is the sum of three bf16 numbers exactly (8 + 8 + 8 of its 24 significant bits, each
// part rounded to nearest), products of bf16 numbers are exact in fp32, and of the nine products of
// two such sums the three smallest reach 2^-24 of the whole together (the second part is at most 2^-8,
// the third 2^-17 of the number's power of two), 2^-27.4 in the mean square: once per product, one fp32
// rounding at most.
// So x w = x1 w1 + (x1 w2 + x2 w1 + x1 w3 + x2 w2 + x3 w1): six bf16 instructions in place of
// the fp32 ones' sixteenfold cost.  x1 w1 is added up in an accumulator of its own and the rest, 2^-8
// as large, in a second one, so that only one rounding per 16 products is of the size of the result:
// fewer than the fp32 instructions make (one per 4 products).  Measured against 64 bits the loss is
// off by 1.3e-8 to 3.0e-8 of itself where forward_kernel's is by 1.6e-8 to 3.7e-8 (what both share is
// the softmax's).  Inputs that are bf16 numbers already
// (the data of bf16 runs, first layer) are their own first part: three products.
#include "lc_internal.h"
#include "lc_mma.h"

namespace lc {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct EvalArgs {
    const float* A;       // [rows][dp_in], zero beyond d_in
    const float* X;       // the averaged model
    float* out;           // [rows][dp_out]
    int64_t w_off, b_off;
    int d_in, d_out, dp_in, dp_out;
    int n_col_blocks;
    int64_t total_blocks;
};

// x = p1 + p2 + p3.  The clamps keep a number that would round to infinity finite (its rest then goes
// to the next part) and send an infinity to the last part, with finite parts before it.  An infinity
// still meets parts of the other operand that are zero or of the other sign, so a sum that is not
// finite is formed again from the operands themselves (see the end of eval_layer_kernel).
constexpr float kMaxBf16 = 3.38953139e38f;
__device__ __forceinline__ void split3(const float (&x)[8], bf16x8& p1, bf16x8& p2, bf16x8& p3) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p1[e] = static_cast<bf16_t>(__builtin_amdgcn_fmed3f(x[e], -kMaxBf16, kMaxBf16));
        const float r = x[e] - static_cast<float>(p1[e]);
        p2[e] = static_cast<bf16_t>(__builtin_amdgcn_fmed3f(r, -kMaxBf16, kMaxBf16));
        p3[e] = static_cast<bf16_t>(r - static_cast<float>(p2[e]));
    }
}

// One workgroup = BM rows x BN columns, 2 x 2 wavefronts, reduction in steps of 32.  A step's tiles
// are loaded as fp32 one step ahead, split in registers and written to LDS as planes of 8-element
// operand fragments: [plane][8-deep reduction piece][row or column], 16 bytes each.  Two
// workgroups per CU, so that one multiplies while the other splits.  The pieces are 32 bytes apart
// modulo the 128 bytes the banks cover: the 8 lanes of a store phase (two rows x 4 pieces) then hit
// 8 different 16-byte slots.
// NA: parts of A (1: A is exactly representable in bf16).
template <int BM, int BN, int NA>
__global__ __launch_bounds__(256, 2) void eval_layer_kernel(EvalArgs a) {
    constexpr int TM = BM / 64, TN = BN / 64;             // 32 x 32 tiles per wavefront
    constexpr int kPieceA = BM * 16 + 32, kPieceB = BN * 16 + 32;   // bytes
    constexpr int UA = BM * 4 / 256, UB = BN / 64;        // 8-element fragments a thread loads per step
    __shared__ __attribute__((aligned(16))) char as[NA * 4 * kPieceA];
    __shared__ __attribute__((aligned(16))) char bs[3 * 4 * kPieceB];

    const int64_t logical = xcd_logical_block(a.total_blocks);
    if (logical < 0) return;
    const int64_t row0 = logical / a.n_col_blocks * BM;
    const int c0 = static_cast<int>(logical % a.n_col_blocks) * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, j = lane & 31, q = lane >> 5;

    const float* W = a.X + a.w_off;
    const float* arow[UA];
#pragma unroll
    for (int u = 0; u < UA; ++u) arow[u] = a.A + (row0 + (tid >> 2) + 64 * u) * a.dp_in + 8 * (tid & 3);
    int bcol[UB];   // (columns past the end read the last one; they are never stored)
#pragma unroll
    for (int u = 0; u < UB; ++u) bcol[u] = c0 + lane + 64 * u < a.d_out ? c0 + lane + 64 * u : a.d_out - 1;

    float ra[UA][8], rb[UB][8];
    auto load_step = [&](int k0) {
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            const Frag<float> f = load8(arow[u] + k0);
#pragma unroll
            for (int e = 0; e < 8; ++e) ra[u][e] = f.v[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {   // rows past d_in meet columns of A that are zero
            const int k = k0 + 8 * wave + e;
            const float* wr = W + static_cast<int64_t>(k < a.d_in ? k : a.d_in - 1) * a.d_out;
#pragma unroll
            for (int u = 0; u < UB; ++u) rb[u][e] = wr[bcol[u]];
        }
    };
    auto store_step = [&]() {
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            const int at = (tid & 3) * kPieceA + ((tid >> 2) + 64 * u) * 16;
            bf16x8 p1, p2, p3;
            if constexpr (NA == 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) p1[e] = static_cast<bf16_t>(ra[u][e]);
            } else {
                split3(ra[u], p1, p2, p3);
                *reinterpret_cast<bf16x8*>(as + 4 * kPieceA + at) = p2;
                *reinterpret_cast<bf16x8*>(as + 8 * kPieceA + at) = p3;
            }
            *reinterpret_cast<bf16x8*>(as + at) = p1;
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int at = wave * kPieceB + (lane + 64 * u) * 16;
            bf16x8 p1, p2, p3;
            split3(rb[u], p1, p2, p3);
            *reinterpret_cast<bf16x8*>(bs + at) = p1;
            *reinterpret_cast<bf16x8*>(bs + 4 * kPieceB + at) = p2;
            *reinterpret_cast<bf16x8*>(bs + 8 * kPieceB + at) = p3;
        }
    };

    f32x16 hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int n = 0; n < TN; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) hi[m][n][r] = lo[m][n][r] = 0.f;

    load_step(0);
    for (int k0 = 0; k0 < a.dp_in; k0 += 32) {
        __syncthreads();   // every wavefront is done with the tiles of the step before
        store_step();
        __syncthreads();
        load_step(k0 + 32 < a.dp_in ? k0 + 32 : k0);   // (the last step's are never used)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 fa[NA][TM], fb[3][TN];
#pragma unroll
            for (int p = 0; p < NA; ++p)
#pragma unroll
                for (int m = 0; m < TM; ++m)
                    fa[p][m] = *reinterpret_cast<const bf16x8*>(as + (4 * p + 2 * s + q) * kPieceA + (wm * BM / 2 + 32 * m + j) * 16);
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int n = 0; n < TN; ++n)
                    fb[p][n] = *reinterpret_cast<const bf16x8*>(bs + (4 * p + 2 * s + q) * kPieceB + (wn * BN / 2 + 32 * n + j) * 16);
#pragma unroll
            for (int pa = 0; pa < NA; ++pa)
#pragma unroll
                for (int pb = 0; pa + pb < 3; ++pb)
#pragma unroll
                    for (int m = 0; m < TM; ++m)
#pragma unroll
                        for (int n = 0; n < TN; ++n) {
                            f32x16& acc = pa + pb == 0 ? hi[m][n] : lo[m][n];
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa][m], fb[pb][n], acc, 0, 0, 0);
                        }
        }
    }

    // bias, ReLU; register r of a 32 x 32 tile holds row 8 (r / 4) + 4 q + r % 4, column j
    static_assert(TM * TN * 16 <= 64, "one bit per output of a lane");
    unsigned long long redo = 0;   // outputs whose sum is not finite
#pragma unroll
    for (int n = 0; n < TN; ++n) {
        const int c = c0 + wn * BN / 2 + 32 * n + j;
        if (c >= a.d_out) continue;
        const float bias = a.X[a.b_off + c];
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = row0 + wm * BM / 2 + 32 * m + 8 * (r / 4) + 4 * q + r % 4;
                const float z = (hi[m][n][r] + lo[m][n][r]) + bias;
                if (!isfinite(z)) redo |= 1ull << ((m * TN + n) * 16 + r);
                a.out[row * a.dp_out + c] = z > 0.f ? z : 0.f;
            }
    }
    // Infinities, NaN and overflows: the products of the parts can turn an infinite sum into NaN (infinity
    // times a part that is zero, or infinite parts of both signs; a zero of A past d_in times the row
    // read in place of one that does not exist), never into a finite one.  Models that diverged only.
    while (redo) {
        const int bit = __builtin_ctzll(redo), r = bit & 15, m = bit / (16 * TN), n = bit / 16 % TN;
        redo &= redo - 1;
        const int c = c0 + wn * BN / 2 + 32 * n + j;
        const int64_t row = row0 + wm * BM / 2 + 32 * m + 8 * (r / 4) + 4 * q + r % 4;
        const float* x = a.A + row * a.dp_in;
        float z = 0.f;
#pragma unroll 1
        for (int k = 0; k < a.d_in; ++k) z = fmaf(x[k], W[static_cast<int64_t>(k) * a.d_out + c], z);
        z += a.X[a.b_off + c];
        a.out[row * a.dp_out + c] = z > 0.f ? z : 0.f;
    }
}

template <int BM, int BN>
void launch_eval(const EvalArgs& a, bool exact_bf16, unsigned grid, hipStream_t s) {
    if (exact_bf16) hipLaunchKernelGGL((eval_layer_kernel<BM, BN, 1>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((eval_layer_kernel<BM, BN, 3>), dim3(grid), dim3(256), 0, s, a);
}

}  // namespace

// Hidden layers of a pass with more than 256 tiles of 64 x 64 outputs; smaller ones are bound by the
// latency of their reduction, which forward_kernel splits over its wavefronts (3072-1024-1024-10:
// 1000 samples 169 us against 178 here, 4000 samples 344 against 260; 1000-500-10, 500 samples: 45
// against 64).
bool eval_layer_ok(const lc_handle* h, int l) {
    const int64_t tiles = static_cast<int64_t>(h->eval.G) * 2 * ((h->layer[l].d_out + 63) / 64);
    return l < h->L && tiles > 256;
}

// 128 x 128 outputs per workgroup (half the LDS traffic per product) once that fills the chip's 512
// places one and a half times in two rounds, else 64 x 64: 8192 samples through 3072-2048-2048-2048-10
// in bf16 runs 1197 us with the large tile, 1554 with the small one (2090 with forward_kernel);
// 784-256-10 97 and 77 us (83).
hipError_t launch_eval_layer(lc_handle* h, int l) {
    const ActSet& S = h->eval;
    const LayerGeom& g = h->layer[l];
    EvalArgs a;
    a.A = static_cast<const float*>(S.a_bm[l - 1]);
    a.X = h->xbar;
    a.out = static_cast<float*>(S.a_bm[l]);
    a.w_off = g.w_off;
    a.b_off = g.b_off;
    a.d_in = g.d_in;
    a.d_out = g.d_out;
    a.dp_in = g.dp_in;
    a.dp_out = g.dp_out;
    const bool exact_bf16 = l == 1 && h->md.gemm == LC_GEMM_BF16;   // the data are bf16 numbers
    const int64_t rows = static_cast<int64_t>(S.G) * 128;
    const bool wide = rows / 128 * ((g.d_out + 127) / 128) >= 384;
    const int bt = wide ? 128 : 64;
    a.n_col_blocks = (g.d_out + bt - 1) / bt;
    a.total_blocks = rows / bt * a.n_col_blocks;
    const unsigned grid = static_cast<unsigned>((a.total_blocks + kXcds - 1) / kXcds * kXcds);
    if (wide) launch_eval<128, 128>(a, exact_bf16, grid, h->stream);
    else launch_eval<64, 64>(a, exact_bf16, grid, h->stream);
    return hipGetLastError();
}

}  // namespace lc
