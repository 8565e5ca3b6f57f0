// Device-side building blocks shared by the MLP kernels: MFMA operand fragments for bf16 and
// fp32 operands, their loads, stores and conversions, weight-row access helpers and the
// XCD-aware block index.  Internal linkage: every translation unit gets its own copy.
#pragma once
#include "lc_internal.h"

namespace lc {
namespace {

// ------------------------------------------------------------------ fragments

template <typename OT>
struct Frag;
template <>
struct Frag<float> {
    float v[8];
};
template <>
struct Frag<bf16_t> {
    bf16x8 v;
};

__device__ __forceinline__ Frag<float> load8(const float* p) {
    Frag<float> f;
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    f.v[0] = a.x; f.v[1] = a.y; f.v[2] = a.z; f.v[3] = a.w;
    f.v[4] = b.x; f.v[5] = b.y; f.v[6] = b.z; f.v[7] = b.w;
    return f;
}
__device__ __forceinline__ Frag<bf16_t> load8(const bf16_t* p) {
    Frag<bf16_t> f;
    f.v = *reinterpret_cast<const bf16x8*>(p);
    return f;
}

// A lane's 8 values of a fragment that is laid out in fragment order (see kFragElems).
__device__ __forceinline__ Frag<float> load_frag(const float* p, int lane) {
    Frag<float> f;
    const float4 a = *reinterpret_cast<const float4*>(p + 4 * lane);
    const float4 b = *reinterpret_cast<const float4*>(p + 256 + 4 * lane);
    f.v[0] = a.x; f.v[1] = a.y; f.v[2] = a.z; f.v[3] = a.w;
    f.v[4] = b.x; f.v[5] = b.y; f.v[6] = b.z; f.v[7] = b.w;
    return f;
}
__device__ __forceinline__ Frag<bf16_t> load_frag(const bf16_t* p, int lane) { return load8(p + 8 * lane); }

// Marks the point where prefetched registers are consumed.  Without it the compiler moves the
// conversion of a prefetched weight row up to its load, which makes every trip wait for the loads
// it has just issued (loads retire in order) and turns the prefetch queue into a plain load.
__device__ __forceinline__ void consume_here(float4& x) {
    asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
}
__device__ __forceinline__ void consume_here(Frag<float>& f) {
    asm volatile("" : "+v"(f.v[0]), "+v"(f.v[1]), "+v"(f.v[2]), "+v"(f.v[3]), "+v"(f.v[4]), "+v"(f.v[5]),
                      "+v"(f.v[6]), "+v"(f.v[7]));
}
__device__ __forceinline__ void consume_here(Frag<bf16_t>& f) {
    f32x4 t = __builtin_bit_cast(f32x4, f.v);
    asm volatile("" : "+v"(t));
    f.v = __builtin_bit_cast(bf16x8, t);
}

__device__ __forceinline__ void pack8(Frag<float>& f, const float (&x)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f.v[e] = x[e];
}
__device__ __forceinline__ void pack8(Frag<bf16_t>& f, const float (&x)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f.v[e] = static_cast<bf16_t>(x[e]);  // round to nearest even
}

__device__ __forceinline__ f32x4 mma8(const Frag<float>& a, const Frag<float>& b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[e], b.v[e], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ f32x4 mma8(const Frag<bf16_t>& a, const Frag<bf16_t>& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

// operand fragments of the 16-deep product: 4 consecutive reduction indices per lane
template <typename OT>
struct Frag4;
template <>
struct Frag4<float> {
    float v[4];
};
template <>
struct Frag4<bf16_t> {
    bf16x4 v;
};
__device__ __forceinline__ Frag4<float> load4(const float* p) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    return Frag4<float>{{a.x, a.y, a.z, a.w}};
}
__device__ __forceinline__ Frag4<bf16_t> load4(const bf16_t* p) {
    Frag4<bf16_t> f;
    f.v = *reinterpret_cast<const bf16x4*>(p);
    return f;
}
__device__ __forceinline__ void pack4(Frag4<float>& f, float a, float b, float c, float d) {
    f.v[0] = a; f.v[1] = b; f.v[2] = c; f.v[3] = d;
}
__device__ __forceinline__ void pack4(Frag4<bf16_t>& f, float a, float b, float c, float d) {
    f.v[0] = static_cast<bf16_t>(a); f.v[1] = static_cast<bf16_t>(b);
    f.v[2] = static_cast<bf16_t>(c); f.v[3] = static_cast<bf16_t>(d);
}
__device__ __forceinline__ f32x4 mma4(const Frag4<float>& a, const Frag4<float>& b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[e], b.v[e], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ f32x4 mma4(const Frag4<bf16_t>& a, const Frag4<bf16_t>& b, f32x4 c) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a.v), __builtin_bit_cast(s16x4, b.v), c,
                                                     0, 0, 0);
}

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return static_cast<float>(x); }

template <typename OT>
__device__ __forceinline__ void store4(OT* p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
    bf16x4 v;
    v[0] = static_cast<bf16_t>(a); v[1] = static_cast<bf16_t>(b);
    v[2] = static_cast<bf16_t>(c); v[3] = static_cast<bf16_t>(d);
    *reinterpret_cast<bf16x4*>(p) = v;
}

// 8 consecutive outputs at a 16-byte aligned address
__device__ __forceinline__ void store8(float* p, const float (&y)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(y[0], y[1], y[2], y[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(y[4], y[5], y[6], y[7]);
}
__device__ __forceinline__ void store8(bf16_t* p, const float (&y)[8]) {
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = static_cast<bf16_t>(y[i]);
    *reinterpret_cast<bf16x8*>(p) = v;
}

__device__ __forceinline__ void store_frag(float* p, int lane, const float (&y)[8]) {
    *reinterpret_cast<float4*>(p + 4 * lane) = make_float4(y[0], y[1], y[2], y[3]);
    *reinterpret_cast<float4*>(p + 256 + 4 * lane) = make_float4(y[4], y[5], y[6], y[7]);
}
__device__ __forceinline__ void store_frag(bf16_t* p, int lane, const float (&y)[8]) { store8(p + 8 * lane, y); }

// Four consecutive floats of a weight row, zero outside [0, d_out).  When the
// state of all replicas is far larger than the caches, each weight is touched
// once per kernel and the loads and stores carry the non-temporal hint; small
// models, whose weights stay cache-resident between kernels, use plain accesses.
__device__ __forceinline__ float4 load_w4(const float* row, int c, int d_out, bool vec, bool stream) {
    if (vec && c + 3 < d_out) {
        if (!stream) return *reinterpret_cast<const float4*>(row + c);
        const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(row + c));
        return make_float4(t[0], t[1], t[2], t[3]);
    }
    // unaligned or ragged rows, element by element.  (Loading unconditionally from clamped
    // positions instead was measured and is slower: the cost of these loads grows with the
    // number of active lanes, and most lanes are past the end of a narrow row.)
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < d_out) r.x = row[c];
    if (c + 1 < d_out) r.y = row[c + 1];
    if (c + 2 < d_out) r.z = row[c + 2];
    if (c + 3 < d_out) r.w = row[c + 3];
    return r;
}
__device__ __forceinline__ void store_w4(float* row, int c, int d_out, bool vec, bool stream, float4 v) {
    if (vec && c + 3 < d_out) {
        if (stream) __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4*>(row + c));
        else *reinterpret_cast<float4*>(row + c) = v;
        return;
    }
    if (c < d_out) row[c] = v.x;
    if (c + 1 < d_out) row[c + 1] = v.y;
    if (c + 2 < d_out) row[c + 2] = v.z;
    if (c + 3 < d_out) row[c + 3] = v.w;
}

// Row `row` of a d_in x d_out matrix, columns c .. c+3, zero beyond either end -- without a branch
// around the loads (rows past the end read the last row and are zeroed afterwards).
__device__ __forceinline__ float4 load_w4_rows(const float* base, int row, int d_in, int c, int d_out, bool vec,
                                               bool stream) {
    const int rr = row < d_in ? row : d_in - 1;
    const float4 x = load_w4(base + static_cast<int64_t>(rr) * d_out, c, d_out, vec, stream);
    return row < d_in ? x : make_float4(0.f, 0.f, 0.f, 0.f);
}

// Weight access mode of a kernel instance.  kWGeneric checks every element against the row end
// (any d_out, any alignment).  kWVector* are for layers whose rows are 16-byte aligned and a
// multiple of 64 columns long: every access is one unconditional 16-byte instruction, which lets
// the compiler issue a trip's loads back to back with no control flow between them.
// kWRagged does the same for every other layer of at least 64 columns.  A load is one unconditional
// 16-byte instruction at 4-byte alignment (which global memory instructions take); in the last
// column chunk it may run over the end of the row, by at most 63 columns: into the next row, or
// behind the last row into the layer's biases, of which there are at least 64 -- always inside the
// replica's own parameters.  What it finds there is never used: the kernels zero those columns
// where they are an operand of a sum, and the stores stop at the row end.  Such rows share cache
// lines with their neighbours, so they are never accessed with the streaming hint (with it:
// 3072-1500-1000-100, 16 workers, batch 100: 2887 instead of 2671 us for 5 steps; 3072-2000x3-10, 32
// workers, batch 32: 9286 instead of 8784).
constexpr int kWGeneric = 0, kWVector = 1, kWVectorStream = 2, kWRagged = 3;
typedef f32x4 f32x4_u __attribute__((aligned(4)));   // four floats at any float address

template <int WM>
__device__ __forceinline__ float4 load_wm(const float* row, int c, int d_out, bool vec) {
    if constexpr (WM == kWVector) {
        return *reinterpret_cast<const float4*>(row + c);
    } else if constexpr (WM == kWVectorStream) {
        const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(row + c));
        return make_float4(t[0], t[1], t[2], t[3]);
    } else if constexpr (WM == kWRagged) {
        const f32x4 t = *reinterpret_cast<const f32x4_u*>(row + c);
        return make_float4(t[0], t[1], t[2], t[3]);
    } else {
        return load_w4(row, c, d_out, vec, false);
    }
}
template <int WM>
__device__ __forceinline__ void store_wm(float* row, int c, int d_out, bool vec, float4 v) {
    if constexpr (WM == kWVector) {
        *reinterpret_cast<float4*>(row + c) = v;
    } else if constexpr (WM == kWVectorStream) {
        __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4*>(row + c));
    } else if constexpr (WM == kWRagged) {
        if (c + 3 < d_out) {
            *reinterpret_cast<f32x4_u*>(row + c) = f32x4{v.x, v.y, v.z, v.w};
        } else {
            if (c < d_out) row[c] = v.x;
            if (c + 1 < d_out) row[c + 1] = v.y;
            if (c + 2 < d_out) row[c + 2] = v.z;
        }
    } else {
        store_w4(row, c, d_out, vec, false, v);
    }
}

// The momentum-SGD update with its roundings spelled out: v' = fma(beta, v, fma(wd, w, g)) and
// w' = fma(-lr, v', w).  Kernels whose results are compared bit for bit (the backward kernel, the
// tau = 1 first-layer kernel, the averaging kernels that form x_bar - lr v themselves) must not
// leave the choice of which products are fused to the compiler's contraction pass.
// Softmax cross-entropy of one sample from e_c = exp(z_c - max z), without the cancellation of
// "p_y - 1" and "log(sum)" when the label's class holds almost all of the mass (a well-fitted
// sample: p_y = 1 - 1e-5 in fp32 leaves three digits of p_y - 1).  With s the sum of e_c over the
// classes OTHER than the label y:
//     p_y - 1 = -s / (s + e_y),      -log p_y = log1p(s / e_y)   (while s < e_y; else the plain form).
__device__ __forceinline__ float xent_loss(float s_other, float e_y, float zy_minus_max) {
    return s_other < e_y ? log1pf(s_other / e_y) : logf(s_other + e_y) - zy_minus_max;
}
__device__ __forceinline__ float xent_delta(float e_c, bool is_label, float s_other, float inv_sum) {
    return (is_label ? -s_other : e_c) * inv_sum;
}

__device__ __forceinline__ float momentum_update(float beta, float v, float g, float wd, float w) {
    return __builtin_fmaf(beta, v, __builtin_fmaf(wd, w, g));
}
__device__ __forceinline__ float weight_update(float w, float lr, float v) { return __builtin_fmaf(-lr, v, w); }

// Sums and maxima across a wavefront without going through LDS.  Quarters: over the four lanes j, j + 16,
// j + 32, j + 48; row: over the 16 lanes of a quarter.  Every lane receives the same value.
// (The two swaps exchange the odd rows of one register with the even rows of the other, and its upper half
// with the other's lower half; the wait states stand for a register that the instruction before has written.
// In inline asm because the builtins' second result comes out as the first here.)
__device__ __forceinline__ void swap_rows(float& x, float& y) { asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(x), "+v"(y)); }
__device__ __forceinline__ void swap_halves(float& x, float& y) { asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(x), "+v"(y)); }
__device__ __forceinline__ float sum_over_quarters(float x) {
    float y = x;
    swap_rows(x, y);
    x += y;
    y = x;
    swap_halves(x, y);
    return x + y;
}
__device__ __forceinline__ float max_over_quarters(float x) {
    float y = x;
    swap_rows(x, y);
    x = fmaxf(x, y);
    y = x;
    swap_halves(x, y);
    return fmaxf(x, y);
}
template <int N>
__device__ __forceinline__ float rotated_in_row(float x) {   // DPP row_ror:N
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_over_row(float x) {
    x += rotated_in_row<8>(x);
    x += rotated_in_row<4>(x);
    x += rotated_in_row<2>(x);
    return x + rotated_in_row<1>(x);
}

__device__ __forceinline__ float max_over_row(float x) {
    x = fmaxf(x, rotated_in_row<8>(x));
    x = fmaxf(x, rotated_in_row<4>(x));
    x = fmaxf(x, rotated_in_row<2>(x));
    return fmaxf(x, rotated_in_row<1>(x));
}

template <int N>
__device__ __forceinline__ float rotated_in_quad(float x) {   // DPP quad_perm
    constexpr int kPerm = N | (N + 1) % 4 << 2 | (N + 2) % 4 << 4 | (N + 3) % 4 << 6;
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kPerm, 0xf, 0xf, false));
}
__device__ __forceinline__ float max_over_quad(float x) {   // over 4 neighbouring lanes
    x = fmaxf(x, rotated_in_quad<2>(x));
    return fmaxf(x, rotated_in_quad<1>(x));
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ----------------------------------------------------------------- index hash

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}
__device__ __forceinline__ int64_t batch_index(uint64_t seed, int i, int64_t k, int b, int64_t N) {
    const uint64_t gamma = 0x9E3779B97F4A7C15ULL;
    uint64_t hsh = mix64(seed + gamma * (static_cast<uint64_t>(k) + 1));
    hsh = mix64(hsh + gamma * (static_cast<uint64_t>(i) + 1));
    hsh = mix64(hsh + gamma * (static_cast<uint64_t>(b) + 1));
    return static_cast<int64_t>(hsh % static_cast<uint64_t>(N));
}

// Partition sampler: bijection of [0, n) by a 4-round balanced Feistel network on 2w bits with
// cycle walking.  The network permutes its 2w-bit domain, so a walk that starts below n returns
// below n after finitely many rounds (fewer than four on average, as the domain is < 4 n).
__device__ __forceinline__ uint64_t feistel_permute(uint64_t x, uint64_t n, uint64_t key) {
    int w = 1;
    while ((1ULL << (2 * w)) < n) ++w;
    const uint64_t mask = (1ULL << w) - 1;
    const uint64_t gamma = 0x9E3779B97F4A7C15ULL;
    do {
        uint64_t l = x >> w, r = x & mask;
#pragma unroll
        for (int round = 0; round < 4; ++round) {
            const uint64_t f = mix64(key + gamma * static_cast<uint64_t>(round + 1) + r) & mask;
            const uint64_t t = l ^ f;
            l = r;
            r = t;
        }
        x = (l << w) | r;
    } while (x >= n);
    return x;
}
__device__ __forceinline__ int64_t partition_index(uint64_t seed, int i, int64_t k, int b, int64_t N, int m, int B) {
    const int64_t lo = static_cast<int64_t>(i) * N / m, hi = static_cast<int64_t>(i + 1) * N / m;
    const int64_t S = (N / m) / B;   // >= 1, checked by lc_init
    const int64_t epoch = k / S, pos = (k % S) * B + b;
    const uint64_t gamma = 0x9E3779B97F4A7C15ULL;
    uint64_t key = mix64(seed + gamma * (static_cast<uint64_t>(epoch) + 1));
    key = mix64(key + gamma * (static_cast<uint64_t>(i) + 1));
    return lo + static_cast<int64_t>(feistel_permute(static_cast<uint64_t>(pos), static_cast<uint64_t>(hi - lo), key));
}

// Workgroups are handed to the 8 XCDs round-robin.  This maps the hardware
// block id to a logical one such that each XCD works on a contiguous range of
// logical blocks (consecutive blocks of one replica then share that XCD's L2
// for the replica's activations).  Returns -1 for the padding blocks.
__device__ __forceinline__ int64_t xcd_logical_block(int64_t total) {
    const int64_t per = (total + kXcds - 1) / kXcds;
    const int64_t bid = blockIdx.x;
    const int64_t logical = (bid % kXcds) * per + bid / kXcds;
    return logical < total ? logical : -1;
}

// Logical block -> (replica g, tile rem of the per_group tiles of a replica).
//   set == 0  replica-major: a replica's blocks are neighbours and share its activations in the L2
//   set >= 1  tile-major inside sets of `set` replicas (set divides n_groups): neighbouring blocks
//             take the same weight tile for different replicas
__device__ __forceinline__ void shared_order(int64_t logical, int per_group, int set, int& g, int& rem) {
    if (set > 0) {
        const int64_t per_set = static_cast<int64_t>(per_group) * set;
        const int within = static_cast<int>(logical % per_set);
        g = static_cast<int>(logical / per_set) * set + within % set;
        rem = within / set;
    } else {
        g = static_cast<int>(logical / per_group);
        rem = static_cast<int>(logical % per_group);
    }
}

}  // namespace
}  // namespace lc
