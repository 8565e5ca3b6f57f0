// Backward pass of the first layer, with the forward pass of the NEXT local step folded in.
//
// Between two averaging steps a worker's local updates touch only its own model (Sec. 2), so the
// first layer's weights after the update of step k are exactly the weights the forward pass of
// step k+1 multiplies its mini-batch with -- and that mini-batch does not depend on the model.
// The first layer needs no dA, so its rows can be shared out any way: here a workgroup owns 64
// COLUMNS of W_1 over all rows (the forward pass's decomposition).  While a tile of W_1, V_1 is
// in registers for
//     dW_1 = A_0^T dZ_1,   v <- beta v + dW_1 + wd w,   w <- w - lr v        (step k)
// the updated tile is used at once as the operand of
//     Z_1' = A_0' W_1 + b_1                                                  (step k+1)
// and W_1 crosses the memory system 16 instead of 20 bytes per parameter and step (12 instead of
// 16 where the momentum is implicit, see FirstArgs::Aux).
//
// This needs no exchange between lanes: the dW tile comes out of the matrix cores in accumulator
// layout (lane (j, q) holds rows 4q..4q+3 of a 16-row block, column j), and a matrix instruction
// with a reduction length of 16 takes its weight operand in exactly that shape (4 consecutive
// reduction indices per lane).  A step of the walk is therefore one 16-row block: the updated
// rows go from the update straight into the forward product, the activation operand is 4
// consecutive entries per lane.
#include "lc_internal.h"
#include "lc_mma.h"

#include <type_traits>

namespace lc {

namespace {

// Wavefronts of a workgroup, and partial sums of Z_1'.  Up to 64 samples two workgroups share a CU; where the whole grid is
// no more than one per CU, fp32 operands at 33 to 64 samples take twice as many (PAIRS), since such a wavefront requests
// nothing ahead (see FlBudget) and needs another one's loads under way beside its matrix instructions.  Five steps with
// four and eight: 3072-1024-1024-10, 16 workers of 64, 1879 and 1797 us; 1500-800-800-10, 16 of 50, 1264 and 1141;
// 784-1000-300-10, 14 of 64, 676 and 641; 2000-777-300-10, 18 of 40, 1337 and 1207; 300-1024-10, 12 of 60, 264 and 236.
// Below 256 inputs, 14 of 60: 64-1024-10 160 and 164, 100 inputs 180 and 173, 160 200 and 203, 192 205 and 207, 224 224 and 220.
// bf16 operands and up to 32 samples, which have a step ahead: 0.99 to 1.04 times as fast.
constexpr int kFlWaves = 4;

struct FirstArgs {
    float* X;             // where the new parameters are written
    float* V;             // where the new momentum is written, or null (implicit momentum, see BwdArgs::Aux)
    int64_t x_stride;
    const float* Xr;      // where the weights are read: X, the one averaged model (stride 0), or the other row buffer
    int64_t xr_stride;
    const float* Aux;     // the momentum rows, or (imp_in) the parameters of one step earlier
    int64_t aux_stride;
    int imp_in;
    float inv_lr;
    int shared_w;         // > 0: block order of steps in which all replicas read one model (see shared_order)
    int64_t w_off, b_off;
    int d_in, d_out, dp_in, dp_out;
    int B;
    const void* a_fm;     // A_0^T of this step, tiles of 16 features in fragment order
    const void* dz_fm;    // dZ_1 of this step, feature-major [G][dp_out][Bp]
    float lr, beta, wd;
    const void* an_bm;    // A_0 of the next step, batch-major [G][Bp][dp_in]
    void* out_bm;         // A_1 of the next step [G][Bp][dp_out]
    void* out_fm;         //                      [G][dp_out][Bp]
    int n_chunks;         // column chunks per replica
    int chunk_cols, wavefronts;   // see FirstLayerPlan
    int64_t total_blocks;
};

// Steps a wavefront requests ahead of the one it works on, and wavefronts per SIMD the register
// budget is set for.  Up to 64 samples two workgroups share a CU (256 registers per lane) with one
// step ahead: what the walk responds to is the number of wavefronts that can issue, not the depth
// of a wavefront's queue (two steps ahead at one workgroup per CU: 1072 us on the 3072x2048 layer
// of 64 replicas, one or two steps ahead at two per CU: 900 us, none ahead at three or four per
// CU: 920 us -- measured while the weight-read mode was still a per-load choice, see WMR below;
// 887 us since).  At 128 samples the 32 accumulator tiles of the forward product leave room for one
// workgroup per CU only.  (fp32 operands at 64 samples spill at 256 registers with a step ahead.)
template <typename OT, int NT>
struct FlBudget {
    static constexpr int kWavesPerSimd = NT >= 8 ? 1 : 2;
    static constexpr int kAhead = (NT == 4 && sizeof(OT) == 4) ? 0 : 1;
};

// One workgroup = one replica x 64 columns of W_1; its 4 wavefronts take the 16-row steps
// wave, wave + 4, ... and never synchronise inside the walk: the dZ_1 slice is staged once, the
// A_0 tiles go from memory straight into operand registers.  The loads of a wavefront's next PD
// steps are in flight while it works on the current one (PD + 1 register sets, addressed
// statically); a step is small enough (about 20 memory instructions with its stores) that the
// steps in flight stay below the 64 outstanding memory instructions a wavefront can have.
// Every weight access is one unconditional 16-byte instruction: of aligned rows that are a multiple of
// 64 columns long and a d_in that is a multiple of 16, or (WM == kWRagged, see lc_mma.h) of any rows
// of at least 64 columns and any d_in.  In those instances the last steps read the last row in place of
// rows that do not exist, the stores leave out what does not exist, and such rows enter the
// forward product as zeros.
// WM is the access mode of the state that streams (momentum or older model, all stores), WMR that of
// the weights read: cached where all replicas read one model, which the neighbouring blocks want in
// the L2.  (A template parameter, not a run-time flag: with the choice made per load the compiler
// waited for each load before it issued the next.)
// PAIRS: 8 wavefronts, of which u and u + 4 take the steps that wavefront u of four would take, in turn, and add up that
// wavefront's share of Z_1' in the same order, each for half of the samples: the same bits.  (Eight shares, added up at the
// end, round otherwise, and a ReLU gate that one of two such sums opens is amplified by later steps: the momentum of
// 3072-1024-1024-10, 16 workers of 64, differed by up to 2.4e-3 after three calls of five steps.)  The updated tiles go
// through LDS, 8 of them between two barriers; a wavefront then holds half of the sums, which leaves registers for a step
// ahead.  (With a share of the columns for either half, rows whose length is no multiple of 32 floats have twice as many
// cache lines that two wavefronts write in part: 2000-777-300-10 1430 us instead of 1207.)
template <typename OT, int NT, int WM, int WMR, bool PAIRS>
__global__ __launch_bounds__(PAIRS ? 512 : 256, (FlBudget<OT, NT>::kWavesPerSimd)) void first_layer_kernel(FirstArgs a) {
    constexpr int NW = PAIRS ? 2 * kFlWaves : kFlWaves;
    constexpr int SW = NW / kFlWaves, MW = NT / SW;   // steps of a round and tiles of samples that a wavefront multiplies
    constexpr int kPad = sizeof(OT) == 2 ? 8 : 4;
    constexpr int Bp = 16 * NT;
    constexpr int NS = Bp / 32;
    constexpr int PD = PAIRS ? 1 : FlBudget<OT, NT>::kAhead;
    // the dZ^T slice during the walk; the wavefronts' partial Z_1' tiles after it
    constexpr size_t kSliceBytes = sizeof(OT) * kColChunk * (Bp + kPad);
    constexpr size_t kPartBytes = sizeof(float) * kFlWaves * Bp * (kColChunk + 4);
    constexpr size_t kTileBytes = PAIRS ? 2 * NW * 4 * 64 * sizeof(Frag4<OT>) : 0;
    constexpr size_t kWalkBytes = kSliceBytes + kTileBytes;
    __shared__ __attribute__((aligned(16))) char smem[kWalkBytes > kPartBytes ? kWalkBytes : kPartBytes];
    __shared__ float bias_s[kColChunk];
    // row (c % 4) * 16 + c / 4 holds column c0 + c: the 16 lanes of an operand read (columns
    // 4 j + t) then hit 16 consecutive LDS rows
    OT (*dzt)[Bp + kPad] = reinterpret_cast<OT (*)[Bp + kPad]>(smem);
    // PAIRS: [buffer][wavefront][t][lane], a lane's 4 x 4 block of an updated tile as operands (columns 4 j + t, rows 4 q ..)
    Frag4<OT> (*wt)[NW][4][64] = reinterpret_cast<Frag4<OT> (*)[NW][4][64]>(smem + kSliceBytes);

    const int64_t logical = xcd_logical_block(a.total_blocks);
    if (logical < 0) return;
    int g, chunk;
    shared_order(logical, a.n_chunks, a.shared_w, g, chunk);
    const int c0 = chunk * kColChunk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: step bases live in scalar registers
    const int turn = wave % kFlWaves, mt0 = wave / kFlWaves * MW;
    const int j = lane & 15, q = lane >> 4;

    float* W = a.X + g * a.x_stride + a.w_off;
    const float* Wr = a.Xr + g * a.xr_stride + a.w_off;
    float* Vw = a.V ? a.V + g * a.x_stride + a.w_off : nullptr;
    const float* Va = a.Aux + g * a.aux_stride + a.w_off;
    const OT* AT = static_cast<const OT*>(a.a_fm) + static_cast<int64_t>(g) * a.dp_in * Bp;
    const OT* AN = static_cast<const OT*>(a.an_bm) + static_cast<int64_t>(g) * Bp * a.dp_in;
    constexpr bool RAG = WM == kWRagged;
    const int n_steps = RAG ? (a.d_in + 15) / 16 : a.d_in / 16;
    const int left = RAG ? a.d_out - (c0 + 4 * j) : 4;   // columns that exist from this lane's first one on

    struct Set {
        float4 w[4], v[4];      // rows k0 + 4 q + r, columns c0 + 4 j ..
        Frag<OT> af[NS];        // A_0^T tile of the 16 rows
        Frag4<OT> an[SW][MW];   // next step's A_0, 4 entries of each batch row
    };
    Set set[PD + 1];

    // A step's addresses are a base that is the same for the whole wavefront (scalar registers)
    // plus byte offsets that a lane keeps for the whole walk: 4 registers serve the loads and the
    // stores of W and V alike.
    unsigned woff[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) woff[r] = 4u * static_cast<unsigned>((4 * q + r) * a.d_out + c0 + 4 * j);
    // fragments of A_0^T; of A_0' one half of a 32-deep fragment per step (see InputLayout)
    constexpr int kHalf = sizeof(OT) == 4 ? 256 : 4;
    const unsigned atoff = static_cast<unsigned>(sizeof(OT)) * static_cast<unsigned>((sizeof(OT) == 4 ? 4 : 8) * lane);
    auto at_byte = [](auto* base, unsigned off) {
        using T = std::remove_pointer_t<decltype(base)>;
        using C = std::conditional_t<std::is_const_v<T>, const char, char>;
        return reinterpret_cast<T*>(reinterpret_cast<C*>(base) + off);
    };

    auto past_end = [&](int row) { return row < a.d_in ? 0 : row - (a.d_in - 1); };   // rows back to the last one
    auto load_step = [&](int s, Set& x) {
        // steps past the end are never used: a valid step is read for them, so that no branch
        // sits between the loads
        const int k0 = 16 * (s < n_steps ? s : n_steps - 1);
        const float* wb = Wr + static_cast<int64_t>(k0) * a.d_out;
        const float* vb = Va + static_cast<int64_t>(k0) * a.d_out;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            unsigned at = woff[r];
            if constexpr (RAG) at -= 4u * static_cast<unsigned>(a.d_out) * static_cast<unsigned>(past_end(k0 + 4 * q + r));
            x.w[r] = load_wm<WMR>(at_byte(wb, at), 0, a.d_out, true);
            x.v[r] = load_wm<WM>(at_byte(vb, at), 0, a.d_out, true);
        }
        const OT* ab = AT + static_cast<int64_t>(k0) * Bp;
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            if constexpr (sizeof(OT) == 4) {
                const float4 lo = *reinterpret_cast<const float4*>(at_byte(ab + kFragElems * st, atoff));
                const float4 hi = *reinterpret_cast<const float4*>(at_byte(ab + kFragElems * st + 256, atoff));
                x.af[st] = Frag<OT>{{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}};
            } else {
                x.af[st] = load8(at_byte(ab + kFragElems * st, atoff));
            }
        }
#pragma unroll
        for (int i = 0; i < SW; ++i) {
            const int si = s - wave + turn + i * kFlWaves, n0 = PAIRS ? (si < n_steps ? si : n_steps - 1) : k0 / 16;
            const OT* nb = AN + (n0 / 2) * kFragElems + (n0 % 2) * kHalf;
#pragma unroll
            for (int mt = 0; mt < MW; ++mt)
                x.an[i][mt] = load4(at_byte(nb + static_cast<int64_t>(16 * (mt0 + mt)) * a.dp_in, atoff));
        }
    };

    // first loads, then the staging of the slice (its own round trip overlaps with them)
#pragma unroll
    for (int p = 0; p < PD; ++p) load_step(wave + p * NW, set[p]);
    {
        const OT* ZT = static_cast<const OT*>(a.dz_fm) + (static_cast<int64_t>(g) * a.dp_out + c0) * Bp;
        for (int p = tid; p < kColChunk * (Bp / 8); p += 64 * NW) {
            const int c = p / (Bp / 8), seg = p % (Bp / 8);
            *reinterpret_cast<Frag<OT>*>(&dzt[(c & 3) * 16 + (c >> 2)][seg * 8]) = load8(ZT + static_cast<int64_t>(p) * 8);
        }
    }
    __syncthreads();
    // bias of these columns: db_1 = sum_b dZ_1, the same update; kept for the forward epilogue
    if (tid < kColChunk && (WM != kWRagged || c0 + tid < a.d_out)) {
        float* bx = a.X + g * a.x_stride + a.b_off + c0 + tid;
        const float x = a.Xr[g * a.xr_stride + a.b_off + c0 + tid];
        float vb0 = a.Aux[g * a.aux_stride + a.b_off + c0 + tid];
        if (a.imp_in) vb0 = (vb0 - x) * a.inv_lr;
        const OT* zr = dzt[(tid & 3) * 16 + (tid >> 2)];
        float sb = 0.f;
        for (int b = 0; b < a.B; ++b) sb += to_f32(zr[b]);
        const float vb = a.beta * vb0 + (sb + a.wd * x);
        if (a.V) a.V[g * a.x_stride + a.b_off + c0 + tid] = vb;
        *bx = x - a.lr * vb;
        bias_s[tid] = x - a.lr * vb;
    }

    f32x4 facc[MW][4];
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int t = 0; t < 4; ++t) facc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto process = [&](int s, Set& x) {
        float* ws = W + static_cast<int64_t>(16 * s) * a.d_out;
        float* vs = Vw ? Vw + static_cast<int64_t>(16 * s) * a.d_out : nullptr;
        // dW tile: sum over the batch of A_0^T[k][b] dZ_1^T[c][b]
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const Frag<OT> zf = *reinterpret_cast<const Frag<OT>*>(&dzt[t * 16 + j][32 * st + 8 * q]);
                acc[t] = mma8(x.af[st], zf, acc[t]);
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            consume_here(x.w[r]);
            consume_here(x.v[r]);
            if (a.imp_in) {   // the tile holds the parameters of one step earlier: v = (x_prev - x) / lr
                x.v[r].x = (x.v[r].x - x.w[r].x) * a.inv_lr;
                x.v[r].y = (x.v[r].y - x.w[r].y) * a.inv_lr;
                x.v[r].z = (x.v[r].z - x.w[r].z) * a.inv_lr;
                x.v[r].w = (x.v[r].w - x.w[r].w) * a.inv_lr;
            }
            x.v[r].x = a.beta * x.v[r].x + (acc[0][r] + a.wd * x.w[r].x);
            x.v[r].y = a.beta * x.v[r].y + (acc[1][r] + a.wd * x.w[r].y);
            x.v[r].z = a.beta * x.v[r].z + (acc[2][r] + a.wd * x.w[r].z);
            x.v[r].w = a.beta * x.v[r].w + (acc[3][r] + a.wd * x.w[r].w);
            x.w[r].x -= a.lr * x.v[r].x;
            x.w[r].y -= a.lr * x.v[r].y;
            x.w[r].z -= a.lr * x.v[r].z;
            x.w[r].w -= a.lr * x.v[r].w;
            const bool in = RAG ? 16 * s + 4 * q + r < a.d_in : !PAIRS || s < n_steps;
            if (in) {
                if (vs) store_wm<WM>(at_byte(vs, woff[r]), 0, left, true, x.v[r]);
                store_wm<WM>(at_byte(ws, woff[r]), 0, left, true, x.w[r]);
            } else {
                x.w[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        // Z_1' += A_0'[:, k0 .. k0+15] W_1[k0 .. k0+15, :] with the tile just updated
        Frag4<OT> bf[4];
        pack4(bf[0], x.w[0].x, x.w[1].x, x.w[2].x, x.w[3].x);
        pack4(bf[1], x.w[0].y, x.w[1].y, x.w[2].y, x.w[3].y);
        pack4(bf[2], x.w[0].z, x.w[1].z, x.w[2].z, x.w[3].z);
        pack4(bf[3], x.w[0].w, x.w[1].w, x.w[2].w, x.w[3].w);
        if constexpr (PAIRS) {
            // (the buffer's readers of two rounds ago have passed the barrier of the last one)
            const int buf = s / NW % 2;
#pragma unroll
            for (int t = 0; t < 4; ++t) wt[buf][wave][t][lane] = bf[t];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SW; ++i) {
                if (s - wave + turn + i * kFlWaves >= n_steps) break;   // uniform over the wavefront
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    bf[t] = wt[buf][turn + i * kFlWaves][t][lane];
#pragma unroll
                    for (int mt = 0; mt < MW; ++mt) facc[mt][t] = mma4(x.an[i][mt], bf[t], facc[mt][t]);
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) facc[mt][t] = mma4(x.an[0][mt], bf[t], facc[mt][t]);
        }
    };

    // groups of PD + 1 steps without control flow in between (a branch would make the compiler
    // drain the loads in flight where the paths meet), then the steps whose loads are under way
    // (PAIRS: as many rounds for every wavefront; steps past the end change nothing)
    int s0 = wave;
    const int s_end = PAIRS ? (n_steps + NW - 1) / NW * NW : n_steps;
    for (; s0 + PD * NW < s_end; s0 += NW * (PD + 1)) {
#pragma unroll
        for (int u = 0; u <= PD; ++u) {
            const int s = s0 + u * NW;
            load_step(s + PD * NW, set[(u + PD) % (PD + 1)]);
            process(s, set[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < PD; ++u) {
        const int s = s0 + u * NW;
        if (s < s_end) process(s, set[u]);   // uniform over the wavefront
    }

    // A_1' = ReLU(Z_1' + b_1): the wavefronts' partial tiles are added in wavefront order
    __syncthreads();   // every wavefront is done with the slice that shares this memory
    float (*part)[Bp][kColChunk + 4] = reinterpret_cast<float (*)[Bp][kColChunk + 4]>(smem);
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<float4*>(&part[turn][16 * (mt0 + mt) + 4 * q + r][4 * j]) =
                make_float4(facc[mt][0][r], facc[mt][1][r], facc[mt][2][r], facc[mt][3][r]);
    __syncthreads();
    for (int f = tid; f < Bp * (kColChunk / 4); f += 64 * NW) {
        const int b = f / (kColChunk / 4), c4 = (f % (kColChunk / 4)) * 4;
        float4 z = *reinterpret_cast<const float4*>(&part[0][b][c4]);
#pragma unroll
        for (int wv = 1; wv < kFlWaves; ++wv) {
            const float4 o = *reinterpret_cast<const float4*>(&part[wv][b][c4]);
            z.x += o.x; z.y += o.y; z.z += o.z; z.w += o.w;
        }
        z.x += bias_s[c4]; z.y += bias_s[c4 + 1]; z.z += bias_s[c4 + 2]; z.w += bias_s[c4 + 3];
        *reinterpret_cast<float4*>(&part[0][b][c4]) =
            make_float4(z.x > 0.f ? z.x : 0.f, z.y > 0.f ? z.y : 0.f, z.z > 0.f ? z.z : 0.f, z.w > 0.f ? z.w : 0.f);
    }
    __syncthreads();
    OT* obm = static_cast<OT*>(a.out_bm) + static_cast<int64_t>(g) * Bp * a.dp_out;
    OT* ofm = static_cast<OT*>(a.out_fm) + static_cast<int64_t>(g) * a.dp_out * Bp;
    auto value = [&](int b, int c) { return part[0][b][c]; };
    // 8 outputs per thread and pass, one vector store each: along the columns for the
    // batch-major copy, along the batch for the feature-major one; only batch rows below B
    // are written, so the zero padding of the buffers is preserved
    for (int e = tid; e < Bp * (kColChunk / 8); e += 64 * NW) {
        const int b = e / (kColChunk / 8), cl = (e % (kColChunk / 8)) * 8;
        if (b >= a.B) continue;
        float y[8];   // (columns that do not exist keep the zeros of the padding)
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = (!RAG || c0 + cl + i < a.d_out) ? value(b, cl + i) : 0.f;
        store8(obm + static_cast<int64_t>(b) * a.dp_out + c0 + cl, y);
    }
    for (int e = tid; e < kColChunk * (Bp / 8); e += 64 * NW) {
        const int c = e / (Bp / 8), bl = (e % (Bp / 8)) * 8;
        if (bl >= a.B || (RAG && c0 + c >= a.d_out)) continue;
        float y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = bl + i < a.B ? value(bl + i, c) : 0.f;
        if (bl + 8 <= a.B) {
            store8(ofm + static_cast<int64_t>(c0 + c) * Bp + bl, y);
        } else {
            for (int i = 0; bl + i < a.B; ++i) ofm[static_cast<int64_t>(c0 + c) * Bp + bl + i] = static_cast<OT>(y[i]);
        }
    }
}


// The same step at 128 samples.  Sharing out the rows alone leaves each wavefront with the whole
// 128 x 64 tile of Z_1' (128 accumulator registers per lane), so four wavefronts fill a CU's register
// file with two steps in flight each, and the walk waits for memory.  Here a workgroup has 8
// wavefronts that share out BOTH: wavefront w updates the 16-row steps 8 r + w (r = 0, 1, ... :
// "rounds") as above, publishes each updated tile in LDS in operand precision, and after one
// barrier per round multiplies all 8 tiles of the round with ITS 16 samples of A_0' -- 4
// accumulator tiles per wavefront, complete at the end of the walk, nothing to add up across
// wavefronts.  Two sets of loads per wavefront, twice the wavefronts (3072x1024, 16 replicas: 161 ->
// 148 us; a third set changes nothing, nor does leaving out either product: what remains is the
// memory system's rate for 256 column walks).
// The tiles are double-buffered: a wavefront can only write round r + 1's buffer (that of round
// r - 1) after the barrier of round r, which every reader of round r - 1 has passed.
constexpr int kWideWaves = 8;

// CPL: columns of a lane, four or (ragged rows, see wide_columns) six; the chunk is 16 CPL columns wide.
template <typename OT, int WM, int WMR, int CPL = 4, int PD = 1>
__global__ __launch_bounds__(64 * kWideWaves) void first_layer_wide_kernel(FirstArgs a) {
    static_assert(sizeof(OT) == 2, "operand fragments of fp32 do not fit the register budget here");
    static_assert(CPL == 4 || (CPL == 6 && WM == kWRagged && WMR == kWRagged), "six columns: 16 and 8 bytes at any float address");
    constexpr int NC = 16 * CPL;
    constexpr int kPad = 8;
    constexpr int Bp = 128, NS = Bp / 32, NTH = 64 * kWideWaves;
    constexpr size_t kSliceBytes = sizeof(OT) * NC * (Bp + kPad);
    constexpr size_t kTileBytes = 2 * kWideWaves * CPL * 64 * sizeof(Frag4<OT>);
    constexpr size_t kPartBytes = sizeof(float) * Bp * (NC + 4);
    constexpr size_t kWalkBytes = kSliceBytes + kTileBytes;
    __shared__ __attribute__((aligned(16))) char smem[kWalkBytes > kPartBytes ? kWalkBytes : kPartBytes];
    __shared__ float bias_s[NC];
    OT (*dzt)[Bp + kPad] = reinterpret_cast<OT (*)[Bp + kPad]>(smem);
    // [buffer][wavefront][pair][lane]: a lane's 4 x 4 block of the tile as 4 operand fragments
    // (columns 4 j + t, rows 4 q ..), 16 bytes per lane and pair: consecutive lanes, no bank conflicts
    bf16x8 (*wt)[kWideWaves][2][64] = reinterpret_cast<bf16x8 (*)[kWideWaves][2][64]>(smem + kSliceBytes);
    // six columns: [buffer][pair of wavefronts][t][lane], rows 4 q .. of the first's tile and of the second's
    bf16x8 (*wt32)[kWideWaves / 2][CPL][64] = reinterpret_cast<bf16x8 (*)[kWideWaves / 2][CPL][64]>(smem + kSliceBytes);

    const int64_t logical = xcd_logical_block(a.total_blocks);
    if (logical < 0) return;
    int g, chunk;
    shared_order(logical, a.n_chunks, a.shared_w, g, chunk);
    const int c0 = chunk * NC;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, q = lane >> 4;

    float* W = a.X + g * a.x_stride + a.w_off;
    const float* Wr = a.Xr + g * a.xr_stride + a.w_off;
    float* Vw = a.V ? a.V + g * a.x_stride + a.w_off : nullptr;
    const float* Va = a.Aux + g * a.aux_stride + a.w_off;
    const OT* AT = static_cast<const OT*>(a.a_fm) + static_cast<int64_t>(g) * a.dp_in * Bp;
    // this wavefront's 16 samples of the next step's input
    const OT* AN = static_cast<const OT*>(a.an_bm) + (static_cast<int64_t>(g) * Bp + 16 * wave) * a.dp_in;
    constexpr bool RAG = WM == kWRagged;
    const int n_rounds = (a.d_in + 16 * kWideWaves - 1) / (16 * kWideWaves);   // (divides unless RAG)
    const int left = RAG ? a.d_out - (c0 + CPL * j) : CPL;   // columns that exist from this lane's first one on
    const int c_own = RAG && left < 1 ? a.d_out - 1 : c0 + CPL * j;   // (a lane without columns reads, and never uses, the last ones)

    struct Set {
        float w[4][CPL], v[4][CPL];   // rows k0 + 4 q + r, columns c0 + CPL j ..
        Frag<OT> af[NS];              // A_0^T tile of this wavefront's 16 rows
        Frag<OT> an[kWideWaves / 2];  // A_0' of this wavefront's samples, 4 entries for each of two tiles of the round
    };
    Set set[PD + 1];

    const unsigned woff = 4u * static_cast<unsigned>(4 * q * a.d_out + c_own);   // (row 4 q of a step; the others by their base)
    const unsigned atoff = static_cast<unsigned>(sizeof(OT)) * static_cast<unsigned>(8 * lane);   // in a fragment
    auto at_byte = [](auto* base, unsigned off) {
        using T = std::remove_pointer_t<decltype(base)>;
        using C = std::conditional_t<std::is_const_v<T>, const char, char>;
        return reinterpret_cast<T*>(reinterpret_cast<C*>(base) + off);
    };

    typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));
    auto load_columns = [&](auto mode, const float* p, float (&to)[CPL]) {
        const float4 f = load_wm<decltype(mode)::value>(p, 0, a.d_out, true);
        to[0] = f.x; to[1] = f.y; to[2] = f.z; to[3] = f.w;
        if constexpr (CPL == 6) {
            const f32x2_u g = *reinterpret_cast<const f32x2_u*>(p + 4);
            to[4] = g[0]; to[5] = g[1];
        }
    };
    auto store_columns = [&](float* p, const float (&from)[CPL]) {
        store_wm<WM>(p, 0, left, true, make_float4(from[0], from[1], from[2], from[3]));
        if constexpr (CPL == 6) {
            if (left > 5) {
                *reinterpret_cast<f32x2_u*>(p + 4) = f32x2_u{from[4], from[5]};
            } else if (left > 4) {
                p[4] = from[4];
            }
        }
    };
    constexpr std::integral_constant<int, WM> kState{};
    constexpr std::integral_constant<int, WMR> kWeights{};
    auto load_round = [&](int r, Set& x) {
        // rounds past the end are never used: the last one is read for them (no branch between the loads)
        const int rr = r < n_rounds ? r : n_rounds - 1;
        const int k0 = 16 * (kWideWaves * rr + wave);
        const int kb = RAG && k0 > a.d_in - 1 ? a.d_in - 1 : k0;
        const float* wb = Wr + static_cast<int64_t>(kb) * a.d_out;
        const float* vb = Va + static_cast<int64_t>(kb) * a.d_out;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            if constexpr (RAG) {   // (rows that do not exist: the last one)
                const int row = k0 + 4 * q + r4, last = a.d_in - 1;
                const unsigned at = 4u * (static_cast<unsigned>((row < last ? row : last) - kb) * static_cast<unsigned>(a.d_out) + c_own);
                load_columns(kWeights, at_byte(wb, at), x.w[r4]);
                load_columns(kState, at_byte(vb, at), x.v[r4]);
            } else {
                load_columns(kWeights, at_byte(wb + r4 * a.d_out, woff), x.w[r4]);
                load_columns(kState, at_byte(vb + r4 * a.d_out, woff), x.v[r4]);
            }
        }
        // (inputs have dp_in rows and columns; a step beyond them reads the last 16 instead, for rows
        // of the tile that are not stored and enter the forward product as zeros)
        const int ka = RAG && k0 > a.dp_in - 16 ? a.dp_in - 16 : k0;
        const OT* ab = AT + static_cast<int64_t>(ka) * Bp;
#pragma unroll
        for (int st = 0; st < NS; ++st) x.af[st] = load8(at_byte(ab + kFragElems * st, atoff));
        const int sn = kWideWaves / 2 * rr;
#pragma unroll
        for (int u = 0; u < kWideWaves / 2; ++u) {
            const int sc = RAG && sn + u >= a.dp_in / 32 ? a.dp_in / 32 - 1 : sn + u;
            x.an[u] = load8(at_byte(AN + sc * kFragElems, atoff));
        }
    };

#pragma unroll
    for (int p = 0; p < PD; ++p) load_round(p, set[p]);
    {
        const OT* ZT = static_cast<const OT*>(a.dz_fm) + (static_cast<int64_t>(g) * a.dp_out + c0) * Bp;
        for (int p = tid; p < NC * (Bp / 8); p += NTH) {
            const int c = p / (Bp / 8), seg = p % (Bp / 8);
            // (six columns a lane: the last chunk may reach past the deltas' padded rows)
            const bool in = CPL == 4 || c0 + c < a.dp_out;
            Frag<OT> f = load8(ZT + (in ? static_cast<int64_t>(p) * 8 : 0));
            if (!in) f.v = bf16x8{};
            *reinterpret_cast<Frag<OT>*>(&dzt[c % CPL * 16 + c / CPL][seg * 8]) = f;
        }
    }
    __syncthreads();
    if (tid < NC && (WM != kWRagged || c0 + tid < a.d_out)) {
        float* bx = a.X + g * a.x_stride + a.b_off + c0 + tid;
        const float x = a.Xr[g * a.xr_stride + a.b_off + c0 + tid];
        float vb0 = a.Aux[g * a.aux_stride + a.b_off + c0 + tid];
        if (a.imp_in) vb0 = (vb0 - x) * a.inv_lr;
        const OT* zr = dzt[tid % CPL * 16 + tid / CPL];
        float sb = 0.f;
        for (int b = 0; b < a.B; ++b) sb += to_f32(zr[b]);
        const float vb = a.beta * vb0 + (sb + a.wd * x);
        if (a.V) a.V[g * a.x_stride + a.b_off + c0 + tid] = vb;
        *bx = x - a.lr * vb;
        bias_s[tid] = x - a.lr * vb;
    }

    f32x4 facc[CPL];
#pragma unroll
    for (int t = 0; t < CPL; ++t) facc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto process = [&](int r, Set& x) {
        const int64_t row0 = static_cast<int64_t>(16 * (kWideWaves * r + wave)) * a.d_out;
        float* ws = W + row0;
        float* vs = Vw ? Vw + row0 : nullptr;
        f32x4 acc[CPL];
#pragma unroll
        for (int t = 0; t < CPL; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                const Frag<OT> zf = *reinterpret_cast<const Frag<OT>*>(&dzt[t * 16 + j][32 * st + 8 * q]);
                acc[t] = mma8(x.af[st], zf, acc[t]);
            }
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
#pragma unroll
            for (int t = 0; t < CPL; ++t) asm volatile("" : "+v"(x.w[r4][t]), "+v"(x.v[r4][t]));   // (see consume_here)
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                float& w = x.w[r4][t];
                float& v = x.v[r4][t];
                if (a.imp_in) v = (v - w) * a.inv_lr;   // (v held the parameters of one step earlier: v = (x_prev - x) / lr)
                v = a.beta * v + (acc[t][r4] + a.wd * w);
                w -= a.lr * v;
            }
            if (!RAG || 16 * (kWideWaves * r + wave) + 4 * q + r4 < a.d_in) {
                if (vs) store_columns(at_byte(vs + r4 * a.d_out, woff), x.v[r4]);
                store_columns(at_byte(ws + r4 * a.d_out, woff), x.w[r4]);
            } else {
#pragma unroll
                for (int t = 0; t < CPL; ++t) x.w[r4][t] = 0.f;
            }
        }
        // the updated tile as operand fragments of this lane, then
        // Z_1'[these 16 samples] += A_0'[.., the round's 128 rows] W_1[the round's 128 rows, :]
        if constexpr (CPL == 6) {
            // 32-deep products of two tiles at a time, each round's sum formed from zero.  (In one sum over all inputs, as below,
            // X and V were 1.024 and 1.038 times as far from 64 bits as with the launches per layer, 1.03 and 1.05 from 1700
            // inputs on; now 0.996 and 0.993, 0.985 and 0.982: 300 drawn models, two seeds.  3072-1500-1000-100, 16 workers of 100,
            // 5 steps: 2254 us either way.  Sums of four rounds added up in LDS: no nearer, 2264 us.)
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                Frag4<OT> b;
                pack4(b, x.w[0][t], x.w[1][t], x.w[2][t], x.w[3][t]);
                reinterpret_cast<bf16x4*>(&wt32[r & 1][wave / 2][t][lane])[wave % 2] = b.v;
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < CPL; t += 2) {
                f32x4 z0{}, z1{};
#pragma unroll
                for (int u = 0; u < kWideWaves / 2; ++u) {
                    z0 = mma8(x.an[u], Frag<OT>{wt32[r & 1][u][t][lane]}, z0);
                    z1 = mma8(x.an[u], Frag<OT>{wt32[r & 1][u][t + 1][lane]}, z1);
                }
                facc[t] += z0;
                facc[t + 1] += z1;
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                Frag4<OT> b0, b1;
                pack4(b0, x.w[0][2 * h], x.w[1][2 * h], x.w[2][2 * h], x.w[3][2 * h]);
                pack4(b1, x.w[0][2 * h + 1], x.w[1][2 * h + 1], x.w[2][2 * h + 1], x.w[3][2 * h + 1]);
                bf16x8 both;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    both[e] = b0.v[e];
                    both[4 + e] = b1.v[e];
                }
                wt[r & 1][wave][h][lane] = both;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kWideWaves; ++u) {
                Frag4<OT> an;
#pragma unroll
                for (int e = 0; e < 4; ++e) an.v[e] = x.an[u / 2].v[4 * (u % 2) + e];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bf16x8 both = wt[r & 1][u][h][lane];
                    Frag4<OT> f0, f1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        f0.v[e] = both[e];
                        f1.v[e] = both[4 + e];
                    }
                    facc[2 * h] = mma4(an, f0, facc[2 * h]);
                    facc[2 * h + 1] = mma4(an, f1, facc[2 * h + 1]);
                }
            }
        }
    };

    // groups of PD + 1 rounds without control flow in between, then the rounds whose loads are under way
    int r0 = 0;
    for (; r0 + PD < n_rounds; r0 += PD + 1) {
#pragma unroll
        for (int u = 0; u <= PD; ++u) {
            load_round(r0 + u + PD, set[(u + PD) % (PD + 1)]);
            process(r0 + u, set[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < PD; ++u)
        if (r0 + u < n_rounds) process(r0 + u, set[u]);   // uniform over the workgroup

    // A_1' = ReLU(Z_1' + b_1), through LDS for the two layouts of the stores
    __syncthreads();   // every wavefront is done with the slice and the tiles that share this memory
    float (*part)[NC + 4] = reinterpret_cast<float (*)[NC + 4]>(smem);
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            const float z = facc[t][r4] + bias_s[CPL * j + t];
            part[16 * wave + 4 * q + r4][CPL * j + t] = z > 0.f ? z : 0.f;
        }
    __syncthreads();
    OT* obm = static_cast<OT*>(a.out_bm) + static_cast<int64_t>(g) * Bp * a.dp_out;
    OT* ofm = static_cast<OT*>(a.out_fm) + static_cast<int64_t>(g) * a.dp_out * Bp;
    for (int e = tid; e < Bp * (NC / 8); e += NTH) {
        const int b = e / (NC / 8), cl = (e % (NC / 8)) * 8;
        if (b >= a.B || (CPL != 4 && c0 + cl >= a.dp_out)) continue;
        float y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = (!RAG || c0 + cl + i < a.d_out) ? part[b][cl + i] : 0.f;
        store8(obm + static_cast<int64_t>(b) * a.dp_out + c0 + cl, y);
    }
    for (int e = tid; e < NC * (Bp / 8); e += NTH) {
        const int c = e / (Bp / 8), bl = (e % (Bp / 8)) * 8;
        if (bl >= a.B || (RAG && c0 + c >= a.d_out)) continue;
        float y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = bl + i < a.B ? part[bl + i][c] : 0.f;
        if (bl + 8 <= a.B) {
            store8(ofm + static_cast<int64_t>(c0 + c) * Bp + bl, y);
        } else {
            for (int i = 0; bl + i < a.B; ++i) ofm[static_cast<int64_t>(c0 + c) * Bp + bl + i] = static_cast<OT>(y[i]);
        }
    }
}

// whole 64-column chunks of 16-byte aligned rows, and whole 16-row steps
bool whole_tiles(const FirstArgs& a) { return a.d_out % kColChunk == 0 && a.w_off % 4 == 0 && a.d_in % 16 == 0; }

template <typename OT, int NT, bool PAIRS>
void launch_fl_pairs(const FirstArgs& a, bool stream_w, unsigned grid, hipStream_t st) {
    const dim3 block(PAIRS ? 512 : 256);
    if constexpr (NT < 8) {   // (at 128 samples other layers go to the wide kernel)
        if (!whole_tiles(a)) {
            hipLaunchKernelGGL((first_layer_kernel<OT, NT, kWRagged, kWRagged, PAIRS>), dim3(grid), block, 0, st, a);
            return;
        }
    }
    if (stream_w && !a.shared_w)
        hipLaunchKernelGGL((first_layer_kernel<OT, NT, kWVectorStream, kWVectorStream, PAIRS>), dim3(grid), block, 0, st, a);
    else if (stream_w) hipLaunchKernelGGL((first_layer_kernel<OT, NT, kWVectorStream, kWVector, PAIRS>), dim3(grid), block, 0, st, a);
    else hipLaunchKernelGGL((first_layer_kernel<OT, NT, kWVector, kWVector, PAIRS>), dim3(grid), block, 0, st, a);
}

template <typename OT, int NT>
void launch_fl_wm(const FirstArgs& a, bool stream_w, unsigned grid, hipStream_t st) {
    if constexpr (NT == 4 && sizeof(OT) == 4) {
        if (a.wavefronts == 2 * kFlWaves) {
            launch_fl_pairs<OT, NT, true>(a, stream_w, grid, st);
            return;
        }
    }
    launch_fl_pairs<OT, NT, false>(a, stream_w, grid, st);
}

template <typename OT>
hipError_t launch_fl(const FirstArgs& a, int nt, bool stream_w, unsigned grid, hipStream_t st) {
    if (nt == 2) launch_fl_wm<OT, 2>(a, stream_w, grid, st);
    else if (nt == 4) launch_fl_wm<OT, 4>(a, stream_w, grid, st);
    else if constexpr (sizeof(OT) == 2) {
        const dim3 block(64 * kWideWaves);
        if (a.chunk_cols == 96) hipLaunchKernelGGL((first_layer_wide_kernel<OT, kWRagged, kWRagged, 6>), dim3(grid), block, 0, st, a);
        else if (!whole_tiles(a)) hipLaunchKernelGGL((first_layer_wide_kernel<OT, kWRagged, kWRagged>), dim3(grid), block, 0, st, a);
        else if (a.wavefronts == kFlWaves) launch_fl_wm<OT, 8>(a, stream_w, grid, st);
        else if (stream_w && !a.shared_w)
            hipLaunchKernelGGL((first_layer_wide_kernel<OT, kWVectorStream, kWVectorStream>), dim3(grid), block, 0, st, a);
        else if (stream_w) hipLaunchKernelGGL((first_layer_wide_kernel<OT, kWVectorStream, kWVector>), dim3(grid), block, 0, st, a);
        else hipLaunchKernelGGL((first_layer_wide_kernel<OT, kWVector, kWVector>), dim3(grid), block, 0, st, a);
    } else {
        return hipErrorInvalidValue;   // (fp32 operands at 128 samples: first_layer_kernel_ok refuses)
    }
    return hipGetLastError();
}

}  // namespace

// Columns of a chunk: 96 instead of 64 in the 128-sample kernel on ragged rows where the rounds of workgroups then cost
// less, a workgroup of 96 columns taking 1.5 times as long.  5 steps of 7238 drawn models (64 .. 3072 inputs, 65 .. 4096
// columns, 8 .. 250 workers of 65 .. 128 samples), times as fast as with 64 columns by rounds, median (least .. most), state
// that streams / cached:
//   2 -> 1   1.107 (1.056 .. 1.163) / 1.045 (0.988 .. 1.112)      2 -> 2   0.85 (0.81 .. 0.91) / 0.90 (0.82 .. 0.97)
//   4 -> 2   1.06 (1.04 .. 1.08) / 1.02 (1.02 .. 1.04)            3 -> 2   0.991 (0.92 .. 1.016) / 0.99 (0.95 .. 1.02)
//   5 -> 3   1.02 (0.96 .. 1.04) / 1.00 (0.98 .. 1.03)            4 -> 3   0.95 (0.92 .. 0.98) / 0.97 (0.94 .. 1.00)
//   8 -> 5, 11 -> 7, 14 -> 9   1.00 .. 1.01 (0.99 .. 1.02)        6 -> 4, 9 -> 6, 12 -> 8   0.99 (0.95 .. 1.01)
// 3072-1500-1000-100, 16 of 100, two rounds of 64 columns, one of 96: 2408 and 2252 us.
static int wide_columns(const lc_handle* h, bool whole) {
    const LayerGeom& g = h->layer[1];
    if (h->train.Bp != 128 || h->md.gemm != LC_GEMM_BF16 || whole) return kColChunk;
    const int64_t cus = compute_units(), m = h->train.G;
    const int64_t r64 = (m * ((g.d_out + 63) / 64) + cus - 1) / cus, r96 = (m * ((g.d_out + 95) / 96) + cus - 1) / cus;
    return 6 * r96 < 4 * r64 ? 96 : kColChunk;
}

struct FirstLayerPlan {
    int columns, wavefronts;   // of a workgroup; 0: the layer keeps the separate launches
};

// The kernel serves layer 1 of models with at least two layers whose first-layer rows are at least one
// column chunk long, when there are enough (replica, column chunk) pairs to fill the chip; everything
// else keeps the row-owner backward kernel and the separate forward launch.
static FirstLayerPlan first_layer_plan(const lc_handle* h) {
    const FirstLayerPlan none{0, 0};
    if (h->md.kind != LC_KIND_MLP || h->L < 2) return none;
    const LayerGeom& g = h->layer[1];
    const ActSet& S = h->train;
    const bool bf16 = h->md.gemm == LC_GEMM_BF16;
    if (g.d_out < kColChunk) return none;
    if (S.Bp != 32 && S.Bp != 64 && S.Bp != 128) return none;
    if (g.d_in < 16 * kFlWaves) return none;
    // fp32 operands at 128 samples: the operand fragments of two steps and the 32 accumulator tiles
    // do not fit the register file
    if (!bf16 && S.Bp == 128) return none;
    // Every workgroup walks a whole column chunk, so a last round of few workgroups takes as long as a
    // full one (3072x1024, batch 128: 147 us a step with 16 replicas = 256 workgroups, 250 with 20, 288
    // with 32).  How many times as fast whole runs are than with the separate launches, median (least)
    // of 1709 models of d0 = 128 .. 3072, d1 = 256 .. 2048, by how full the rounds are on average:
    //   one round (192 workgroups and more) 1.02 .. 1.17 everywhere
    //   up to 64 samples, state cached or whole tiles: 50 .. 60 % 0.98 .. 1.10 (0.94), 60 .. 100 % 1.01 .. 1.17
    //   up to 64 samples, ragged rows that stream: fp32 operands 0.86 .. 0.99 (0.85) below 80 %, 1.01 up to
    //   90 %; bf16 0.90 .. 1.01 (0.89) below 70 %, 1.04 up to 80 %
    //   128 samples: below 70 % 0.84 .. 1.01 (0.84), to 75 % 0.95 .. 1.02, to 80 % 0.97 .. 1.03 (ragged
    //   and cached 0.97), above 0.99 .. 1.11
    // Counted are the workgroups that will be launched.  Where those have 96 columns, whole runs are 1.14 times as fast as
    // with the separate launches with a state that streams (median of 1265 models, least 1.04) and 1.13 cached (2093 models,
    // least 1.00); of the rounds of 64 columns 706 and 2008 of these models would fill less than 75 and 80 %.
    const bool whole = g.d_out % kColChunk == 0 && g.w_off % 4 == 0 && g.d_in % 16 == 0;
    FirstLayerPlan p{wide_columns(h, whole), kFlWaves};
    const int64_t blocks = static_cast<int64_t>(S.G) * ((g.d_out + p.columns - 1) / p.columns);
    const int64_t cus = compute_units(), rounds = (blocks + cus - 1) / cus;
    if (blocks < 192) return none;
    int full = 0;   // per cent
    if (rounds == 1) full = 0;
    else if (S.Bp == 128) full = whole || h->stream_weights ? 75 : 80;
    else if (!whole && h->stream_weights) full = bf16 ? 70 : 85;
    if (100 * blocks < full * cus * rounds) return none;
    // 128 samples: the wide kernel.  (Whole tiles whose height is no multiple of the 128 rows that its wavefronts
    // take together stay with the other one: cut off as ragged rows are, they run 0.94 .. 1.0 times as fast up
    // to 784 inputs of a cached state, 1.0 .. 1.03 from 1040 inputs on.)
    if (S.Bp == 128 && !(whole && g.d_in % (16 * kWideWaves) != 0)) p.wavefronts = kWideWaves;
    if (S.Bp == 64 && !bf16 && blocks <= cus && g.d_in >= 256) p.wavefronts = 2 * kFlWaves;   // (see kFlWaves)
    return p;
}

bool first_layer_kernel_ok(const lc_handle* h) { return first_layer_plan(h).columns != 0; }

// Backward pass and update of layer 1 for the step in slot train.cur_slot, and A_1 of the step in
// the next slot (which must have been gathered already).
hipError_t launch_first_layer(lc_handle* h) {
    const ActSet& S = h->train;
    const LayerGeom& g = h->layer[1];
    const bool bf16 = h->md.gemm == LC_GEMM_BF16;
    const size_t es = bf16 ? 2 : 4;
    const size_t slot_bytes = static_cast<size_t>(S.G) * S.Bp * g.dp_in * es;
    const FirstLayerPlan plan = first_layer_plan(h);
    if (!plan.columns) return hipErrorInvalidValue;
    if (S.cur_slot + 1 >= S.slots || h->a0_layout != kInputsLayers) return hipErrorInvalidValue;
    FirstArgs a;
    const StepBufs sb = plan_step_buffers(h, 1);
    a.X = sb.ox;
    a.V = sb.ov;
    a.x_stride = h->Ps;
    a.Xr = sb.xr;
    a.xr_stride = sb.xr_stride;
    a.Aux = sb.aux;
    a.aux_stride = sb.aux_stride;
    a.imp_in = sb.imp_in;
    a.inv_lr = 1.f / h->md.lr;
    a.shared_w = (sb.xr_stride == 0 && shared_weight_order(h, g)) ? shared_set(h, S.G) : 0;
    a.w_off = g.w_off;
    a.b_off = g.b_off;
    a.d_in = g.d_in;
    a.d_out = g.d_out;
    a.dp_in = g.dp_in;
    a.dp_out = g.dp_out;
    a.B = S.B;
    a.a_fm = static_cast<const char*>(S.a_fm[0]) + static_cast<size_t>(S.cur_slot) * slot_bytes;
    a.dz_fm = S.dz_fm[1];
    a.lr = h->md.lr;
    a.beta = effective_beta(h);
    a.wd = h->md.wd;
    a.an_bm = static_cast<const char*>(S.a_bm[0]) + static_cast<size_t>(S.cur_slot + 1) * slot_bytes;
    a.out_bm = S.a_bm[1];
    a.out_fm = S.a_fm[1];
    a.chunk_cols = plan.columns;
    a.wavefronts = plan.wavefronts;
    a.n_chunks = (g.d_out + a.chunk_cols - 1) / a.chunk_cols;
    a.total_blocks = static_cast<int64_t>(S.G) * a.n_chunks;
    const unsigned grid = static_cast<unsigned>((a.total_blocks + kXcds - 1) / kXcds * kXcds);
    timing_start(h, kTimeBwd, 1, kBwdFirstLayer);
    const hipError_t e = bf16 ? launch_fl<bf16_t>(a, S.Bp / 16, h->stream_weights, grid, h->stream)
                              : launch_fl<float>(a, S.Bp / 16, h->stream_weights, grid, h->stream);
    timing_stop(h, kTimeBwd, 1, kBwdFirstLayer);
    if (e == hipSuccess) h->imp[1] = sb.next;
    return e;
}

}  // namespace lc

extern "C" int lc_first_layer_workgroup(const lc_handle* h, int32_t* columns, int32_t* wavefronts) {
    if (!h || !columns || !wavefronts) return LC_ERR_ARG;
    const lc::FirstLayerPlan p = h->fl_on ? lc::first_layer_plan(h) : lc::FirstLayerPlan{0, 0};
    *columns = p.columns;
    *wavefronts = p.wavefronts;
    return LC_OK;
}
