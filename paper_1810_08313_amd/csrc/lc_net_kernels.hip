// Local steps of small networks of any depth with the whole model on one compute unit.
//
// A PASGD worker touches nothing but its own model between two averaging steps (Sec. 2).  Where a
// replica's weights, one batch's activations and its deltas fit the LDS of a compute unit together,
// one workgroup takes a whole run of local steps: the weights stay in LDS, the momentum in
// registers, and what the launch-per-layer kernels hand each other through memory stays in LDS.
// Those kernels need 2 L launches per step of 6 to 20 us each at this size, nearly all of it launch
// and dependent memory round trips; here a step is 2 L + 1 phases between workgroup barriers, each a
// chain of LDS reads and matrix instructions (in the case below the compute unit's matrix cores are
// busy a quarter of the time, LDS bank conflicts take a tenth).
// (130-70-33-7, 3 workers, batch 48, fp32, two periods of 3 steps: 346 -> 130 us, 16 us a step; with a memory
// round trip per tile at the start, the layers' descriptions read in every tile and the loss in every step 136.)
//
// One step, 16 wavefronts sharing out 16 x 16 tiles of every product:
//   A_l = ReLU(A_{l-1} W_l + b_l) for l = 1 .. L (the last one without ReLU)
//   softmax cross-entropy, dZ_L
//   dZ_{l-1} = (dZ_l W_l^T) .* [A_{l-1} > 0] for l = L .. 2, with the weights of before the update
//   dW_l = A_{l-1}^T dZ_l, db_l and the momentum update of all layers
// LDS holds fp32 values throughout (with bf16 operands values that bf16 holds exactly, for activations
// and deltas; the masters for weights): W_l transposed, [column][row], A_l and dZ_l feature-major,
// [unit][sample].  With that every store of a result tile is one 16-byte access, and of the six
// operand reads three are (the others are four 4-byte reads of 16 consecutive lanes each).
//
// No workgroup waits for another: a launch ends with its period, and the averaging step is a launch
// of its own.  (Averaging inside the launch, behind a barrier of all replicas, can time out where other
// streams keep workgroups of the launch off the chip; the case above took 142 us with it.)
#include "lc_internal.h"
#include "lc_mma.h"

namespace lc {

namespace {

constexpr int kNetWaves = 16, kNetThreads = 64 * kNetWaves;
constexpr int kNetTiles = 8;            // 16 x 16 weight tiles per wavefront (4 momentum registers each)
constexpr int kNetFloats = 40704;       // LDS of a workgroup (159 KB of 160)
constexpr int kNetMaxClasses = 64;
constexpr int kTileBias = 1 << 14;      // in the tile table: first tile of its columns
static_assert(kNetFloats <= 1 << 16 && LC_MAX_LAYERS <= 16, "the tile table's fields: LDS offsets of 16 bits, layers of 4");
constexpr int kNetStage = 4;            // pieces of 4 values of A_0 per thread, where A_0 is kept in LDS

struct NetLayer {
    int d_in, d_out, kp, np;   // kp, np: padded to multiples of 16
    int ws;                    // floats between the columns of W^T in LDS
    int w, act, dz, bias;      // LDS offsets: W^T, A_l (l < L), dZ_l, b_l (the bias momentum np further on)
    int tile0;                 // first weight tile
    int64_t w_off, b_off;
};

struct NetArgs {
    float* X;
    float* V;
    int64_t x_stride;
    const float* Xr;      // where the weights are read at the start: X, or the one averaged model
    int64_t xr_stride;
    NetLayer layer[LC_MAX_LAYERS];
    int L, n_tiles;
    int B, Bq, Bp, dp0, G;   // Bq: batch padded to a multiple of 16 (LDS), Bp: as the gathered inputs have it
    int bs;                  // floats between the units of A and dZ in LDS
    int lred, tiles;         // LDS offsets: losses by sample, tile table
    int a0;                  // LDS offset of A_0, or -1: read from memory
    const void* a0_bm;       // [slots][G][Bp][dp0] of OT
    const void* a0_fm;       // [slots][G][dp0][Bp] of OT
    int64_t a0_slot;
    const int32_t* labels;   // [slots][G][Bp]
    int slot0, n_steps;
    float lr, beta_first, beta, wd;
    float* loss;             // [G][kLossParts], slot 0 written
};

__device__ __forceinline__ float net_round(float x, bf16_t) { return static_cast<float>(static_cast<bf16_t>(x)); }
__device__ __forceinline__ float net_round(float x, float) { return x; }

// IN_LDS: A_0 of the step is kept in LDS too (where it fits), else its operands come from memory.
template <typename OT, bool IN_LDS>
__global__ __launch_bounds__(kNetThreads) void net_kernel(NetArgs a) {
    __shared__ __attribute__((aligned(16))) float s[kNetFloats];
    // of every weight tile: (in s: layer, column tile, kTileBias, rows and columns that exist); LDS offsets of
    // its operands of dZ and A (of A_0 in memory: its first feature); of its weights, and what lies between columns
    __shared__ int tile_za[kNetWaves * kNetTiles], tile_w[kNetWaves * kNetTiles];
    const int g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, q = lane >> 4;
    float* Xg = a.X + g * a.x_stride;
    float* Vg = a.V + g * a.x_stride;
    const float* Xrg = a.Xr + g * a.xr_stride;
    const int BS = a.bs, nbt = a.Bq / 16;

    // ---- the tile table: what the steps need to know of a weight tile, without the layer's description
    int* tiles = reinterpret_cast<int*>(s + a.tiles);
    for (int l = 0; l < a.L; ++l) {
        const NetLayer& y = a.layer[l];
        const int nt = y.np / 16, n = nt * (y.kp / 16), in_at = l > 0 ? a.layer[l - 1].act : a.a0;
        for (int i = tid; i < n; i += kNetThreads) {
            const int kt = i / nt, ct = i % nt, t = y.tile0 + i, rows = y.d_in - 16 * kt, cols = y.d_out - 16 * ct;
            tiles[t] = l << 16 | ct << 24 | (kt == 0 ? kTileBias : 0) | (rows < 16 ? rows : 16) << 8 | (cols < 16 ? cols : 16);
            tile_za[t] = (y.dz + 16 * ct * BS) | (!IN_LDS && l == 0 ? 16 * kt : in_at + 16 * kt * BS) << 16;
            tile_w[t] = (y.w + 16 * ct * y.ws + 16 * kt) | y.ws << 16;
        }
    }
    __syncthreads();
    // ---- load the state; entries beyond the layer's sizes are zero and stay zero under the update.
    // All tiles' loads first: one memory round trip instead of one per tile (12400 -> 5000 clocks at four).
    f32x4 v[kNetTiles];
    {
        f32x4 w[kNetTiles];
#pragma unroll
        for (int i = 0; i < kNetTiles; ++i) {
            const int t = wave + kNetWaves * i;
            v[i] = w[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (t < a.n_tiles) {
                const int e = __builtin_amdgcn_readfirstlane(tiles[t]), o = __builtin_amdgcn_readfirstlane(tile_w[t]);
                const NetLayer& y = a.layer[e >> 16 & 15];
                const int n = 16 * (e >> 24 & 63) + j, k0 = ((o & 0xffff) - y.w) % y.ws + 4 * q;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // (entries that do not exist read the first one and are zeroed: no branch around the loads)
                    const bool in = 4 * q + r < (e >> 8 & 31) && j < (e & 31);
                    const int64_t at = y.w_off + (in ? static_cast<int64_t>(k0 + r) * y.d_out + n : 0);
                    w[i][r] = Xrg[at];
                    v[i][r] = Vg[at];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kNetTiles; ++i) {
            const int t = wave + kNetWaves * i;
            if (t < a.n_tiles) {
                const int e = __builtin_amdgcn_readfirstlane(tiles[t]), o = __builtin_amdgcn_readfirstlane(tile_w[t]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = 4 * q + r < (e >> 8 & 31) && j < (e & 31);
                    w[i][r] = in ? w[i][r] : 0.f;
                    v[i][r] = in ? v[i][r] : 0.f;
                }
                *reinterpret_cast<f32x4*>(s + (o & 0xffff) + j * (o >> 16) + 4 * q) = w[i];
            }
        }
    }
    for (int l = 0; l < a.L; ++l) {
        const NetLayer& y = a.layer[l];
        for (int n = tid; n < y.np; n += kNetThreads) {
            const bool in = n < y.d_out;
            s[y.bias + n] = in ? Xrg[y.b_off + n] : 0.f;
            s[y.bias + y.np + n] = in ? Vg[y.b_off + n] : 0.f;
        }
    }

    // A_0 in LDS (where it fits): thread t moves pieces t, t + 1024, ... of 4 samples of one feature
    const int n_stage = a.layer[0].kp * (a.Bq / 4), per_k = a.Bq / 4;
    const unsigned inv_k = ((1u << 20) + per_k - 1) / per_k;   // e / per_k = e inv_k >> 20 for e < 4096, per_k <= 32
    auto request = [&](const OT* from, int t, Frag4<OT> (&f)[kNetStage]) {
#pragma unroll
        for (int u = 0; u < kNetStage; ++u) {
            const int e = t + kNetThreads * u, k = static_cast<int>(static_cast<unsigned>(e) * inv_k >> 20), b4 = (e - k * per_k) * 4;
            if (kNetThreads * u < n_stage) f[u] = load4(from + (e < n_stage ? k * a.Bp + b4 : 0));
        }
    };
    auto place = [&](int t, const Frag4<OT> (&f)[kNetStage]) {
#pragma unroll
        for (int u = 0; u < kNetStage; ++u) {
            const int e = t + kNetThreads * u, k = static_cast<int>(static_cast<unsigned>(e) * inv_k >> 20), b4 = (e - k * per_k) * 4;
            if (e < n_stage)
                *reinterpret_cast<float4*>(s + a.a0 + k * BS + b4) =
                    make_float4(to_f32(f[u].v[0]), to_f32(f[u].v[1]), to_f32(f[u].v[2]), to_f32(f[u].v[3]));
        }
    };
    Frag4<OT> next_in[kNetStage];
    if constexpr (IN_LDS) {
        request(static_cast<const OT*>(a.a0_fm) + a.slot0 * a.a0_slot + static_cast<int64_t>(g) * a.dp0 * a.Bp, tid, next_in);
        place(tid, next_in);
    }
    __syncthreads();

    for (int step = 0; step < a.n_steps; ++step) {
        // What a step derives from the thread's id and from the layer table is derived afresh from
        // opaque copies, so that none of it is held in registers across the steps.
        int tid_o = threadIdx.x, zero = 0;
        asm volatile("" : "+v"(tid_o));
        asm volatile("" : "+s"(zero));
        const NetLayer* const layer = a.layer + zero;
        const int tid = tid_o, lane = tid & 63, j = lane & 15, q = lane >> 4;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const float beta = step == 0 ? a.beta_first : a.beta, lr = a.lr, wd = a.wd;
        const int slot = a.slot0 + step;
        const OT* A0 = static_cast<const OT*>(a.a0_bm) + slot * a.a0_slot + static_cast<int64_t>(g) * a.Bp * a.dp0;
        const OT* A0T = static_cast<const OT*>(a.a0_fm) + slot * a.a0_slot + static_cast<int64_t>(g) * a.dp0 * a.Bp;
        const int32_t* lab = a.labels + (static_cast<int64_t>(slot) * a.G + g) * a.Bp;

        const int yl = (tid >> 3) < a.B ? lab[tid >> 3] : -1;   // (asked for here: the softmax does not wait for it)

        // ---- forward
        for (int l = 0; l < a.L; ++l) {
            const NetLayer& y = layer[l];
            const bool last = l == a.L - 1;
            const int n_t = nbt * (y.np / 16), n_s = y.kp / 16;
            for (int t = wave; t < n_t; t += kNetWaves) {
                const int b0 = 16 * (t % nbt), n = 16 * (t / nbt) + j;
                const float* wt = s + y.w + n * y.ws + 4 * q;
                // sums of 32 products, added up: one accumulator over the whole reduction is off by 1.23
                // times (up to 1.95) as much in the gradients as the launches per layer, whose
                // wavefronts share out the reduction
                const f32x4 zeros = f32x4{0.f, 0.f, 0.f, 0.f};
                f32x4 acc = zeros;
                if (!IN_LDS && l == 0) {
                    // the input rows come from memory: four steps' operands in flight
                    const OT* ar = A0 + static_cast<int64_t>(b0 + j) * a.dp0 + 4 * q;
                    constexpr int kF = 4;
                    Frag4<OT> cur[kF], nxt[kF];
#pragma unroll
                    for (int u = 0; u < kF; ++u) cur[u] = load4(ar + 16 * (u < n_s ? u : 0));
                    for (int s0 = 0; s0 < n_s; s0 += kF) {
#pragma unroll
                        for (int u = 0; u < kF; ++u) {
                            const int st = s0 + kF + u;
                            nxt[u] = load4(ar + 16 * (st < n_s ? st : 0));
                        }
                        f32x4 part = zeros;
#pragma unroll
                        for (int u = 0; u < kF; ++u) {
                            if (s0 + u < n_s) {   // uniform
                                const float4 w = *reinterpret_cast<const float4*>(wt + 16 * (s0 + u));
                                Frag4<OT> bf;
                                pack4(bf, w.x, w.y, w.z, w.w);
                                part = mma4(cur[u], bf, u % 2 == 0 ? zeros : part);
                                if (u % 2 == 1 || s0 + u + 1 == n_s) acc += part;
                            }
                        }
#pragma unroll
                        for (int u = 0; u < kF; ++u) cur[u] = nxt[u];
                    }
                } else {
                    const float* ap = s + (l == 0 ? a.a0 : layer[l - 1].act) + 4 * q * BS + b0 + j;
                    auto product = [&](const float* x, const float* wr, f32x4 c) {
                        const float4 w = *reinterpret_cast<const float4*>(wr);
                        Frag4<OT> af, bf;
                        pack4(af, x[0], x[BS], x[2 * BS], x[3 * BS]);
                        pack4(bf, w.x, w.y, w.z, w.w);
                        return mma4(af, bf, c);
                    };
#pragma unroll 1
                    for (int st = 1; st < n_s; st += 2, ap += 32 * BS, wt += 32)
                        acc += product(ap + 16 * BS, wt + 16, product(ap, wt, zeros));
                    if (n_s & 1) acc += product(ap, wt, zeros);
                }
                const float bias = s[y.bias + n];
                f32x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float z = acc[r] + bias;
                    if (last) o[r] = z;
                    else o[r] = (b0 + 4 * q + r < a.B && z > 0.f) ? net_round(z, OT()) : 0.f;   // (batch padding stays zero)
                }
                *reinterpret_cast<f32x4*>(s + (last ? y.dz : y.act) + n * BS + b0 + 4 * q) = o;
            }
            __syncthreads();
        }

        // ---- the next step's inputs (the gather kernel left them in other XCDs' memory, two microseconds
        //      away): into registers where A_0 is kept in LDS, else into the L2, one 4-byte load per cache
        //      line.  Behind the loads of the forward pass, since loads retire in order.
        const bool more = step + 1 < a.n_steps;
        float touched[4] = {0.f, 0.f, 0.f, 0.f};
        if (IN_LDS && more) request(A0T + a.a0_slot, tid, next_in);
        if (!IN_LDS && more) {
            const int n_lines = a.Bp * a.dp0 * static_cast<int>(sizeof(OT)) / 128;
            const float* nt = reinterpret_cast<const float*>(A0T + a.a0_slot);
            const float* nb = reinterpret_cast<const float*>(A0 + a.a0_slot);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = tid + kNetThreads * u;
                if (e < n_lines) {
                    touched[u] = nt[32 * e];
                    touched[2 + u] = nb[32 * e];
                }
            }
        }

        // ---- softmax cross-entropy, 8 lanes per sample; dZ_L over the logits
        {
            const NetLayer& y = layer[a.L - 1];
            const int b = tid >> 3, u8 = tid & 7;
            if (b < a.Bq) {   // (whole groups of 8 lanes)
                float* z = s + y.dz + b;
                float zc[kNetMaxClasses / 8], zmax = -INFINITY;
#pragma unroll
                for (int u = 0; u < kNetMaxClasses / 8; ++u) {
                    const int c = u8 + 8 * u;
                    zc[u] = c < y.d_out ? z[c * BS] : -INFINITY;
                    zmax = fmaxf(zmax, zc[u]);
                }
#pragma unroll
                for (int o = 4; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 8));
                float s_other = 0.f, e_y = 0.f, z_y = 0.f;
#pragma unroll
                for (int u = 0; u < kNetMaxClasses / 8; ++u) {
                    const int c = u8 + 8 * u;
                    if (c >= y.d_out) continue;
                    const float e = expf(zc[u] - zmax);
                    if (c == yl) {
                        e_y = e;
                        z_y = zc[u] - zmax;
                    } else {
                        s_other += e;
                    }
                    zc[u] = e;
                }
#pragma unroll
                for (int o = 4; o > 0; o >>= 1) {
                    s_other += __shfl_xor(s_other, o, 8);
                    e_y += __shfl_xor(e_y, o, 8);
                    z_y += __shfl_xor(z_y, o, 8);
                }
                const float inv = 1.f / (s_other + e_y), invB = 1.f / static_cast<float>(a.B);
#pragma unroll
                for (int u = 0; u < kNetMaxClasses / 8; ++u) {
                    const int c = u8 + 8 * u;
                    if (c < y.np)
                        z[c * BS] = (c < y.d_out && yl >= 0) ? net_round(xent_delta(zc[u], c == yl, s_other, inv) * invB, OT()) : 0.f;
                }
                if (!more && u8 == 0) s[a.lred + b] = yl >= 0 ? xent_loss(s_other, e_y, z_y) : 0.f;
            }
        }
        __syncthreads();

        // ---- deltas of the layers below, with the weights of before the update
        for (int l = a.L - 1; l >= 1; --l) {
            const NetLayer& y = layer[l];
            const NetLayer& p = layer[l - 1];
            const int n_t = nbt * (p.np / 16), n_s = y.np / 16;
            for (int t = wave; t < n_t; t += kNetWaves) {
                const int b0 = 16 * (t % nbt), k = 16 * (t / nbt) + j;
                const float* zp = s + y.dz + 4 * q * BS + b0 + j;
                const float* wp = s + y.w + 4 * q * y.ws + k;
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int st = 0; st < n_s; ++st, zp += 16 * BS, wp += 16 * y.ws) {
                    Frag4<OT> af, bf;
                    pack4(af, zp[0], zp[BS], zp[2 * BS], zp[3 * BS]);
                    pack4(bf, wp[0], wp[y.ws], wp[2 * y.ws], wp[3 * y.ws]);
                    acc = mma4(af, bf, acc);
                }
                const f32x4 act = *reinterpret_cast<const f32x4*>(s + p.act + k * BS + b0 + 4 * q);
                f32x4 d;
#pragma unroll
                for (int r = 0; r < 4; ++r) d[r] = act[r] > 0.f ? net_round(acc[r], OT()) : 0.f;
                *reinterpret_cast<f32x4*>(s + p.dz + k * BS + b0 + 4 * q) = d;
            }
            __syncthreads();
        }

        // ---- weight gradients and updates, biases, the step's loss
#pragma unroll
        for (int i = 0; i < kNetTiles; ++i) {
            const int t = wave + kNetWaves * i;
            if (t < a.n_tiles) {
                const int e = __builtin_amdgcn_readfirstlane(tiles[t]);
                const unsigned za = __builtin_amdgcn_readfirstlane(tile_za[t]);
                const int ow = __builtin_amdgcn_readfirstlane(tile_w[t]);
                const float* zt = s + (za & 0xffffu) + j * BS + 4 * q;
                const float* at = s + (za >> 16) + j * BS + 4 * q;
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
                float db = 0.f;   // column sum of dZ_l over this lane's samples
                if (!IN_LDS && (e >> 16 & 15) == 0) {
                    const OT* ar = A0T + (static_cast<int>(za >> 16) + j) * a.Bp + 4 * q;
                    Frag4<OT> af[8];
#pragma unroll
                    for (int st = 0; st < 8; ++st) af[st] = load4(ar + 16 * (st < nbt ? st : 0));
#pragma unroll
                    for (int st = 0; st < 8; ++st)
                        if (st < nbt) {   // uniform
                            const float4 z = *reinterpret_cast<const float4*>(zt + 16 * st);
                            Frag4<OT> bf;
                            pack4(bf, z.x, z.y, z.z, z.w);
                            db += (z.x + z.y) + (z.z + z.w);
                            acc = mma4(af[st], bf, acc);
                        }
                } else {
#pragma unroll 1
                    for (int st = 0; st < nbt; ++st, at += 16, zt += 16) {
                        const float4 z = *reinterpret_cast<const float4*>(zt);
                        const float4 x = *reinterpret_cast<const float4*>(at);
                        Frag4<OT> af, bf;
                        pack4(af, x.x, x.y, x.z, x.w);
                        pack4(bf, z.x, z.y, z.z, z.w);
                        db += (z.x + z.y) + (z.z + z.w);
                        acc = mma4(af, bf, acc);
                    }
                }
                if (e & kTileBias) {   // the bias of these columns, by the wavefront of their first tile
                    const NetLayer& y = layer[e >> 16 & 15];
                    db += __shfl_xor(db, 16, 64);
                    db += __shfl_xor(db, 32, 64);
                    if (q == 0 && j < (e & 31)) {
                        float* bp = s + y.bias + 16 * (e >> 24 & 63) + j;
                        const float vb = momentum_update(beta, bp[y.np], db, wd, *bp);
                        bp[y.np] = vb;
                        *bp = weight_update(*bp, lr, vb);
                    }
                }
                f32x4* wp = reinterpret_cast<f32x4*>(s + (ow & 0xffff) + j * (ow >> 16) + 4 * q);
                f32x4 w = *wp;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // (an entry that does not exist must stay zero also where its zero operand meets an infinity)
                    const float gw = 4 * q + r < (e >> 8 & 31) && j < (e & 31) ? acc[r] : 0.f;
                    v[i][r] = momentum_update(beta, v[i][r], gw, wd, w[r]);
                    w[r] = weight_update(w[r], lr, v[i][r]);
                }
                *wp = w;
            }
        }
        if (!more && wave == 0) {   // (the losses that are kept are those of the last step)
            float sum = (lane < a.Bq ? s[a.lred + lane] : 0.f) + (lane + 64 < a.Bq ? s[a.lred + lane + 64] : 0.f);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
            if (lane == 0) a.loss[static_cast<int64_t>(g) * kLossParts] = sum / static_cast<float>(a.B);
        }
        __syncthreads();

        asm volatile("" : : "v"(touched[0]), "v"(touched[1]), "v"(touched[2]), "v"(touched[3]));
        if (IN_LDS && more) {
            place(tid, next_in);
            __syncthreads();
        }
    }
    // ---- write the state back
#pragma unroll
    for (int i = 0; i < kNetTiles; ++i) {
        const int t = wave + kNetWaves * i;
        if (t < a.n_tiles) {
            const int e = __builtin_amdgcn_readfirstlane(tiles[t]), o = __builtin_amdgcn_readfirstlane(tile_w[t]);
            const NetLayer& y = a.layer[e >> 16 & 15];
            const int n = 16 * (e >> 24 & 63) + j, k0 = ((o & 0xffff) - y.w) % y.ws + 4 * q;
            const f32x4 w = *reinterpret_cast<const f32x4*>(s + (o & 0xffff) + j * y.ws + 4 * q);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * q + r < (e >> 8 & 31) && j < (e & 31)) {
                    const int64_t at = y.w_off + static_cast<int64_t>(k0 + r) * y.d_out + n;
                    Xg[at] = w[r];
                    Vg[at] = v[i][r];
                }
        }
    }
    for (int l = 0; l < a.L; ++l) {
        const NetLayer& y = a.layer[l];
        for (int n = tid; n < y.d_out; n += kNetThreads) {
            Xg[y.b_off + n] = s[y.bias + n];
            Vg[y.b_off + n] = s[y.bias + y.np + n];
        }
    }
}

// LDS layout of a model; false where it does not fit (or has more classes or tiles than the kernel takes).
bool net_layout(const lc_handle* h, NetArgs& a) {
    if (h->md.kind != LC_KIND_MLP || h->L < 1) return false;
    if (h->layer[h->L].d_out > kNetMaxClasses) return false;
    a.L = h->L;
    a.B = h->md.B;
    a.Bq = static_cast<int>(round_up(a.B, 16));
    a.bs = a.Bq + 4;   // (a multiple of 4 floats that spreads consecutive units over the banks)
    int64_t off = 0;
    int n_tiles = 0;
    for (int l = 0; l < a.L; ++l) {
        const LayerGeom& g = h->layer[l + 1];
        if (g.d_in > 1024 || g.d_out > 1024) return false;   // (column tiles have 6 bits in the tile table, and such layers do not fit anyway)
        NetLayer& y = a.layer[l];
        y.d_in = g.d_in;
        y.d_out = g.d_out;
        y.kp = static_cast<int>(round_up(g.d_in, 16));
        y.np = static_cast<int>(round_up(g.d_out, 16));
        y.ws = y.kp + 4;
        y.w_off = g.w_off;
        y.b_off = g.b_off;
        y.tile0 = n_tiles;
        n_tiles += (y.kp / 16) * (y.np / 16);
        y.w = static_cast<int>(off);
        off += static_cast<int64_t>(y.np) * y.ws;
        y.act = static_cast<int>(off);
        if (l < a.L - 1) off += static_cast<int64_t>(y.np) * a.bs;
        y.dz = static_cast<int>(off);
        off += static_cast<int64_t>(y.np) * a.bs;
        y.bias = static_cast<int>(off);
        off += 2 * y.np;
        if (off > kNetFloats) return false;
    }
    a.lred = static_cast<int>(off);
    off += 128;
    a.tiles = static_cast<int>(off);
    off += n_tiles;
    a.n_tiles = n_tiles;
    off = round_up(off, 4);
    const int64_t in = static_cast<int64_t>(a.layer[0].kp) * a.bs;
    a.a0 = off + in <= kNetFloats && a.layer[0].kp * (a.Bq / 4) <= kNetStage * kNetThreads ? static_cast<int>(off) : -1;
    return n_tiles <= kNetWaves * kNetTiles && off <= kNetFloats;
}

}  // namespace

// A model that fits takes this route where one compute unit per replica is the faster way at any number of
// steps per call.  Measured against the launches per layer on 1493 models (inputs 16 .. 640, up to three
// hidden layers of 16 .. 256, 2 .. 512 replicas of 8 .. 128 samples; calls of 1, 5 and 16 steps; the figures
// are the slowest of the three):
//   A_0 kept in LDS: 1.03 .. 5.8 times as fast, except one layer of few classes (launches of 12 us a
//   step) and two layers with many weight tiles, where loading the state costs a call of one step: 0.95 on.
//   A_0 read from memory, twice per step, at 0.2 (bf16) to 0.4 us per row of 16 x 16 tiles in the first
//   layer where LDS takes 0.04 to 0.1: one layer 0.61 on; two layers of few tiles 1.07 on, of more from
//   0.58 (limit twice as high, 1.16 on, below 0.71 on, where the first hidden layer is narrower than a
//   column chunk, whose rows the launches read element by element); three layers of few tiles 1.01 on,
//   of more 0.83; more layers 1.07 on.
bool net_shape_ok(const lc_handle* h) {
    if (resident_shape_ok(h)) return false;
    NetArgs a;
    if (!net_layout(h, a)) return false;
    if (a.L >= 4) return true;
    const bool narrow = a.layer[0].d_out < kColChunk;
    if (a.a0 >= 0) return a.L == 3 || (a.L == 2 ? narrow || a.n_tiles < 88 : a.layer[0].d_out > 16 || a.n_tiles < 24);
    return (a.L == 2 && a.n_tiles < (narrow ? 64 : 40)) || (a.L == 3 && a.n_tiles < (narrow ? 112 : 80));
}

hipError_t launch_net(lc_handle* h, int slot0, int n_steps) {
    const ActSet& S = h->train;
    NetArgs a;
    if (!net_layout(h, a)) return hipErrorInvalidValue;
    a.X = h->X;
    a.V = h->V;
    a.x_stride = h->Ps;
    a.Xr = h->lazy_rows ? h->xbar : h->X;
    a.xr_stride = h->lazy_rows ? 0 : h->Ps;
    a.Bp = S.Bp;
    a.dp0 = h->layer[1].dp_in;
    a.G = S.G;
    a.a0_bm = S.a_bm[0];
    a.a0_fm = S.a_fm[0];
    a.a0_slot = static_cast<int64_t>(S.G) * S.Bp * a.dp0;
    a.labels = S.labels;
    a.slot0 = slot0;
    a.n_steps = n_steps;
    a.lr = h->md.lr;
    a.beta_first = effective_beta(h);
    a.beta = h->md.beta;
    a.wd = h->md.wd;
    a.loss = S.loss;
    if (slot0 < 0 || n_steps < 1 || slot0 + n_steps > S.slots || a.Bq > S.Bp) return hipErrorInvalidValue;
    timing_start(h, kTimeBwd, 0, kBwdResident);
    const dim3 grid(S.G), block(kNetThreads);
    if (h->md.gemm == LC_GEMM_BF16) {
        if (a.a0 >= 0) hipLaunchKernelGGL((net_kernel<bf16_t, true>), grid, block, 0, h->stream, a);
        else hipLaunchKernelGGL((net_kernel<bf16_t, false>), grid, block, 0, h->stream, a);
    } else {
        if (a.a0 >= 0) hipLaunchKernelGGL((net_kernel<float, true>), grid, block, 0, h->stream, a);
        else hipLaunchKernelGGL((net_kernel<float, false>), grid, block, 0, h->stream, a);
    }
    h->loss_parts_train = 1;
    timing_stop(h, kTimeBwd, 0, kBwdResident);
    return hipGetLastError();
}

}  // namespace lc
