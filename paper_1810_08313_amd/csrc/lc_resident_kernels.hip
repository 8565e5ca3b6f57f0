// Local steps of small two-layer models with the weights resident on chip.
//
// Between two averaging steps a PASGD worker touches nothing but its own model (Sec. 2:
// tau local mini-batch SGD updates, then one averaging step).  When a replica's first layer,
// cut into slices of 16 hidden units, fits the LDS of the compute units, a whole run of local
// steps is one kernel launch: every workgroup loads its slice of W_1 (into LDS) and of the
// momentum V_1 (into registers) once, takes all the steps on them, and writes them back once.
// The streaming kernels need four launches per step and move W and V through the memory
// system in every one of them; at this size those launches, not the arithmetic, are the cost.
//
// Work split for a model d0 -> d1 -> d2 (d2 <= 16), replica g, workgroup cb of the NB slices of 16 hidden units:
//   owns   hidden units C = [16 cb, 16 cb + 16): columns C of W_1, V_1, entries C of b_1, and the
//          matching ROWS C of W_2, V_2 -- every weight of the model has exactly one owner;
//   keeps  a private copy of b_2 (d2 values), updated identically by every workgroup.
// One step:
//   (1) A_0 W_1[:, C]                                      MFMA; the 16 wavefronts split batch tiles and K
//   then one wavefront per tile of 16 samples, in registers from here to dZ_1:
//   (2) A_1[:, C] = ReLU(. + b_1[C]) and this slice's share of the logits, A_1[:, C] W_2[C, :] (16 x 16
//       values), handed to the replica; barrier with the same tile's wavefronts of the other slices
//   (3) Z_2 = sum of the NB shares in slice order + b_2, softmax cross-entropy, dZ_2
//       (redundantly in every workgroup: a few hundred values)
//   (4) dZ_1[:, C] = (dZ_2 W_2[C, :]^T) .* [A_1[:, C] > 0]  with the weights of before the update
//   and with all wavefronts again
//   (5) dW_2[C, :] = A_1[:, C]^T dZ_2, db_2 and their momentum updates (one wavefront each)
//   (6) dW_1[:, C] = A_0^T dZ_1[:, C], db_1[C] and the momentum update of the slice
// The only communication is the share of the logits (Bp x 16 values per workgroup and step), into a
// region of the step's own.  (Exchanging the logit shares instead of the activations is what lets W_2 be
// partitioned: with the activations exchanged every workgroup had to keep and update a full
// copy of W_2, and the second layer's products, done 16 times over, were a quarter of the step.)
//
// What bounds it is the chain of phases.  784-256-10, 8 replicas, batch 64, fp32, in clocks of a step of
// 30000 (12.5 us): (1) 10000, of which 6300 are matrix instructions, (2) 1500, barrier 2500, (3) 4500,
// (4) 900, (5) and (6) 10500, of which 6300 matrix instructions.  It was 42000 with the phases (2) to (5)
// spread over all threads and LDS (a 64-term sum per thread for dW_2 alone made the step wait for 8000,
// the shuffles of the softmax and an L2 invalidation per barrier for 3000) and the inputs in plain rows:
// 461 us for 4 periods of 5 steps then, 341 us now.
//
// The barrier is a counter per replica and batch tile in device memory (arrive_and_wait_step); the
// counters are never reset, each launch is told their value at its start.  All workgroups of a launch are
// co-resident (the launcher refuses grids above one workgroup per compute unit), and the
// poll loop is bounded: a wavefront that runs out of polls raises the error flag, stops
// waiting for good and finishes its steps, so the grid always drains.  (A cooperative launch
// would have the runtime vouch for the co-residency, but costs 18 us more per launch here, a
// tenth of the throughput at five steps per launch; the bounded wait covers the same case.)
// Where an XCD has compute units for an eighth of the replicas, a replica's workgroups all go to one
// XCD, and shares and counters stay in its L2: up to 64 replicas of 64 hidden
// units, 16 of 256.
//
// A launch may also hold several whole communication periods: after every `period` steps the
// averaging step of Sec. 2 is taken inside the kernel (average_resident), with one barrier over
// all workgroups of all replicas, always at agent scope.
#include "lc_internal.h"
#include "lc_mma.h"

namespace lc {

namespace {

constexpr int kResMaxD0 = 1024;   // padded input width the LDS slice is sized for
constexpr int kResMaxD1 = 256;    // padded hidden width: at most kResMaxSlices shares of the logits are requested at once
constexpr int kResMaxSlices = 16;
static_assert(kResMaxD1 <= 16 * kResMaxSlices, "a slice whose share nobody adds would be missing from the logits");
constexpr int kResShare = 16 * 16;   // a slice's share of the logits of one batch tile, floats
static_assert(kResShare * sizeof(float) % 128 == 0, "shares in whole cache lines, see arrive_and_wait_step");
constexpr int kResK1P = kResMaxD0 + 4;
constexpr int kResWaves = 16;                    // wavefronts per workgroup: four per SIMD hide each other's waits
constexpr int kResThreads = kResWaves * 64;
constexpr int kResTiles = kResMaxD0 / 16 / kResWaves;   // 16-row tiles of W_1 per wavefront

struct ResArgs {
    float* X;
    float* V;
    int64_t x_stride;
    const float* Xr;      // where the weights are read at the start: X, or the one averaged model
    int64_t xr_stride;
    int64_t w1_off, b1_off, w2_off, b2_off;
    int d0, d1, d2, dp0, dp1;
    int B, G, NB;
    const void* a0_bm;    // [slots][G] A_0 in fragment order, tiles of 16 samples
    const void* a0_fm;    // [slots][G] A_0^T in fragment order, tiles of 16 features
    int64_t a0_slot;      // elements per slot
    const int32_t* labels;  // [slots][G][Bp]
    int slot0, n_steps;
    float lr, beta_first, beta, wd;
    int vec;              // rows of W_1 may be accessed 16 bytes at a time
    float* zx;            // [steps][G][NB][Bp][16] exchange buffer: the slices' shares of the logits, by step of the launch
    unsigned* ctr;        // [G][MT][kCtrTile] arrivals since attach, by batch tile: every workgroup arrives once per step, whatever
                          // happens.  (One slice has nobody to wait for: nobody arrives and nobody looks)
    unsigned ctr_base;    // their value when this launch starts
    unsigned* err;        // set to 1 when a barrier wait ran out of polls
    int spin_limit;       // polls one barrier wait may take
    float* loss;          // [G][kLossParts], slot 0 written
    int local_xcd;        // every replica's workgroups share one XCD (one L2): exchange through that L2
    unsigned xcc_of;      // 4 bits per residue of the hardware block id mod 8: the XCD such blocks run on
    int period;           // averaging step after every `period` steps inside the launch; 0: none
    float* avx;           // [2][G][x_stride] models handed over at an averaging step, by parity of the period
    unsigned* gctr;       // arrivals of all workgroups at averaging steps since attach
    unsigned gctr_base;   // its value when this launch starts
};

// Barrier among the workgroups that add to *ctr, called by one thread per workgroup after a
// workgroup barrier: what the workgroup wrote before is visible to every workgroup that leaves
// the wait.  The wait is bounded; a workgroup that runs out of polls raises the error flag and
// never waits again (it still arrives, so the counts stay right), so the grid always drains.
__device__ __forceinline__ void arrive_and_wait(unsigned* ctr, unsigned target, int spin_limit, unsigned* err,
                                                bool& gave_up) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int polls = 0;
    while (!gave_up) {
        if (polls++ >= spin_limit) {   // a limit of 0 gives up without looking: the host's way to force this path
            gave_up = true;
            atomicOr(err, 1u);
            break;
        }
        const unsigned seen = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (static_cast<int>(seen - target) >= 0) break;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// The barrier of a step, among the wavefronts of one batch tile: no cache is written back or invalidated.
// What it orders are the shares of the logits, and those (a) have been stored through to the scope that the
// readers share, and have arrived there (the caller waits for its stores), (b) lie in a region of the step's
// own, whose lines nobody has read before in this launch -- and a launch begins with the caches clean -- so
// no reader holds an older copy.  (A share is whole cache lines of its own: kResShare, and the buffer is aligned
// to 256 bytes.  Another layout has to keep that.  The agent-scope acquire invalidates the L2 as well: 3000 clocks of a step
// of 42000 with one per workgroup, 10000 with one per wavefront.)
//
// local: the wavefronts run on one XCD, i.e. behind one L2, and counter and data need not leave it.
// Read-modify-write atomics without the device-scope bit are performed in the L2, so the counter is
// added to and polled there (the poll is a compare-and-swap that never matches: a workgroup-scope LOAD
// may be served by the compute unit's L1 and then never sees the count move -- measured), where the
// agent-scope form sends data and counter to the memory side and back.  Valid only while the participants
// really share an L2: the launcher checks the placement rule once with a probe kernel, and every
// workgroup checks its own XCD id against it.
__device__ __forceinline__ void arrive_and_wait_step(unsigned* ctr, unsigned target, int spin_limit, unsigned* err,
                                                     bool local, bool& gave_up) {
    if (local) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int polls = 0;
    while (!gave_up) {
        if (polls++ >= spin_limit) {
            gave_up = true;
            atomicOr(err, 1u);
            break;
        }
        unsigned seen = 0xFFFFFFFFu;   // (were the count ever this, the swap would write the same value back)
        if (local)
            __hip_atomic_compare_exchange_strong(ctr, &seen, 0xFFFFFFFFu, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            seen = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (static_cast<int>(seen - target) >= 0) break;
    }
}

// The XCD this wavefront runs on: hardware register XCC_ID (number 20), bits 3:0.  The operand
// of s_getreg is (size - 1) << 11 | offset << 6 | register.
__device__ __forceinline__ unsigned this_xcd() { return __builtin_amdgcn_s_getreg(((4 - 1) << 11) | (0 << 6) | 20); }

__global__ void xcd_probe_kernel(unsigned* out) {
    if (threadIdx.x == 0) out[blockIdx.x] = this_xcd();
}

// x_bar = (1/m) sum_i x^(i) of one entry (Sec. 2, the averaging step), summed in double in
// replica order and rounded once: the same arithmetic, bit for bit, as the averaging kernels.
__device__ __forceinline__ float mean_of_replicas(const float* p, int64_t stride, int G) {
    double s = 0.0;
    for (int i0 = 0; i0 < G; i0 += 4) {   // four loads in flight, added in replica order
        float r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u < G) r[u] = p[(i0 + u) * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u < G) s += static_cast<double>(r[u]);
    }
    return static_cast<float>(s / static_cast<double>(G));
}

__device__ __forceinline__ float round_operand(float x, bf16_t) { return static_cast<float>(static_cast<bf16_t>(x)); }
__device__ __forceinline__ float round_operand(float x, float) { return x; }

// The averaging step inside a resident launch (Sec. 2: after tau local updates the models are
// replaced by their mean; the momentum buffers stay local).  Every workgroup hands over its part
// of the model, waits for all workgroups of all replicas, and forms the mean of its own part from
// the m copies.  Two buffers, by parity of the period: a workgroup overwrites a buffer only after
// the barrier of the period in between, which every reader of the older contents has reached by
// then.
__device__ __forceinline__ void average_resident(const ResArgs& a, int tid, int pi, int g, int cb,
                                                 float (*w1s)[kResK1P], float (*w2s)[17], float* b1s,
                                                 float* b2s, bool& gave_up) {
    const int wave = tid >> 6, j = tid & 15, q = (tid >> 4) & 3;
    const int c_base = 16 * cb, n_kt = a.dp0 / 16;
    const bool vec = a.vec != 0;
    float* all = a.avx + static_cast<int64_t>(pi & 1) * a.G * a.x_stride;
    float* mine = all + g * a.x_stride;
    for (int kt = wave; kt < n_kt; kt += kResWaves) {
        const int k = 16 * kt + j, c = c_base + 4 * q;
        if (k < a.d0) {
            const float4 w = make_float4(w1s[4 * q + 0][k], w1s[4 * q + 1][k], w1s[4 * q + 2][k], w1s[4 * q + 3][k]);
            store_w4(mine + a.w1_off + static_cast<int64_t>(k) * a.d1, c, a.d1, vec, false, w);
        }
    }
    if (tid < 16 && c_base + tid < a.d1) mine[a.b1_off + c_base + tid] = b1s[tid];
    if (tid >= 64 && tid < 320) {   // own rows of the second layer
        const int kk = (tid - 64) >> 4, c2 = tid & 15;
        if (c_base + kk < a.d1 && c2 < a.d2) mine[a.w2_off + static_cast<int64_t>(c_base + kk) * a.d2 + c2] = w2s[c2][kk];
    }
    if (cb == 0 && tid < a.d2) mine[a.b2_off + tid] = b2s[tid];
    __builtin_amdgcn_s_waitcnt(0);   // this wavefront's stores have left before the workgroup arrives
    __syncthreads();
    if (tid == 0)
        arrive_and_wait(a.gctr, a.gctr_base + static_cast<unsigned>(pi + 1) * static_cast<unsigned>(a.G * a.NB),
                        a.spin_limit, a.err, gave_up);
    __syncthreads();
    for (int kt = wave; kt < n_kt; kt += kResWaves) {
        const int k = 16 * kt + j, c = c_base + 4 * q;
        if (k < a.d0) {
            const float* src = all + a.w1_off + static_cast<int64_t>(k) * a.d1;
            double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
            for (int g0 = 0; g0 < a.G; g0 += 8) {
                float4 r[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (g0 + u < a.G) r[u] = load_w4(src + (g0 + u) * a.x_stride, c, a.d1, vec, false);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (g0 + u < a.G) {
                        s0 += static_cast<double>(r[u].x);
                        s1 += static_cast<double>(r[u].y);
                        s2 += static_cast<double>(r[u].z);
                        s3 += static_cast<double>(r[u].w);
                    }
            }
            const double dm = static_cast<double>(a.G);
            w1s[4 * q + 0][k] = static_cast<float>(s0 / dm);
            w1s[4 * q + 1][k] = static_cast<float>(s1 / dm);
            w1s[4 * q + 2][k] = static_cast<float>(s2 / dm);
            w1s[4 * q + 3][k] = static_cast<float>(s3 / dm);
        }
    }
    // the second layer and the biases, an entry at a time (its m loads together): this phase must
    // stay light in registers, the step loop around it has none to spare
    if (tid >= 128 && tid < 384) {
        const int kk = (tid - 128) >> 4, c2 = tid & 15;
        if (c_base + kk < a.d1 && c2 < a.d2)
            w2s[c2][kk] = mean_of_replicas(all + a.w2_off + static_cast<int64_t>(c_base + kk) * a.d2 + c2, a.x_stride, a.G);
    }
    if (tid < 16 && c_base + tid < a.d1) b1s[tid] = mean_of_replicas(all + a.b1_off + c_base + tid, a.x_stride, a.G);
    if (tid >= 64 && tid < 64 + a.d2) b2s[tid - 64] = mean_of_replicas(all + a.b2_off + tid - 64, a.x_stride, a.G);
    __syncthreads();
}

template <typename OT, int MT>
__global__ __launch_bounds__(kResThreads) void resident_kernel(ResArgs args) {
    const ResArgs& a = args;
    constexpr int Bp = 16 * MT;
    constexpr int NS = Bp / 32;   // 32-wide steps over the batch
    constexpr int KP = kResWaves / MT;   // wavefronts that share one batch tile and split the reduction
    __shared__ __attribute__((aligned(16))) float w1s[16][kResK1P];    // W_1[:, C]^T
    __shared__ float w2s[16][17], v2s[16][17];                          // W_2[C, :]^T, V_2[C, :]^T: [class][own hidden unit]
    __shared__ __attribute__((aligned(16))) float part[KP - 1][Bp][20];
    __shared__ float a1s[Bp][17];                                       // own slice of A_1
    __shared__ float z2s[Bp][17];                                       // dZ_2
    __shared__ __attribute__((aligned(16))) OT dz1t[16][Bp + 8];        // dZ_1[:, C]^T
    __shared__ float b1s[16], vb1s[16], b2s[16], vb2s[16];
    __shared__ float lred[Bp];
    __shared__ float colsum1[MT][16], colsum2[MT][16];

    // Blocks are dealt to the XCDs round-robin.  Replica g has its blocks on XCD g mod 8 where each XCD has
    // compute units enough for that; else the replicas' blocks simply follow each other.
    int g, cb;
    if (a.local_xcd) {
        const int i = blockIdx.x / kXcds;
        g = blockIdx.x % kXcds + kXcds * (i / a.NB);
        cb = i % a.NB;
        if (g >= a.G) return;
    } else {
        const int64_t logical = xcd_logical_block(static_cast<int64_t>(a.G) * a.NB);
        if (logical < 0) return;
        g = static_cast<int>(logical / a.NB);
        cb = static_cast<int>(logical % a.NB);
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, q = lane >> 4;
    const int c_base = 16 * cb;
    const int n_kt = a.dp0 / 16;
    const bool vec = a.vec != 0;

    float* Xg = a.X + g * a.x_stride;
    float* Vg = a.V + g * a.x_stride;
    const float* Xrg = a.Xr + g * a.xr_stride;
    // ---- load the resident state
    f32x4 v1[kResTiles];   // V_1 at rows 16 kt + j, columns c_base + 4 q .. + 3, kt = wave + 16 i
    {
        // all tiles' loads first, with no branch around them (rows that do not exist read the last
        // row and are zeroed): one memory round trip instead of one per tile
        float4 wl[kResTiles], vl[kResTiles];
        if (vec && c_base + 16 <= a.d1) {   // the whole slice exists and is aligned (uniform over the workgroup)
#pragma unroll
            for (int i = 0; i < kResTiles; ++i) {
                const int k = 16 * (wave + kResWaves * i) + j, kc = k < a.d0 ? k : a.d0 - 1;
                const int64_t at = a.w1_off + static_cast<int64_t>(kc) * a.d1 + c_base + 4 * q;
                wl[i] = *reinterpret_cast<const float4*>(Xrg + at);
                vl[i] = *reinterpret_cast<const float4*>(Vg + at);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kResTiles; ++i) {
                const int k = 16 * (wave + kResWaves * i) + j, kc = k < a.d0 ? k : a.d0 - 1;
                wl[i] = load_w4(Xrg + a.w1_off + static_cast<int64_t>(kc) * a.d1, c_base + 4 * q, a.d1, vec, false);
                vl[i] = load_w4(Vg + a.w1_off + static_cast<int64_t>(kc) * a.d1, c_base + 4 * q, a.d1, vec, false);
            }
        }
#pragma unroll
        for (int i = 0; i < kResTiles; ++i) {
            const int kt = wave + kResWaves * i, k = 16 * kt + j;
            const bool in = k < a.d0;
            v1[i] = in ? f32x4{vl[i].x, vl[i].y, vl[i].z, vl[i].w} : f32x4{0.f, 0.f, 0.f, 0.f};
            if (kt < n_kt) {
                w1s[4 * q + 0][k] = in ? wl[i].x : 0.f;
                w1s[4 * q + 1][k] = in ? wl[i].y : 0.f;
                w1s[4 * q + 2][k] = in ? wl[i].z : 0.f;
                w1s[4 * q + 3][k] = in ? wl[i].w : 0.f;
            }
        }
    }
    if (tid < 256) {   // own rows of the second layer
        const int kk = tid >> 4, c2 = tid & 15;
        const bool in = c_base + kk < a.d1 && c2 < a.d2;
        const int64_t at = a.w2_off + (in ? static_cast<int64_t>(c_base + kk) * a.d2 + c2 : 0);
        const float w = Xrg[at], v = Vg[at];
        w2s[c2][kk] = in ? w : 0.f;
        v2s[c2][kk] = in ? v : 0.f;
    }
    if (tid < 16) {
        const bool in1 = c_base + tid < a.d1, in2 = tid < a.d2;
        b1s[tid] = in1 ? Xrg[a.b1_off + c_base + tid] : 0.f;
        vb1s[tid] = in1 ? Vg[a.b1_off + c_base + tid] : 0.f;
        b2s[tid] = in2 ? Xrg[a.b2_off + tid] : 0.f;
        vb2s[tid] = in2 ? Vg[a.b2_off + tid] : 0.f;
    }
    __syncthreads();
    bool gave_up = false;   // first lane of a wavefront: one of its barrier waits ran out of polls
    if (a.local_xcd && threadIdx.x == 0 && this_xcd() != ((a.xcc_of >> (4 * (blockIdx.x % kXcds))) & 15u))
        atomicOr(a.err, 2u);   // not where the probe saw such blocks run: the exchange cannot be trusted
    // the input rows of batch tile mt, and where a wavefront's share of their fragments begins
    auto input_tile = [&](const ResArgs& a, int slot, int mt) {
        return static_cast<const OT*>(a.a0_bm) + slot * a.a0_slot + (static_cast<int64_t>(g) * MT + mt) * (a.dp0 / 32) * kFragElems;
    };
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    const int first_st = uwave / MT < (a.d0 + 31) / 32 ? uwave / MT : 0;
    for (int s = 0; s < a.n_steps;) {
    // One period (the whole launch when it has no averaging steps).
    const int s_end = a.period > 0 ? s + a.period : a.n_steps;
    const int s_begin = s;
    Frag<OT> af;
    for (; s < s_end; ++s) {
        // What a step derives from the thread's id is derived afresh from an opaque copy, so that none of
        // it is held in registers across the steps and the averaging step, which need them for their loads.
        int tid_o = threadIdx.x;
        asm volatile("" : "+v"(tid_o));
        const int tid = tid_o, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 15, q = lane >> 4;
        int zero = 0;   // ... and what it takes from the arguments is read afresh, for the scalar registers' sake
        asm volatile("" : "+s"(zero));
        const ResArgs& a = (&args)[zero];
        const float beta = s == 0 ? a.beta_first : a.beta, lr = a.lr, wd = a.wd;
        const int d1 = a.d1, d2 = a.d2, NB = a.NB;
        const int slot = a.slot0 + s;
        const OT* A0T = static_cast<const OT*>(a.a0_fm) + slot * a.a0_slot + static_cast<int64_t>(g) * a.dp0 * Bp;
        const int32_t* lab = a.labels + (static_cast<int64_t>(slot) * a.G + g) * Bp;
        float* xp = a.zx + (static_cast<int64_t>(s) * a.G + g) * Bp * a.dp1;   // [NB][Bp][16] of [dp1 / 16][Bp][16]
        // ---- (1) Z_1[:, C]^T: wavefront (mt, kpart) takes batch tile mt and the 32-wide k steps
        //      kpart, kpart + KP, ...  A lane ends up with hidden units 4 q .. 4 q + 3 of sample 16 mt + j.
        const int mt = wave % MT, kpart = wave / MT;
        f32x4 z1 = f32x4{0.f, 0.f, 0.f, 0.f};
        const int y = kpart == 0 && 16 * mt + j < a.B ? lab[16 * mt + j] : -1;
        {
            const OT* atile = input_tile(a, slot, mt);
            if (s == s_begin) af = load_frag(atile + kFragElems * first_st, lane);
            const int n_st = (a.d0 + 31) / 32;   // (steps that hold only padding rows are skipped)
            for (int st = kpart; st < n_st; st += KP) {
                const int k0 = 32 * st + 8 * q;
                const int nx = st + KP < n_st ? st + KP : st;
                const Frag<OT> af_next = load_frag(atile + kFragElems * nx, lane);   // next step's operand in flight
                const float4 x0 = *reinterpret_cast<const float4*>(&w1s[j][k0]);
                const float4 x1 = *reinterpret_cast<const float4*>(&w1s[j][k0 + 4]);
                const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
                Frag<OT> bf;
                pack8(bf, x);
                z1 += mma8(bf, af, f32x4{0.f, 0.f, 0.f, 0.f});   // (sums of 32, added up: no error of a long chain)
                af = af_next;
            }
        }
        if (kpart > 0) *reinterpret_cast<f32x4*>(&part[kpart - 1][16 * mt + j][4 * q]) = z1;
        // (operands of what follows the barrier)
        float w2a[4];   // W_2[own unit 4 q + i, class j]
        if (wave < MT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w2a[i] = round_operand(w2s[j][4 * q + i], OT());
        }
        __syncthreads();
        // ---- (2) to (4): wavefront mt takes batch tile mt from the partial sums to dZ_1 in registers.  The
        //      16 x 16 products have their reduction index in the order the results before them are in:
        //      instruction i sums over units (classes) 4 q + i, which a lane holds in register i.
        if (wave < MT) {
            const int b = 16 * mt + j;
            f32x4 a1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 1; p < KP; ++p) z1 += *reinterpret_cast<const f32x4*>(&part[p - 1][b][4 * q]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float z = z1[r] + b1s[4 * q + r];
                if (b < a.B && c_base + 4 * q + r < d1) a1[r] = round_operand(z > 0.f ? z : 0.f, OT());
                a1s[b][4 * q + r] = a1[r];
            }
            // ---- (2) this slice's share of the logits, (A_1[:, C] W_2[C, :])^T, handed to the replica
            f32x4 zp = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                zp = __builtin_amdgcn_mfma_f32_16x16x4f32(w2a[i], a1[i], zp, 0, 0, 0);
            float* px = xp + static_cast<int64_t>(cb) * (MT * kResShare) + b * 16 + 4 * q;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (a.local_xcd) __hip_atomic_store(px + r, zp[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);   // as far as the XCD's L2
                else __hip_atomic_store(px + r, zp[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // written through to device scope
            }
            // ---- replica-wide barrier of the wavefronts of this batch tile: nothing else is exchanged
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);   // the whole wavefront's stores have arrived before it does
            if (NB > 1 && lane == 0) {
                const unsigned target = a.ctr_base + static_cast<unsigned>(s + 1) * static_cast<unsigned>(NB);
                arrive_and_wait_step(a.ctr + (g * MT + mt) * kCtrTile, target, a.spin_limit, a.err, a.local_xcd != 0, gave_up);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            // ---- (3) logits = sum of the slices' shares in slice order + b_2; softmax cross-entropy and
            //      dZ_2 (redundantly in every workgroup: a few hundred values).  Classes 4 q .. 4 q + 3 of
            //      sample b in a lane; all shares are requested at once.
            f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
            {
                const float* sx = xp + b * 16 + 4 * q;
                f32x4 r[kResMaxSlices];
#pragma unroll
                for (int o = 0; o < kResMaxSlices; ++o) r[o] = *reinterpret_cast<const f32x4*>(sx + (o < NB ? o : 0) * (MT * kResShare));
#pragma unroll
                for (int o = 0; o < kResMaxSlices; ++o) z += o < NB ? r[o] : f32x4{0.f, 0.f, 0.f, 0.f};
            }
            float zmax = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                z[r] += b2s[4 * q + r];
                if (4 * q + r < d2) zmax = fmaxf(zmax, z[r]);
            }
            zmax = max_over_quarters(zmax);
            f32x4 ex;
            float s_other = 0.f, e_y = 0.f, z_y = 0.f;   // (over the classes other than the label, see xent_loss)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 4 * q + r;
                ex[r] = c < d2 ? expf(z[r] - zmax) : 0.f;
                s_other += c == y ? 0.f : ex[r];
                e_y += c == y ? ex[r] : 0.f;
                z_y += c == y ? z[r] : 0.f;
            }
            s_other = sum_over_quarters(s_other);
            const float sum = s_other + sum_over_quarters(e_y), inv = 1.f / sum, invB = 1.f / static_cast<float>(a.B);
            f32x4 dz2, dz1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 4 * q + r;
                dz2[r] = y >= 0 && c < d2 ? round_operand(xent_delta(ex[r], c == y, s_other, inv) * invB, OT()) : 0.f;
                z2s[b][c] = dz2[r];
            }
            if (cb == 0) {   // (the step's own loss is a by-product here: the plain form, without the log1p of xent_loss)
                z_y = sum_over_quarters(z_y);
                if (q == 0) lred[b] = y >= 0 ? -(z_y - zmax - logf(sum)) : 0.f;
            }
            // ---- (4) dZ_1[:, C]^T from the second layer's weights of before this step's update, and this
            //      tile's sums of dZ_1[:, C] and dZ_2 (bias gradients)
#pragma unroll
            for (int i = 0; i < 4; ++i) dz1 = __builtin_amdgcn_mfma_f32_16x16x4f32(round_operand(w2s[4 * q + i][j], OT()), dz2[i], dz1, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const OT d = static_cast<OT>(a1[r] > 0.f ? dz1[r] : 0.f);   // rounds in bf16 mode
                dz1t[4 * q + r][b] = d;
                const float s1 = sum_over_row(to_f32(d)), s2 = sum_over_row(dz2[r]);
                if (j == 0) {
                    colsum1[mt][4 * q + r] = s1;
                    colsum2[mt][4 * q + r] = s2;
                }
            }
        }
        __syncthreads();
        // ---- the step's loss and the bias updates.  These small jobs go to the last wavefronts: when the
        //      tiles of step (6) do not divide evenly, those have one tile less to do
        if (cb == 0 && wave == kResWaves - 3) {
            float v = lane < Bp ? lred[lane] : 0.f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (lane == 0) a.loss[static_cast<int64_t>(g) * kLossParts] = v / static_cast<float>(a.B);
        }
        if (wave == kResWaves - 2 && lane < 32) {
            const int c = lane & 15;
            const bool first = lane < 16;
            float db = 0.f;
#pragma unroll
            for (int w = 0; w < MT; ++w) db += first ? colsum1[w][c] : colsum2[w][c];
            if (first) {
                if (c_base + c < d1) {
                    const float vb = momentum_update(beta, vb1s[c], db, wd, b1s[c]);
                    vb1s[c] = vb;
                    b1s[c] = weight_update(b1s[c], lr, vb);
                }
            } else if (c < d2) {
                const float vb = momentum_update(beta, vb2s[c], db, wd, b2s[c]);
                vb2s[c] = vb;
                b2s[c] = weight_update(b2s[c], lr, vb);
            }
        }
        // ---- (5) dW_2[C, :] = A_1[:, C]^T dZ_2 and the update of the own rows
        if (wave == kResWaves - 1) {
            __builtin_amdgcn_s_setprio(3);   // (its own tiles wait for this, and the step for them)
            f32x4 gw = f32x4{0.f, 0.f, 0.f, 0.f};
            float x[Bp / 4], y[Bp / 4];
#pragma unroll
            for (int i = 0; i < Bp / 4; ++i) {
                x[i] = a1s[4 * i + q][j];
                y[i] = z2s[4 * i + q][j];
            }
            __builtin_amdgcn_sched_barrier(0);   // all reads before the chain of products, not one pair after the other
#pragma unroll
            for (int i = 0; i < Bp / 4; ++i) gw = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], gw, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kk = 4 * q + r;   // (entries that do not exist are zero and stay zero)
                const float w = w2s[j][kk];
                const float v = momentum_update(beta, v2s[j][kk], c_base + kk < d1 && j < d2 ? gw[r] : 0.f, wd, w);
                v2s[j][kk] = v;
                w2s[j][kk] = weight_update(w, lr, v);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        // ---- (6) dW_1[:, C] = A_0^T dZ_1[:, C] and the update of the slice
#pragma unroll
        for (int i = 0; i < kResTiles; ++i) {
            const int kt = wave + kResWaves * i;
            if (16 * kt < a.d0) {   // (tiles that hold only padding rows have nothing to update)
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < NS; ++st) {
                    const int b0 = 32 * st + 8 * q;
                    const Frag<OT> af = *reinterpret_cast<const Frag<OT>*>(&dz1t[j][b0]);
                    const Frag<OT> bf = load_frag(A0T + static_cast<int64_t>(kt * NS + st) * kFragElems, lane);
                    acc = mma8(af, bf, acc);
                }
                const int k = 16 * kt + j;
                // rows k >= d0 and columns beyond d1 have zero gradient, weight and momentum,
                // and stay zero under the update
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float w = w1s[4 * q + r][k];
                    const float v = momentum_update(beta, v1[i][r], acc[r], wd, w);
                    v1[i][r] = v;
                    w1s[4 * q + r][k] = weight_update(w, lr, v);
                }
            }
        }
        if (s + 1 < s_end) af = load_frag(input_tile(a, slot + 1, mt) + kFragElems * first_st, lane);   // on its way across the barrier
        __syncthreads();
    }
    int tid_a = threadIdx.x;
    asm volatile("" : "+v"(tid_a));
    if (a.period > 0) average_resident(a, tid_a, s / a.period - 1, g, cb, w1s, w2s, b1s, b2s, gave_up);
    }

    // ---- write the state back
    int tid_w = threadIdx.x;
    asm volatile("" : "+v"(tid_w));
    {
    const int tid = tid_w, wave = tid >> 6, j = tid & 15, q = (tid >> 4) & 3;
#pragma unroll
    for (int i = 0; i < kResTiles; ++i) {
        const int kt = wave + kResWaves * i;
        if (kt < n_kt) {
            const int k = 16 * kt + j, c = c_base + 4 * q;
            if (k < a.d0) {
                const float4 w = make_float4(w1s[4 * q + 0][k], w1s[4 * q + 1][k], w1s[4 * q + 2][k], w1s[4 * q + 3][k]);
                const float4 v = make_float4(v1[i][0], v1[i][1], v1[i][2], v1[i][3]);
                store_w4(Xg + a.w1_off + static_cast<int64_t>(k) * a.d1, c, a.d1, vec, false, w);
                store_w4(Vg + a.w1_off + static_cast<int64_t>(k) * a.d1, c, a.d1, vec, false, v);
            }
        }
    }
    if (tid < 16 && c_base + tid < a.d1) {
        Xg[a.b1_off + c_base + tid] = b1s[tid];
        Vg[a.b1_off + c_base + tid] = vb1s[tid];
    }
    if (tid >= 64 && tid < 320) {   // own rows of the second layer
        const int kk = (tid - 64) >> 4, c2 = tid & 15;
        if (c_base + kk < a.d1 && c2 < a.d2) {
            const int64_t at = a.w2_off + static_cast<int64_t>(c_base + kk) * a.d2 + c2;
            Xg[at] = w2s[c2][kk];
            Vg[at] = v2s[c2][kk];
        }
    }
    if (cb == 0 && tid < a.d2) {
        Xg[a.b2_off + tid] = b2s[tid];
        Vg[a.b2_off + tid] = vb2s[tid];
    }
    }
}

// Softmax regression (one layer, d0 -> d1 with d1 <= 16 classes): the same idea without any
// exchange.  One workgroup per replica takes all the steps of a launch, and selects and fetches the
// mini-batches itself.  Wavefront w owns the weights and momentum of features 16 w .. 16 w + 15, in registers
// (class 4 q + r of feature 16 w + j in register r); LDS holds a copy of W^T for the logits and the batch.
// One step:
//   logits, the wavefronts sharing out batch tiles and the reduction; every wavefront also takes its operand
//     of the weight gradient, A_0 of its features, into registers
//   one wavefront per batch tile: softmax cross-entropy and dZ; all: a batch that was requested a step ago
//     into LDS, and another one requested
//   dW = A_0^T dZ and the update of the own tile
// What bounds it is latency: 64-10, 4 workers, batch 32, one period of 4 steps, 14.2 us -- 1.7 us a step (1 to 16
// steps: 9.1 to 34.7 us), 2.5 us for the averaging step in the launch (1 to 4 periods: 14.2 to 42.3 us), 4.9 us for the
// launch itself, the indices' hash and one round trip for rows, state and labels.  With a gather kernel before it, W in
// LDS only and the softmax through LDS it was 18.2 us.
struct Res1Args {
    float* X;
    float* V;
    int64_t x_stride;
    const float* Xr;
    int64_t xr_stride;
    int64_t w_off, b_off;
    int d0, d1, dp0;
    int B, G;
    const void* data;       // [N][d0] of OT
    const int32_t* labels;  // [N]
    int32_t* idx_out;       // [steps][G][Bp] of the launch
    int64_t N;
    uint64_t seed;
    int64_t k;              // local iteration of the launch's first step
    int sampler, m;
    int n_steps, ring;      // batches the ring holds
    float lr, beta_first, beta, wd;
    float* loss;            // [G][kLossParts], slot 0 written
    int period;             // averaging step after every `period` steps inside the launch; 0: none
    float* avx;             // [2][G][x_stride] models handed over at an averaging step
    unsigned* gctr;         // arrivals at averaging steps since attach
    unsigned gctr_base;
    unsigned* err;
    int spin_limit;
};

constexpr int kRes1Steps = 4 * kGatherSlots;   // most steps of a launch
constexpr int kRes1Ring = 96 * 1024;           // bytes of the ring of batches
constexpr int kRes1First = 6;                  // rounds of fetches at the start
constexpr int kRes1K = 256;                    // padded inputs: 16 features for each of the 16 wavefronts

template <typename OT, int MT>
__global__ __launch_bounds__(kResThreads) void resident1_kernel(Res1Args a) {
    constexpr int Bp = 16 * MT;
    constexpr int NS = Bp / 32;
    constexpr int KP = kResWaves / MT;
    constexpr int NP = MT;   // rounds of fetches for a batch: each takes at least a row per wavefront
    __shared__ __attribute__((aligned(16))) OT ring[kRes1Ring / sizeof(OT)];   // A_0 of several steps
    __shared__ __attribute__((aligned(16))) float ws[16][kRes1K + 4];   // W^T (row = class)
    __shared__ __attribute__((aligned(16))) float part[KP - 1][Bp][20];
    __shared__ __attribute__((aligned(16))) OT dzt[16][Bp + 8];         // dZ^T
    __shared__ int idxs[kRes1Steps * Bp], labs[kRes1Steps * Bp];        // [step][Bp], -1: no sample
    __shared__ float bs[16], vbs[16];
    __shared__ float lred[Bp];

    const int g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, q = lane >> 4;
    float* Xg = a.X + g * a.x_stride;
    float* Vg = a.V + g * a.x_stride;
    const float* Xrg = a.Xr + g * a.xr_stride;
    const int d0 = a.d0, d1 = a.d1, dp0 = a.dp0;
    const float lr = a.lr, wd = a.wd;

    // ---- the launch's mini-batches
    for (int e = tid; e < a.n_steps * Bp; e += kResThreads) {
        const int s = e / Bp, b = e % Bp;
        int64_t idx = -1;
        if (b < a.B)
            idx = a.sampler ? partition_index(a.seed, g, a.k + s, b, a.N, a.m, a.B) : batch_index(a.seed, g, a.k + s, b, a.N);
        idxs[e] = static_cast<int>(idx);
        a.idx_out[(static_cast<int64_t>(s) * a.G + g) * Bp + b] = static_cast<int>(idx);
    }
    __syncthreads();
    // The ring holds R batches.  The first `lead - 1` are fetched together; the one after them is on its way
    // when the steps begin, and step s places batch s + lead - 1 and requests batch s + lead.
    const OT* data = static_cast<const OT*>(a.data);
    const int row = dp0 + 16 / static_cast<int>(sizeof(OT)), R = a.ring, lead = R > 1 ? R : 2;
    // A lane fetches 4 features; a wavefront takes as many whole rows at a time as it has lanes for.
    const bool vec = d0 % 4 == 0;   // row pieces are whole and aligned
    const int per_row = dp0 / 4, rows = 64 / per_row, lane_row = lane / per_row, c = 4 * (lane - per_row * lane_row);
    const int my_row = lane_row < rows ? wave * rows + lane_row : -(1 << 20);   // of the 16 * rows of a round
    auto fetch = [&](int idx) {   // features c .. c + 3 of a sample, zero where there are none
        const bool in = idx >= 0 && c < d0;
        const OT* p = data + (in ? static_cast<int64_t>(idx) * d0 + c : 0);
        Frag4<OT> f;
        if (vec) {
            f = load4(p);
            if (!in) pack4(f, 0.f, 0.f, 0.f, 0.f);
        } else {
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = to_f32(p[in && c + i < d0 ? i : 0]);
            pack4(f, in ? x[0] : 0.f, in && c + 1 < d0 ? x[1] : 0.f, in && c + 2 < d0 ? x[2] : 0.f, in && c + 3 < d0 ? x[3] : 0.f);
        }
        return f;
    };
    auto put = [&](OT* to, const Frag4<OT>& f) { store4(to, to_f32(f.v[0]), to_f32(f.v[1]), to_f32(f.v[2]), to_f32(f.v[3])); };
    Frag4<OT> next[NP];
    auto request = [&](int s) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int b = my_row + kResWaves * rows * u;
            if (kResWaves * rows * u < Bp) next[u] = fetch(b >= 0 && b < Bp ? idxs[s * Bp + b] : -1);
        }
    };
    auto place = [&](int s) {
        OT* to = ring + s % R * (Bp * row) + c;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int b = my_row + kResWaves * rows * u;
            if (b >= 0 && b < Bp) put(to + b * row, next[u]);
        }
    };
    const int n_first = (lead - 1 < a.n_steps ? lead - 1 : a.n_steps) * Bp;   // rows
    Frag4<OT> first[kRes1First];
#pragma unroll
    for (int u = 0; u < kRes1First; ++u) {
        const int r = my_row + kResWaves * rows * u;
        if (kResWaves * rows * u < n_first) first[u] = fetch(r >= 0 && r < n_first ? idxs[r] : -1);
    }
    // ---- the own tile of the state (entries that do not exist read the first one and are zeroed), the labels
    const int k_own = 16 * wave + j;
    float w[4], v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool in = k_own < d0 && 4 * q + r < d1;
        const int64_t at = a.w_off + (in ? k_own * d1 + 4 * q + r : 0);
        w[r] = Xrg[at];
        v[r] = Vg[at];
    }
    const bool has_bias = tid < d1;
    const float b_in = Xrg[a.b_off + (has_bias ? tid : 0)], vb_in = Vg[a.b_off + (has_bias ? tid : 0)];
    for (int e = tid; e < a.n_steps * Bp; e += kResThreads) {
        const int idx = idxs[e], y = a.labels[idx >= 0 ? idx : 0];
        labs[e] = idx >= 0 ? y : -1;
    }
#pragma unroll
    for (int u = 0; u < kRes1First; ++u) {
        const int r = my_row + kResWaves * rows * u;
        if (r >= 0 && r < n_first) put(ring + r * row + c, first[u]);
    }
    if (lead - 1 < a.n_steps) request(lead - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const bool in = k_own < d0 && 4 * q + r < d1;
        w[r] = in ? w[r] : 0.f;
        v[r] = in ? v[r] : 0.f;
        ws[4 * q + r][k_own] = w[r];
    }
    if (tid < 16) {
        bs[tid] = has_bias ? b_in : 0.f;
        vbs[tid] = has_bias ? vb_in : 0.f;
    }
    __syncthreads();

    const int mt = wave % MT, kpart = wave / MT;
    bool gave_up = false;   // thread 0: a barrier wait ran out of polls
    for (int s = 0; s < a.n_steps; ++s) {
        int tid_o = threadIdx.x;   // (addresses are derived afresh in every step instead of held in registers)
        asm volatile("" : "+v"(tid_o));
        const int tid = tid_o, lane = tid & 63, j = lane & 15, q = lane >> 4, k_own = 16 * wave + j;
        const float beta = s == 0 ? a.beta_first : a.beta;
        const OT* as = ring + s % R * (Bp * row);
        // ---- logits^T, partial over this wavefront's share of d0: class 4 q + r of sample 16 mt + j
        f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int st = kpart; st < dp0 / 32; st += KP) {
            const int k0 = 32 * st + 8 * q;
            const Frag<OT> af = load8(as + (16 * mt + j) * row + k0);
            const float4 x0 = *reinterpret_cast<const float4*>(&ws[j][k0]);
            const float4 x1 = *reinterpret_cast<const float4*>(&ws[j][k0 + 4]);
            const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            Frag<OT> bf;
            pack8(bf, x);
            z = mma8(bf, af, z);
        }
        if (kpart > 0) *reinterpret_cast<f32x4*>(&part[kpart - 1][16 * mt + j][4 * q]) = z;
        // ---- A_0 of the own features, operand of dW
        Frag<OT> own[NS];
        if (16 * wave < dp0) {
#pragma unroll
            for (int st = 0; st < NS; ++st)
#pragma unroll
                for (int e = 0; e < 8; ++e) own[st].v[e] = as[(32 * st + 8 * q + e) * row + k_own];
        }
        __syncthreads();
        // ---- a place of the ring has become free (with R = 1 this step's, else that of the step before)
        if (s + lead - 1 < a.n_steps) {
            place(s + lead - 1);
            if (s + lead < a.n_steps) request(s + lead);
        }
        // ---- softmax cross-entropy and dZ, one wavefront per batch tile
        if (wave < MT) {
            const int b = 16 * mt + j, y = labs[s * Bp + b];
#pragma unroll
            for (int p = 1; p < KP; ++p) z += *reinterpret_cast<const f32x4*>(&part[p - 1][b][4 * q]);
            float zmax = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                z[r] += bs[4 * q + r];
                if (4 * q + r < d1) zmax = fmaxf(zmax, z[r]);
            }
            zmax = max_over_quarters(zmax);
            f32x4 ex;
            float s_other = 0.f, e_y = 0.f, z_y = 0.f;   // (over the classes other than the label, see xent_loss)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 4 * q + r;
                ex[r] = c < d1 ? expf(z[r] - zmax) : 0.f;
                s_other += c == y ? 0.f : ex[r];
                e_y += c == y ? ex[r] : 0.f;
                z_y += c == y ? z[r] : 0.f;
            }
            s_other = sum_over_quarters(s_other);
            const float sum = s_other + sum_over_quarters(e_y), inv = 1.f / sum, invB = 1.f / static_cast<float>(a.B);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = 4 * q + r;
                const OT dz = static_cast<OT>(y >= 0 && c < d1 ? xent_delta(ex[r], c == y, s_other, inv) * invB : 0.f);
                dzt[c][b] = dz;
            }
            if (s + 1 == a.n_steps) {   // (the losses that are kept are those of the last step)
                z_y = sum_over_quarters(z_y);
                if (q == 0) lred[b] = y >= 0 ? -(z_y - zmax - logf(sum)) : 0.f;
            }
        }
        __syncthreads();
        if (s + 1 == a.n_steps && wave == kResWaves - 1) {
            float l = lane < Bp ? lred[lane] : 0.f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
            if (lane == 0) a.loss[static_cast<int64_t>(g) * kLossParts] = l / static_cast<float>(a.B);
        }
        if (wave == kResWaves - 2) {   // column sums of dZ, a quarter of the batch per lane
            float db = 0.f;
#pragma unroll
            for (int i = 0; i < Bp / 32; ++i) {
                const Frag<OT> f = load8(&dzt[j][32 * i + 8 * q]);
#pragma unroll
                for (int e = 0; e < 8; ++e) db += to_f32(f.v[e]);
            }
            db = sum_over_quarters(db);
            if (lane < d1) {
                const float vb = momentum_update(beta, vbs[lane], db, wd, bs[lane]);
                vbs[lane] = vb;
                bs[lane] = weight_update(bs[lane], lr, vb);
            }
        }
        // ---- dW^T = dZ^T A_0 of the own features and the update
        if (16 * wave < dp0) {
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < NS; ++st) {
                const Frag<OT> zf = *reinterpret_cast<const Frag<OT>*>(&dzt[j][32 * st + 8 * q]);
                acc = mma8(zf, own[st], acc);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // (an entry that does not exist must stay zero also where its zero operand meets an infinity)
                const float gw = k_own < d0 && 4 * q + r < d1 ? acc[r] : 0.f;
                v[r] = momentum_update(beta, v[r], gw, wd, w[r]);
                w[r] = weight_update(w[r], lr, v[r]);
                ws[4 * q + r][k_own] = w[r];
            }
        }
        __syncthreads();
        if (a.period == 0 || (s + 1) % a.period != 0) continue;
        // ---- averaging step, as in the two-layer kernel: hand over the model, wait for all
        //      replicas, take the mean of the m copies
        const int pi = (s + 1) / a.period - 1;
        float* all = a.avx + static_cast<int64_t>(pi & 1) * a.G * a.x_stride;
        float* mine = all + g * a.x_stride;
        for (int e = tid; e < d0 * d1; e += kResThreads) mine[a.w_off + e] = ws[e % d1][e / d1];
        if (tid < d1) mine[a.b_off + tid] = bs[tid];
        __builtin_amdgcn_s_waitcnt(0);   // this wavefront's stores have left before the workgroup arrives
        __syncthreads();
        if (tid == 0)
            arrive_and_wait(a.gctr, a.gctr_base + static_cast<unsigned>(pi + 1) * static_cast<unsigned>(a.G),
                            a.spin_limit, a.err, gave_up);
        __syncthreads();
        for (int e = tid; e < d0 * d1; e += kResThreads)
            ws[e % d1][e / d1] = mean_of_replicas(all + a.w_off + e, a.x_stride, a.G);
        if (tid < d1) bs[tid] = mean_of_replicas(all + a.b_off + tid, a.x_stride, a.G);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = ws[4 * q + r][k_own];
    }

#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (k_own < d0 && 4 * q + r < d1) {
            const int64_t at = a.w_off + k_own * d1 + 4 * q + r;
            Xg[at] = w[r];
            Vg[at] = v[r];
        }
    }
    if (tid < d1) {
        Xg[a.b_off + tid] = bs[tid];
        Vg[a.b_off + tid] = vbs[tid];
    }
}

}  // namespace

size_t resident_exchange_floats(const lc_handle* h) {
    // steps of a launch x (replicas x padded batch x padded hidden width); the single-layer form
    // exchanges nothing (a token amount keeps the buffer pointer non-null)
    if (h->L == 1) return 64;
    return static_cast<size_t>(h->train.slots) * h->m * h->train.Bp * h->layer[1].dp_out;
}

// Compute units of the current device: 256 on the MI355X this is written for, fewer on a partition of it.
// That many workgroups of the resident kernel can be on the chip at the same time (16 wavefronts and
// 66 KB and more of LDS each), and launches of one workgroup per CU take rounds of that many.  Without a
// device (host-only use of the library) the full chip is assumed; the kernel's bounded barrier wait remains the last line of defence.
int compute_units() {
    static const int units = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) return 256;
        return cus < 256 ? cus : 256;   // (the exchange buffers and counters are sized for 256)
    }();
    return units;
}

static int resident_slices(const lc_handle* h) { return (h->layer[1].d_out + 15) / 16; }   // workgroups of a replica

bool exchange_is_local(const lc_handle* h) {
    if (h->L != 2 || !h->res_a1x || !h->res_on || !h->res_local_on || !h->res_xcc_known) return false;
    // a replica's workgroups on one XCD, which has room for an eighth of the chip's
    return (h->m + kXcds - 1) / kXcds * resident_slices(h) <= compute_units() / kXcds;
}

// Two layers, at most 16 classes and 64 samples, widths within the LDS budget, and few enough
// workgroups that all of them are on the chip at the same time (one per compute unit); or one
// layer of at most 256 (padded) inputs and 16 classes.
bool resident_shape_ok(const lc_handle* h) {
    if (h->md.kind != LC_KIND_MLP || h->md.B > 64) return false;
    if (h->L == 1) return h->layer[1].d_out <= 16 && h->layer[1].dp_in <= kRes1K;
    if (h->L != 2) return false;
    if (h->layer[2].d_out > 16) return false;
    if (h->layer[1].dp_in > kResMaxD0 || h->layer[1].dp_out > kResMaxD1) return false;
    return h->m <= 64 && static_cast<int64_t>(h->m) * (h->layer[1].dp_out / 16) <= compute_units();
}

namespace {

hipError_t launch_resident1(lc_handle* h, int slot0, int n_steps, int period) {
    const ActSet& S = h->train;
    const bool bf16 = h->md.gemm == LC_GEMM_BF16;
    Res1Args a;
    a.X = h->X;
    a.V = h->V;
    a.x_stride = h->Ps;
    a.Xr = h->lazy_rows ? h->xbar : h->X;
    a.xr_stride = h->lazy_rows ? 0 : h->Ps;
    a.w_off = h->layer[1].w_off;
    a.b_off = h->layer[1].b_off;
    a.d0 = h->layer[1].d_in;
    a.d1 = h->layer[1].d_out;
    a.dp0 = h->layer[1].dp_in;
    a.B = S.B;
    a.G = S.G;
    a.data = h->data;
    a.labels = h->labels;
    a.idx_out = S.idx + static_cast<size_t>(slot0) * S.G * S.Bp;
    a.N = h->md.N;
    a.seed = h->seed;
    a.k = h->k;
    a.sampler = h->md.sampler;
    a.m = h->m;
    a.n_steps = n_steps;
    {
        const int batch = S.Bp * (a.dp0 * (bf16 ? 2 : 4) + 16), per_round = kResWaves * (64 / (a.dp0 / 4));
        int ring = kRes1Ring / batch;
        if (ring > 1 + kRes1First * per_round / S.Bp) ring = 1 + kRes1First * per_round / S.Bp;
        a.ring = ring < n_steps ? ring : n_steps;
    }
    a.lr = h->md.lr;
    a.beta_first = effective_beta(h);
    a.beta = h->md.beta;
    a.wd = h->md.wd;
    a.loss = S.loss;
    a.period = period;
    a.avx = h->res_avx;
    a.gctr = h->res_ctr + kCtrAll;
    a.gctr_base = h->res_garrivals;
    a.err = h->res_ctr + kCtrErr;
    a.spin_limit = h->res_spin_limit;
    if (slot0 < 0 || n_steps < 1 || slot0 + n_steps > S.slots || n_steps > kRes1Steps) return hipErrorInvalidValue;
    if (period < 0 || (period > 0 && (n_steps % period != 0 || !h->res_avx || S.G > compute_units()))) return hipErrorInvalidValue;
    if (S.Bp != 32 && S.Bp != 64) return hipErrorInvalidValue;
    if (a.dp0 > kRes1K || a.d1 > 16) return hipErrorInvalidValue;
    timing_start(h, kTimeBwd, 0, kBwdResident);
    const dim3 grid(static_cast<unsigned>(S.G)), block(kResThreads);
    if (S.Bp == 32) {
        if (bf16) hipLaunchKernelGGL((resident1_kernel<bf16_t, 2>), grid, block, 0, h->stream, a);
        else hipLaunchKernelGGL((resident1_kernel<float, 2>), grid, block, 0, h->stream, a);
    } else {
        if (bf16) hipLaunchKernelGGL((resident1_kernel<bf16_t, 4>), grid, block, 0, h->stream, a);
        else hipLaunchKernelGGL((resident1_kernel<float, 4>), grid, block, 0, h->stream, a);
    }
    h->loss_parts_train = 1;
    if (period > 0) h->res_garrivals += static_cast<unsigned>(n_steps / period) * static_cast<unsigned>(S.G);
    timing_stop(h, kTimeBwd, 0, kBwdResident);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_resident(lc_handle* h, int slot0, int n_steps, int period) {
    if (h->L == 1) return launch_resident1(h, slot0, n_steps, period);
    const ActSet& S = h->train;
    const bool bf16 = h->md.gemm == LC_GEMM_BF16;
    ResArgs a;
    a.X = h->X;
    a.V = h->V;
    a.x_stride = h->Ps;
    a.Xr = h->lazy_rows ? h->xbar : h->X;
    a.xr_stride = h->lazy_rows ? 0 : h->Ps;
    a.w1_off = h->layer[1].w_off;
    a.b1_off = h->layer[1].b_off;
    a.w2_off = h->layer[2].w_off;
    a.b2_off = h->layer[2].b_off;
    a.d0 = h->layer[1].d_in;
    a.d1 = h->layer[1].d_out;
    a.d2 = h->layer[2].d_out;
    a.dp0 = h->layer[1].dp_in;
    a.dp1 = h->layer[1].dp_out;
    a.B = S.B;
    a.G = S.G;
    a.NB = resident_slices(h);
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
    a.vec = (a.d1 % 4 == 0 && a.w1_off % 4 == 0) ? 1 : 0;
    a.zx = h->res_a1x;
    a.ctr = h->res_ctr + kCtrReplica;
    a.ctr_base = h->res_arrivals;
    a.err = h->res_ctr + kCtrErr;
    a.spin_limit = h->res_spin_limit;
    a.loss = S.loss;
    a.period = period;
    a.avx = h->res_avx;
    a.gctr = h->res_ctr + kCtrAll;
    a.gctr_base = h->res_garrivals;
    a.local_xcd = exchange_is_local(h) ? 1 : 0;
    a.xcc_of = h->res_xcc_of;
    if (slot0 < 0 || n_steps < 1 || slot0 + n_steps > S.slots) return hipErrorInvalidValue;
    if (period < 0 || (period > 0 && (n_steps % period != 0 || !h->res_avx))) return hipErrorInvalidValue;
    const int64_t total = static_cast<int64_t>(a.G) * a.NB;
    if (total > compute_units() || a.G > 64 || !h->res_a1x) return hipErrorInvalidValue;
    const unsigned grid = static_cast<unsigned>(a.local_xcd ? (a.G + kXcds - 1) / kXcds * kXcds * a.NB
                                                            : (total + kXcds - 1) / kXcds * kXcds);
    if (S.Bp != 32 && S.Bp != 64) return hipErrorInvalidValue;
    timing_start(h, kTimeBwd, 0, kBwdResident);
    if (S.Bp == 32) {
        if (bf16) hipLaunchKernelGGL((resident_kernel<bf16_t, 2>), dim3(grid), dim3(kResThreads), 0, h->stream, a);
        else hipLaunchKernelGGL((resident_kernel<float, 2>), dim3(grid), dim3(kResThreads), 0, h->stream, a);
    } else {
        if (bf16) hipLaunchKernelGGL((resident_kernel<bf16_t, 4>), dim3(grid), dim3(kResThreads), 0, h->stream, a);
        else hipLaunchKernelGGL((resident_kernel<float, 4>), dim3(grid), dim3(kResThreads), 0, h->stream, a);
    }
    h->loss_parts_train = 1;
    h->res_arrivals += static_cast<unsigned>(n_steps) * static_cast<unsigned>(a.NB);   // wraps like the counters do
    if (period > 0) h->res_garrivals += static_cast<unsigned>(n_steps / period) * static_cast<unsigned>(total);
    timing_stop(h, kTimeBwd, 0, kBwdResident);
    return hipGetLastError();
}

// Where do blocks run?  Hardware block ids are dealt to the XCDs round-robin; the resident kernel's
// XCD-local exchange needs exactly that, so it is observed once per handle instead of assumed:
// 256 one-thread blocks report their XCD, and the rule holds if blocks with the same id mod 8
// agree and the 8 residues name 8 different XCDs.
hipError_t probe_block_placement(lc_handle* h) {
    h->res_xcc_known = false;
    h->res_xcc_of = 0;
    if (!h->res_ctr) return hipSuccess;
    unsigned* dev = h->res_ctr + kCtrProbe;
    unsigned host[256];
    hipLaunchKernelGGL(xcd_probe_kernel, dim3(256), dim3(64), 0, h->stream, dev);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(host, dev, sizeof(host), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return e;
    unsigned seen = 0, packed = 0;
    for (int r = 0; r < kXcds; ++r) {
        for (int b = r; b < 256; b += kXcds)
            if (host[b] != host[r] || host[b] > 15u) return hipSuccess;   // no such rule here: agent-scope exchange
        if (seen & (1u << host[r])) return hipSuccess;
        seen |= 1u << host[r];
        packed |= host[r] << (4 * r);
    }
    h->res_xcc_known = true;
    h->res_xcc_of = packed;
    return hipSuccess;
}

}  // namespace lc
