// bf16 expert products for the big chunks of a batch (experts with more rows
// of the call than a small chunk holds; every expert of a prefill batch), for
// weights in tiled order.
//
// A workgroup of 8 waves computes 256 weight rows x up to 128 tokens of one
// chunk over the whole contraction, 128 bytes of each row (two 16x16x32 bf16
// MFMAs deep) per pipeline stage:
//   * each wave owns two 16-row weight tiles, which nobody else reads: they go
//     global -> registers three stages ahead of their MFMAs (four register
//     sets) and never pass through LDS;
//   * the chunk's token rows go global -> LDS with the 16-byte direct-to-LDS
//     loads, each load 8 whole 128-byte row blocks, three stages ahead in a
//     ring of four; every wave reads every token fragment from LDS.
// Every wave issues the same loads per stage, so it waits for its oldest stage
// with a constant vmcnt, and one barrier per stage publishes the ring's slot.
// An item is compiled for its chunk's token-tile count (1 .. 8), so each stage
// is straight-line code.
//
// Bound by the weight stream (HBM).  Against a kernel that staged the weights
// in LDS too (three stages of 48 KB, two in flight), R1-shaped layer, one box:
// T = 600 3955 -> 3569 us, T = 2048 4503 -> 4164 us (its gate/up 2839 -> 2530
// us, 5.6 -> 6.3 TB/s), skewed T = 1000 2458 -> 2310 us.  Two workgroups of 4
// waves per CU (128 weight rows each, twice the token loads): 4365 us at
// T = 2048; runs of two or four down groups through one pipeline: equal.
//
//   gate/up: wave w takes feature tile w of the item's 128 features (its gate
//            and its up rows) -> bf16 SwiGLU rows;
//   down:    wave w takes row tiles 2w, 2w + 1 of the item's 256 rows -> fp32
//            expert output rows.
// (The 8-bit products of prefill batches run ffn_prefill8.h.)
#include "caee_internal.h"

#include <type_traits>

namespace caee {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) u32x4_t g_u32x4_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kGemmWaves = 8;
constexpr int kGemmThreads = kGemmWaves * kWave;
constexpr int kNT = 8;                 // token tiles of an item at most (16 tokens each)
constexpr int kBufWord3 = 0x00020000;   // buffer descriptor word 3: 32-bit data format, raw access
constexpr int kNoVmem = 0x7FF & ~0x071;  // scheduling barrier that vector memory operations do not cross
// Workgroups of the launch per CU (one runs at a time; a CU that is done
// early takes the next: 2 per CU measured 1 % slower at T = 2048, 2 % at 600).
constexpr int kGridPerCu = 32;

// One slot of the token ring: row t's 128-byte block at f[t / 8][8 (t % 8) ..],
// its 16-byte piece c in position c ^ (t % 8) (an XOR swizzle: the 8 lanes of
// a fragment read that take one piece each of 8 consecutive rows hit 8
// different bank groups).
struct TokStage {
    u32x4_t f[2 * kNT][kWave];
};

// Weight pieces of one stage in registers: [tile][half].
struct WReg {
    u32x4_t v[2][2];
};

__device__ inline float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

// Waits until at most N of this wave's vector memory loads are outstanding and
// its LDS reads are done, so that a slot is free once every wave has passed
// the barrier behind it (gfx9 s_waitcnt: vmcnt in bits 3:0 and 15:14, expcnt
// in 6:4, not waited, lgkmcnt in 11:8).
template <int N>
__device__ inline void wait_stage() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | (((N >> 4) & 3) << 14));
}

// Workgroup barrier without the memory fence of __syncthreads (which would
// wait for every load in flight); the empty asm keeps the compiler from
// moving memory accesses across it.
__device__ inline void stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int N>
using IntC = std::integral_constant<int, N>;

template <bool kGateUp>
__global__ __launch_bounds__(kGemmThreads, 2) void k_gemm(FfnParams p) {
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-descriptor type exists for the GPU target only
    // The ring's slots are separate LDS objects (and the code below names
    // each statically), so the compiler can tell a read of one slot from the
    // loads still filling the others and does not wait for those.
    __shared__ TokStage st0, st1, st2, st3;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int K = kGateUp ? p.d : p.f;                 // contraction length
    const int nblk = K * 2 / 128;                      // pipeline stages (128 bytes of each row)
    const size_t ksteps = (size_t)K * 2 / 64;          // 64-byte steps per weight row
    const size_t row_units = (size_t)K * 2 / 16;       // 16-byte pieces per token row
    const int groups = kGateUp ? p.f / (16 * kGemmWaves) : p.d / (32 * kGemmWaves);
    const int n_chunks = ffn_list_size(p);
    const size_t expert_bytes = (kGateUp ? (size_t)2 * p.f * p.d : (size_t)p.d * p.f) * 2;
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    const bool by_xcd = items_by_xcd(p, groups);
    const int xcd = by_xcd ? blockIdx.x % kXcds : 0, xcds = by_xcd ? kXcds : 1;
    const int n_local = (n_chunks - xcd + xcds - 1) / xcds * groups;
    for (int it = blockIdx.x / xcds; it < n_local; it += gridDim.x / xcds) {
        const int c = xcd + xcds * (it / groups), grp = it % groups;
        const ChunkRef ck = ffn_chunk(p, c);
        const int xs = ck.xs;
        if (ffn_skip(p, xs)) continue;   // uniform over the workgroup
        const int row0 = ck.row0, ntok = ck.ntok;
        const u32x4_t* wb = (const u32x4_t*)ffn_weights(p, xs, !kGateUp, expert_bytes);
        const int t0 = kGateUp ? grp * kGemmWaves + wave : (grp * kGemmWaves + wave) * 2;
        const int t1 = kGateUp ? p.f / 16 + t0 : t0 + 1;
        const u32x4_t* const wsrc[2] = {wb + (size_t)t0 * ksteps * 64 + lane, wb + (size_t)t1 * ksteps * 64 + lane};

        // Token rows: x, or the chunk's SwiGLU rows; buffer loads, whose waits
        // the compiler counts apart from the LDS reads of the multiply (with
        // global_load_lds it drained every load once per loop body).
        const char* tbase = kGateUp ? (const char*)p.x : (const char*)p.h + (size_t)row0 * row_units * 16;
        const uint32_t tbytes = (uint32_t)((size_t)(kGateUp ? p.T : ntok) * row_units * 16);
        const __amdgpu_buffer_rsrc_t tbuf =
            __builtin_amdgcn_make_buffer_rsrc((void*)tbase, 0, (int)tbytes, kBufWord3);

        // The item for NB token tiles (its chunk's count); kKeep: its weights
        // are read again by the expert's other chunks and stay in the caches
        // (streamed past them, skewed T = 1000 took 2540 us instead of 2375;
        // kept for every chunk, evenly used experts at T = 600 3822 instead
        // of 3636).
        auto run = [&](auto nbc, auto kc) __attribute__((always_inline)) {
            constexpr int NB = decltype(nbc)::value;
            constexpr bool kKeep = decltype(kc)::value;
            // Token loads of a stage: 2 NB of 8 rows each, kTok per wave
            // (past 2 NB: a valid row into slots nobody reads).
            constexpr int kTok = (2 * NB + kGemmWaves - 1) / kGemmWaves;
            constexpr int kLoads = kTok + 4;
            static_assert(kTok * kGemmWaves <= 2 * kNT, "ring slots");
            uint32_t toff[kTok];
#pragma unroll
            for (int i = 0; i < kTok; ++i) {
                int n = 8 * (kTok * wave + i) + (lane >> 3);   // lane l: piece (l % 8) ^ (l / 8) of its row
                n = n < ntok ? n : 0;          // padded token columns read a valid row; results dropped
                const uint32_t row = kGateUp ? (uint32_t)ffn_token(p, xs, row0 + n) : (uint32_t)n;
                toff[i] = (row * (uint32_t)row_units + (uint32_t)((lane & 7) ^ (lane >> 3))) * 16u;
            }
            // This lane's B fragment of token tile n, half h: token 16n + r,
            // piece 4h + g of its block, at f[2n] + fo[h].
            const int fo[2] = {(r >> 3) * kWave + (r & 7) * 8 + (g ^ (r & 7)),
                               (r >> 3) * kWave + (r & 7) * 8 + ((4 + g) ^ (r & 7))};
            f32x4_t acc[2][NB];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int n = 0; n < NB; ++n) acc[t][n] = zero;

            auto issue_tok = [&](int kb, TokStage& s) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < kTok; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(tbuf, (lds_void_t*)&s.f[kTok * wave + i][0], 16, toff[i],
                                                             kb * 128, 0, 0);
                // The waits count loads in the order written here.
                __builtin_amdgcn_sched_barrier(kNoVmem);
            };
            auto issue_w = [&](int kb, WReg& w) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        g_u32x4_t* src = (g_u32x4_t*)(wsrc[t] + (size_t)kb * 128 + h * 64);
                        w.v[t][h] = kKeep ? *src : __builtin_nontemporal_load(src);
                    }
                __builtin_amdgcn_sched_barrier(kNoVmem);
            };
            // One stage: the token fragments of the first half, then each tile's
            // two MFMAs of it with the read of its second half between them,
            // then the second half's (left to itself the compiler reads a
            // fragment or two, waits, multiplies).
            auto compute = [&](const TokStage& s, const WReg& w) __attribute__((always_inline)) {
                bf16x8_t b[2][NB], a[2][2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int n = 0; n < NB; ++n) b[h][n] = __builtin_bit_cast(bf16x8_t, (&s.f[2 * n][0])[fo[h]]);
                    a[0][h] = __builtin_bit_cast(bf16x8_t, w.v[0][h]);
                    a[1][h] = __builtin_bit_cast(bf16x8_t, w.v[1][h]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        acc[0][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][h], b[h][n], acc[0][n], 0, 0, 0);
                        acc[1][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][h], b[h][n], acc[1][n], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 2 * NB, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto slot = [&](auto jc) -> TokStage& {
                constexpr int J = decltype(jc)::value & 3;
                if constexpr (J == 0) return st0;
                else if constexpr (J == 1) return st1;
                else if constexpr (J == 2) return st2;
                else return st3;
            };
            WReg w0, w1, w2, w3;
            auto wset = [&](auto jc) -> WReg& {
                constexpr int J = decltype(jc)::value & 3;
                if constexpr (J == 0) return w0;
                else if constexpr (J == 1) return w1;
                else if constexpr (J == 2) return w2;
                else return w3;
            };
            // Step v (J = v mod 4) issues the weights of block v + 1 (their
            // registers held block v - 3, which this wave multiplied in the
            // step before), waits until its tokens and weights of block v - 2
            // have landed, passes the barrier that makes every wave's tokens
            // of that block visible and after which all are done with block
            // v - 3, whose ring slot the tokens of block v + 1 then refill,
            // and multiplies block v - 2.  Steps past the last block re-read
            // it, so the waits are constants.  The remaining steps after the
            // loop (three at most) wait for all but the token loads of the two
            // steps before: nothing multiplies the weights that are re-read,
            // so the compiler may leave those loads out of what a count would
            // include.
            auto step = [&](int v, auto jc, auto mc, auto tc) __attribute__((always_inline)) {
                constexpr int J = decltype(jc)::value;
                const int u = v + 1 < nblk ? v + 1 : nblk - 1;
                issue_w(u, wset(IntC<J + 1>{}));
                if constexpr (decltype(tc)::value) wait_stage<2 * kTok>();
                else wait_stage<2 * kLoads + 4>();
                stage_barrier();
                issue_tok(u, slot(IntC<J + 1>{}));
                if constexpr (decltype(mc)::value) compute(slot(IntC<J + 2>{}), wset(IntC<J + 2>{}));
            };
            // Steps 0 and 1 only load; steps 2 .. nblk + 1 multiply.
            const int vend = nblk + 2;
            issue_w(0, w0);
            issue_tok(0, st0);
            step(0, IntC<0>{}, std::false_type{}, std::false_type{});
            step(1, IntC<1>{}, std::false_type{}, std::false_type{});
            int v = 2;
#pragma clang loop unroll(disable)
            for (; v + 4 <= vend; v += 4) {
                step(v, IntC<2>{}, std::true_type{}, std::false_type{});
                step(v + 1, IntC<3>{}, std::true_type{}, std::false_type{});
                step(v + 2, IntC<4>{}, std::true_type{}, std::false_type{});
                step(v + 3, IntC<5>{}, std::true_type{}, std::false_type{});
            }
            if (v < vend) {
                step(v, IntC<2>{}, std::true_type{}, std::true_type{});
                if (v + 1 < vend) {
                    step(v + 1, IntC<3>{}, std::true_type{}, std::true_type{});
                    if (v + 2 < vend) step(v + 2, IntC<4>{}, std::true_type{}, std::true_type{});
                }
            }
            wait_stage<0>();   // the re-reads past the last block have landed
            stage_barrier();   // all waves are done with the ring before the next item refills it
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                int tn = 16 * n + r;
                asm volatile("" : "+v"(tn));   // keeps the row arithmetic here, out of the stage loop
                if (tn >= ntok) continue;
                if constexpr (kGateUp) {
                    float h[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[e] = silu_mul(acc[0][n][e], acc[1][n][e]);
                    // bf16 SwiGLU rows, rounded to nearest even
                    uint2 pk;
                    pk.x = bf16_rne(h[0]) | (bf16_rne(h[1]) << 16);
                    pk.y = bf16_rne(h[2]) | (bf16_rne(h[3]) << 16);
                    *(uint2*)((uint16_t*)p.h + (size_t)(row0 + tn) * p.f + t0 * 16 + 4 * g) = pk;
                } else {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        store_y4(p, (size_t)(row0 + tn), (t ? t1 : t0) * 16 + 4 * g, acc[t][n][0], acc[t][n][1],
                                 acc[t][n][2], acc[t][n][3]);
                }
            }
        };
        // Near-equal pieces of more than 128 rows have more than 64 each.
        const int nb = (ntok + 15) >> 4;
        if (ck.multi && nb > kNT / 2) {
            switch (nb) {
                case 5: run(IntC<5>{}, std::true_type{}); break;
                case 6: run(IntC<6>{}, std::true_type{}); break;
                case 7: run(IntC<7>{}, std::true_type{}); break;
                default: run(IntC<8>{}, std::true_type{}); break;
            }
        } else {
            switch (nb) {
                case 1: run(IntC<1>{}, std::false_type{}); break;
                case 2: run(IntC<2>{}, std::false_type{}); break;
                case 3: run(IntC<3>{}, std::false_type{}); break;
                case 4: run(IntC<4>{}, std::false_type{}); break;
                case 5: run(IntC<5>{}, std::false_type{}); break;
                case 6: run(IntC<6>{}, std::false_type{}); break;
                case 7: run(IntC<7>{}, std::false_type{}); break;
                default: run(IntC<8>{}, std::false_type{}); break;
            }
        }
    }
#endif
}

}  // namespace

int gemm_bf16_blocks() { return kNT; }

// Gate/up groups of 128 features, down groups of 256 rows; x within the reach
// of a buffer descriptor.
static bool gemm_fits(long long T, int d, int f) {
    return d % 256 == 0 && f % 128 == 0 && T * d * 2 < (1LL << 32);
}

bool gemm_bf16_supports(const FfnParams& p, int nb) { return nb == kNT && p.tiled && gemm_fits(p.T, p.d, p.f); }

bool gemm_bf16_applies(const caee_layer_desc_t& d, bool tiled) {
    return d.w_dtype == CAEE_BF16 && tiled && gemm_fits(d.T, d.d, d.f);
}

hipError_t launch_gemm(const FfnParams& p, bool gate_up, int max_chunks, hipStream_t s) {
    const int groups = gate_up ? p.f / (16 * kGemmWaves) : p.d / (32 * kGemmWaves);
    long long items = (long long)((max_chunks + kXcds - 1) / kXcds * kXcds) * groups;
    const long long cap = (long long)device_cu_count() * kGridPerCu;
    if (items > cap) items = cap;
    const dim3 grid((unsigned)((items + kXcds - 1) / kXcds * kXcds)), block(kGemmThreads);
    if (gate_up) ffn_launch(k_gemm<true>, grid, block, s, p);
    else ffn_launch(k_gemm<false>, grid, block, s, p);
    return hipGetLastError();
}

}  // namespace caee
