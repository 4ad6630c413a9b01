// Host side of the 8-bit prefill products, the gather of x's block scales,
// and the gate/up kernel (ffn_prefill8.h; the down kernel is compiled in
// ffn_prefill8_down.hip, next to this file: each takes over a minute).
#include "ffn_prefill8.h"

namespace caee {
namespace {

// Block scales of x for the rows of the big chunks, transposed and in
// permuted row order: xst[b][row] = xs[token of row][b].  One workgroup per
// chunk and kXsBlocks blocks, one thread per row: each reads kXsBlocks scales
// of its token (one line) and stores them to rows of consecutive lanes.
// Bound by latency (one round trip for the token, one for the scales); with
// one workgroup per chunk walking all blocks it took 90-107 us next to the
// small-chunk kernels of an R1-shaped layer (T = 128, 600), 11 us alone.
constexpr int kXsBlocks = 8;
__global__ __launch_bounds__(256) void k_gather_xs(FfnParams p) {
    const int nblk = p.d / 128;
    const int b0 = blockIdx.y * kXsBlocks;
    const int list = ffn_list_size(p);
    for (int c = blockIdx.x; c < list; c += gridDim.x) {
        const ChunkRef ck = ffn_chunk(p, c);
        for (int n = threadIdx.x; n < ck.ntok; n += blockDim.x) {
            const int row = ck.row0 + n;
            const float* src = p.xs + (size_t)ffn_token(p, ck.xs, row) * nblk + b0;
            float v[kXsBlocks];
#pragma unroll
            for (int b = 0; b < kXsBlocks; ++b) v[b] = b0 + b < nblk ? src[b] : 0.0f;
#pragma unroll
            for (int b = 0; b < kXsBlocks; ++b)
                if (b0 + b < nblk) p.xst[(size_t)(b0 + b) * p.P + row] = v[b];
        }
    }
}

}  // namespace

hipError_t launch_gather_xs(const FfnParams& p, int max_chunks, hipStream_t s) {
    const int blocks = max_chunks > 0 ? max_chunks : 1;
    const int nblk = p.d / 128;
    hipLaunchKernelGGL(k_gather_xs, dim3((unsigned)blocks, (unsigned)((nblk + kXsBlocks - 1) / kXsBlocks)), dim3(256),
                       0, s, p);
    return hipGetLastError();
}

// The buffers the kernel reads through buffer descriptors (token codes and
// block scales of x and of the SwiGLU rows) must hold fewer than 2^31 bytes.
static bool p8_buffers_fit(long long T, long long P, long long d, long long f) {
    const long long lim = 1LL << 31;
    return T * d < lim && P * f < lim && (d / 128) * P * 4 < lim && (f / 128) * P * 4 < lim;
}

bool gemm_fp8_supports(const FfnParams& p, int nb) {
    return nb == kP8NT && p.tiled && p.f % 128 == 0 && p.d % 256 == 0 && p.d / 128 <= kP8MaxKBlocks &&
           p.f / 128 <= kP8MaxKBlocks && p8_buffers_fit(p.T, p.P, p.d, p.f);
}

bool gemm_fp8_applies(const caee_layer_desc_t& d, bool tiled) {
    return d.w_dtype == CAEE_FP8_E4M3 && d.T > kGemmT && tiled && d.f % 128 == 0 &&
           d.d % 256 == 0 && d.d / 128 <= kP8MaxKBlocks && d.f / 128 <= kP8MaxKBlocks &&
           p8_buffers_fit(d.T, (long long)d.T * (d.k + d.n_shared), d.d, d.f);
}

int gemm_fp8_blocks() { return kP8NT; }

hipError_t launch_prefill8(const FfnParams& p, bool gate_up, int max_chunks, hipStream_t s) {
    const int groups = gate_up ? p.f / 128 : p.d / 256;
    // One workgroup per CU at a time (the ring takes most of the LDS); two
    // per CU in the grid, so that a CU whose items end early takes more.
    long long items = (long long)max_chunks * groups;
    const long long cap = (long long)device_cu_count() * CAEE_P8_GRID_PER_CU;
    if (items > cap) items = cap;
    if (items < 1) items = 1;
    if (!gate_up) return launch_prefill8_down(p, (unsigned)items, s);
    ffn_launch(k_prefill8<true>, dim3((unsigned)items), dim3(kP8Threads), s, p);
    return hipGetLastError();
}

}  // namespace caee
