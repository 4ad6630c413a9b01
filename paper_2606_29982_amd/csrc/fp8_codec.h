// OCP E4M3 (fn) encoding shared by the 8-bit kernels.
#pragma once

#include <stdint.h>

namespace caee {

constexpr float kE4M3Max = 448.0f;   // largest finite E4M3 magnitude

// OCP E4M3 (fn) codes of a and b (a in bits 7:0, b in bits 15:8, the rest of
// `old` kept; HI = true puts them in bits 23:16 and 31:24 instead): nearest
// representable value, ties to the even code, magnitudes above 448 saturate
// to 448.  gfx950's packed conversion rounds to nearest even (subnormal
// codes included); clamping to +-448 first gives the saturation.  Checked
// bit for bit against the branch-by-branch definition (code = round(|v| /
// 2^(e - 3)) within binade e, 2^-9 steps below 2^-6, sign bit 0x80) over
// every fp32 value of magnitude up to 448.5, both signs.
template <bool HI = false>
__device__ inline uint32_t e4m3_code2(float a, float b, uint32_t old = 0u) {
    const float ca = fminf(fmaxf(a, -kE4M3Max), kE4M3Max), cb = fminf(fmaxf(b, -kE4M3Max), kE4M3Max);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(ca, cb, (int)old, HI);
}

// Four codes packed little-endian into one word.
__device__ inline uint32_t e4m3_code4(float a, float b, float c, float d) {
    return e4m3_code2<true>(c, d, e4m3_code2(a, b));
}

constexpr int kQuantLanes = 16;   // lanes that quantise one 128-value block

// Quantisation of one block of 128 consecutive values by 16 lanes, lane l
// holding values 8l .. 8l + 7: scale = amax / 448 (1 for an all-zero block),
// code = e4m3(value / scale), all in fp32.  Returns the scale.
__device__ inline float quant_block(const float (&v)[8], uint8_t* q, int l) {
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(v[i]));
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    const float sc = amax > 0.0f ? amax / kE4M3Max : 1.0f;
    uint2 c;
    c.x = e4m3_code4(v[0] / sc, v[1] / sc, v[2] / sc, v[3] / sc);
    c.y = e4m3_code4(v[4] / sc, v[5] / sc, v[6] / sc, v[7] / sc);
    *(uint2*)(q + 8 * l) = c;
    return sc;
}

__device__ inline void load8(const float* src, float (&v)[8]) {
    const float4 a = *(const float4*)src, b = *(const float4*)(src + 4);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
    v[4] = b.x;
    v[5] = b.y;
    v[6] = b.z;
    v[7] = b.w;
}
__device__ inline void load8(const uint16_t* src, float (&v)[8]) {   // bf16
    const uint4 w = *(const uint4*)src;
    const uint32_t p[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(p[i] << 16);
        v[2 * i + 1] = __uint_as_float(p[i] & 0xFFFF0000u);
    }
}

}  // namespace caee
