// Per-row absmax int8 quantization arithmetic on bf16 inputs, shared by the row
// quantizer and by the small fused linear (which quantizes its own token rows): both
// must give the same codes and scales bit for bit.
//   a = max_k |v[k]|, s = a / 127, q[k] = clamp(rne(v[k] * (127 / a)), -127, 127);
// a row with a == 0, or with 127/a overflowing float32, gets s = 0 and q = 0.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace w8a8 {

// 16 and 8 bytes at any address, as one global load or store (the hardware takes any
// alignment).
struct __attribute__((packed, aligned(1))) Bytes16 {
    uint32_t w[4];
};
struct __attribute__((packed, aligned(1))) Bytes8 {
    uint32_t w[2];
};

namespace qmath {

__device__ __forceinline__ float bf16_to_f32(uint32_t h) {
    return __uint_as_float(h << 16);
}

// Largest |v| bit pattern among the 8 bf16 values in a 16-byte vector.
__device__ __forceinline__ uint32_t absmax8(uint4 d) {
    uint32_t w[4] = {d.x, d.y, d.z, d.w};
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t lo = w[i] & 0x7FFFu, hi = (w[i] >> 16) & 0x7FFFu;
        m = max(m, max(lo, hi));
    }
    return m;
}

// Maximum over the wavefront, the same in every lane: four steps inside the rows of 16
// lanes, two across them (lane 63 then holds the maximum), all in DPP operands; a shuffle
// tree goes through LDS six times.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    const auto step = [&](auto ctrl) {
        v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF,
                                                         0xF, true));
    };
    step(std::integral_constant<int, 0x111>{});   // row_shr:1
    step(std::integral_constant<int, 0x112>{});   // row_shr:2
    step(std::integral_constant<int, 0x114>{});   // row_shr:4
    step(std::integral_constant<int, 0x118>{});   // row_shr:8
    step(std::integral_constant<int, 0x142>{});   // row_bcast:15
    step(std::integral_constant<int, 0x143>{});   // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Sum over the wavefront, by the same steps.
__device__ __forceinline__ int wave_sum(int v) {
    const auto step = [&](auto ctrl) {
        v += __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xF, 0xF, true);
    };
    step(std::integral_constant<int, 0x111>{});   // row_shr:1
    step(std::integral_constant<int, 0x112>{});   // row_shr:2
    step(std::integral_constant<int, 0x114>{});   // row_shr:4
    step(std::integral_constant<int, 0x118>{});   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, true);   // row_bcast:15, rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, true);   // row_bcast:31, rows 2, 3
    return __builtin_amdgcn_readlane(v, 63);
}

// Codes of four values: clamp(rne(v * inv), -127, 127) as bytes, the first lowest. The
// product is clamped (the same as clamping its rounding: the bounds are integers) and
// 1.5 * 2^23 added, which rounds it to the nearest even integer and leaves the code in
// the sum's low byte; three byte permutations pack four of them. inv is 0 for a zero row,
// which yields zero codes (never 0 * inf).
__device__ __forceinline__ uint32_t code4(float v0, float v1, float v2, float v3, float inv) {
    const auto one = [&](float v) {
        return __float_as_uint(__builtin_amdgcn_fmed3f(v * inv, -127.0f, 127.0f) + 12582912.0f);
    };
    const uint32_t lo = __builtin_amdgcn_perm(one(v1), one(v0), 0x0C0C0400u);
    const uint32_t hi = __builtin_amdgcn_perm(one(v3), one(v2), 0x0C0C0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Code of one bf16 element.
__device__ __forceinline__ uint32_t code(uint32_t h, float inv) {
    const float r = __builtin_rintf(__builtin_amdgcn_fmed3f(bf16_to_f32(h) * inv, -127.0f, 127.0f));
    return (uint32_t)((int)r) & 0xFFu;
}

// 8 codes of a 16-byte bf16 vector packed into 8 bytes.
__device__ __forceinline__ uint2 code8(uint4 d, float inv) {
    const auto lo = [](uint32_t w) { return __uint_as_float(w << 16); };
    const auto hi = [](uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); };
    return make_uint2(code4(lo(d.x), hi(d.x), lo(d.y), hi(d.y), inv),
                      code4(lo(d.z), hi(d.z), lo(d.w), hi(d.w), inv));
}

struct RowScale {
    float inv;    // 127 / a, or 0 for a zero row
    float scale;  // a / 127, or 0 for a zero row
};

__device__ __forceinline__ RowScale row_scale_f(float a) {
    float inv = 127.0f / a;     // correctly rounded (no fast-math)
    float s = a / 127.0f;
    bool zero = !(a > 0.0f) || !__builtin_isfinite(inv);
    RowScale r;
    r.inv = zero ? 0.0f : inv;
    r.scale = zero ? 0.0f : s;
    return r;
}

__device__ __forceinline__ RowScale row_scale(uint32_t amax_bits) {
    return row_scale_f(bf16_to_f32(amax_bits));
}

}  // namespace qmath
}  // namespace w8a8
