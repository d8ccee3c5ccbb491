// Per-row symmetric absmax int8 quantizer for gfx950.
//
// One rule serves both operands of the W8A8 linear (Section 3, "The quantization
// recipe (reused)"): per output channel for the weight W [N,K] (offline) and per token
// for the activation X [M,K] (online, every forward; "The fused kernel"). For a row v:
//   a = max_k |v[k]|, s = a / 127, q[k] = clamp(rne(v[k] * (127 / a)), -127, 127),
// and a row with a == 0 or with 127/a overflowing float32 gets s = 0, q = 0.
//
// The rule can run on transformed values v[k] = T(x[k]) * c[k] instead of the bf16
// inputs themselves: T is the identity or the exact GELU x * Phi(x) (the activation in
// front of the MLP down-projection, applied here so that it costs no pass of its own),
// and c is a per-input-channel multiplier, the run-time half of SmoothQuant (the recipe
// of Section 3 smooths the activations by 1/s[k] and folds s[k] into the weights).
// Both are evaluated in float32; the row maximum is then taken on float32 values.
//
// The kernel is HBM-bound (3 bytes moved per element: 2 read, 1 written). Rows whose K fits
// the register file (K <= 65536 for the plain rule) are read once with 16-byte loads, kept in
// VGPRs for the second (quantizing) pass and written with 16-byte stores, streaming where
// alignment allows, by a persistent grid that prefetches the next rows while it finishes the
// current ones; the row maximum is taken on the bf16 bit patterns (|v| ordered as an unsigned
// integer, exact for finite values) with a wavefront reduction and, for rows of several
// wavefronts, one LDS exchange. Longer rows are read twice by a looped kernel.
#include "w8a8_internal.hpp"
#include "quant_math.hpp"

namespace w8a8 {
namespace {

using namespace qmath;

typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

// Buffer-resource word 3 for gfx9 (raw 32-bit data format, no swizzle), an offset beyond any
// row (loads give zero, stores are dropped), and the streaming cache policy of a store.
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kOutside = 0x7FFFFF00;
constexpr int kStreaming = 2;

// Swap with the neighbouring lane (lane l <-> l ^ 1) by a DPP quad permutation [1,0,3,2].
__device__ __forceinline__ uint32_t swap_lane_pair(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
}


// erfc(z) for z >= 0 by the Chebyshev fit of Numerical Recipes (Press, Teukolsky,
// Vetterling, Flannery, "erfcc"): t = 1 / (1 + z/2), erfc(z) ~ t exp(-z^2 + P(t)) with a
// degree-9 polynomial P, fractional error below 1.2e-7 for every z >= 0. One hardware
// reciprocal, one hardware exp2 and ten FMAs: the quantizer stays near the HBM bound.
__device__ __forceinline__ float erfc_nonneg(float z) {
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.5f, z, 1.0f));
    float p = 0.17087277f;
    p = __builtin_fmaf(t, p, -0.82215223f);
    p = __builtin_fmaf(t, p, 1.48851587f);
    p = __builtin_fmaf(t, p, -1.13520398f);
    p = __builtin_fmaf(t, p, 0.27886807f);
    p = __builtin_fmaf(t, p, -0.18628806f);
    p = __builtin_fmaf(t, p, 0.09678418f);
    p = __builtin_fmaf(t, p, 0.37409196f);
    p = __builtin_fmaf(t, p, 1.00002368f);
    const float arg = __builtin_fmaf(t, p, __builtin_fmaf(-z, z, -1.26551223f));
    return t * __builtin_amdgcn_exp2f(arg * 1.44269504088896341f);
}

// GELU(x) = x * Phi(x) with 2 Phi(x) = erfc(-x / sqrt(2)): for x < 0 that is
// erfc(|x| / sqrt(2)) (no cancellation in the left tail), for x >= 0 it is 2 - erfc.
__device__ __forceinline__ float gelu_f32(float x) {
    const float e = erfc_nonneg(__builtin_fabsf(x) * 0.70710678118654752440f);
    return 0.5f * x * (x < 0.0f ? e : 2.0f - e);
}

// The same factor from a table: the inputs are bf16, so h = erfc(|x| / sqrt(2)) / 2 takes one
// value per magnitude. From 16 up it is 0; below 2^-8 it is 1/2 - |x| / sqrt(2 pi) to within
// |x|^3 / 15 (4e-9). The 12 binades between (128 magnitudes each) and the end make 6 KB, which
// every block copies to LDS: with 28 binades (down to 2^-24, where h is 1/2) the copy cost
// short calls 0.3 us more. The entries are computed here at compile time in double: a series
// up to z = 1.5, the continued fraction of erfc above.
constexpr int kGeluLo = (127 - 8) << 7, kGeluHi = (127 + 4) << 7;   // bf16 magnitude bits
constexpr int kGeluN = kGeluHi - kGeluLo + 1;

constexpr double exp_nonpos(double x) {
    int n = 0;
    for (; x < -0.01; x *= 0.5)
        ++n;
    double s = 1.0, term = 1.0;
    for (int i = 1; i <= 7; ++i) {
        term *= x / i;
        s += term;
    }
    for (; n > 0; --n)
        s *= s;
    return s;
}

constexpr double erfc_const(double z) {
    constexpr double kInvSqrtPi = 0.56418958354775628695;
    if (z < 1.5) {
        double sum = z, term = z;
        for (int n = 1; n < 60 && (term > 1e-19 || term < -1e-19); ++n) {
            term *= -z * z / n;
            sum += term / (2 * n + 1);
        }
        return 1.0 - 2.0 * kInvSqrtPi * sum;
    }
    double f = z;
    for (int n = 60; n >= 1; --n)
        f = z + 0.5 * n / f;
    return exp_nonpos(-z * z) * kInvSqrtPi / f;
}
static_assert(erfc_const(1.0) > 0.157299207050 && erfc_const(1.0) < 0.157299207051, "series");
static_assert(erfc_const(2.0) > 0.004677734981047 && erfc_const(2.0) < 0.004677734981048, "fraction");

struct alignas(16) GeluTable {
    float h[(kGeluN + 3) / 4 * 4];   // erfc(|x| / sqrt(2)) / 2 at magnitude kGeluLo + i
};

constexpr GeluTable make_gelu_table() {
    GeluTable t{};
    for (int i = 0; i + 1 < kGeluN; ++i) {
        double x = 1.0 + (i & 127) / 128.0;
        for (int e = i >> 7; e < 8; ++e)
            x *= 0.5;
        for (int e = 8; e < (i >> 7); ++e)
            x *= 2.0;
        const double h = 0.5 * erfc_const(x * 0.70710678118654752440);
        t.h[i] = h < 1e-45 ? 0.0f : (float)h;
    }
    return t;   // the last entry (|x| >= 16) is 0
}
__device__ const GeluTable kGeluTable = make_gelu_table();

// GELU of a bf16 value given by its bits h (0 .. 0xFFFF): x * Phi(x) with Phi(x) = h(|x|)
// for x < 0 and 1 - h(|x|) otherwise, the table in LDS.
__device__ __forceinline__ float gelu_lookup(uint32_t h, const float *table) {
    const float x = bf16_to_f32(h);
    const int mag = (int)(h & 0x7FFFu);
    const float tail = table[min(max(mag, kGeluLo), kGeluHi) - kGeluLo];
    const float e = mag < kGeluLo
                        ? __builtin_fmaf(__builtin_fabsf(x), -0.39894228040143267794f, 0.5f)
                        : tail;
    return x * (x < 0.0f ? e : 1.0f - e);
}

// The value the row rule sees: T(x), times the channel multiplier c when there is one.
template <int ACT, bool CM>
__device__ __forceinline__ float transform(float x, float c) {
    float t = x;
    if constexpr (ACT == ACT_GELU)
        t = gelu_f32(x);
    if constexpr (CM)
        t = t * c;
    return t;
}

// Code of a float32 value (transformed rows).
__device__ __forceinline__ uint32_t code_f(float v, float inv) {
    const float r = __builtin_amdgcn_fmed3f(__builtin_rintf(v * inv), -127.0f, 127.0f);
    return (uint32_t)((int)r) & 0xFFu;
}

__device__ __forceinline__ uint32_t abs_bits(float v) {
    return __float_as_uint(v) & 0x7FFFFFFFu;
}

// Elements [8 vi, min(8 vi + 8, K)) of a row of K >= 8 at any alignment, zeros behind K.
__device__ __forceinline__ uint4 load8_any(const uint16_t *row, int64_t vi, int64_t nwhole,
                                           int64_t K) {
    const int64_t at = vi < nwhole ? vi * 8 : K - 8;
    const Bytes16 b = *reinterpret_cast<const Bytes16 *>(row + at);
    uint4 d = make_uint4(b.w[0], b.w[1], b.w[2], b.w[3]);
    if (vi >= nwhole) {
        const int sh = (int)(vi * 8 - at) * 16;       // 16 .. 112 bits
        uint64_t lo = d.x | (uint64_t)d.y << 32, hi = d.z | (uint64_t)d.w << 32;
        if (sh < 64) {
            lo = lo >> sh | hi << (64 - sh);
            hi >>= sh;
        } else {
            lo = hi >> (sh - 64);
            hi = 0;
        }
        d = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
    return d;
}

// Register-resident path, persistent and software-pipelined: TPR threads per row
// (64 = one wavefront, up to 1024 = the block), NV 16-byte vectors per thread (K % 8 ==
// 0, v 16-byte and q 8-byte aligned). Blocks have max(TPR, 256) threads. Row group j of
// a block holds rows j*RPB .. j*RPB + RPB - 1; block b handles row groups b, b + G, b +
// 2G, ... (G = gridDim.x) and loads
// group j + G while it reduces, quantizes and stores group j, so the HBM reads of the
// next rows overlap the work and the stores of the current ones.
// With a transform (ACT != ACT_NONE or a multiplier), each thread's columns are the
// same for every row, so its multipliers are loaded once into registers; the
// transformed row is held as float32 between the maximum and the coding pass.
//
// Loads and stores go through a buffer descriptor of the row (lanes past its end, and rows
// past the last, read zeros and store nothing) and so need no branches: with a branch around
// a load the compiler cannot count the loads in flight and waits for all of them, the next
// row's included. With that, the wavefront maximum in DPP operands and one barrier per row
// instead of two, us for branches and shuffles -> now: 4096 x 2048 6.7 -> 5.6, 2048 x 4096
// 7.0 -> 5.9, 77 x 4096 3.1 -> 2.7, 4096 x 7696 22.1 -> 19.6 (4.8 TB/s); with GELU and the
// multiplier 4096 x 16384 47 -> 42.
//
// ANY: rows at any alignment and any K >= 8, by the same 16-byte loads and 8-byte stores
// at the rows' own alignment. The vector that crosses the row's end is read as the row's
// last 8 elements shifted down, zeros behind, and its codes are stored one by one.
template <int TPR>
constexpr int reg_block_threads() { return TPR > 256 ? TPR : 256; }

template <int TPR, int NV, int ACT, bool CM, bool ANY = false>
__global__ void __launch_bounds__(reg_block_threads<TPR>())
quant_rows_reg(const uint16_t *__restrict__ v, int64_t rows, int64_t K,
               const float *__restrict__ colmul, int8_t *__restrict__ q,
               float *__restrict__ scale) {
    constexpr bool PLAIN = ACT == ACT_NONE && !CM;
    constexpr int BS = reg_block_threads<TPR>();
    constexpr int RPB = BS / TPR;
    constexpr int WPR = TPR / 64;              // wavefronts per row
    const int t = threadIdx.x % TPR;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave / WPR;
    const int64_t nvec = (K + 7) >> 3;
    const int64_t nwhole = K >> 3;             // vectors that lie wholly in the row
    const int64_t groups = (rows + RPB - 1) / RPB;
    const bool wide = (K % 16 == 0) && (reinterpret_cast<uintptr_t>(q) % 16 == 0);
    __shared__ uint32_t part[2][RPB][WPR];     // in turn, so one barrier per row will do
    constexpr bool GELU = ACT == ACT_GELU;
    __shared__ __attribute__((aligned(16))) float gelu[GELU ? sizeof(GeluTable) / 4 : 1];

    float cmr[CM ? NV : 1][8];
    if constexpr (CM) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int64_t vi = (int64_t)j * TPR + t;
            if constexpr (ANY) {
                if (vi < nwhole) {
                    const Bytes16 *c = reinterpret_cast<const Bytes16 *>(colmul + vi * 8);
                    const Bytes16 lo = c[0], hi = c[1];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        cmr[j][e] = __uint_as_float(e < 4 ? lo.w[e & 3] : hi.w[e & 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        cmr[j][e] = vi * 8 + e < K ? colmul[vi * 8 + e] : 0.0f;
                }
                continue;
            }
            const float4 *c4 = reinterpret_cast<const float4 *>(colmul) + 2 * vi;
            const float4 lo = vi < nvec ? c4[0] : make_float4(0, 0, 0, 0);
            const float4 hi = vi < nvec ? c4[1] : make_float4(0, 0, 0, 0);
            cmr[j][0] = lo.x; cmr[j][1] = lo.y; cmr[j][2] = lo.z; cmr[j][3] = lo.w;
            cmr[j][4] = hi.x; cmr[j][5] = hi.y; cmr[j][6] = hi.z; cmr[j][7] = hi.w;
        }
    }

    auto load = [&](uint4 (&d)[NV], int64_t grp) __attribute__((always_inline)) {
        const int64_t row = grp * RPB + sub;
        const bool live = row < rows;
        const uint16_t *base = v + (live ? row : 0) * K;
        const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
            (void *)base, (short)0, live ? (int)(2 * K) : 0, kRsrcWord3);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if constexpr (ANY) {
                const int64_t vi = (int64_t)j * TPR + t;
                d[j] = make_uint4(0, 0, 0, 0);
                if (live && vi < nvec)
                    d[j] = load8_any(base, vi, nwhole, K);
            } else {
                const u32x4v w = __builtin_amdgcn_raw_buffer_load_b128(src, (j * TPR + t) * 16, 0, 0);
                d[j] = make_uint4(w.x, w.y, w.z, w.w);
            }
        }
    };
    int turn = 0;
    auto process = [&](const uint4 (&d)[NV], int64_t grp) __attribute__((always_inline)) {
        const int64_t row = grp * RPB + sub;
        uint32_t m = 0;
        float f[PLAIN ? 1 : NV][8];
        if constexpr (PLAIN) {
#pragma unroll
            for (int j = 0; j < NV; ++j)
                m = max(m, absmax8(d[j]));
        } else {
            float fm = 0.0f;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const uint32_t w[4] = {d[j].x, d[j].y, d[j].z, d[j].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t h = (e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu);
                    f[j][e] = GELU ? gelu_lookup(h, gelu) : bf16_to_f32(h);
                    if constexpr (CM)
                        f[j][e] *= cmr[j][e];
                    fm = fmaxf(fm, __builtin_fabsf(f[j][e]));
                }
            }
            m = __float_as_uint(fm);   // |v| >= 0: its bit pattern orders like the value
        }
        m = wave_max(m);
        if constexpr (WPR > 1) {
            if ((threadIdx.x & 63) == 0)
                part[turn][sub][wave % WPR] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < WPR; ++w)
                m = max(m, part[turn][sub][w]);
            turn ^= 1;
        }
        const RowScale rs = PLAIN ? row_scale(m) : row_scale_f(__uint_as_float(m));
        // Codes of vector j of this lane (8 bytes).
        auto codes = [&](int j) __attribute__((always_inline)) {
            uint2 o;
            if constexpr (PLAIN) {
                o = code8(d[j], rs.inv);
            } else {
                o.x = code4(f[j][0], f[j][1], f[j][2], f[j][3], rs.inv);
                o.y = code4(f[j][4], f[j][5], f[j][6], f[j][7], rs.inv);
            }
            return o;
        };
        const bool live = row < rows;
        if constexpr (ANY) {
            if (!live)
                return;
            if (t == 0)
                scale[row] = rs.scale;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int64_t vi = (int64_t)j * TPR + t;
                if (vi >= nvec)
                    continue;
                const uint2 c = codes(j);
                int8_t *o = q + row * K + vi * 8;
                if (vi < nwhole) {
                    *reinterpret_cast<Bytes8 *>(o) = Bytes8{{c.x, c.y}};
                } else {
#pragma unroll
                    for (int e = 0; e < 7; ++e)
                        if (vi * 8 + e < K)
                            o[e] = (int8_t)((e < 4 ? c.x : c.y) >> (8 * (e & 3)));
                }
            }
        } else {
            // Only lane 0 of the row lies inside the 4 bytes of its scale.
            const __amdgpu_buffer_rsrc_t sdst = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(scale + (live ? row : 0)), (short)0, live ? 4 : 0, kRsrcWord3);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(rs.scale), sdst, t * 4, 0, 0);
            const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(q + (live ? row : 0) * K), (short)0, live ? (int)K : 0, kRsrcWord3);
            // 16-byte stores, one pair of vectors at a time. Vectors j and j+1 of lane t are
            // j*TPR + t and (j+1)*TPR + t; neighbouring lanes swap one code word pair so that
            // the even lane holds vectors j*TPR + t, +1 and the odd lane (j+1)*TPR + t - 1,
            // +1. Streaming stores where rows are 16-byte aligned: they leave no dirty lines
            // in this XCD's L2 for the kernel's end to write back before the consumer starts
            // (plain stores, and 8-byte streaming ones, delayed the next kernel by 1.5-2.5
            // us). A row's last vector without a partner (K % 16 == 8) goes out alone.
            constexpr int NP = (NV + 1) / 2;
            u32x4v o[NP];
            int v0[NP];
            const bool odd = t & 1;
#pragma unroll
            for (int j = 0; j + 1 < NV; j += 2) {
                // Selects on scalars (a select between array elements would put the
                // array in memory).
                const uint2 ca = codes(j), cb = codes(j + 1);
                const uint32_t a0 = ca.x, a1 = ca.y, b0 = cb.x, b1 = cb.y;
                const uint32_t r0 = swap_lane_pair(odd ? a0 : b0);
                const uint32_t r1 = swap_lane_pair(odd ? a1 : b1);
                o[j / 2] = odd ? u32x4v{r0, r1, b0, b1} : u32x4v{a0, a1, r0, r1};
                v0[j / 2] = odd ? (j + 1) * TPR + t - 1 : j * TPR + t;
            }
            if constexpr (NV % 2 == 1) {
                // The last vector of an odd count: the even lane of each pair takes its
                // neighbour's codes (vector j*TPR + t + 1) and stores both.
                const uint2 c = codes(NV - 1);
                o[NP - 1] = u32x4v{c.x, c.y, swap_lane_pair(c.x), swap_lane_pair(c.y)};
                v0[NP - 1] = odd ? kOutside / 8 : (NV - 1) * TPR + t;
            }
            if (wide) {
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    __builtin_amdgcn_raw_buffer_store_b128(o[p], dst, v0[p] * 8, 0, kStreaming);
            } else {
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    __builtin_amdgcn_raw_buffer_store_b128(
                        o[p], dst, v0[p] + 1 < (int)nvec ? v0[p] * 8 : kOutside, 0, 0);
                if (nvec & 1) {
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        __builtin_amdgcn_raw_buffer_store_b64(
                            u32x2v{o[p].x, o[p].y}, dst,
                            v0[p] + 1 == (int)nvec ? v0[p] * 8 : kOutside, 0, 0);
                }
            }
        }
    };

    uint4 a[NV], b[NV];
    int64_t grp = blockIdx.x;
    load(a, grp);
    if constexpr (GELU) {
        // All of a thread's share of the table is requested before any of it is stored.
        constexpr int N4 = sizeof(GeluTable) / 16, PER = (N4 + BS - 1) / BS;
        float4 h[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            h[i] = reinterpret_cast<const float4 *>(&kGeluTable)[min(i * BS + (int)threadIdx.x, N4 - 1)];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i * BS + (int)threadIdx.x < N4)
                reinterpret_cast<float4 *>(gelu)[i * BS + threadIdx.x] = h[i];
        __syncthreads();
    }
    // The last row group is processed outside the loop, so that inside it every load and
    // store is unconditional.
    for (;;) {
        if (grp + gridDim.x >= groups)
            break;
        load(b, grp + gridDim.x);
        __builtin_amdgcn_sched_barrier(0);
        process(a, grp);
        grp += gridDim.x;
        if (grp + gridDim.x >= groups) {
#pragma unroll
            for (int j = 0; j < NV; ++j)
                a[j] = b[j];
            break;
        }
        load(a, grp + gridDim.x);
        __builtin_amdgcn_sched_barrier(0);
        process(b, grp);
        grp += gridDim.x;
    }
    process(a, grp);
}

// General path: a 256-thread block per row (a block takes every G-th row when there are
// more rows than the grid's G blocks), two passes over the row (the second re-reads it,
// normally from L2). VEC selects 16-byte loads and 8-byte stores (K % 8 ==
// 0; v and colmul 16-byte, q 8-byte aligned); a transform is then evaluated on the 8
// values of a vector in both passes. Otherwise every element is loaded and stored on
// its own, for any K and any alignment.
template <bool VEC, int ACT, bool CM>
__global__ void __launch_bounds__(256)
quant_rows_loop(const uint16_t *__restrict__ v, int64_t rows, int64_t K,
                const float *__restrict__ colmul, int8_t *__restrict__ q,
                float *__restrict__ scale) {
    constexpr bool PLAIN = ACT == ACT_NONE && !CM;
    const int t = threadIdx.x;
    const int64_t nvec = K >> 3;
    __shared__ uint32_t part[4];
    // Block b takes rows b, b + G, b + 2G, ... (G = gridDim.x, at most 65536 blocks).
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        const uint16_t *src = v + row * K;
        auto value = [&](int64_t k) {
            return transform<ACT, CM>(bf16_to_f32(src[k]), CM ? colmul[k] : 1.0f);
        };
        // The 8 transformed values of vector vi.
        auto values8 = [&](int64_t vi, float (&f)[8]) __attribute__((always_inline)) {
            const uint4 d = reinterpret_cast<const uint4 *>(src)[vi];
            float c[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
            if constexpr (CM) {
                const float4 *c4 = reinterpret_cast<const float4 *>(colmul) + 2 * vi;
                const float4 lo = c4[0], hi = c4[1];
                c[0] = lo.x; c[1] = lo.y; c[2] = lo.z; c[3] = lo.w;
                c[4] = hi.x; c[5] = hi.y; c[6] = hi.z; c[7] = hi.w;
            }
            const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t h = (e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu);
                f[e] = transform<ACT, CM>(bf16_to_f32(h), c[e]);
            }
        };
        uint32_t m = 0;
        if constexpr (VEC && PLAIN) {
            const uint4 *s4 = reinterpret_cast<const uint4 *>(src);
            for (int64_t vi = t; vi < nvec; vi += 256)
                m = max(m, absmax8(s4[vi]));
        } else if constexpr (VEC) {
            float fm = 0.0f;
            for (int64_t vi = t; vi < nvec; vi += 256) {
                float f[8];
                values8(vi, f);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    fm = fmaxf(fm, __builtin_fabsf(f[e]));
            }
            m = abs_bits(fm);
        } else if constexpr (PLAIN) {
            for (int64_t k = t; k < K; k += 256)
                m = max(m, (uint32_t)src[k] & 0x7FFFu);
        } else {
            for (int64_t k = t; k < K; k += 256)
                m = max(m, abs_bits(value(k)));
        }
        m = wave_max(m);
        if ((t & 63) == 0)
            part[t >> 6] = m;
        __syncthreads();
        m = max(max(part[0], part[1]), max(part[2], part[3]));
        __syncthreads();   // part is rewritten for the next row
        const RowScale rs = PLAIN ? row_scale(m) : row_scale_f(__uint_as_float(m));
        if (t == 0)
            scale[row] = rs.scale;
        int8_t *dst = q + row * K;
        if constexpr (VEC && PLAIN) {
            const uint4 *s4 = reinterpret_cast<const uint4 *>(src);
            uint2 *d2 = reinterpret_cast<uint2 *>(dst);
            for (int64_t vi = t; vi < nvec; vi += 256)
                d2[vi] = code8(s4[vi], rs.inv);
        } else if constexpr (VEC) {
            uint2 *d2 = reinterpret_cast<uint2 *>(dst);
            for (int64_t vi = t; vi < nvec; vi += 256) {
                float f[8];
                values8(vi, f);
                d2[vi] = make_uint2(code4(f[0], f[1], f[2], f[3], rs.inv),
                                    code4(f[4], f[5], f[6], f[7], rs.inv));
            }
        } else if constexpr (PLAIN) {
            for (int64_t k = t; k < K; k += 256)
                dst[k] = (int8_t)code((uint32_t)src[k], rs.inv);
        } else {
            for (int64_t k = t; k < K; k += 256)
                dst[k] = (int8_t)code_f(value(k), rs.inv);
        }
    }
}

template <int TPR, int NV, int ACT, bool CM, bool ANY = false>
hipError_t launch_reg(const uint16_t *v, int64_t rows, int64_t K, const float *colmul,
                      int8_t *q, float *scale, hipStream_t s) {
    constexpr int BS = reg_block_threads<TPR>();
    constexpr int RPB = BS / TPR;
    const int64_t groups = (rows + RPB - 1) / RPB;
    // Persistent grid: up to 2048 threads per CU, each block walking row groups with
    // prefetch.
    const int64_t max_blocks = 256 * 2048 / BS;
    const int64_t blocks = groups < max_blocks ? groups : max_blocks;
    hipLaunchKernelGGL((quant_rows_reg<TPR, NV, ACT, CM, ANY>), dim3((unsigned)blocks), dim3(BS),
                       0, s, v, rows, K, colmul, q, scale);
    return hipGetLastError();
}

template <int ACT, bool CM>
hipError_t launch_rows(const uint16_t *v, int64_t rows, int64_t K, const float *colmul,
                       int8_t *q, float *scale, hipStream_t s) {
    constexpr bool PLAIN = ACT == ACT_NONE && !CM;
    const bool vec = (K % 8 == 0) && (reinterpret_cast<uintptr_t>(v) % 16 == 0) &&
                     (reinterpret_cast<uintptr_t>(q) % 8 == 0) &&
                     (reinterpret_cast<uintptr_t>(colmul) % 16 == 0);
    const int64_t nvec = K / 8;
    // Threads per row and vectors per thread, from sweeps of both over rows x K with the
    // matrices rotated through HBM. The vector count per thread is the smallest that
    // covers the row, so few lanes idle (at K = 4608 a 256 x 4 row leaves 44% of them
    // idle: 11-24% slower than 128 x 5 for the plain rule); fewer rows spread a row over
    // more threads.
    if constexpr (PLAIN) {
        if (vec && nvec > 256 && nvec <= 2048) {
            if (nvec <= 512) {
                if (rows < 1024)
                    return launch_reg<512, 1, ACT, CM>(v, rows, K, colmul, q, scale, s);
                // One wavefront per row with exactly the vectors the row needs.
                if (nvec <= 320)
                    return launch_reg<64, 5, ACT, CM>(v, rows, K, colmul, q, scale, s);
                if (nvec <= 384)
                    return launch_reg<64, 6, ACT, CM>(v, rows, K, colmul, q, scale, s);
                if (rows < 4096)
                    return launch_reg<128, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
                if (nvec <= 448)
                    return launch_reg<64, 7, ACT, CM>(v, rows, K, colmul, q, scale, s);
                return launch_reg<64, 8, ACT, CM>(v, rows, K, colmul, q, scale, s);
            }
            if (nvec <= 768 && rows < 1024)
                return launch_reg<256, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 640)
                return launch_reg<128, 5, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 768)
                return launch_reg<128, 6, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 1024)
                return rows >= 4096 ? launch_reg<128, 8, ACT, CM>(v, rows, K, colmul, q, scale, s)
                                    : launch_reg<256, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
            // Long rows: 512 threads each while the rows are few (512 x 12288: 5.3 us, 5.8 on
            // 256 x 6; 512 x 16384: 6.1, 6.6 on 256 x 8).
            if (nvec <= 1536)
                return rows < 1536 ? launch_reg<512, 3, ACT, CM>(v, rows, K, colmul, q, scale, s)
                                   : launch_reg<256, 6, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (rows < 768)
                return launch_reg<512, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
            return rows >= 4096 ? launch_reg<1024, 2, ACT, CM>(v, rows, K, colmul, q, scale, s)
                                : launch_reg<256, 8, ACT, CM>(v, rows, K, colmul, q, scale, s);
        }
    } else {
        // Transformed rows hold the float32 row too, so more threads with fewer vectors each
        // pay; GELU rows also spread the copy of the table to LDS over more threads (us, GELU:
        // 128 x 2560 3.3 on 512 x 1 against 3.9 on 128 x 3, 4608 x 2560 10.9 against 12.2 on
        // 256 x 2, 2048 x 4096 7.9 on 512 x 1 against 8.6 on 256 x 2, 2048 x 16384 22.1 on
        // 1024 x 2 against 24.8 on 512 x 4; with the multiplier 4608 x 16384 49.4 on 512 x 4,
        // 54.6 on 256 x 8, 57.6 on 1024 x 2; multiplier alone: 512 x 16384 6.5 on 512 x 4,
        // 7.0 on 256 x 8, 4608 x 16384 43.0 on 256 x 8, 43.9 on 512 x 4).
        constexpr bool GELU = ACT == ACT_GELU;
        if (vec && nvec > 192 && nvec <= 2048 && (nvec > 256 || rows >= 1024)) {
            if (nvec <= 256)
                return launch_reg<128, 2, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 512 && rows < (nvec <= 384 ? 1024 : 4096))
                return launch_reg<512, 1, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (GELU && nvec <= 384)
                return launch_reg<128, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 512)
                return launch_reg<256, 2, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 768)
                return launch_reg<256, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 1024)
                return launch_reg<512, 2, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 1536)
                return launch_reg<512, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (GELU && !CM && rows < 4096)
                return launch_reg<1024, 2, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (GELU || rows < 768)
                return launch_reg<512, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
            return launch_reg<256, 8, ACT, CM>(v, rows, K, colmul, q, scale, s);
        }
    }
    if (vec && K > 0) {
        // K <= 2048: below 1024 rows a row takes 128 or 256 threads with one vector each
        // (8-13% faster than a wavefront per row at K = 1536-2048, 32% with GELU);
        // from 1024 rows up a wavefront per row with exactly the row's vectors.
        if (nvec <= 64)
            return launch_reg<64, 1, ACT, CM>(v, rows, K, colmul, q, scale, s);
        if (nvec <= 128)
            return rows < 1024 ? launch_reg<128, 1, ACT, CM>(v, rows, K, colmul, q, scale, s)
                               : launch_reg<64, 2, ACT, CM>(v, rows, K, colmul, q, scale, s);
        if (nvec <= 256) {
            if (rows < 1024)
                return launch_reg<256, 1, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if (nvec <= 192)
                return launch_reg<64, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
            if constexpr (PLAIN)
                return launch_reg<64, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
        }
        // Long rows (K up to 65536 for the plain rule, e.g. a 53248-wide projection
        // input; 32768 for transformed rows, whose float32 copy of 8 vectors per thread
        // would not fit 128 VGPRs): a 1024-thread block per row, still read once. The
        // looped kernel below reads such rows twice, the second time mostly from the
        // MALL, since 32 CUs' rows overflow an XCD's L2.
        // Up to K = 24576 three vectors a thread, so that few lanes work on nothing
        // (4608 x 16400 with the multiplier: 47.8 us, 50.6 on four; 7-13% over K = 16400,
        // 18432, 20480 and 24576, 1 to 4608 rows and every transform).
        if (nvec <= 3072)
            return launch_reg<1024, 3, ACT, CM>(v, rows, K, colmul, q, scale, s);
        if (nvec <= 4096)
            return launch_reg<1024, 4, ACT, CM>(v, rows, K, colmul, q, scale, s);
        if constexpr (PLAIN)
            if (nvec <= 8192)
                return launch_reg<1024, 8, ACT, CM>(v, rows, K, colmul, q, scale, s);
    }
    // Any alignment: a coarser choice of the same mappings (4000 x 4097: 15.0 us, against
    // 10.5 at K = 4096; 600 x 20001: 12.5 us). The looped kernel below, one element per
    // load and store, takes 21.2 and 39.7 us there and is left for K < 8 and the longest
    // rows.
    if (!vec && K >= 8 && K <= 32768) {
        const int64_t n = (K + 7) / 8;
        if (n <= 64)
            return launch_reg<64, 1, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        if (n <= 128)
            return launch_reg<64, 2, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        if (n <= 256)
            return launch_reg<128, 2, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        if (n <= 512)
            return launch_reg<256, 2, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        if (n <= 1024)
            return launch_reg<512, 2, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        if (n <= 2048)
            return launch_reg<512, 4, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
        return launch_reg<1024, 4, ACT, CM, true>(v, rows, K, colmul, q, scale, s);
    }
    const unsigned grid = (unsigned)(rows < 65536 ? rows : 65536);
    if (vec)
        hipLaunchKernelGGL((quant_rows_loop<true, ACT, CM>), dim3(grid), dim3(256), 0, s, v,
                           rows, K, colmul, q, scale);
    else
        hipLaunchKernelGGL((quant_rows_loop<false, ACT, CM>), dim3(grid), dim3(256), 0, s, v,
                           rows, K, colmul, q, scale);
    return hipGetLastError();
}

// Calibration: per-column max |T(x)|. Bound by reading the matrix once: 16-byte loads, eight
// in flight per lane, at the rows' own alignment, and the maxima kept as bf16 bit patterns
// (two per register) until the end. A block takes up to 512 columns and rows_per_block
// rows: lpr lanes (a power of two) cover the columns of a row, blockDim / lpr rows at a time;
// the row groups meet in LDS, blocks by an unsigned atomic maximum on the float32 bit
// pattern (monotone for values >= 0), skipped where the column already holds as much; a
// single block of rows that need not be merged (store) writes its maxima straight away.
// 16384 x 4096 takes 34.4 us (3.9 TB/s), 4608 x 16384 35.5 us, with GELU 38.5 us; one element
// per load and evaluating GELU for each took 71.7, 84.3 and 93.4 us.
//
// |GELU| needs no evaluation per element. It grows with x > 0; for x < 0 it grows with |x|
// up to 0.75 and falls from the next bf16 value on (|x| Phi(-|x|) peaks at 0.7518). So the
// column's maximum is at one of: its largest positive x, its largest |x| <= 0.75 and its
// smallest |x| > 0.75 among the negative ones. The negative x of largest magnitude is
// evaluated too, so that an infinity or NaN shows.
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef int16_t s16x8 __attribute__((ext_vector_type(8)));

template <int ACT>
struct ColMax {
    u16x8 m = {};                       // plain: |x|
    __device__ __forceinline__ void add(u16x8 x) {
        m = __builtin_elementwise_max(m, x & (uint16_t)0x7FFF);
    }
    __device__ __forceinline__ void merge(const ColMax &o) {
        m = __builtin_elementwise_max(m, o.m);
    }
    __device__ __forceinline__ uint32_t result(int e) const { return (uint32_t)m[e] << 16; }
};

template <>
struct ColMax<ACT_GELU> {
    // u = x - kSplit modulo 2^16 orders the bit patterns: negative x beyond -0.75 first
    // (from 0, by magnitude), then every positive x, then negative x up to -0.75 (from
    // kSmall, by magnitude).
    static constexpr uint16_t kSplit = 0xBF41, kLarge = 0x7FFF - 0x3F41, kSmall = 0x8000 - 0xBF41;
    s16x8 pos = {};                     // largest x >= 0
    u16x8 lo = ~u16x8{};                // min u: the smallest |x| > 0.75 if it is <= kLarge
    u16x8 hi = {};                      // max u: the largest |x| <= 0.75 if it is >= kSmall
    u16x8 neg = {};                     // x < 0 of the largest magnitude if it is >= 0x8000
    __device__ __forceinline__ void add(u16x8 x) {
        const u16x8 u = x - kSplit;
        pos = __builtin_elementwise_max(pos, (s16x8)x);
        lo = __builtin_elementwise_min(lo, u);
        hi = __builtin_elementwise_max(hi, u);
        neg = __builtin_elementwise_max(neg, x);
    }
    __device__ __forceinline__ void merge(const ColMax &o) {
        pos = __builtin_elementwise_max(pos, o.pos);
        lo = __builtin_elementwise_min(lo, o.lo);
        hi = __builtin_elementwise_max(hi, o.hi);
        neg = __builtin_elementwise_max(neg, o.neg);
    }
    __device__ __forceinline__ uint32_t result(int e) const {
        auto at = [](uint16_t h) { return abs_bits(gelu_f32(bf16_to_f32(h))); };
        uint32_t r = at((uint16_t)pos[e]);
        if (lo[e] <= kLarge)
            r = max(r, at((uint16_t)(lo[e] + kSplit)));
        if (hi[e] >= kSmall)
            r = max(r, at((uint16_t)(hi[e] + kSplit)));
        if (neg[e] >= 0x8000)
            r = max(r, at(neg[e]));
        return r;
    }
};

constexpr int kColThreads = 1024;

template <int ACT>
__global__ void __launch_bounds__(kColThreads)
col_absmax_kernel(const uint16_t *__restrict__ v, int64_t rows, int64_t K, int lpr_log2,
                  int64_t rows_per_block, bool store, uint32_t *amax) {
    constexpr int U = 8;                            // rows in flight per lane
    const int lpr = 1 << lpr_log2;
    const int rpp = (int)blockDim.x >> lpr_log2;                // rows covered by one load of the block
    const int t = threadIdx.x & (lpr - 1), sub = threadIdx.x >> lpr_log2;
    const int64_t vi = (int64_t)blockIdx.x * lpr + t, nwhole = K >> 3;
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_block;
    const int64_t r1 = r0 + rows_per_block < rows ? r0 + rows_per_block : rows;
    __shared__ __attribute__((aligned(16))) char part_bytes[kColThreads * sizeof(ColMax<ACT>)];
    ColMax<ACT> *const part = reinterpret_cast<ColMax<ACT> *>(part_bytes);

    ColMax<ACT> cm;
    if (vi * 8 < K) {
        auto load = [&](int64_t r) {
            const uint16_t *row = v + r * K;
            if (K >= 8)
                return __builtin_bit_cast(u16x8, load8_any(row, vi, nwhole, K));
            u16x8 x = {};
            for (int e = 0; e < (int)K; ++e)
                x[e] = row[e];
            return x;
        };
        int64_t r = r0 + sub;
        for (; r + (U - 1) * rpp < r1; r += U * rpp) {
            u16x8 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                x[u] = load(r + u * rpp);
#pragma unroll
            for (int u = 0; u < U; ++u)
                cm.add(x[u]);
        }
        for (; r < r1; r += rpp)
            cm.add(load(r));
    }
    part[threadIdx.x] = cm;
    __syncthreads();
    // Column c of the block: entry c % 8 of lane c / 8 of every row group.
    for (int c = threadIdx.x; c < lpr; c += blockDim.x) {
        for (int g = 1; g < rpp; ++g)
            cm.merge(part[g * lpr + c]);
        part[c] = cm;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < lpr * 8; c += blockDim.x) {
        const int64_t k = (int64_t)blockIdx.x * lpr * 8 + c;
        if (k >= K)
            break;
        const uint32_t m = part[c >> 3].result(c & 7);
        if (store)
            amax[k] = m;
        else if (m > __hip_atomic_load(amax + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(amax + k, m);
    }
}

__global__ void __launch_bounds__(256) fill_zero_u32(uint32_t *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        p[i] = 0u;
}

// SmoothQuant factors: s = ax^alpha / aw^(1 - alpha) (alpha = 1/2: sqrtf / sqrtf, each
// correctly rounded); channels without a positive, finite pair, or whose factor is 0
// or infinite, stay unsmoothed (s = 1). s_inv = 1 / s is the activation multiplier.
__global__ void __launch_bounds__(256)
smooth_factors_kernel(const float *__restrict__ ax, const float *__restrict__ aw, int64_t K,
                      float alpha, float *__restrict__ s, float *__restrict__ s_inv) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= K)
        return;
    const float a = ax[k], b = aw[k];
    float f = 1.0f;
    if (a > 0.0f && b > 0.0f && __builtin_isfinite(a) && __builtin_isfinite(b)) {
        f = alpha == 0.5f ? sqrtf(a) / sqrtf(b) : powf(a, alpha) / powf(b, 1.0f - alpha);
        if (!(f > 0.0f) || !__builtin_isfinite(f))
            f = 1.0f;
    }
    s[k] = f;
    s_inv[k] = 1.0f / f;
}

}  // namespace

hipError_t launch_quant_rows(const uint16_t *v, int64_t rows, int64_t K, int act,
                             const float *colmul, int8_t *q, float *scale, hipStream_t s) {
    if (rows <= 0)
        return hipSuccess;
    if (act == ACT_GELU)
        return colmul ? launch_rows<ACT_GELU, true>(v, rows, K, colmul, q, scale, s)
                      : launch_rows<ACT_GELU, false>(v, rows, K, colmul, q, scale, s);
    return colmul ? launch_rows<ACT_NONE, true>(v, rows, K, colmul, q, scale, s)
                  : launch_rows<ACT_NONE, false>(v, rows, K, colmul, q, scale, s);
}

hipError_t launch_col_absmax(const uint16_t *v, int64_t rows, int64_t K, int act,
                             float *amax, bool accumulate, hipStream_t s) {
    if (K <= 0)
        return hipSuccess;
    uint32_t *bits = reinterpret_cast<uint32_t *>(amax);
    const auto fill = [&]() {
        hipLaunchKernelGGL(fill_zero_u32, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, s, bits,
                           K);
    };
    if (rows > 0) {
        const int64_t nvec = (K + 7) / 8;
        int lpr_log2 = 0;
        while (lpr_log2 < 6 && (1 << lpr_log2) < nvec)
            ++lpr_log2;
        const int64_t kb = (nvec + (1 << lpr_log2) - 1) >> lpr_log2;
        // Eight rows in flight per thread (figures: matrices in turn from 300 MB). One block for
        // all rows where it can hold them: it
        // needs no zeroing before it (128 x 4096: 5.0 us, 6.1 on blocks of 512). It takes as
        // few threads as leave four rows for each, since the merge walks a column's row
        // groups one by one: at least 16 groups or 512 threads (1 x 4096 with GELU: 3.8 us,
        // 4.5 on 1024; 1 x 64 with GELU: 3.7 on 128, 10.2 on 1024), at most 64 groups. Beyond, blocks
        // of 1024 threads, two per CU (the chip's resident threads), so that few atomics
        // meet on a column (16384 x 4096: 32.0 us, 36.9 on 256); 256 threads where that
        // leaves few row blocks and the loads' latency counts (300 x 1000: 6.2 against 7.2
        // us), 512 between, up to 48 blocks of 1024 (1000 x 1001: 7.4 us, 8.5 on 1024, 7.6 on
        // 256), all with at most 16 row groups (16384 x 64: 7.9 us on 128, 9.7 on 1024).
        const int64_t batch = 8 * (kColThreads >> lpr_log2);
        const int merge16 = 16 << lpr_log2, merge64 = 64 << lpr_log2;
        int threads = merge16 < 64 ? 64 : merge16 < 512 ? merge16 : 512;
        while (threads < kColThreads && threads < merge64 && 4 * (threads >> lpr_log2) < rows)
            threads *= 2;
        if (8 * (threads >> lpr_log2) < rows) {
            threads = rows <= 4 * batch ? 256 : kb * rows <= 48 * batch ? 512 : kColThreads;
            threads = threads < merge16 ? threads : merge16 < 64 ? 64 : merge16;
        }
        const int64_t unit = 8 * (threads >> lpr_log2);
        const int64_t want = kb < 512 ? 512 / kb : 1;
        int64_t rpb = ((rows + want - 1) / want + unit - 1) / unit * unit;
        while ((rows + rpb - 1) / rpb > 65535)
            rpb *= 2;
        const dim3 grid((unsigned)kb, (unsigned)((rows + rpb - 1) / rpb));
        const bool store = grid.y == 1 && !accumulate;
        if (!accumulate && !store)
            fill();
        if (act == ACT_GELU)
            hipLaunchKernelGGL(col_absmax_kernel<ACT_GELU>, grid, dim3(threads), 0, s, v, rows, K,
                               lpr_log2, rpb, store, bits);
        else
            hipLaunchKernelGGL(col_absmax_kernel<ACT_NONE>, grid, dim3(threads), 0, s, v, rows, K,
                               lpr_log2, rpb, store, bits);
    } else if (!accumulate) {
        fill();
    }
    return hipGetLastError();
}

hipError_t launch_smooth_factors(const float *ax, const float *aw, int64_t K, float alpha,
                                 float *smooth, float *smooth_inv, hipStream_t s) {
    if (K <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(smooth_factors_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0,
                       s, ax, aw, K, alpha, smooth, smooth_inv);
    return hipGetLastError();
}

}  // namespace w8a8
