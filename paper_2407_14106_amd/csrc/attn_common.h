// Helpers shared by the attention kernels: per-lane feature slices of bf16 or
// fp32 rows, dot products with fp32 accumulation, and the (dtype, d, H)
// dispatch.
#pragma once

#include "common.h"

namespace gt {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// exp2 as the hardware gives it (v_exp_f32: results below 2^-126 become 0).
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// Lane layout of the edge kernels: each (node, head) is owned by L = D / F
// consecutive lanes, each holding F features (32 bytes; 64 of fp32 where the
// node's features would not fit one wavefront otherwise), which keeps the
// per-lane register footprint small enough for several resident wavefronts
// per SIMD to overlap their gathers.  A bf16 lane's features are consecutive.
// An fp32 lane's come in 16-byte pieces dealt round-robin over the L lanes: a
// run of 64 bytes a lane has each of its four loads touch every cache line of
// a row (gathering 512-byte rows of a clustered graph: 14.2 TB/s in runs of 64
// bytes, 19.9 TB/s dealt; with 32 bytes a lane 20.3 and 20.7 TB/s, and the column
// pass measured 4% slower dealt, so bf16 keeps its runs).
template <typename T, int D, int H>
struct EdgeCfg {
    static constexpr int F = sizeof(T) == 4 && H * D / 8 <= kWave ? 8 : 16;  // features per lane
    static constexpr int L = D / F;                     // lanes per (node, head)
    static constexpr int G = H * L;                     // lanes per node
    static constexpr int NPW = kWave / G;               // nodes per wavefront
    static constexpr int RUN = sizeof(T) == 4 ? 4 : F;  // consecutive features of a lane
    static constexpr int STR = L * RUN;                 // features between a lane's runs
    static_assert(D % F == 0 && F % RUN == 0 && G <= kWave && kWave % G == 0, "unsupported (d, H)");
};

// F features of one row slice, stored packed as loaded: a run of 16 (bf16), or
// runs of 4 features STR apart (fp32).
template <typename T, int F, int STR>
struct Slice;

template <int F, int STR>
struct Slice<uint16_t, F, STR> {
    uint32_t w[F / 2];
    __device__ __forceinline__ void load(const uint16_t* p) {
#pragma unroll
        for (int i = 0; i < F / 8; ++i) {
            const uint4 v = *reinterpret_cast<const uint4*>(p + 8 * i);
            w[4 * i + 0] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
    __device__ __forceinline__ float f(int i) const { return (i & 1) ? bf16hi(w[i >> 1]) : bf16lo(w[i >> 1]); }
    __device__ __forceinline__ float dot(const Slice& o) const {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int i = 0; i < F / 2; i += 2) {
            a0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[i]),
                                                 __builtin_bit_cast(bf16x2_t, o.w[i]), a0, false);
            a1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w[i + 1]),
                                                 __builtin_bit_cast(bf16x2_t, o.w[i + 1]), a1, false);
        }
        return a0 + a1;
    }
    // acc[2i] += p * lo(w[i]), acc[2i+1] += p * hi(w[i]) with p given as the
    // bf16 pairs (p, 0) and (0, p): one dot2 per element, no conversion.
    __device__ __forceinline__ void axpy_w(float (&acc)[F], uint32_t p_lo, uint32_t p_hi) const {
#pragma unroll
        for (int i = 0; i < F / 2; ++i) {
            const bf16x2_t x = __builtin_bit_cast(bf16x2_t, w[i]);
            acc[2 * i] = __builtin_amdgcn_fdot2_f32_bf16(x, __builtin_bit_cast(bf16x2_t, p_lo), acc[2 * i], false);
            acc[2 * i + 1] =
                __builtin_amdgcn_fdot2_f32_bf16(x, __builtin_bit_cast(bf16x2_t, p_hi), acc[2 * i + 1], false);
        }
    }
};

template <int F, int STR>
struct Slice<float, F, STR> {
    float w[F];
    __device__ __forceinline__ void load(const float* p) {
#pragma unroll
        for (int i = 0; i < F / 4; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(p + i * STR);
            w[4 * i + 0] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
    __device__ __forceinline__ float f(int i) const { return w[i]; }
    __device__ __forceinline__ float dot(const Slice& o) const {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int i = 0; i < F; i += 2) {
            a0 = fmaf(w[i], o.w[i], a0);
            a1 = fmaf(w[i + 1], o.w[i + 1], a1);
        }
        return a0 + a1;
    }
};

template <typename T, int D, int H>
using SliceOf = Slice<T, EdgeCfg<T, D, H>::F, EdgeCfg<T, D, H>::STR>;

// Store a lane's F fp32 values, times scale, as T (bf16: round to nearest
// even), laid out like Slice.
template <typename T, int F, int STR>
__device__ __forceinline__ void store_slice(T* p, const float (&v)[F], float scale) {
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < F / 8; ++i) {
            uint4 o;
            o.x = pack_bf16x2(v[8 * i + 0] * scale, v[8 * i + 1] * scale);
            o.y = pack_bf16x2(v[8 * i + 2] * scale, v[8 * i + 3] * scale);
            o.z = pack_bf16x2(v[8 * i + 4] * scale, v[8 * i + 5] * scale);
            o.w = pack_bf16x2(v[8 * i + 6] * scale, v[8 * i + 7] * scale);
            *reinterpret_cast<uint4*>(p + 8 * i) = o;
        }
    } else {
#pragma unroll
        for (int i = 0; i < F / 4; ++i)
            *reinterpret_cast<float4*>(p + i * STR) =
                make_float4(v[4 * i] * scale, v[4 * i + 1] * scale, v[4 * i + 2] * scale, v[4 * i + 3] * scale);
    }
}

// Sum over the L lanes (2, 4 or 8) that share one (node, head): DPP exchanges
// inside a quad (xor 1, xor 2), then the mirrored lane of the other quad; every
// lane of a group is active whenever one is.
template <int Ctrl>
__device__ __forceinline__ float dpp_f32(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), Ctrl, 0xF, 0xF, true));
}
template <int L>
__device__ __forceinline__ float group_sum(float x) {
    static_assert(L == 2 || L == 4 || L == 8, "lanes per (node, head)");
    x += dpp_f32<0xB1>(x);                           // quad_perm 1,0,3,2
    if constexpr (L >= 4) x += dpp_f32<0x4E>(x);     // quad_perm 2,3,0,1
    if constexpr (L >= 8) x += dpp_f32<0x141>(x);    // row_half_mirror
    return x;
}

}  // namespace gt

// Dispatch a templated launcher over (dtype, d, H).  FN<T, D, H>(args...) must
// return gt_status.
#define GT_DISPATCH_ATTN(dtype, d, H, FN, ...)                                               \
    [&]() -> gt_status {                                                                     \
        if ((dtype) == GT_BF16) {                                                            \
            if ((d) == 32) {                                                                 \
                switch (H) {                                                                 \
                    case 1: return FN<uint16_t, 32, 1>(__VA_ARGS__);                         \
                    case 2: return FN<uint16_t, 32, 2>(__VA_ARGS__);                         \
                    case 4: return FN<uint16_t, 32, 4>(__VA_ARGS__);                         \
                    case 8: return FN<uint16_t, 32, 8>(__VA_ARGS__);                         \
                    case 16: return FN<uint16_t, 32, 16>(__VA_ARGS__);                       \
                }                                                                            \
            } else if ((d) == 64) {                                                          \
                switch (H) {                                                                 \
                    case 1: return FN<uint16_t, 64, 1>(__VA_ARGS__);                         \
                    case 2: return FN<uint16_t, 64, 2>(__VA_ARGS__);                         \
                    case 4: return FN<uint16_t, 64, 4>(__VA_ARGS__);                         \
                    case 8: return FN<uint16_t, 64, 8>(__VA_ARGS__);                         \
                    case 16: return FN<uint16_t, 64, 16>(__VA_ARGS__);                       \
                }                                                                            \
            }                                                                                \
        } else if ((dtype) == GT_F32) {                                                      \
            if ((d) == 32) {                                                                 \
                switch (H) {                                                                 \
                    case 1: return FN<float, 32, 1>(__VA_ARGS__);                            \
                    case 2: return FN<float, 32, 2>(__VA_ARGS__);                            \
                    case 4: return FN<float, 32, 4>(__VA_ARGS__);                            \
                    case 8: return FN<float, 32, 8>(__VA_ARGS__);                            \
                    case 16: return FN<float, 32, 16>(__VA_ARGS__);                          \
                }                                                                            \
            } else if ((d) == 64) {                                                          \
                switch (H) {                                                                 \
                    case 1: return FN<float, 64, 1>(__VA_ARGS__);                            \
                    case 2: return FN<float, 64, 2>(__VA_ARGS__);                            \
                    case 4: return FN<float, 64, 4>(__VA_ARGS__);                            \
                    case 8: return FN<float, 64, 8>(__VA_ARGS__);                            \
                    case 16: return FN<float, 64, 16>(__VA_ARGS__);                          \
                }                                                                            \
            }                                                                                \
        }                                                                                    \
        return gt::fail(GT_ERR_UNSUPPORTED, "attention: unsupported (dtype, d, H)");         \
    }()
