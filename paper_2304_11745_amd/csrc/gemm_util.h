// Device helpers shared by the matrix-core kernels: element types, epilogue arithmetic, tile numbering over the XCDs.
#pragma once
#include "device_util.h"
#include "kernels.h"

// the address of a __shared__ object as the direct-to-LDS load builtins take it
#define GACER_LDS(p) ((__attribute__((address_space(3))) void *)(p))

namespace gacer {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf16_to_f32(unsigned short v) { return __uint_as_float(((unsigned)v) << 16); }
__device__ __forceinline__ unsigned short f32_to_bf16(float f)     // round to nearest even (hardware conversion)
{
    return __builtin_bit_cast(unsigned short, (__bf16)f);
}

// exact (erf) GELU; kept out of line so that the unrolled epilogues stay small
static __device__ __attribute__((noinline)) float gelu_erf(float v)
{
    return __fmul_rn(__fmul_rn(0.5f, v), __fadd_rn(1.f, erff(__fmul_rn(v, 0.70710678118654752440f))));
}

__device__ __forceinline__ float gelu_erf_inl(float v)
{
    return __fmul_rn(__fmul_rn(0.5f, v), __fadd_rn(1.f, erff(__fmul_rn(v, 0.70710678118654752440f))));
}

__device__ __forceinline__ float act_apply(float v, int act)
{
    if (act == ACT_RELU) return __builtin_fmaxf(v, 0.f);
    if (act == ACT_RELU6) return __builtin_amdgcn_fmed3f(v, 0.f, 6.f);
    if (act == ACT_GELU) return gelu_erf(v);
    if (act == ACT_HSWISH || act == ACT_HSIGMOID) return hard_act(v, act);
    return v;
}

template <int DT> struct El;
template <> struct El<DT_F32> { typedef float T; static constexpr int VEC = 4; };
template <> struct El<DT_BF16> { typedef unsigned short T; static constexpr int VEC = 8; };

template <typename T> __device__ __forceinline__ void store_out(T *y, int64_t o, float v);
template <> __device__ __forceinline__ void store_out<float>(float *y, int64_t o, float v) { y[o] = v; }
template <> __device__ __forceinline__ void store_out<unsigned short>(unsigned short *y, int64_t o, float v) { y[o] = f32_to_bf16(v); }
__device__ __forceinline__ float load_in(const float *p, int64_t o) { return p[o]; }
__device__ __forceinline__ float load_in(const unsigned short *p, int64_t o) { return bf16_to_f32(p[o]); }

// Activation of EV values; `act` is uniform over the launch, so the branch is taken once per vector.
template <int EV> __device__ __forceinline__ void act_vec(float *v, int act)
{
    if (act == ACT_RELU) {                        // clamps as single v_max / v_med3 instructions, no divergent branches
#pragma unroll
        for (int q = 0; q < EV; ++q) v[q] = __builtin_fmaxf(v[q], 0.f);
    } else if (act == ACT_RELU6) {
#pragma unroll
        for (int q = 0; q < EV; ++q) v[q] = __builtin_amdgcn_fmed3f(v[q], 0.f, 6.f);
    } else if (act == ACT_GELU) {
#pragma unroll
        for (int q = 0; q < EV; ++q) v[q] = gelu_erf(v[q]);
    } else if (act == ACT_HSWISH || act == ACT_HSIGMOID) {
#pragma unroll
        for (int q = 0; q < EV; ++q) v[q] = hard_act(v[q], act);
    }
}

// Epilogue of EV consecutive output channels of one row, all inside the launched range and 16-byte aligned:
// y = act(alpha * v + bias + res).  Bias and residual arrive preloaded (their loads are issued before the accumulators
// are turned through LDS, so that no global round trip sits between the last MFMA and the output store).
template <int DT>
__device__ __forceinline__ void finish_vec(const GemmArgs &a, float *v, const float *bv, bool has_res, const uint4 &rv,
                                           typename El<DT>::T *yg, int64_t o)
{
    constexpr int EV = DT == DT_BF16 ? 8 : 4;
#pragma unroll
    for (int q = 0; q < EV; ++q) v[q] = __fmaf_rn(v[q], a.alpha, bv[q]);
    if (has_res) {
        const unsigned rw[4] = {rv.x, rv.y, rv.z, rv.w};
        if constexpr (DT == DT_BF16) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[2 * q] = __fadd_rn(v[2 * q], __uint_as_float(rw[q] << 16));
                v[2 * q + 1] = __fadd_rn(v[2 * q + 1], __uint_as_float(rw[q] & 0xFFFF0000u));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = __fadd_rn(v[q], __uint_as_float(rw[q]));
        }
    }
    act_vec<EV>(v, a.act);
    if constexpr (DT == DT_BF16)
        *(uint4 *)(yg + o) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    else
        *(float4 *)(yg + o) = make_float4(v[0], v[1], v[2], v[3]);
}

// bias of EV consecutive channels (zeros without a bias pointer); n is a multiple of 4 and the pointer 16-byte aligned
template <int EV> __device__ __forceinline__ void load_bias_vec(const float *bias, int n, bool ok, float *bv)
{
#pragma unroll
    for (int q = 0; q < EV; ++q) bv[q] = 0.f;
    if (bias && ok) {
#pragma unroll
        for (int q = 0; q < EV; q += 4) {
            const float4 b4 = *(const float4 *)(bias + n + q);
            bv[q] = b4.x; bv[q + 1] = b4.y; bv[q + 2] = b4.z; bv[q + 3] = b4.w;
        }
    }
}

// four consecutive elements as floats, and back (8-byte vectors for bf16, 16-byte for fp32)
__device__ __forceinline__ void load_vec4(const float *p, float *v)
{
    const float4 t = *(const float4 *)p;
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load_vec4(const unsigned short *p, float *v)
{
    const uint2 t = *(const uint2 *)p;
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xFFFF0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xFFFF0000u);
}
__device__ __forceinline__ void store_vec4(float *p, const float *v) { *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void store_vec4(unsigned short *p, const float *v) { *(uint2 *)p = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])); }

// The arithmetic of a stand-alone per-channel affine operator on one 16-byte vector: one FMA, the clamp (none, ReLU or
// ReLU6), one rounding to the element type.
template <int DT> __device__ __forceinline__ uint4 affine_vec(uint4 x, const float *sc, const float *sh, int act)
{
    constexpr int VEC = El<DT>::VEC;
    float v[VEC];
    if constexpr (DT == DT_BF16) {
        const unsigned x4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) { v[2 * q] = __uint_as_float(x4[q] << 16); v[2 * q + 1] = __uint_as_float(x4[q] & 0xFFFF0000u); }
    } else {
        v[0] = __uint_as_float(x.x); v[1] = __uint_as_float(x.y); v[2] = __uint_as_float(x.z); v[3] = __uint_as_float(x.w);
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
        const float t = __fmaf_rn(v[q], sc[q], sh[q]);
        v[q] = act == ACT_RELU ? __builtin_fmaxf(t, 0.f) : act == ACT_RELU6 ? __builtin_amdgcn_fmed3f(t, 0.f, 6.f) : t;
    }
    if constexpr (DT == DT_BF16) return make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    else return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
}

// Ragged or unaligned tail: element by element (rare: odd channel counts, unaligned channel chunks).
template <int DT>
__device__ __noinline__ void finish_one(float v, float alpha, const float *bias, int act, const typename El<DT>::T *rg,
                                        typename El<DT>::T *yg, int64_t o, int n, int n_hi)
{
    if (n >= n_hi) return;
    float t = __fmaf_rn(v, alpha, bias ? bias[n] : 0.f);
    if (rg) t = __fadd_rn(t, load_in(rg, o));
    // leaf function (no nested call, hence no stack): the activation is expanded in place
    if (act == ACT_RELU) t = __builtin_fmaxf(t, 0.f);
    else if (act == ACT_RELU6) t = __builtin_amdgcn_fmed3f(t, 0.f, 6.f);
    else if (act == ACT_GELU) t = gelu_erf_inl(t);
    else if (act == ACT_HSWISH || act == ACT_HSIGMOID) t = hard_act(t, act);
    store_out<typename El<DT>::T>(yg, o, t);
}
template <int DT>
__device__ __forceinline__ void finish_scalar(const GemmArgs &a, const float *v, const typename El<DT>::T *rg, typename El<DT>::T *yg, int64_t o, int n)
{
    constexpr int EV = DT == DT_BF16 ? 8 : 4;
#pragma unroll
    for (int q = 0; q < EV; ++q) finish_one<DT>(v[q], a.alpha, a.bias, a.act, rg, yg, o + q, n + q, a.n_hi);
}

// Workgroups are handed to the 8 XCDs round-robin by their index, and each XCD has its own L2.  Neighbouring tiles share
// operand rows (the halo of a k x k window, the A rows of tiles that differ only in n, the B rows of tiles that differ
// only in m), so tile numbers are dealt such that every XCD works on one contiguous run of them: workgroup b -> XCD
// b % 8 -> the (b / 8)-th tile of that XCD's run.  Whether the runs are bands of m or bands of n is tile_order()'s choice.
__device__ __forceinline__ int xcd_contiguous(int b, int n)
{
    const int q = n >> 3, r = n & 7, x = b & 7;
    return __builtin_amdgcn_readfirstlane(x * q + min(x, r) + (b >> 3));
}

}  // namespace gacer
