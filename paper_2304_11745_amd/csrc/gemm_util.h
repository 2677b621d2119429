// Device helpers shared by the matrix-core kernels: element types, epilogue arithmetic, tile numbering over the XCDs.
#pragma once
#include <type_traits>
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
static inline __device__ __attribute__((noinline)) float gelu_erf(float v)
{
    return __fmul_rn(__fmul_rn(0.5f, v), __fadd_rn(1.f, erff(__fmul_rn(v, 0.70710678118654752440f))));
}

__device__ __forceinline__ float gelu_erf_inl(float v)
{
    return __fmul_rn(__fmul_rn(0.5f, v), __fadd_rn(1.f, erff(__fmul_rn(v, 0.70710678118654752440f))));
}

template <int DT> struct El;
template <> struct El<DT_F32> { typedef float T; static constexpr int VEC = 4; };
template <> struct El<DT_BF16> { typedef unsigned short T; static constexpr int VEC = 8; };

// The wait states that the result of a 32x32 MFMA takes (its passes and two more, bf16 another two).  hipcc puts them in front of whatever
// reads or overwrites the result first, but where several ways lead on from a loop of MFMAs it has counted one to three too few on one of
// them; so they stand behind such loops.
template <int DT> __device__ __forceinline__ void mfma_settle()
{
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DT == DT_BF16) asm volatile("s_nop 11");
    else asm volatile("s_nop 15\n\ts_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}

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

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000);
}

// `width` bits from bit `at` on (none for width <= 0, whatever `at`)
__device__ __forceinline__ unsigned bit_run(int width, int at) { return width > 0 ? ((1u << width) - 1u) << at : 0u; }

// One bit per tap (bit r * kw + q, kh * kw <= 31) of a window whose origin is (ih0, iw0), set where the tap lies in the image.
// `rows`: bit r * kw of every tap row r (tap_rows).
__device__ __forceinline__ unsigned taps_inside(int ih0, int iw0, int H, int W, int kh, int kw, unsigned rows)
{
    const int r0 = max(-ih0, 0), r1 = min(H - ih0, kh), q0 = max(-iw0, 0), q1 = min(W - iw0, kw);
    return bit_run(q1 - q0, q0) * (rows & bit_run((r1 - r0) * kw, r0 * kw));
}
inline unsigned tap_rows(int kh, int kw)
{
    unsigned rows = 0;
    for (int r = 0; r < kh && r * kw < 31; ++r) rows |= 1u << (r * kw);
    return rows;
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

// ---- epilogue of the tiled kernels ----
// The kernels hand the weights to the MFMA as its first operand: element e of a 32x32 tile is then row lane % 32 and channel
// (e / 4) * 8 + (lane / 32) * 4 + e % 4, i.e. a lane owns one output row and four consecutive channels at a time.  Bias and
// residual are read in that layout, all at once (turned through LDS as fp32 first, each tile waited for its own), the finished
// elements pass through the wave's patch of LDS (4608 bytes) in their own type, two bf16 tiles side by side where there are two,
// and are stored as 16-byte vectors along the channels; the residual comes the same way back.  (Before, fp32 accumulators were
// turned through LDS and each 32x32 tile waited for its own bias and residual.)  One launch, us, before / with this and 32-bit
// addresses: bf16 16x56x56 256->128 14.6 / 12.5, 32x28x28 512->128 13.6 / 11.7, 32x28x28 128->128 3x3 17.5 / 14.8, 64x7x7 320->1280 11.8 /
// 9.9, 16x28x28 128->512 with a residual 11.2 / 10.3; fp32 8x14x14 96->576 6.8 / 6.1, 8x112x112 64->128 3x3 132 / 129.
// `row_at(i, r, pos)` gives the output position of row r of row tile i and whether it is stored; rows_inside: all of them are.
// RES: 0 no residual, 1 a residual, 2 to be seen at run time
template <int DT, int TM, int TN, int RES, typename RowAt>
__device__ __forceinline__ void store_tiles_as(const GemmArgs &a, f32x16 (&acc)[TM][TN], unsigned char *patch, int n_wave, int lane, unsigned y_off,
                                            bool rows_inside, RowAt row_at)
{
    typedef typename El<DT>::T T;
    constexpr int ESZ = (int)sizeof(T), VE = 16 / ESZ;
    constexpr int JT = DT == DT_BF16 && TN % 2 == 0 ? 2 : 1;                    // tiles side by side in the patch
    constexpr int PROW = JT * 32 * ESZ + 16;
    constexpr int CPR = JT * 32 / VE, ITER = 32 * CPR / 64;
    static_assert(32 * PROW <= 4608, "patch");
    typedef typename std::conditional<DT == DT_BF16, uint2, uint4>::type R;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const unsigned y_row = (unsigned)a.y_row;
    const bool vec = y_row % VE == 0 && a.n_lo % VE == 0 && y_off % VE == 0 && ((uintptr_t)a.y & 15) == 0;
    // a vector that reaches over the end of a descriptor's range would read as zero
    const bool bias_vec = a.n_lo % 4 == 0 && a.n_hi % 4 == 0 && ((uintptr_t)a.bias & 15) == 0;
    const bool res_vec = vec && a.n_hi % VE == 0 && ((uintptr_t)a.res & 15) == 0;
    const __amdgpu_buffer_rsrc_t br = rsrc_of(a.bias, a.bias ? (unsigned)a.n_hi * 4u : 0u), rr = rsrc_of(a.res, 0x7FFFFFFFu);
    uint4 bias[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned bo = (unsigned)(n_wave + j * 32 + q * 8 + lhalf * 4) * 4u;
            if (bias_vec) {
                bias[j][q] = buf_load16(br, bo);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) ((float *)&bias[j][q])[e] = buf_load1<float>(br, bo + 4u * e);
            }
        }
    constexpr int PASSES = TN / JT;
    uint4 res[TM][PASSES][ITER];                // requested one row tile ahead
    auto request_res = [&](int i) {
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int idx = it * 64 + lane;
            unsigned pos;
            const bool ok = row_at(i, idx / CPR, pos);
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                const int n = n_wave + p * JT * 32 + idx % CPR * VE;
                res[i][p][it] = buf_load16(rr, ok && n < a.n_hi ? (pos * y_row + (unsigned)n + y_off) * ESZ : OOB);
            }
        }
    };
    const bool has_res = RES == 2 ? a.res != nullptr : RES == 1;
    if (has_res && res_vec) request_res(0);
    const bool inside = rows_inside && vec && n_wave + TN * 32 <= a.n_hi;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM && has_res && res_vec) request_res(i + 1);
        unsigned out[ITER];                     // byte offset of the lane's vectors, without the channel of the pass
        bool ok[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int idx = it * 64 + lane;
            unsigned pos;
            ok[it] = row_at(i, idx / CPR, pos);
            out[it] = (pos * y_row + (unsigned)(n_wave + idx % CPR * VE) + y_off) * ESZ;
        }
#pragma unroll
        for (int j0 = 0; j0 < TN; j0 += JT) {
            R rl[JT][4];                        // residual in the accumulators' layout
            if (has_res) {
                if (res_vec) {
#pragma unroll
                    for (int it = 0; it < ITER; ++it) *(uint4 *)(patch + (it * 64 + lane) / CPR * PROW + (it * 64 + lane) % CPR * 16) = res[i][j0 / JT][it];
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int j = 0; j < JT; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) rl[j][q] = *(const R *)(patch + lrow * PROW + (j * 32 + q * 8 + lhalf * 4) * ESZ);
                    __builtin_amdgcn_wave_barrier();
                } else {
                    unsigned pos;
                    const bool row_ok = row_at(i, lrow, pos);
#pragma unroll
                    for (int j = 0; j < JT; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int n = n_wave + (j0 + j) * 32 + q * 8 + lhalf * 4 + e;
                                ((T *)&rl[j][q])[e] = buf_load1<T>(rr, row_ok && n < a.n_hi ? (pos * y_row + (unsigned)n + y_off) * ESZ : OOB);
                            }
                }
            }
#pragma unroll
            for (int j = j0; j < j0 + JT; ++j) {
                float v[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[4 * q] = __fmaf_rn(acc[i][j][4 * q], a.alpha, __uint_as_float(bias[j][q].x));
                    v[4 * q + 1] = __fmaf_rn(acc[i][j][4 * q + 1], a.alpha, __uint_as_float(bias[j][q].y));
                    v[4 * q + 2] = __fmaf_rn(acc[i][j][4 * q + 2], a.alpha, __uint_as_float(bias[j][q].z));
                    v[4 * q + 3] = __fmaf_rn(acc[i][j][4 * q + 3], a.alpha, __uint_as_float(bias[j][q].w));
                }
                if (has_res) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float r[4];
                        load_vec4((const T *)&rl[j - j0][q], r);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[4 * q + e] = __fadd_rn(v[4 * q + e], r[e]);
                    }
                }
                act_vec<16>(v, a.act);
#pragma unroll
                for (int q = 0; q < 4; ++q) store_vec4((T *)(patch + lrow * PROW + ((j - j0) * 32 + q * 8 + lhalf * 4) * ESZ), v + 4 * q);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int idx = it * 64 + lane, n = n_wave + j0 * 32 + idx % CPR * VE;
                const unsigned char *from = patch + idx / CPR * PROW + idx % CPR * 16;
                char *to = (char *)a.y + (out[it] + (unsigned)(j0 * 32 * ESZ));
                if (inside) {
                    *(uint4 *)to = *(const uint4 *)from;
                } else if (ok[it] && n < a.n_hi) {
                    if (vec && n + VE <= a.n_hi) {
                        *(uint4 *)to = *(const uint4 *)from;
                    } else {
                        for (int e = 0; e < VE; ++e)
                            if (n + e < a.n_hi) ((T *)to)[e] = ((const T *)from)[e];
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

template <int DT, int TM, int TN, typename RowAt>
__device__ __forceinline__ void store_tiles(const GemmArgs &a, f32x16 (&acc)[TM][TN], unsigned char *patch, int n_wave, int lane, unsigned y_off,
                                            bool rows_inside, RowAt row_at)
{
    // one tile per wave: code of its own for each; with more tiles two copies cost registers (bf16 128x128: a wave per SIMD, 12.3 -> 15.7 us)
    if constexpr (TM * TN > 1) store_tiles_as<DT, TM, TN, 2>(a, acc, patch, n_wave, lane, y_off, rows_inside, row_at);
    else if (a.res) store_tiles_as<DT, TM, TN, 1>(a, acc, patch, n_wave, lane, y_off, rows_inside, row_at);
    else store_tiles_as<DT, TM, TN, 0>(a, acc, patch, n_wave, lane, y_off, rows_inside, row_at);
}

}  // namespace gacer
