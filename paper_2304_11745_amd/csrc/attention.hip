// Attention of one head as one launch: scores = alpha * Q K^T, probabilities = softmax(scores), context = probabilities * V, each
// tensor rounded to bf16 and written, with the bits of the three stand-alone kernels.
//
// A workgroup owns 32 queries of one head.  Q and all K rows go into LDS by direct loads (128-byte rows, swizzled as in
// slices_kernel), V through registers into a transposed copy (the product over V wants eight consecutive keys per lane).  Scores of 32x32
// tiles are formed with swapped operands, so that a lane holds four consecutive keys of one query, and stay in LDS; each row is
// normalised in place by 16 lanes, and two waves multiply with V.  The arithmetic is that of the stand-alone
// operators: one MFMA chain over ascending 32-byte k groups, the softmax of softmax_vec_kernel (more lanes than it uses add exact zeros), a
// chain over the keys.
//
// What bounds it: the length of one wave's chain around one round trip to memory, which three launches paid three times.  A layer of
// BERT's round, us less than with three launches: 1 image of 16 tokens 4.9, 2 of 72 6.2, 8 of 128 6.0, 32 of 128 7.6, 64 of 64 7.3.
// Up to 128 keys: with room for 256 in LDS one workgroup fits a unit and K and V are read once per 32 queries (4 images of 200 tokens
// 1.1 us more than three launches, 16 of 256 15.5 us more).
#include <hip/hip_runtime.h>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"

namespace gacer {

struct AttnKernelArgs {
    const void *qkv;
    void *scores, *probs, *ctx;
    unsigned qkv_bytes;
    int S, heads, tiles, z_lo;         // keys, heads, query tiles per head, first image
    float alpha;
    unsigned div_tiles[2], div_heads[2];
};

__global__ __launch_bounds__(256) void attention_kernel(AttnKernelArgs a)
{
    constexpr int SMAX = ATTENTION_KEYS_MAX;
    constexpr int PROW = SMAX * 2 + 16;                // bytes of a row of scores and of the transposed V: 4 banks on from row to row
    constexpr int G = SMAX / 8, RPW = 64 / G;          // lanes per row of the softmax, rows per pass of a wave
    constexpr int VIT = SMAX / 64;                     // V items (two keys x eight features) per thread
    __shared__ __align__(1024) unsigned char qs[32 * 128];
    __shared__ __align__(1024) unsigned char ks[SMAX * 128];
    __shared__ __align__(16) unsigned char vt[64 * PROW];
    __shared__ __align__(16) unsigned char ps[32 * PROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int z = div_by((int)blockIdx.x, a.div_tiles), q0 = ((int)blockIdx.x - z * a.tiles) * 32;
    const int zi = div_by(z, a.div_heads), head = z - zi * a.heads, img = a.z_lo + zi;
    const unsigned S = (unsigned)a.S, D2 = (unsigned)a.heads * 128u, pitch = 3u * D2;        // bytes: one of q / k / v, one row of qkv
    const __amdgpu_buffer_rsrc_t r = rsrc_of(a.qkv, a.qkv_bytes);
    const unsigned base = (unsigned)img * S * pitch + (unsigned)head * 128u;

    // a wave load fills eight rows: lane l row l / 8, slot l % 8, which holds chunk (l % 8) ^ ((row / 2) % 8)
    const int frow = lane >> 3;
    const unsigned chunk[2] = {(unsigned)((lane & 7) ^ (lane >> 4)) * 16u, (unsigned)((lane & 7) ^ (lane >> 4) ^ 4) * 16u};   // by the parity of the load
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, GACER_LDS(qs + wave * 1024), 16, (int)(base + (unsigned)(q0 + wave * 8 + frow) * pitch + chunk[wave & 1]), 0, 0, 0);
    const int key_tiles = (a.S + 31) / 32;
    for (int l = wave; l < key_tiles * 4; l += 4)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, GACER_LDS(ks + l * 1024), 16, (int)(base + D2 + (unsigned)(l * 8 + frow) * pitch + chunk[wave & 1]), 0, 0, 0);
    uint4 v0[VIT], v1[VIT];                            // keys 2 j and 2 j + 1, features 8 c .. 8 c + 7; beyond the keys zeros
#pragma unroll
    for (int u = 0; u < VIT; ++u) {
        const unsigned item = (unsigned)(u * 256 + tid), j2 = item >> 3 << 1, at = base + 2u * D2 + j2 * pitch + (item & 7u) * 16u;
        v0[u] = buf_load16(r, j2 < S ? at : OOB);
        v1[u] = buf_load16(r, j2 + 1u < S ? at + pitch : OOB);
    }
#pragma unroll
    for (int u = 0; u < VIT; ++u) {
        const unsigned item = (unsigned)(u * 256 + tid), j = item >> 3, c = item & 7u;
        const unsigned lo[4] = {v0[u].x, v0[u].y, v0[u].z, v0[u].w}, hi[4] = {v1[u].x, v1[u].y, v1[u].z, v1[u].w};
        if (j * 2u >= (S + 15u) / 16u * 16u) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            *(unsigned *)(vt + (c * 8u + 2u * q) * PROW + j * 4u) = (lo[q] & 0xFFFFu) | (hi[q] << 16);
            *(unsigned *)(vt + (c * 8u + 2u * q + 1u) * PROW + j * 4u) = (lo[q] >> 16) | (hi[q] & 0xFFFF0000u);
        }
    }
    __builtin_amdgcn_s_waitcnt((7 << 4));              // vmcnt(0), lgkmcnt(0)
    asm volatile("" ::: "memory");
    __syncthreads();

    const int sw = (lrow >> 1) & 7;
    bf16x8 fq[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) fq[g] = *(const bf16x8 *)(qs + lrow * 128 + (((2 * g + lhalf) ^ sw) * 16));
    for (int t = wave; t < key_tiles; t += 4) {
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(ks + (t * 32 + lrow) * 128 + (((2 * g + lhalf) ^ sw) * 16)), fq[g], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __fmaf_rn(acc[4 * q + e], a.alpha, 0.f);
            store_vec4((unsigned short *)(ps + lrow * PROW + (t * 32 + q * 8 + lhalf * 4) * 2), v);
        }
    }
    __syncthreads();

    // softmax of rows 8 wave .. 8 wave + 7; a lane holds eight keys
    const int sub = lane % G;
    const bool ok = sub * 8 < a.S;
#pragma unroll
    for (int p = 0; p < 8 / RPW; ++p) {
        const int row = wave * 8 + p * RPW + lane / G;
        unsigned char *at = ps + row * PROW + sub * 16;
        Vec<unsigned short, 8> x;
        x.raw = *(const uint4 *)at;
        float e[8], m = -INFINITY;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            e[q] = ok ? x.get(q) : -INFINITY;
            m = fmaxf(m, e[q]);
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            e[q] = ok ? expf(__fsub_rn(e[q], m)) : 0.f;
            s = __fadd_rn(s, e[q]);
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) s = __fadd_rn(s, __shfl_xor(s, o, 64));
        Vec<unsigned short, 8> y;
        y.raw = make_uint4(0u, 0u, 0u, 0u);            // beyond the keys: zeros for the padded end of the chain over them
        if (ok) {
#pragma unroll
            for (int q = 0; q < 8; ++q) y.set(q, __fdiv_rn(e[q], s));
        }
        *(uint4 *)at = y.raw;
        if (ok && q0 + row < a.S) {
            const unsigned o = (((unsigned)(img * a.heads + head) * S + (unsigned)(q0 + row)) * S + (unsigned)(sub * 8)) * 2u;
            *(uint4 *)((char *)a.scores + o) = x.raw;
            *(uint4 *)((char *)a.probs + o) = y.raw;
        }
    }
    __syncthreads();

    if (wave >= 2) return;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const int groups = (a.S + 15) / 16;
    const unsigned char *va = vt + (wave * 32 + lrow) * PROW + lhalf * 16, *pa = ps + lrow * PROW + lhalf * 16;
    for (int g = 0; g < groups; ++g) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(va + g * 32), *(const bf16x8 *)(pa + g * 32), acc, 0, 0, 0);
    if (q0 + lrow >= a.S) return;
    char *o = (char *)a.ctx + (((unsigned)img * S + (unsigned)(q0 + lrow)) * D2 + (unsigned)(head * 128 + wave * 64 + lhalf * 8));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        store_vec4((unsigned short *)(o + q * 16), v);
    }
}

LaunchInfo launch_attention(const GemmArgs &a, hipStream_t s, bool dry)
{
    constexpr int SMAX = ATTENTION_KEYS_MAX;
    const int tiles = (a.H + 31) / 32;
    LaunchInfo li;
    li.workgroups = tiles * a.zh * a.zb;
    li.threads = 256;
    li.lds_bytes = 4096 + SMAX * 128 + 96 * (SMAX * 2 + 16);
    li.wg_per_cu = 160 * 1024 / li.lds_bytes;
    li.kernel = "attention_bf16";
    li.phases = 1;
    if (dry || !li.workgroups) return li;
    AttnKernelArgs b;
    b.qkv = a.x; b.scores = a.attn_scores; b.probs = a.attn_probs; b.ctx = a.y;
    b.qkv_bytes = (unsigned)a.x_bytes;
    b.S = a.H; b.heads = a.zh; b.tiles = tiles; b.z_lo = a.z_lo; b.alpha = a.alpha;
    divisor(tiles, b.div_tiles);
    divisor(a.zh, b.div_heads);
    GACER_LAUNCH(attention_kernel, dim3(li.workgroups), dim3(256), 0, s, b);
    return li;
}

}  // namespace gacer
