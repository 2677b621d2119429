// A pointwise convolution and the depthwise convolution that reads it (the first two of an inverted residual block) as one launch, bf16.
//
// A workgroup owns one image, a band of output rows and 32 channels.  The input pixels under the band (whole image rows, the halo of
// the window included) go into LDS by direct loads with the 32 weight rows, all requested at once, in blocks of ROWB bytes of K; each
// wave multiplies tiles of 32 positions, finishes them as the pointwise operator does (bias, activation, one rounding) and puts them
// into LDS, channels in rows, with a border of zeros where the window leaves the image.  The rows that the band owns go on to the
// pointwise operator's output tensor, the depthwise sums are formed from LDS.  The halo is computed twice: its products cost less
// than reading the wide tensor back (K is a sixth of it).
//
// What bounds it: with few images one round trip to memory and one wave's chain of instructions, which two launches paid twice; with many
// the vector instructions of the two epilogues and the window.  Us of the pair, two launches / here: one image 28x28 32->192 5.42 /
// 4.19, 14x14 64->384 5.33 / 4.28, 56x56 24->144 6.05 / 5.46, 7x7 160->960 5.62 / 5.10; 8 images 7.82 / 6.01, 6.49 / 5.19, -, 6.81 / 5.30; 32
// images 12.1 / 10.9, 9.44 / 7.72, -, 9.48 / 8.04.  What is left to two launches: see expand_dw_takes.  In fp32 the halo's products are not
// cheap and LDS holds half as many rows: 8 images 14x14 96->576 9.95 / 12.4, 56x56 24->144 16.0 / 28.2.
//
// Both operators keep their own arithmetic: one MFMA chain over ascending 32-byte k groups per slice of K (slices as slices_kernel has
// them, added in ascending order), then one FMA chain over the window, row-major from zero, the border multiplied like the rest.
#include <hip/hip_runtime.h>
#include <string>
#include "device_util.h"
#include "gemm_util.h"
#include "expand_geom.h"
#include "kernels.h"

namespace gacer {

struct ExpandArgs {
    const void *x, *w1, *w2;
    const float *b1, *b2;
    void *mid, *y;
    unsigned x_bytes, w1_bytes, w2_bytes, b1_bytes, b2_bytes;
    unsigned x_pitch, x_img, w1_pitch, k_bytes;    // bytes between input pixels, images, weight rows; bytes of K
    int H, W, Ho, Wo, C;
    int rows, bands, blocks;                       // output rows per band, bands per image, blocks of 32 channels
    int k_blocks, per;                             // blocks of K, of which a slice has `per`
    int tiles, n_lo;                               // tiles of 32 positions that a band fills at most, first image
    int act1, act2;
    unsigned mid_at;                               // LDS offset of the pointwise result
    unsigned div_w[2], div_blocks[2], div_bands[2], div_wt[2];
};

template <int KD, int S, int ROWB>
__global__ __launch_bounds__(256, 2) void expand_dw_kernel(ExpandArgs a)
{
    typedef unsigned short T;
    constexpr int ESZ = (int)sizeof(T), KC = ROWB / 16, SWZ = 256 / ROWB, RPL = 64 / KC, G = ROWB / 32, PAD = KD / 2;
    constexpr int PROW = ExpandGeom::PROW, CPR = 32 * ESZ / 16, ITER = 32 * CPR / 64;
    constexpr int TW = ExpandGeom::TW, NC = (TW - 1) * S + KD;
    extern __shared__ __align__(1024) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int own = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int t0 = div_by(own, a.div_blocks), n0 = __builtin_amdgcn_readfirstlane((own - t0 * a.blocks) * 32);
    const int t1 = div_by(t0, a.div_bands), band = __builtin_amdgcn_readfirstlane(t0 - t1 * a.bands);
    const int img = __builtin_amdgcn_readfirstlane(a.n_lo + t1);
    const int oh0 = band * a.rows, oh1 = min(oh0 + a.rows, a.Ho);                      // output rows of the band
    const int top = oh0 * S - PAD, ih0 = max(top, 0), ih1 = min((oh1 - 1) * S - PAD + KD, a.H);   // input rows under it
    const int P = (ih1 - ih0) * a.W, W2 = a.W + 2 * PAD;
    const __amdgpu_buffer_rsrc_t xr = rsrc_of(a.x, a.x_bytes), wr = rsrc_of(a.w1, a.w1_bytes), br = rsrc_of(a.b1, a.b1_bytes);
    const __amdgpu_buffer_rsrc_t dr = rsrc_of(a.w2, a.w2_bytes), cr = rsrc_of(a.b2, a.b2_bytes);
    const int a_block = a.tiles * 32 * ROWB;       // bytes of a K block of A
    unsigned char *As = smem, *Bs = smem + a.k_blocks * a_block, *mid = smem + a.mid_at;

    // a wave load fills RPL rows: lane l row l / KC, slot l % KC, which holds chunk (l % KC) ^ ((row / SWZ) % KC)
    const int lr = lane / KC;
    const unsigned x0 = (unsigned)img * a.x_img + (unsigned)(ih0 * a.W) * a.x_pitch;
    const int tiles = (P + 31) / 32;
    for (int kb = 0; kb < a.k_blocks; ++kb) {
        for (int l = wave; l < tiles * (32 / RPL); l += 4) {
            const int row = l * RPL + lr;
            const unsigned c = (unsigned)(kb * ROWB) + (unsigned)((lane % KC) ^ ((row / SWZ) % KC)) * 16u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GACER_LDS(As + kb * a_block + l * 1024), 16, (int)(c < a.k_bytes ? x0 + (unsigned)row * a.x_pitch + c : OOB), 0, 0, 0);
        }
        for (int l = wave; l < 32 / RPL; l += 4) {
            const int row = l * RPL + lr;
            const unsigned c = (unsigned)(kb * ROWB) + (unsigned)((lane % KC) ^ ((row / SWZ) % KC)) * 16u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, GACER_LDS(Bs + kb * 32 * ROWB + l * 1024), 16, (int)(c < a.k_bytes ? (unsigned)(n0 + row) * a.w1_pitch + c : OOB), 0, 0, 0);
        }
    }
    uint4 bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = buf_load16(br, (unsigned)(n0 + q * 8 + lhalf * 4) * 4u);
    // depthwise weights and bias of this thread's four channels
    const int cv = tid & 7, slot = tid >> 3;
    const unsigned c4 = (unsigned)(n0 + cv * 4);
    uint2 wraw[KD][KD];
#pragma unroll
    for (int r = 0; r < KD; ++r)
#pragma unroll
        for (int q = 0; q < KD; ++q) wraw[r][q] = buf_load8(dr, (int)c4 < a.C ? ((unsigned)((r * KD + q) * a.C) + c4) * ESZ : OOB);
    const uint4 dbias = buf_load16(cr, c4 * 4u);
    // the border: zeros left and right of every row, and whole rows above and below the image
    {
        const int lds_rows = (oh1 - oh0 - 1) * S + KD, c16 = PROW / 16;
        for (int i = tid; i < lds_rows * 2 * PAD * c16; i += 256) {
            const int px = i / c16, row = px / (2 * PAD), col = px - row * (2 * PAD);
            *(uint4 *)(mid + (row * W2 + (col < PAD ? col : a.W + col)) * PROW + (i - px * c16) * 16) = make_uint4(0u, 0u, 0u, 0u);
        }
        const int above = ih0 - top, below = lds_rows - above - (ih1 - ih0);
        for (int i = tid; i < (above + below) * W2 * c16; i += 256) {
            const int at = i < above * W2 * c16 ? i : i + (ih1 - ih0) * W2 * c16;
            *(uint4 *)(mid + at * 16) = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    __builtin_amdgcn_s_waitcnt((7 << 4));          // vmcnt(0), lgkmcnt(0)
    asm volatile("" ::: "memory");
    __syncthreads();

    const int sw = (lrow / SWZ) % KC;
    // rows of the pointwise output that this band stores
    const int own0 = oh0 * S, own1 = band == a.bands - 1 ? a.H : min(oh1 * S, a.H);
    const unsigned m_pitch = (unsigned)a.C * ESZ, m_img = (unsigned)img * (unsigned)(a.H * a.W) * m_pitch + (unsigned)n0 * ESZ;
    for (int t = wave; t < tiles; t += 4) {
        f32x16 sum;
        for (int kb = 0; kb < a.k_blocks;) {                                           // slices of K
            f32x16 acc;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.f;
            const int first = kb, end = min(kb + a.per, a.k_blocks);
            for (; kb < end; ++kb) {
                const unsigned char *fa0 = As + kb * a_block + (t * 32 + lrow) * ROWB, *fb0 = Bs + (kb * 32 + lrow) * ROWB;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int c = ((2 * g + lhalf) ^ sw) * 16;
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(fb0 + c), *(const bf16x8 *)(fa0 + c), acc, 0, 0, 0);
                }
            }
            mfma_settle<DT_BF16>();
            if (first == 0) {
                sum = acc;
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[e] = __fadd_rn(sum[e], acc[e]);
            }
        }
        float v[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[4 * q] = __fmaf_rn(sum[4 * q], 1.f, __uint_as_float(bias[q].x));
            v[4 * q + 1] = __fmaf_rn(sum[4 * q + 1], 1.f, __uint_as_float(bias[q].y));
            v[4 * q + 2] = __fmaf_rn(sum[4 * q + 2], 1.f, __uint_as_float(bias[q].z));
            v[4 * q + 3] = __fmaf_rn(sum[4 * q + 3], 1.f, __uint_as_float(bias[q].w));
        }
        act_vec<16>(v, a.act1);
        const int p = t * 32 + lrow, r = div_by(p, a.div_w);
        unsigned char *to = mid + ((ih0 - top + r) * W2 + PAD + p - r * a.W) * PROW + lhalf * (4 * ESZ);
        if (p < P) {
#pragma unroll
            for (int q = 0; q < 4; ++q) store_vec4((T *)(to + q * 8 * ESZ), v + 4 * q);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int idx = it * 64 + lane, pp = t * 32 + idx / CPR, ch = idx % CPR;
            const int pr = div_by(pp, a.div_w), ih = ih0 + pr, iw = pp - pr * a.W;
            if (pp < P && ih >= own0 && ih < own1 && n0 + ch * (16 / ESZ) < a.C)
                *(uint4 *)((char *)a.mid + (m_img + (unsigned)(ih * a.W + iw) * m_pitch + (unsigned)ch * 16u)) =
                    *(const uint4 *)(mid + ((ih - top) * W2 + PAD + iw) * PROW + ch * 16);
        }
    }
    __syncthreads();

    if ((int)c4 >= a.C) return;
    const int WT = (a.Wo + TW - 1) / TW, items = (oh1 - oh0) * WT;
    const float db[4] = {__uint_as_float(dbias.x), __uint_as_float(dbias.y), __uint_as_float(dbias.z), __uint_as_float(dbias.w)};
    const unsigned char *from0 = mid + cv * (4 * ESZ);
    for (int i = slot; i < items; i += 32) {
        const int oh = div_by(i, a.div_wt), ow = (i - oh * WT) * TW;
        const unsigned char *from = from0 + (oh * S * W2 + ow * S) * PROW;
        float acc[TW][4];
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t][e] = 0.f;
#pragma unroll
        for (int r = 0; r < KD; ++r) {
            float in[NC][4];
#pragma unroll
            for (int j = 0; j < NC; ++j) load_vec4((const T *)(from + (r * W2 + j) * PROW), in[j]);
#pragma unroll
            for (int q = 0; q < KD; ++q) {
                float wf[4];
                load_vec4((const T *)&wraw[r][q], wf);
#pragma unroll
                for (int t = 0; t < TW; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t][e] = __fmaf_rn(in[t * S + q][e], wf[e], acc[t][e]);
            }
        }
        if (a.b2_bytes) {
#pragma unroll
            for (int t = 0; t < TW; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] = __fadd_rn(acc[t][e], db[e]);
        }
        act_vec<TW * 4>(&acc[0][0], a.act2);
        T *out = (T *)a.y + (((unsigned)(img * a.Ho + oh0 + oh) * (unsigned)a.Wo + (unsigned)ow) * (unsigned)a.C + c4);
#pragma unroll
        for (int t = 0; t < TW; ++t)
            if (ow + t < a.Wo) store_vec4(out + (unsigned)(t * a.C), acc[t]);
    }
}

template <int KD, int S>
static LaunchInfo go(const GemmArgs &g, const StreamArgs &d, hipStream_t s, bool dry)
{
    constexpr int ESZ = 2;
    const ExpandGeom geo = expand_geometry(g, d);
    LaunchInfo li;
    li.workgroups = geo.workgroups;
    li.threads = 256;
    li.lds_bytes = geo.lds;
    li.wg_per_cu = 160 * 1024 / geo.lds < 8 ? 160 * 1024 / geo.lds : 8;
    static const std::string name = "expand_dw_bf16_" + std::to_string(KD) + "x" + std::to_string(KD) + "s" + std::to_string(S);
    li.kernel = name.c_str();
    li.phases = 1;
    if (dry || !li.workgroups) return li;
    ExpandArgs b;
    auto range = [](int64_t bytes) { return (unsigned)(bytes < 0 ? 0 : bytes > 0x7FFFFFFF ? 0x7FFFFFFF : bytes); };
    b.x = g.x; b.w1 = g.w; b.b1 = g.bias; b.mid = g.y;
    b.w2 = d.w; b.b2 = d.bias; b.y = d.y;
    b.x_bytes = range(g.x_bytes);
    b.w1_bytes = range(g.w_bytes);
    b.w2_bytes = (unsigned)(KD * KD * d.C * ESZ);
    b.b1_bytes = g.bias ? (unsigned)d.C * 4u : 0u;
    b.b2_bytes = d.bias ? (unsigned)d.C * 4u : 0u;
    b.x_pitch = (unsigned)(g.x_pix * ESZ);
    b.x_img = (unsigned)(g.x_img * ESZ);
    b.w1_pitch = (unsigned)(g.w_row * ESZ);
    b.k_bytes = (unsigned)(g.K * ESZ);
    b.H = d.H; b.W = d.W; b.Ho = d.Ho; b.Wo = d.Wo; b.C = d.C;
    b.rows = geo.rows; b.bands = geo.bands; b.blocks = geo.blocks;
    b.k_blocks = geo.k_blocks;
    b.per = g.kwaves ? g.kb_per_wave * 64 / geo.rowb : geo.k_blocks;       // a slice: kb_per_wave (an even number of) 64-byte blocks
    b.tiles = geo.tiles;
    b.n_lo = d.n_lo;
    b.act1 = g.act; b.act2 = d.act;
    b.mid_at = (unsigned)geo.mid_at;
    divisor(d.W, b.div_w);
    divisor(geo.blocks, b.div_blocks);
    divisor(geo.bands, b.div_bands);
    divisor((d.Wo + ExpandGeom::TW - 1) / ExpandGeom::TW, b.div_wt);
    const dim3 grid(li.workgroups), block(256);
    if (geo.rowb == 64) GACER_LAUNCH((expand_dw_kernel<KD, S, 64>), grid, block, geo.lds, s, b);
    else GACER_LAUNCH((expand_dw_kernel<KD, S, 128>), grid, block, geo.lds, s, b);
    return li;
}

LaunchInfo launch_expand_dw(const GemmArgs &g, const StreamArgs &d, hipStream_t s, bool dry)
{
    if (d.k == 3) return d.stride == 1 ? go<3, 1>(g, d, s, dry) : go<3, 2>(g, d, s, dry);
    return d.stride == 1 ? go<5, 1>(g, d, s, dry) : go<5, 2>(g, d, s, dry);
}

}  // namespace gacer
