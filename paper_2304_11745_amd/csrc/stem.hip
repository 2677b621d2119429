// Convolutions whose channels do not fill a 16-byte vector (the 3-channel stems of image networks).
//
// A K row of such a convolution is kh short runs: the kw x Cin values under one tap row are contiguous in the channels-last
// image.  Each run is padded to whole 16-byte chunks (7x7x3 bf16: 21 values in 3 chunks), a k group of the matrix
// instruction takes one chunk per lane half, and the run is read from LDS as it lies in the image: a workgroup copies the
// input rows under its 128 output positions into an LDS strip (16-byte loads, zeros for what lies outside the image), keeps
// all weights beside it in the same chunk order, and walks several tiles so that the weights are laid out once.
//
// The weights are the first operand of the product, so a lane ends up with 16 channels of one output position; two
// permlane32 swaps per 32 channels turn them into whole 16-byte vectors.
//
// What bounds it: instruction issue -- about 900 instructions per wave and tile for staging, fragments and epilogue, which is
// why the tile loop has no calls and takes its arguments in a struct small enough for the scalar registers -- and in fp32 the
// matrix cores.  Gathering every element with a load of its own, as the generic loader of igemm_kernel does, is bound by the
// address unit.  Measured there / here, microseconds, 224x224 images: 64x7x7x3 stride 2 bf16, 16 images 55.4 / 21.7; 64x3x3x3
// bf16, 8 images 37.5 / 20.0; 32x3x3x3 stride 2 bf16, 32 images 29.3 / 18.0; 64x11x11x3 stride 4 bf16, 8 images 33.2 / 13.1;
// 64x7x7x3 fp32, 8 images 45.5 / 37.7; 64x3x3x3 fp32, 8 images 47.5 / 38.0.
//
// An output element is one MFMA chain over its tap rows in ascending order; which kernel an operator takes depends on its
// unsplit shape only, so every chunk of it adds alike.
#include <hip/hip_runtime.h>
#include <string>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"
#include "stem_geom.h"

namespace gacer {

static constexpr int STEM_THREADS = 256;
static constexpr int STEM_PATCH_ROW = 128 + 16, STEM_PATCH = 32 * STEM_PATCH_ROW;      // LDS of one wave's epilogue

// What the kernel needs of GemmArgs and StemGeom: few enough values to stay in scalar registers.
struct StemArgs {
    const void *x, *w, *res;
    const float *bias;
    void *y;
    int x_bytes, w_bytes;
    int H, Wo, HoWo, WC, Cin, run, kh, stride, pad;
    int y_row, img_lo, n_lo, n_hi, act;
    int pairs, rowb, rs, lead, shift, cpr, strip_bytes, tiles_img;
    int per_wg, rest;          // workgroup b walks per_wg tiles, one more if b < rest
    unsigned div_wo[2], div_pairs2[2], div_tiles[2];
};

// VEC consecutive elements from element `e` on, zero unless ok: a 16-byte load of whole dwords and, for a bf16 chunk that
// starts on an odd element, one dword more and a funnel shift.  The caller knows that e >= 0 and that 20 bytes from there
// (rounded down to a dword) lie inside the tensor.
template <int DT>
__device__ __forceinline__ uint4 chunk(__amdgpu_buffer_rsrc_t r, int e, bool ok)
{
    const int at = (e * (16 / El<DT>::VEC)) & ~3;
    uint4 v = buf_load16(r, ok ? (unsigned)at : OOB);
    if constexpr (DT == DT_BF16) {
        const unsigned v4 = __float_as_uint(buf_load1<float>(r, ok && (e & 1) ? (unsigned)(at + 16) : OOB));
        const unsigned sh = (unsigned)(e & 1) * 16u;
        v = make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, sh), __builtin_amdgcn_alignbit(v.z, v.y, sh),
                       __builtin_amdgcn_alignbit(v.w, v.z, sh), __builtin_amdgcn_alignbit(v4, v.w, sh));
    }
    return v;
}

// The same element by element, for chunks that may reach over an end of the tensor (what lies outside reads as zero)
template <int DT>
__device__ __forceinline__ uint4 chunk_edge(__amdgpu_buffer_rsrc_t r, int bytes, int e, bool ok)
{
    typedef typename El<DT>::T T;
    constexpr int VEC = El<DT>::VEC, ESZ = (int)sizeof(T);
    unsigned d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
        const T one = buf_load1<T>(r, ok && e + q >= 0 && (e + q + 1) * ESZ <= bytes ? (unsigned)((e + q) * ESZ) : OOB);
        if constexpr (DT == DT_BF16) d[q >> 1] |= (unsigned)one << ((q & 1) * 16);
        else d[q] = __float_as_uint(one);
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// dword q of a chunk of which the first `valid` elements count
template <int DT> __device__ __forceinline__ unsigned valid_mask(int q, int valid)
{
    if constexpr (DT == DT_BF16) return 2 * q + 1 < valid ? 0xFFFFFFFFu : 2 * q < valid ? 0xFFFFu : 0u;
    else return q < valid ? 0xFFFFFFFFu : 0u;
}

// PAIRS: k groups per tap row, 0 = not known at compile time.  ODD: the first element of a position's run may be odd (bf16,
// odd stride * Cin): one dword more per chunk and a funnel shift.  LINES: whole groups of 32 TN channels, 16-byte vectors, no
// residual and an activation of a few instructions; kept apart from the general epilogue because calls and rarely taken
// branches in the tile loop cost it half its speed (instruction fetch and registers saved around calls).
template <int DT, int TN, int PAIRS, bool ODD, bool LINES>
__global__ __launch_bounds__(STEM_THREADS) void stem_kernel(StemArgs a)
{
    typedef typename El<DT>::T T;
    constexpr int VEC = El<DT>::VEC, ESZ = (int)sizeof(T);
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *strip = smem, *Bs = smem + a.strip_bytes;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int n0 = a.n_lo + (int)blockIdx.y * (32 * TN);
    const int pairs = PAIRS ? PAIRS : a.pairs;
    const int run = a.run, HoWo = a.HoWo, WC = a.WC, x_bytes = a.x_bytes, w_bytes = a.w_bytes;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes), wr = make_rsrc(a.w, a.w_bytes);

    for (int r = tid >> 3; r < 32 * TN; r += STEM_THREADS / 8)
        for (int q = tid & 7; q < 2 * pairs * a.kh; q += 8) {
            const int kr = div_by(q, a.div_pairs2), c = q - kr * 2 * pairs, n = n0 + r, valid = run - c * VEC;
            const int e = n * (a.kh * run) + kr * run + c * VEC;
            uint4 v = chunk<DT>(wr, e, n < a.n_hi && valid > 0 && e * ESZ <= w_bytes - 20);
            if (e * ESZ > w_bytes - 20) v = chunk_edge<DT>(wr, w_bytes, e, n < a.n_hi && valid > 0);
            *(uint4 *)(Bs + r * a.rowb + q * 16) = make_uint4(v.x & valid_mask<DT>(0, valid), v.y & valid_mask<DT>(1, valid),
                                                              v.z & valid_mask<DT>(2, valid), v.w & valid_mask<DT>(3, valid));
        }

    float *bias = (float *)(Bs + 32 * TN * a.rowb);
    if (tid < 32 * TN) bias[tid] = a.bias && n0 + tid < a.n_hi ? a.bias[n0 + tid] : 0.f;

    // what follows a run is image data under zero weights: only finite values may meet them, so it is cut off
    unsigned tail[4], right[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        tail[q] = valid_mask<DT>(q, run - (2 * (pairs - 1) + lhalf) * VEC);
        right[q] = valid_mask<DT>(q, WC + a.shift - (a.cpr - 1) * VEC);
    }

    GemmArgs fin;                               // what the general epilogue reads
    fin.alpha = 1.f; fin.bias = nullptr; fin.act = a.act; fin.n_hi = a.n_hi;
    T *yg = (T *)a.y;
    const T *rg = (const T *)a.res;
    const bool vec_out = a.y_row % VEC == 0 && a.n_lo % VEC == 0 && (((uintptr_t)a.y) & 15) == 0 && (((uintptr_t)a.res) & 15) == 0;

    const int wg = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int t_lo = wg * a.per_wg + min(wg, a.rest), t_hi = t_lo + a.per_wg + (wg < a.rest ? 1 : 0);
    // A tile's strip: image, first position, input rows.  A wave copies rows wave, wave + 4, ... of it; three rows and 128 chunks
    // per lane pass through registers, requested while the tile before is computed; what is larger follows after the barrier.
    struct Strip { int img, p0, oh_a, ih0, rows; bool edge; };
    const int border = (a.lead - a.shift) / VEC, per_row = a.rs / 16;           // whole chunks left of the image, chunks per strip row
    auto strip_of = [&](int t) {
        Strip s;
        const int im = __builtin_amdgcn_readfirstlane(div_by(t, a.div_tiles));
        s.img = a.img_lo + im;
        s.p0 = (t - im * a.tiles_img) * STEM_BM;
        s.oh_a = __builtin_amdgcn_readfirstlane(div_by(s.p0, a.div_wo));
        const int oh_b = __builtin_amdgcn_readfirstlane(div_by(min(s.p0 + STEM_BM, HoWo) - 1, a.div_wo));
        s.ih0 = s.oh_a * a.stride - a.pad;
        s.rows = (oh_b - s.oh_a) * a.stride + a.kh;
        s.edge = stem_edge(s.img == 0 && s.ih0 <= 0, s.img * a.H + min(s.ih0 + s.rows, a.H), WC, x_bytes / ESZ, VEC);
        return s;
    };
    auto load = [&](const Strip &s, int r, int k) {
        const int ih = s.ih0 + r, c = k - border;
        return chunk<DT>(xr, (s.img * a.H + ih) * WC - a.shift + c * VEC, r < s.rows && ih >= 0 && ih < a.H && c >= 0 && c < a.cpr);
    };
    auto put = [&](const Strip &s, int r, int k, uint4 v) {
        const int c = k - border;
        if (DT == DT_BF16 && c == 0 && a.shift) v.x &= 0xFFFF0000u;
        if (c == a.cpr - 1) { v.x &= right[0]; v.y &= right[1]; v.z &= right[2]; v.w &= right[3]; }
        if (r < s.rows && k < per_row) *(uint4 *)(strip + r * a.rs + k * 16) = v;
    };
    constexpr int WAVES = STEM_THREADS / 64;
    uint4 ahead[6];
    Strip s = strip_of(t_lo);
    if (!s.edge) {
#pragma unroll
        for (int u = 0; u < 6; ++u) ahead[u] = load(s, wave + (u >> 1) * WAVES, lane + (u & 1) * 64);
    }
    for (int t = t_lo; t < t_hi; ++t) {
        const int img = s.img, p0 = s.p0, oh_a = s.oh_a;
        __syncthreads();                        // the weights are laid out / the previous tile's patches have been read
        if (s.edge) {
            for (int r = wave; r < s.rows; r += WAVES)
                for (int k = lane; k < per_row; k += 64) {
                    const int ih = s.ih0 + r, c = k - border;
                    put(s, r, k, chunk_edge<DT>(xr, x_bytes, (img * a.H + ih) * WC - a.shift + c * VEC, ih >= 0 && ih < a.H && c >= 0 && c < a.cpr));
                }
        } else {
#pragma unroll
            for (int u = 0; u < 6; ++u) put(s, wave + (u >> 1) * WAVES, lane + (u & 1) * 64, ahead[u]);
            for (int r = wave; r < s.rows; r += WAVES)
                for (int k = r < 3 * WAVES ? lane + 128 : lane; k < per_row; k += 64) put(s, r, k, load(s, r, k));
        }
        __syncthreads();
        if (t + 1 < t_hi) {
            s = strip_of(t + 1);
            if (!s.edge) {
#pragma unroll
                for (int u = 0; u < 6; ++u) ahead[u] = load(s, wave + (u >> 1) * WAVES, lane + (u & 1) * 64);
            }
        }

        const int p = p0 + wave * 32 + lrow;
        const bool in = p < HoWo;
        const int oh = in ? div_by(p, a.div_wo) : oh_a, ow = in ? p - oh * a.Wo : 0;
        const int elem = a.lead + (ow * a.stride - a.pad) * a.Cin;              // never negative: lead >= pad * Cin
        const unsigned sh = ODD ? (unsigned)(elem & 1) * 16u : 0u;
        const unsigned char *arow = strip + (oh - oh_a) * a.stride * a.rs + ((elem * ESZ) & ~3) + lhalf * 16;
        const unsigned char *brow = Bs + lrow * a.rowb + lhalf * 16;

        f32x16 acc[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; e += 4) {   // channel 32 j + 2 e + 4 (lane / 32) + q
                const float4 b4 = *(const float4 *)(bias + 32 * j + 2 * e + 4 * lhalf);
                acc[j][e] = b4.x; acc[j][e + 1] = b4.y; acc[j][e + 2] = b4.z; acc[j][e + 3] = b4.w;
            }
        auto group = [&](const unsigned *src, const unsigned char *b, bool last) {
            unsigned d[4] = {src[0], src[1], src[2], src[3]};
            if constexpr (ODD) {
                const unsigned d4 = src[4];
                d[0] = __builtin_amdgcn_alignbit(d[1], d[0], sh);
                d[1] = __builtin_amdgcn_alignbit(d[2], d[1], sh);
                d[2] = __builtin_amdgcn_alignbit(d[3], d[2], sh);
                d[3] = __builtin_amdgcn_alignbit(d4, d[3], sh);
            }
            if (last) {
#pragma unroll
                for (int q = 0; q < 4; ++q) d[q] &= tail[q];
            }
            const uint4 xf = make_uint4(d[0], d[1], d[2], d[3]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const uint4 wf = *(const uint4 *)(b + j * 32 * a.rowb);
                if constexpr (DT == DT_BF16) {
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf), __builtin_bit_cast(bf16x8, xf), acc[j], 0, 0, 0);
                } else {
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wf.x), __uint_as_float(xf.x), acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wf.y), __uint_as_float(xf.y), acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wf.z), __uint_as_float(xf.z), acc[j], 0, 0, 0);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wf.w), __uint_as_float(xf.w), acc[j], 0, 0, 0);
                }
            }
        };
        for (int r = 0; r < a.kh; ++r) {
            if constexpr (PAIRS > 0) {
#pragma unroll
                for (int k = 0; k < PAIRS; ++k) group((const unsigned *)(arow + k * 32), brow + k * 32, k == PAIRS - 1);
            } else {
                for (int k = 0; k < pairs; ++k) group((const unsigned *)(arow + k * 32), brow + k * 32, k == pairs - 1);
            }
            arow += a.rs;
            brow += pairs * 32;
        }

        // Element e of a lane is channel (e/4)*8 + (lane/32)*4 + e%4 of position lane%32.  Swapping the upper half of group
        // 2h with the lower half of group 2h + 1 leaves a lane with eight consecutive channels, 8 (2h + lane/32) onwards.
        // Finished vectors go through a patch of LDS (the strip, which has been consumed) so that a wave stores whole
        // 128-byte lines: stored as they lie, 32 bytes per position, the launch was bound by its stores (2.2 TB/s).
        const int64_t m_img = (int64_t)img * HoWo;
        __syncthreads();                        // the strip has been consumed by all waves
        unsigned char *patch = strip + wave * STEM_PATCH;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[j][8 * h + q]), __float_as_uint(acc[j][8 * h + 4 + q]), false, false);
                    v[q] = __uint_as_float(r[0]);
                    v[4 + q] = __uint_as_float(r[1]);
                }
                const int n = n0 + j * 32 + 8 * (2 * h + lhalf);
                if constexpr (LINES) {
                    if (a.act == ACT_RELU) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = __builtin_fmaxf(v[q], 0.f);
                    } else if (a.act == ACT_RELU6) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = __builtin_amdgcn_fmed3f(v[q], 0.f, 6.f);
                    } else if (a.act != ACT_NONE) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = hard_act(v[q], a.act);
                    }
                    unsigned char *dst = patch + lrow * STEM_PATCH_ROW + (8 * (2 * h + lhalf) + (DT == DT_BF16 ? 32 * j : 0)) * ESZ;
                    if constexpr (DT == DT_BF16) {
                        *(uint4 *)dst = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
                    } else {
                        *(float4 *)dst = make_float4(v[0], v[1], v[2], v[3]);
                        *(float4 *)(dst + 16) = make_float4(v[4], v[5], v[6], v[7]);
                    }
                    continue;
                }
                if (!in || n >= a.n_hi) continue;
#pragma unroll
                for (int u = 0; u < 8; u += VEC) {
                    const int nu = n + u;
                    const int64_t o = (m_img + p) * a.y_row + nu;
                    if (nu >= a.n_hi) break;
                    if (vec_out && nu + VEC <= a.n_hi) {
                        const float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};     // the accumulators started at the bias
                        uint4 rv = make_uint4(0u, 0u, 0u, 0u);
                        if (rg) rv = *(const uint4 *)(rg + o);
                        finish_vec<DT>(fin, v + u, bv, rg != nullptr, rv, yg, o);
                    } else {
                        finish_scalar<DT>(fin, v + u, rg, yg, o, nu);
                    }
                }
            }
            if constexpr (LINES) if (DT != DT_BF16 || j == TN - 1) {
                constexpr int LINE = DT == DT_BF16 ? 32 * TN * 2 : 128, LPR = LINE / 16;        // bytes and lanes per position
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 32 * LPR / 64; ++i) {
                    const int row = i * (64 / LPR) + lane / LPR, pr = p0 + wave * 32 + row, col = (lane % LPR) * 16;
                    const uint4 v = *(const uint4 *)(patch + row * STEM_PATCH_ROW + col);
                    if (pr < HoWo) *(uint4 *)((unsigned char *)(yg + (m_img + pr) * a.y_row + n0 + (DT == DT_BF16 ? 0 : 32 * j)) + col) = v;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

template <int DT, int TN>
static LaunchInfo go_stem(const GemmArgs &a, const StemGeom &g, hipStream_t s, bool dry)
{
    const int groups = (a.n_hi - a.n_lo + 32 * TN - 1) / (32 * TN);
    LaunchInfo li;
    li.threads = STEM_THREADS;
    li.lds_bytes = g.strip_bytes + 32 * TN * (g.rowb + 4);
    li.wg_per_cu = 160 * 1024 / li.lds_bytes < 4 ? 160 * 1024 / li.lds_bytes : 4;
    const int most = 256 * li.wg_per_cu / groups;                               // one resident set of workgroups walks all tiles
    const int wgs = g.tiles < most ? g.tiles : most < 1 ? 1 : most;
    li.workgroups = wgs * groups;
    li.kernel = DT == DT_BF16 ? "stem_bf16" : "stem_f32";
    li.phases = 1;
    if (dry || g.tiles == 0) return li;
    StemArgs b = {a.x, a.w, a.res, a.bias, a.y, (int)a.x_bytes, (int)a.w_bytes, a.H, a.Wo, a.Ho * a.Wo, a.W * a.Cin, a.Cin, a.kw * a.Cin, a.kh,
                  a.stride, a.pad, (int)a.y_row, a.m_lo / (a.Ho * a.Wo), a.n_lo, a.n_hi, a.act, g.pairs, g.rowb, g.rs, g.lead, g.shift, g.cpr,
                  g.strip_bytes, g.tiles_img, g.tiles / wgs, g.tiles % wgs, {0u, 0u}, {0u, 0u}, {0u, 0u}};
    divisor(a.Wo, b.div_wo);
    divisor(2 * g.pairs, b.div_pairs2);
    divisor(g.tiles_img, b.div_tiles);
    const dim3 grid(wgs, groups), block(STEM_THREADS);
    const bool lines = (a.n_hi - a.n_lo) % (32 * TN) == 0 && a.y_row % El<DT>::VEC == 0 && a.n_lo % El<DT>::VEC == 0 && ((uintptr_t)a.y & 15) == 0 &&
                       !a.res && a.act != ACT_GELU;
#define GO(P, O) (lines ? go((stem_kernel<DT, TN, P, O, true>)) : go((stem_kernel<DT, TN, P, O, false>)))
    auto go = [&](void (*kernel)(StemArgs)) { GACER_LAUNCH(kernel, grid, block, li.lds_bytes, s, b); };
    if (DT == DT_BF16 && (a.stride * a.Cin) % 2) { if (g.pairs == 1) GO(1, true); else GO(0, true); }
    else if (g.pairs == 1) GO(1, false);
    else if (g.pairs == 2) GO(2, false);
    else if (g.pairs == 3) GO(3, false);
    else GO(0, false);
#undef GO
    return li;
}

template <int DT>
static LaunchInfo pick_stem(const GemmArgs &a, hipStream_t s, bool dry)
{
    StemGeom g;
    // 64 channels per workgroup share a strip; 32 while the tiles alone do not reach every compute unit (one image, 64x7x7x3
    // bf16, 98 tiles: 9.7 -> 7.5 us)
    if (a.n_hi - a.n_lo > 32 && stem_geometry(a, 2, &g) && g.tiles >= 256) return go_stem<DT, 2>(a, g, s, dry);
    stem_geometry(a, 1, &g);                    // held when the tenant was loaded
    return go_stem<DT, 1>(a, g, s, dry);
}

LaunchInfo launch_stem(const GemmArgs &a, hipStream_t s, bool dry)
{
    return a.dtype == DT_BF16 ? pick_stem<DT_BF16>(a, s, dry) : pick_stem<DT_F32>(a, s, dry);
}

}  // namespace gacer
