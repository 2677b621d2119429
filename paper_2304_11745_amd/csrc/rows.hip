// Row-streaming kernel for pointwise (1x1, unpadded) convolutions and plain GEMMs with a short K (MobileNet's expand layers, the
// 64-channel 1x1 layers of ResNet-50).
//
// A workgroup stages 32 RS rows of A and the B rows of its 32 << LC output channels in LDS, all requested at once by coalesced direct
// loads (rows padded to a power of two of 16-byte chunks, swizzled as in igemm_dma_kernel); beyond K the descriptor fills in
// zeros.  Its four waves stand 1 << LC side by side along the channels; each keeps its B fragments in registers and takes its row
// tiles from the stage.  The operands of the MFMAs are swapped, so that a lane owns one row and four consecutive channels at a
// time: bias, residual and activation are applied in registers, the finished elements pass through a patch of LDS in their
// own type and are stored as whole 64-byte (fp32: 128-byte) pieces of rows.  Every accumulator is the same MFMA chain over ascending
// 32-byte k groups as in igemm_kernel, so both give the same bits.
//
// What bounds it: with many rows the output's way to memory (100352x256x64 bf16: 64 MB in 14.4 us), with few one wave's chain of
// instructions around one round trip.  Before, a wave read its fragments of A straight from global memory (32 pieces of 32 bytes a
// load, 19 bytes per clock and unit) and B was copied to LDS in a loop that waited for each piece.  One launch, us, before / here:
// bf16 196x384x64 4.04 / 3.20, 12544x576x96 13.8 / 8.2, 25088x256x64 with a residual 9.3 / 8.3, 100352x256x64 24.5 / 14.4,
// 401408x96x16 27.0 / 17.2, 401408x16x32 13.2 / 8.7; fp32 (tiled kernel before) 12544x16x32 5.42 / 3.79, 100352x144x24 24.8 / 22.3,
// 401408x16x32 25.2 / 18.5.
#include <hip/hip_runtime.h>
#include <string>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"

namespace gacer {

struct RowsArgs {
    const void *x, *w, *res;
    const float *bias;
    void *y;
    unsigned x_bytes, w_bytes, res_bytes, bias_bytes;
    unsigned x_pitch, w_pitch, y_pitch, k_bytes;       // bytes between input pixels, weight rows, output rows; bytes of K
    int m_lo, m_hi, n_lo, n_hi;
    float alpha;
    int act, vec, in_vec, dense;       // output stored, bias and residual read in whole vectors; one pitch for all input rows
    int HoWo, Wo, W, stride;
    unsigned x_img;
    unsigned div_howo[2], div_wo[2];
};

// Geometry shared with the launcher.  G: 32-byte k groups; ROWB: bytes of an LDS row.
template <int DT, int G, int LC> struct RowsGeom {
    static constexpr int ESZ = DT == DT_BF16 ? 2 : 4;
    static constexpr int RS = LC == 1 ? 2 : 4;         // row tiles of 32 per workgroup
    static constexpr int KC = G == 1 ? 2 : G == 2 ? 4 : G <= 4 ? 8 : 16, ROWB = KC * 16;
    static constexpr int A = 32 * RS * ROWB, B = (32 << LC) * ROWB;
    static constexpr int PROW = 32 * ESZ + 16, PATCH = 4 * 32 * PROW;
    static constexpr bool OVER = LC == 2;              // the patches overlay the weights (costs a barrier, leaves room for a third workgroup)
    static constexpr int LDS = A + (OVER ? (B > PATCH ? B : PATCH) : B + PATCH);
};

template <int DT, int G, int LC>
__global__ __launch_bounds__(256, G == 6 ? 2 : 3) void rowgemm_kernel(RowsArgs a)
{
    typedef typename El<DT>::T T;
    typedef RowsGeom<DT, G, LC> Z;
    constexpr int ESZ = Z::ESZ, VE = 16 / ESZ, RS = Z::RS, KC = Z::KC, ROWB = Z::ROWB, PROW = Z::PROW;
    constexpr int RPL = 64 / KC;                       // rows filled by one wave load
    constexpr int SWZ = ROWB >= 256 ? 1 : 256 / ROWB;  // rows per sweep over the banks
    constexpr int CPR = 32 / VE, ITER = 32 * CPR / 64; // 16-byte chunks per patch row, and of a lane
    constexpr int COLS = 1 << LC, ROWS = 4 >> LC;
    constexpr int A_LOADS = 32 * RS / RPL, B_LOADS = 32 * COLS / RPL;
    __shared__ __align__(1024) unsigned char smem[Z::LDS];
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef typename std::conditional<DT == DT_BF16, bf16x8, f32x4>::type F;
    typedef typename std::conditional<DT == DT_BF16, uint2, uint4>::type R;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5, wcol = wave & (COLS - 1), wrow = wave >> LC;
    const int mb = a.m_lo + (int)blockIdx.x * 32 * RS, nb = a.n_lo + (int)blockIdx.y * 32 * COLS, n0 = nb + wcol * 32;
    auto rsrc = [](const void *p, unsigned bytes) { return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000); };
    const __amdgpu_buffer_rsrc_t xr = rsrc(a.x, a.x_bytes), wr = rsrc(a.w, a.w_bytes), rr = rsrc(a.res, a.res_bytes), br = rsrc(a.bias, a.bias_bytes);
    unsigned char *As = smem, *Bs = smem + Z::A;

    // a wave load fills RPL rows: lane l row l / KC, slot l % KC, which holds chunk (l % KC) ^ ((row / SWZ) % KC)
    auto chunk_of = [&](int row) { return (unsigned)((lane % KC) ^ ((row / SWZ) % KC)) * 16u; };
#pragma unroll
    for (int q = 0; q < (A_LOADS + 3) / 4; ++q) {
        const int l = q * 4 + wave, row = l * RPL + lane / KC, m = mb + row;
        if (A_LOADS % 4 && l >= A_LOADS) break;
        const unsigned c = chunk_of(row);
        unsigned off;
        if (a.dense) {
            off = (unsigned)m * a.x_pitch + c;
        } else {
            const int img = div_by(m, a.div_howo), rem = m - img * a.HoWo;
            const int oh = div_by(rem, a.div_wo), ow = rem - oh * a.Wo;
            off = (unsigned)img * a.x_img + (unsigned)(oh * a.stride * a.W + ow * a.stride) * a.x_pitch + c;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GACER_LDS(As + l * 1024), 16, (int)(c < a.k_bytes ? off : OOB), 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < (B_LOADS + 3) / 4; ++q) {
        const int l = q * 4 + wave, row = l * RPL + lane / KC;
        if (B_LOADS % 4 && l >= B_LOADS) break;
        const unsigned c = chunk_of(row);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, GACER_LDS(Bs + l * 1024), 16, (int)(c < a.k_bytes ? (unsigned)(nb + row) * a.w_pitch + c : OOB), 0, 0, 0);
    }
    // bias and residual in the layout of the accumulators: four channels of row lrow per group of four elements
    uint4 bias[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned bo = (unsigned)(n0 + q * 8 + lhalf * 4) * 4u;
        if (a.in_vec) {
            bias[q] = buf_load16(br, bo);
        } else {                                       // a vector that reaches over the end of the range would read as zero
#pragma unroll
            for (int e = 0; e < 4; ++e) ((float *)&bias[q])[e] = buf_load1<float>(br, bo + 4u * e);
        }
    }
    R res[4];
    auto load_res = [&](R *r, int m0) {
        const unsigned ro = (unsigned)(m0 + lrow) * a.y_pitch + (unsigned)(n0 + lhalf * 4) * ESZ;
        if (a.in_vec) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (DT == DT_BF16) r[q] = buf_load8(rr, ro + (unsigned)(q * 8 * ESZ));
                else r[q] = buf_load16(rr, ro + (unsigned)(q * 8 * ESZ));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) ((T *)&r[q])[e] = buf_load1<T>(rr, ro + (unsigned)((q * 8 + e) * ESZ));
        }
    };
    if (a.res) load_res(res, mb + wrow * 32);
    unsigned lds_off[ITER], out_off[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int idx = it * 64 + lane, row = idx / CPR, ch = idx % CPR;
        lds_off[it] = (unsigned)(row * PROW + ch * 16);
        out_off[it] = (unsigned)row * a.y_pitch + (unsigned)(ch * 16);
    }
    auto meet = [&]() {
        __builtin_amdgcn_s_waitcnt((7 << 4));          // vmcnt(0), lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    meet();
    const int frag = lrow * ROWB, sw = (lrow / SWZ) % KC;
    F fb[G];
#pragma unroll
    for (int g = 0; g < G; ++g) fb[g] = *(const F *)(Bs + wcol * 32 * ROWB + frag + (((2 * g + lhalf) ^ sw) * 16));
    if constexpr (Z::OVER) meet();
    unsigned char *mine = Bs + (Z::OVER ? 0 : Z::B) + wave * 32 * PROW;
    if (n0 >= a.n_hi) return;                          // no barrier below

#pragma unroll
    for (int t = wrow; t < RS; t += ROWS) {
        const int m0 = mb + t * 32;
        if (m0 >= a.m_hi) return;
        F fa[G];
#pragma unroll
        for (int g = 0; g < G; ++g) fa[g] = *(const F *)(As + t * 32 * ROWB + frag + (((2 * g + lhalf) ^ sw) * 16));
        R next[4];
        if (t + ROWS < RS && a.res) load_res(next, m0 + ROWS * 32);
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if constexpr (DT == DT_BF16) {
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[g], fa[g], acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[g][e], fa[g][e], acc, 0, 0, 0);
            }
        }
        float v[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[4 * q] = __fmaf_rn(acc[4 * q], a.alpha, __uint_as_float(bias[q].x));
            v[4 * q + 1] = __fmaf_rn(acc[4 * q + 1], a.alpha, __uint_as_float(bias[q].y));
            v[4 * q + 2] = __fmaf_rn(acc[4 * q + 2], a.alpha, __uint_as_float(bias[q].z));
            v[4 * q + 3] = __fmaf_rn(acc[4 * q + 3], a.alpha, __uint_as_float(bias[q].w));
        }
        if (a.res) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float r[4];
                load_vec4((const T *)&res[q], r);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * q + e] = __fadd_rn(v[4 * q + e], r[e]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) res[q] = next[q];
        }
        act_vec<16>(v, a.act);
#pragma unroll
        for (int q = 0; q < 4; ++q) store_vec4((T *)(mine + lrow * PROW + (q * 8 + lhalf * 4) * ESZ), v + 4 * q);
        __builtin_amdgcn_wave_barrier();
        char *yt = (char *)a.y + ((int64_t)m0 * a.y_pitch + (int64_t)n0 * ESZ);
        if (a.vec && n0 + 32 <= a.n_hi && m0 + 32 <= a.m_hi) {
#pragma unroll
            for (int it = 0; it < ITER; ++it) *(uint4 *)(yt + out_off[it]) = *(const uint4 *)(mine + lds_off[it]);
        } else {
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int idx = it * 64 + lane, row = idx / CPR, n = n0 + idx % CPR * VE;
                if (m0 + row >= a.m_hi || n >= a.n_hi) continue;
                if (a.vec && n + VE <= a.n_hi) {
                    *(uint4 *)(yt + out_off[it]) = *(const uint4 *)(mine + lds_off[it]);
                } else {
                    for (int e = 0; e < VE; ++e)
                        if (n + e < a.n_hi) *((T *)(yt + out_off[it]) + e) = *((const T *)(mine + lds_off[it]) + e);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Single-tap, unpadded, unsplit products whose rows are whole vectors and hold at most 192 bytes of K: properties of the operator, not of
// the launched sub-range, so that every chunk adds alike.  Beyond 192 bytes a workgroup would stage more than it computes on.
bool rows_takes(const GemmArgs &a)
{
    const int esz = a.dtype == DT_BF16 ? 2 : 4, vec = 16 / esz;
    return !a.b_trans && !a.pre_scale && a.ksplit == 1 && a.kh == 1 && a.kw == 1 && a.pad == 0 && a.zb * a.zh == 1 && a.z_lo == 0 &&
           (int64_t)a.K * esz <= 192 && a.Cin % vec == 0 && a.x_pix % vec == 0 && a.x_img % vec == 0 && a.w_row % vec == 0 &&
           (((uintptr_t)a.x | (uintptr_t)a.w) & 15) == 0;
}

template <int DT, int G, int LC>
static LaunchInfo go(const RowsArgs &b, hipStream_t s, bool dry)
{
    typedef RowsGeom<DT, G, LC> Z;
    static const std::string name = std::string("rowgemm_") + (DT == DT_BF16 ? "bf16_x" : "f32_x") + std::to_string(32 << LC);
    const dim3 grid((b.m_hi - b.m_lo + 32 * Z::RS - 1) / (32 * Z::RS), (b.n_hi - b.n_lo + (32 << LC) - 1) / (32 << LC));
    LaunchInfo li;
    li.workgroups = (int)(grid.x * grid.y);
    li.threads = 256;
    li.lds_bytes = Z::LDS;
    li.wg_per_cu = 160 * 1024 / Z::LDS < 4 ? 160 * 1024 / Z::LDS : 4;
    li.kernel = name.c_str();
    li.phases = 1;
    if (!dry && li.workgroups) GACER_LAUNCH((rowgemm_kernel<DT, G, LC>), grid, dim3(256), 0, s, b);
    return li;
}

template <int DT, int LC>
static LaunchInfo go_g(const RowsArgs &b, hipStream_t s, bool dry)
{
    switch ((b.k_bytes + 31) / 32) {
    case 1: return go<DT, 1, LC>(b, s, dry);
    case 2: return go<DT, 2, LC>(b, s, dry);
    case 3: return go<DT, 3, LC>(b, s, dry);
    case 4: return go<DT, 4, LC>(b, s, dry);
    default: return go<DT, 6, LC>(b, s, dry);
    }
}

template <int DT>
static LaunchInfo launch(const GemmArgs &a, hipStream_t s, bool dry)
{
    constexpr int ESZ = DT == DT_BF16 ? 2 : 4;
    RowsArgs b;
    auto range = [](int64_t bytes) { return (unsigned)(bytes < 0 ? 0 : bytes > 0x7FFFFFFF ? 0x7FFFFFFF : bytes); };
    b.x = a.x; b.w = a.w; b.res = a.res; b.bias = a.bias; b.y = a.y;
    b.x_bytes = range(a.x_bytes);
    b.w_bytes = range(a.w_bytes);
    b.res_bytes = a.res ? range(((int64_t)(a.m_hi - 1) * a.y_row + a.n_hi) * ESZ) : 0u;
    b.bias_bytes = a.bias ? (unsigned)a.n_hi * 4u : 0u;
    b.x_pitch = (unsigned)(a.x_pix * ESZ); b.w_pitch = (unsigned)(a.w_row * ESZ); b.y_pitch = (unsigned)(a.y_row * ESZ); b.k_bytes = (unsigned)(a.K * ESZ);
    b.m_lo = a.m_lo; b.m_hi = a.m_hi; b.n_lo = a.n_lo; b.n_hi = a.n_hi;
    b.alpha = a.alpha; b.act = a.act;
    b.vec = a.y_row % (16 / ESZ) == 0 && a.n_lo % (16 / ESZ) == 0 && ((uintptr_t)a.y & 15) == 0;
    b.in_vec = a.n_lo % 4 == 0 && a.n_hi % 4 == 0 && ((uintptr_t)a.bias & 15) == 0 && (!a.res || (a.y_row % 4 == 0 && ((uintptr_t)a.res & (4 * ESZ - 1)) == 0));
    b.dense = a.stride == 1 && a.x_img == (int64_t)a.Ho * a.Wo * a.x_pix;
    b.HoWo = a.Ho * a.Wo; b.Wo = a.Wo; b.W = a.W; b.stride = a.stride;
    b.x_img = (unsigned)(a.x_img * ESZ);
    divisor(b.HoWo, b.div_howo);
    divisor(b.Wo, b.div_wo);
    // One column of 32 channels: four waves along the rows.  More: two by two, which fills the chip from the fewest rows; three columns in
    // fp32 as one (100352x96x16 13.2 / 11.5, 401408x96x16 38.3 / 36.6); bf16 with many tiles in three columns or more: four side by side,
    // which read the rows they share once.  Us two by two / four side by side, by the number of 32x32 tiles: 4704 (25088x192x32)
    // 5.1 / 5.7, 6272 (25088x256x64) 7.1 / 6.7, 7056 (12544x576x96) 8.2 / 8.2, 9408 (100352x96x16) 8.5 / 7.1, 12544
    // (50176x256x64) 10.7 / 8.8, 25088 (100352x256x64) 18.6 / 14.4; two columns (100352x64x64) 7.2 / 8.0.
    const int cols = (a.n_hi - a.n_lo + 31) / 32;
    const int64_t tiles = (int64_t)((a.m_hi - a.m_lo + 31) / 32) * cols;
    if (cols == 1 || (DT == DT_F32 && cols == 3)) return go_g<DT, 0>(b, s, dry);
    if constexpr (DT == DT_BF16)
        if (cols >= 3 && tiles > 6000) return go_g<DT, 2>(b, s, dry);
    return go_g<DT, 1>(b, s, dry);
}

LaunchInfo launch_rows(const GemmArgs &a, hipStream_t s, bool dry)
{
    return a.dtype == DT_BF16 ? launch<DT_BF16>(a, s, dry) : launch<DT_F32>(a, s, dry);
}

}  // namespace gacer
