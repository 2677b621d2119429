// 3x3 convolutions (stride 1, padding 1, bf16) with many output positions: the input is staged once per channel block instead
// of once per tap.
//
// A workgroup owns BM output positions (consecutive in a column strip of at most 56 columns, row by row through all images)
// x BN channels (256x128, 256x64, 128x64, 64x64).  Per block of 32 channels the positions and their one-pixel halo (for 256 positions at most 384 pixels
// of 64 bytes) go into LDS by direct loads (zeros left and right of the image); all nine taps read their A fragments from there, a tap being a fixed
// displacement of the LDS row.  Taps above or below an image read a row of zeros instead.  The weights stream past in stages of
// one tap (BN = 128, three stages) or three taps (BN = 64, three stages, or two where that leaves room for a second workgroup of 256
// positions).  Two input blocks alternate, the next one being
// requested while this one is used.  The step structure is that of igemm_dma_kernel: counted waits, one bare barrier per
// step, fragments one k group ahead, requests spread between the MFMA groups.
//
// What bounds it: igemm_dma_kernel moves every input pixel from L2 into LDS once per tap, 24 KB per 512 clocks of MFMA on its
// 256x128 tile, which is that path's rate; here it is 11 KB.  What is left is the fill of the pipeline and the epilogue of a
// short K (two workgroups per unit cover for each other) and, at 64 channels, the output.  Microseconds there / here, 32 images:
// 224x224 64->64 284.6 / 179.0, 112x112 64->128 110.7 / 80.2, 112x112 128->128 156.4 / 122.2, 56x56 256->256 153.8 / 119.3,
// 28x28 512->512 144.2 / 112.4 (1053 TFLOP/s), 56x56 64->64 22.0 / 16.8.  Outputs finished in registers (store_tiles) took, before / after:
// 16 images 112x112 64->128 49.0 / 44.5, 56x56 64->64 11.1 / 10.4, 224x224 64->64 85.3 / 81.3, 8 images 112x112 128->128 39.2 / 36.9.
//
// A third weight stage where BN = 64, us: 8 images 28x28 512->512 37.7 / 32.3, 16 images 28x28 128->128 10.0 / 8.6 (on the tiled kernels before),
// 14x14 512->512 25.5 / 20.7 (likewise), 32 images 28x28 128->128 14.6 / 12.2.  A workgroup alone on its unit keeps the matrix cores 52 %
// busy; reading fragments two or three k groups ahead, more stages and work put between the MFMAs of a group change that by 1 to 3 %.
//
// An output element is one MFMA chain over channel blocks of 32, in a block over the taps in ascending order, whatever the tile;
// which kernel an operator takes depends on its unsplit shape only, so every chunk of it adds alike.
#include <hip/hip_runtime.h>
#include <string>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"
#include "conv3_geom.h"

namespace gacer {

static constexpr int THREADS = 256;
static constexpr int ROWB = 64;                // bytes of a channel block: one LDS row
static constexpr int PATCH = 4608;             // bytes of a wave's epilogue patch; the patches overlay an input block
constexpr int conv3_input_bytes(int bm)        // LDS of an input block: pixels and rows of zeros, at least the patches of four waves
{
    return (conv3_rows(bm) + 16) * ROWB > 4 * PATCH ? (conv3_rows(bm) + 16) * ROWB : 4 * PATCH;
}

template <int N> __device__ __forceinline__ void wait_loads()       // at most N loads outstanding, own LDS reads done
{
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}

// the wait for N to 0 outstanding loads, `pending` being a constant once the steps are unrolled
template <int N> __device__ __forceinline__ void wait_pending(int pending)
{
    if (pending == N) wait_loads<N>();
    else if constexpr (N > 0) wait_pending<N - 1>(pending);
}

// TPS: taps per step; NSB: weight stages
template <int BM, int BN, int TPS, int NSB>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2 * (2 * conv3_input_bytes(BM) + NSB * TPS * BN * ROWB) <= 160 * 1024 ? 2 : 1)))
void conv3_kernel(GemmArgs a, Conv3Geom geo)
{
    constexpr int WM = BM == 256 && BN == 64 ? 4 : 2, WN = 4 / WM;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int ROWS = conv3_rows(BM);       // input pixels (LDS rows) per tile and channel block
    constexpr int SPB = 9 / TPS;               // steps per channel block (a multiple of NSB over two blocks)
    constexpr int NB = BN * TPS / 64;          // weight loads per thread and step
    constexpr int NA = ROWS / 64;              // input loads per thread and channel block
    constexpr int A_STEPS = TPS == 1 ? NA : 2 - NA % 2, PA = NA / A_STEPS;      // the steps of a block that request inputs, and how many each
    constexpr int G = 2 * TPS;                 // k groups (32 bytes of k) per step
    constexpr int ABYTES = conv3_input_bytes(BM), BBYTES = BN * TPS * ROWB;
    static_assert(NSB <= 3 && 2 * SPB % NSB == 0 && NA % A_STEPS == 0 && A_STEPS <= SPB * 2 / 3, "inputs are requested in the first two thirds of a block");

    // separate arrays named by compile-time indices: the compiler can tell what is being filled from what is being read
    __shared__ __align__(1024) unsigned char a0[ABYTES];
    __shared__ __align__(1024) unsigned char a1[ABYTES];
    __shared__ __align__(1024) unsigned char b0[BBYTES];
    __shared__ __align__(1024) unsigned char b1[BBYTES];
    __shared__ __align__(1024) unsigned char b2[NSB > 2 ? BBYTES : 16];
    auto a_at = [&](int i) -> unsigned char * { return i ? a1 : a0; };
    auto b_at = [&](int i) -> unsigned char * { return i == 0 ? b0 : i == 1 ? b1 : b2; };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int tile = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int by_m = div_by(tile, geo.div_tiles_m), by_n = div_by(tile, geo.div_tiles_n);
    const int tile_m = __builtin_amdgcn_readfirstlane(geo.n_major ? tile - by_m * geo.tiles_m : by_n);
    const int tile_n = __builtin_amdgcn_readfirstlane(geo.n_major ? by_m : tile - by_n * geo.tiles_n);
    const int strip = __builtin_amdgcn_readfirstlane(div_by(tile_m, geo.div_strip));
    const int p0 = (tile_m - strip * geo.tiles_strip) * BM, c0 = strip * geo.tw, n0 = a.n_lo + tile_n * BN;
    const int tw = geo.tw, tw2 = tw + 2;
    const int row0 = __builtin_amdgcn_readfirstlane(div_by(p0, geo.div_tw)), col0 = p0 - row0 * tw;

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes), wr = make_rsrc(a.w, a.w_bytes);

    // Direct loads fill LDS linearly: load p of a thread fills row 64 p + tid / 4, slot tid % 4, which holds logical chunk
    // slot ^ (row / 4) % 4 (fragment reads of 32 rows then meet no bank conflict).
    const int chunk = (tid & 3) ^ ((tid >> 4) & 3);
    const unsigned x_pix = (unsigned)a.x_pix * 2u;
    // LDS row L is pixel (row0 - 1) * tw2 + col0 + L of the strip, its rows padded by one pixel on either side
    unsigned a_off[NA];
#pragma unroll
    for (int p = 0; p < NA; ++p) {
        const int q = row0 * tw2 + col0 + p * 64 + (tid >> 2);                   // counted from row -1
        const int r1 = div_by(q, geo.div_tw2), c = c0 + (q - r1 * tw2) - 1, r = r1 - 1;
        const bool ok = r >= 0 && r < geo.rows && c >= 0 && c < a.W;
        a_off[p] = ok ? (unsigned)((geo.row_lo + r) * a.W + c) * x_pix + (unsigned)(chunk * 16) : OOB;
    }
    unsigned b_off[BN / 64];
#pragma unroll
    for (int i = 0; i < BN / 64; ++i) {
        const int n = n0 + i * 64 + (tid >> 2);
        b_off[i] = n < a.n_hi ? (unsigned)n * ((unsigned)a.w_row * 2u) + (unsigned)(chunk * 16) : OOB;
    }
    const int ncb = a.Cin / 32;                // channel blocks, an even number
    const int wave_slot = wave * 1024;
    // one load each; OOB plus any offset inside a tensor stays out of range.  Blocks beyond the last repeat it, unused.
    auto request_a = [&](unsigned char *dst, int cb, int p) {
        const unsigned d = (unsigned)(min(cb, ncb - 1) * ROWB);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GACER_LDS(dst + p * 4096 + wave_slot), 16, (int)(a_off[p] + d), 0, 0, 0);
    };
    auto request_b = [&](unsigned char *dst, int cb, int tap0, int i) {
        const int tap = TPS == 1 ? tap0 : tap0 + i;
        const unsigned d = (unsigned)((tap * a.Cin + min(cb, ncb - 1) * 32) * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, GACER_LDS(dst + i * 4096 + wave_slot), 16, (int)(b_off[TPS == 1 ? i : 0] + d), 0, 0, 0);
    };

    // this lane's rows of the A fragments: LDS row of tap (0, 0), and whether the rows above and below belong to the image
    const int lrow = lane & 31, lhalf = lane >> 5;
    int f_row[TM];
    bool up[TM], down[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int p = p0 + wm * (BM / WM) + i * 32 + lrow;
        const int r = div_by(p, geo.div_tw), h = r - div_by(r, geo.div_h) * a.H;
        f_row[i] = (r - row0) * tw2 + (p - r * tw) - col0;
        up[i] = h > 0;
        down[i] = h < a.H - 1;
    }
    const int b_row = (wn * (BN / WN) + lrow) * ROWB, b_swz = (lhalf ^ ((lrow >> 2) & 3)) * 16;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    uint4 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[1][i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[1][j] = make_uint4(0u, 0u, 0u, 0u);

    auto mfmas = [&](int set) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[set][j]),
                                                                    __builtin_bit_cast(bf16x8, fa[set][i]), acc[i][j], 0, 0, 0);
    };
    constexpr int SCHED_ALU_MAY_CROSS = 0x2 | 0x4;

    // zero rows of both input blocks (rows ROWS .. + 15, never loaded)
    if (tid < 64) *(uint4 *)(a0 + ROWS * ROWB + tid * 16) = make_uint4(0u, 0u, 0u, 0u);
    else if (tid < 128) *(uint4 *)(a1 + ROWS * ROWB + (tid - 64) * 16) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int p = 0; p < NA; ++p) request_a(a0, 0, p);
#pragma unroll
    for (int u = 0; u < NSB - 1; ++u)
#pragma unroll
        for (int i = 0; i < NB; ++i) request_b(b_at(u), 0, u * TPS, i);
    wait_loads<(NSB - 2) * NB>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // Input loads per step: none in the last third of a block, so that they have landed when the block starts.
    // Two channel blocks per trip: stages and input blocks keep compile-time names.
    for (int cb = 0; cb < ncb; cb += 2) {
#pragma unroll
        for (int u = 0; u < 2 * SPB; ++u) {
            const int blk = u / SPB, t = u % SPB;
            const int na = t < A_STEPS ? PA : 0;
            const int v = u + NSB - 1;                                           // the step whose weights are requested
            const unsigned char *cur_a = a_at(blk), *cur_b = b_at(u % NSB);
            // opaque: the fragment addresses of all nine taps would otherwise be kept in registers around the loop and spill
#pragma unroll
            for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(f_row[i]));
#pragma unroll
            for (int slot = 0; slot < G; ++slot) {
                const int tap = t * TPS + slot / 2, g = slot & 1, set = slot & 1;
                const int r = tap / 3, q = tap % 3;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    int L = f_row[i] + r * tw2 + q;
                    if (r == 0) L = up[i] ? L : ROWS;
                    if (r == 2) L = down[i] ? L : ROWS;
                    fa[set][i] = *(const uint4 *)(cur_a + L * ROWB + (((2 * g + lhalf) ^ ((L >> 2) & 3)) * 16));
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) fb[set][j] = *(const uint4 *)(cur_b + (slot / 2) * (BN * ROWB) + b_row + j * 32 * ROWB + (b_swz ^ (g * 32)));
#pragma unroll
                for (int p = slot * (NB + na) / G; p < (slot + 1) * (NB + na) / G; ++p) {
                    if (p < NB) request_b(b_at(v % NSB), cb + v / SPB, (v % SPB) * TPS, p);
                    else request_a(a_at(blk ^ 1), cb + blk + 1, t * PA + p - NB);
                }
                __builtin_amdgcn_sched_barrier(SCHED_ALU_MAY_CROSS);
                mfmas(set ^ 1);
                __builtin_amdgcn_sched_barrier(SCHED_ALU_MAY_CROSS);
            }
            // The weights of the next step, requested NSB - 2 steps ago, have landed.  Younger than them: the inputs of that step and all
            // requests since (a step requests weights first; ahead of the first block nothing but weights, and counting fewer is safe).  Before a
            // new block its inputs have landed too; younger than those: the weights requested since.
            auto inputs = [&](int step) { return step >= 0 && step % SPB < A_STEPS ? PA : 0; };
            int pending = inputs(u - NSB + 2);
#pragma unroll
            for (int w = u - NSB + 3; w <= u; ++w) pending += NB + inputs(w);
            if (t == SPB - 1 && pending > (SPB - A_STEPS) * NB) pending = (SPB - A_STEPS) * NB;
            wait_pending<(NSB - 2) * (NB + PA) + PA>(pending);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    mfmas(1);
    wait_loads<0>();
    __builtin_amdgcn_s_barrier();              // the epilogue reuses a0
    asm volatile("" ::: "memory");

    // position of a tile row: counted along the strip, then in the tensor
    store_tiles<DT_BF16, TM, TN>(a, acc, a0 + wave * PATCH, n0 + wn * (BN / WN), lane, 0u, p0 + BM <= geo.rows * tw && c0 + tw <= a.W, [&](int i, int r, unsigned &pos) {
        const int p = p0 + wm * (BM / WM) + i * 32 + r, row = div_by(p, geo.div_tw), c = c0 + p - row * tw;
        pos = (unsigned)((geo.row_lo + row) * a.W + c);
        return row < geo.rows && c < a.W;
    });
}

template <int BM, int BN, int TPS, int NSB>
static LaunchInfo go_conv3(const GemmArgs &a, hipStream_t s, bool dry)
{
    Conv3Geom g;
    g.tw = conv3_strip(a.W);
    g.strips = (a.W + g.tw - 1) / g.tw;
    g.rows = (a.m_hi - a.m_lo) / a.W;
    g.row_lo = a.m_lo / a.W;
    g.tiles_strip = (int)(((int64_t)g.rows * g.tw + BM - 1) / BM);
    g.tiles_m = g.strips * g.tiles_strip;
    g.tiles_n = (a.n_hi - a.n_lo + BN - 1) / BN;
    LaunchInfo li;
    li.workgroups = g.tiles_m * g.tiles_n;
    li.threads = THREADS;
    li.lds_bytes = 2 * conv3_input_bytes(BM) + NSB * TPS * BN * ROWB;
    li.wg_per_cu = 160 * 1024 / li.lds_bytes;
    // 256x64 tiles have two forms: with three weight stages, and with two
    static const std::string name = "conv3_bf16_" + std::to_string(BM) + "x" + std::to_string(BN) + (BM == 256 && BN == 64 && NSB == 3 ? "s3" : "");
    li.kernel = name.c_str();
    li.phases = 1;
    if (dry || li.workgroups == 0) return li;
    // An XCD's band of tiles shares weights along m and inputs along n: number along the side that moves fewer bytes
    const double A = (double)(a.m_hi - a.m_lo) * a.Cin, B = (double)(a.n_hi - a.n_lo) * a.K;
    g.n_major = B + (g.tiles_n < 8 ? g.tiles_n : 8) * A < A + (g.tiles_m < 8 ? g.tiles_m : 8) * B ? 1 : 0;
    divisor(g.tw, g.div_tw);
    divisor(g.tw + 2, g.div_tw2);
    divisor(a.H, g.div_h);
    divisor(g.tiles_strip, g.div_strip);
    divisor(g.tiles_m, g.div_tiles_m);
    divisor(g.tiles_n, g.div_tiles_n);
    GACER_LAUNCH((conv3_kernel<BM, BN, TPS, NSB>), dim3(li.workgroups), dim3(THREADS), 0, s, a, g);
    return li;
}

LaunchInfo launch_conv3(const GemmArgs &a, hipStream_t s, bool dry)
{
    const Conv3Tile t = conv3_tile(a);
    if (t.bn == 128) return go_conv3<256, 128, 1, 3>(a, s, dry);
    if (t.bm == 64) return go_conv3<64, 64, 3, 3>(a, s, dry);
    if (t.bm == 128) return go_conv3<128, 64, 3, 3>(a, s, dry);
    // a third weight stage costs the second workgroup its place on the unit: where there is at most one anyway
    if (conv3_wgs(a, 256, 64) <= 256) return go_conv3<256, 64, 3, 3>(a, s, dry);
    return go_conv3<256, 64, 3, 2>(a, s, dry);
}

}  // namespace gacer
