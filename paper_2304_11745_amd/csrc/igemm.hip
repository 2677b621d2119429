// Implicit-GEMM convolution / GEMM / attention products on CDNA4 matrix cores.
//
//   Y[m][n] = act( alpha * sum_k A[m][k] * B[n][k] + bias[n] + res[m][n] )
//
// One 256-thread workgroup (4 wavefronts of 64) owns a BM x BN output tile and walks K in blocks of
// KV 16-byte vectors per row.  Global tiles are prefetched two blocks ahead into registers, staged
// through double-buffered LDS and consumed by 32x32 MFMA tiles:
//   fp32 : v_mfma_f32_32x32x2_f32   (true fp32 multiply-accumulate)
//   bf16 : v_mfma_f32_32x32x16_bf16 (fp32 accumulate)
//
// Bit-exactness across decompositions: each output element is the ordered sum of `ksplit` slice
// accumulators; a slice accumulator is one MFMA chain that walks its k range in ascending groups of
// 32 bytes.  ksplit and the slice length are fixed per operator from its unsplit shape, so the order
// of additions never depends on the tile shape, on the position of the element inside a tile, or on
// the launched sub-range.  K tails are zero filled.  A chunk launch (Eq. 5: part of the batch, or part
// of the output channels) therefore produces exactly the bits the unsplit launch produces.
#include <hip/hip_runtime.h>
#include <string>
#include <type_traits>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"

namespace gacer {

static constexpr int THREADS = 256;
enum { LOAD_VEC = 0, LOAD_GATHER = 1, LOAD_BT = 2, LOAD_TAPS = 3, LOAD_AFFINE = 4 };

// Epilogue of the tiles of one wave (first row m_wave, first channel n_wave): store_tiles, or the partial tiles of a K slice into the
// workspace, turned through the wave's patch of LDS so that they leave as whole rows of 32 floats.
template <int DT, int TM, int TN>
__device__ __forceinline__ void igemm_epilogue(const GemmArgs &a, f32x16 (&acc)[TM][TN], unsigned char *patch, int m_wave, int n_wave, int lane,
                                               int slice, int64_t y_off)
{
    if (a.ksplit == 1) {
        store_tiles<DT, TM, TN>(a, acc, patch, n_wave, lane, (unsigned)y_off, m_wave + TM * 32 <= a.m_hi, [&](int i, int r, unsigned &pos) {
            pos = (unsigned)(m_wave + i * 32 + r);
            return (int)pos < a.m_hi;
        });
        return;
    }
    constexpr int PROW = 144;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int Nl = a.n_hi - a.n_lo;
    float *ws = a.ws + (int64_t)slice * (a.m_hi - a.m_lo) * Nl;
    const bool vec = Nl % 4 == 0 && ((uintptr_t)a.ws & 15) == 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4 *)(patch + lrow * PROW + (q * 8 + lhalf * 4) * 4) = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = it * 8 + (lane >> 3), m = m_wave + i * 32 + row, n = n_wave + j * 32 + (lane & 7) * 4;
                const float4 v = *(const float4 *)(patch + row * PROW + (lane & 7) * 16);
                if (m >= a.m_hi || n >= a.n_hi) continue;
                float *p = ws + (int64_t)(m - a.m_lo) * Nl + (n - a.n_lo);
                if (vec && n + 4 <= a.n_hi) {
                    *(float4 *)p = v;
                } else {
                    const float e[4] = {v.x, v.y, v.z, v.w};
                    for (int q = 0; q < 4; ++q)
                        if (n + q < a.n_hi) p[q] = e[q];
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
}

template <int DT, int BM, int BN, int WM, int WN, int KV, int LOAD>
__global__ __launch_bounds__(THREADS) void igemm_kernel(GemmArgs a)
{
    typedef typename El<DT>::T T;
    constexpr int VEC = El<DT>::VEC;            // elements per 16-byte vector
    constexpr int ESZ = (int)sizeof(T);
    constexpr int BK = KV * VEC;                // elements per K block
    constexpr int ROWB = KV * 16 + 16;          // LDS bytes per tile row (16 bytes of padding)
    constexpr int RPP = THREADS / KV;           // tile rows covered by one pass of all threads
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int AV = (BM + RPP - 1) / RPP;    // 16-byte vectors per thread, A tile
    constexpr int BV = (BN + RPP - 1) / RPP;
    constexpr int NV = BN / VEC;                // LOAD_BT: n-vectors per k row of the B tile
    constexpr int BTV = (BK * NV + THREADS - 1) / THREADS;
    constexpr int BREG = LOAD == LOAD_BT ? BTV : BV;
    constexpr bool TAPS = (LOAD == LOAD_TAPS);  // k walks (tap row, tap col, channel); otherwise one tap
    static_assert(WM * WN == 4 && TM >= 1 && TN >= 1, "tile shape");

    __shared__ __align__(16) unsigned char smem[2 * (BM + BN) * ROWB];
    unsigned char *As = smem, *Bs = smem + 2 * BM * ROWB;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int tile = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int by_m = div_by(tile, a.div_tiles_m), by_n = div_by(tile, a.div_tiles_n);
    const int tile_m = __builtin_amdgcn_readfirstlane(a.n_major ? tile - by_m * a.tiles_m : by_n);
    const int tile_n = __builtin_amdgcn_readfirstlane(a.n_major ? by_m : tile - by_n * a.tiles_n);
    const int m0 = a.m_lo + tile_m * BM, n0 = a.n_lo + tile_n * BN;

    const int z = blockIdx.z;
    const int zq = __builtin_amdgcn_readfirstlane(div_by(z, a.div_zh));
    const int zb = a.z_lo + zq, zh = z - zq * a.zh;
    const int64_t x_zoff = zb * a.x_zb + zh * a.x_zh, w_zoff = zb * a.w_zb + zh * a.w_zh;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc((const T *)a.x + x_zoff, a.x_bytes - x_zoff * ESZ);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc((const T *)a.w + w_zoff, a.w_bytes - w_zoff * ESZ);
    const int64_t y_off = zb * a.y_zb + zh * a.y_zh;

    const int HoWo = a.Ho * a.Wo;
    const unsigned x_img = (unsigned)a.x_img * ESZ, x_pix = (unsigned)a.x_pix * ESZ;         // bytes; offsets fit 32 bits
    const int vcol = tid % KV;                  // which 16-byte vector of the row this thread moves
    const int vrow = tid / KV;

    // ---- per-thread A rows: byte offset of the window origin (or OOB) and validity masks of its taps ----
    unsigned a_off[AV], a_hm[AV], a_wm[AV];
#pragma unroll
    for (int i = 0; i < AV; ++i) {
        const int row = vrow + i * RPP;
        const int m = m0 + row;
        const bool ok = (row < BM) && (m < a.m_hi);
        const int mm = ok ? m : a.m_lo;
        const int img = div_by(mm, a.div_howo), rem = mm - img * HoWo;
        const int oh = div_by(rem, a.div_wo), ow = rem - oh * a.Wo;
        const int ih0 = oh * a.stride - a.pad, iw0 = ow * a.stride - a.pad;
        const unsigned at = (unsigned)img * x_img + (unsigned)(ih0 * a.W + iw0) * x_pix;      // wraps below zero at the border
        a_off[i] = ok ? at : OOB;
        a_hm[i] = ok ? 1u : 0u;
        a_wm[i] = 0u;
        if constexpr (TAPS) {                   // one validity bit per tap (kh*kw <= 31 on this path): bit r*kw + q
            a_hm[i] = ok ? taps_inside(ih0, iw0, a.H, a.W, a.kh, a.kw, a.tap_bits) : 0u;
        } else if constexpr (LOAD == LOAD_GATHER) {     // one bit per tap row and per tap column
            a_hm[i] = ok ? bit_run(min(a.H - ih0, a.kh) - max(-ih0, 0), max(-ih0, 0)) : 0u;
            a_wm[i] = bit_run(min(a.W - iw0, a.kw) - max(-iw0, 0), max(-iw0, 0));
        }
    }
    // ---- per-thread B rows: byte offset of the weight row, and whether the row exists ----
    unsigned b_off[BV];
    bool b_ok[BV];
#pragma unroll
    for (int i = 0; i < BV; ++i) {
        const int row = vrow + i * RPP;
        const int n = n0 + row;
        b_ok[i] = row < BN && n < a.n_hi;
        b_off[i] = b_ok[i] ? (unsigned)n * ((unsigned)a.w_row * ESZ) : 0u;
    }

    // K range of this slice, in blocks of BK (kb_per_slice counts 64-byte blocks)
    const int nkb_all = (a.K + BK - 1) / BK;
    const int per = a.kb_per_slice / (KV / 4);
    const int slice = blockIdx.y;
    const int kb_lo = slice * per;
    const int nkb = min(nkb_all, kb_lo + per);
    const int k_end = min(a.K, nkb * BK);       // loads at or beyond k_end return zeros

    // running position of this thread's vector in K: element index kv and, for tapped walks, (r, s, ci)
    int kv = kb_lo * BK + vcol * VEC;
    int kr = 0, ksx = 0, kci = kv;
    if constexpr (TAPS) {
        const int tap = div_by(kv, a.div_cin);
        kci = kv - tap * a.Cin;
        kr = div_by(tap, a.div_kw);
        ksx = tap - kr * a.kw;
    }

    // gather variant, short K: decode k -> (byte offset inside the window, tap row, tap col) once per workgroup
    constexpr int KTAB = LOAD == LOAD_GATHER ? 256 : 1;
    __shared__ int ktab_delta[KTAB], ktab_rq[KTAB];
    const bool use_ktab = LOAD == LOAD_GATHER && a.K <= KTAB;
    if constexpr (LOAD == LOAD_GATHER) {
        if (use_ktab) {
            for (int k = tid; k < a.K; k += THREADS) {
                const int tap = k / a.Cin, ci = k - tap * a.Cin;
                const int r = tap / a.kw, q = tap - r * a.kw;
                ktab_delta[k] = (int)((unsigned)(r * a.W + q) * x_pix + (unsigned)(ci * ESZ));
                ktab_rq[k] = (r << 8) | q;
            }
            __syncthreads();
        }
    }

    uint4 ra[2][AV], rb[2][BREG];
    // LOAD_AFFINE: scale and shift of this thread's channels of the block in flight, and the block's first channel
    constexpr bool PRE = LOAD == LOAD_AFFINE;
    constexpr int PV = PRE ? 2 * (VEC / 4) : 1;
    uint4 rp[2][PV];
    int rkv[2] = {0, 0};
    const bool pre_store = PRE && n0 == 0;      // the tile column that covers output channel 0 writes the affine tensor

    // loads the next K block of this thread (blocks are requested in ascending order, one call per block)
    auto load_global = [&](uint4 *pa, uint4 *pb, uint4 *pp, int &pkv) {
        if constexpr (LOAD == LOAD_GATHER) {
            // element-wise gather: any Cin, any alignment (stem convolutions, ragged K)
            T ea[AV][VEC], eb[BV][VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const int k = kv + e;
                const bool k_ok = k < k_end;
                int r, q;
                unsigned delta;
                if (use_ktab) {                 // short K (stem convolutions): k -> (offset, taps) from the LDS table
                    const int kc = k < KTAB ? k : KTAB - 1;
                    delta = (unsigned)ktab_delta[kc];
                    r = ktab_rq[kc] >> 8;
                    q = ktab_rq[kc] & 255;
                } else {
                    const int tap = k / a.Cin, ci = k - tap * a.Cin;
                    r = (tap / a.kw) & 31;
                    q = (tap - (tap / a.kw) * a.kw) & 31;
                    delta = (unsigned)(r * a.W + q) * x_pix + (unsigned)(ci * ESZ);
                }
#pragma unroll
                for (int i = 0; i < AV; ++i) {
                    const bool ok = k_ok && ((a_hm[i] >> r) & (a_wm[i] >> q) & 1u);
                    ea[i][e] = buf_load1<T>(xr, ok ? a_off[i] + delta : OOB);
                }
#pragma unroll
                for (int i = 0; i < BV; ++i) eb[i][e] = buf_load1<T>(wr, (k_ok && b_ok[i]) ? b_off[i] + (unsigned)(k * ESZ) : OOB);
            }
#pragma unroll
            for (int i = 0; i < AV; ++i) pa[i] = *(const uint4 *)ea[i];
#pragma unroll
            for (int i = 0; i < BV; ++i) pb[i] = *(const uint4 *)eb[i];
        } else {
            const bool k_ok = kv < k_end;
            if constexpr (TAPS) {
                const unsigned delta = (unsigned)(kr * a.W + ksx) * x_pix + (unsigned)(kci * ESZ);
                const unsigned tp = k_ok ? (unsigned)(kr * a.kw + ksx) : 31u;      // bit 31 is never set
#pragma unroll
                for (int i = 0; i < AV; ++i) pa[i] = buf_load16(xr, ((a_hm[i] >> tp) & 1u) ? a_off[i] + delta : OOB);
            } else {
                const unsigned delta = (unsigned)(kv * ESZ);
#pragma unroll
                for (int i = 0; i < AV; ++i) pa[i] = buf_load16(xr, (k_ok && a_hm[i]) ? a_off[i] + delta : OOB);
            }
            if constexpr (LOAD != LOAD_BT) {
                const unsigned delta = (unsigned)(kv * ESZ);
#pragma unroll
                for (int i = 0; i < BV; ++i) pb[i] = buf_load16(wr, (k_ok && b_ok[i]) ? b_off[i] + delta : OOB);
            } else {
                // B stored [k][n]: vectors run along n
                const int kb0 = kv - vcol * VEC;
#pragma unroll
                for (int i = 0; i < BTV; ++i) {
                    const int idx = tid + i * THREADS;
                    const int kk = idx / NV, nv = idx - kk * NV;
                    const int k = kb0 + kk, n = n0 + nv * VEC;
                    const bool ok = idx < BK * NV && k < k_end && n < a.n_hi;
                    pb[i] = buf_load16(wr, ok ? ((unsigned)k * (unsigned)a.w_row + (unsigned)n) * ESZ : OOB);
                }
            }
        }
        if constexpr (PRE) {                    // beyond K both read zero, so the transformed element is act(0) = 0
            const __amdgpu_buffer_rsrc_t psr = make_rsrc(a.pre_scale, (int64_t)a.Cin * 4), phr = make_rsrc(a.pre_shift, (int64_t)a.Cin * 4);
            const bool k_ok = kv < k_end;
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                pp[q] = buf_load16(psr, k_ok ? (unsigned)((kv + 4 * q) * 4) : OOB);
                pp[VEC / 4 + q] = buf_load16(phr, k_ok ? (unsigned)((kv + 4 * q) * 4) : OOB);
            }
            pkv = kv;
        }
        // advance to the next block
        kv += BK;
        if constexpr (TAPS) {
            kci += BK;
            if (a.Cin >= BK) {                  // at most one tap boundary per block: select-only update
                const bool w1 = kci >= a.Cin;
                kci -= w1 ? a.Cin : 0;
                ksx += w1 ? 1 : 0;
                const bool w2 = ksx == a.kw;
                ksx = w2 ? 0 : ksx;
                kr += w2 ? 1 : 0;
            } else {
                const int tap = div_by(kv, a.div_cin);
                kci = kv - tap * a.Cin;
                kr = div_by(tap, a.div_kw);
                ksx = tap - kr * a.kw;
            }
        }
    };

    auto store_lds = [&](int buf, const uint4 *pa, const uint4 *pb, const uint4 *pp, int pkv) {
        float sc[VEC], sh[VEC];
        if constexpr (PRE) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                sc[4 * q] = __uint_as_float(pp[q].x); sc[4 * q + 1] = __uint_as_float(pp[q].y);
                sc[4 * q + 2] = __uint_as_float(pp[q].z); sc[4 * q + 3] = __uint_as_float(pp[q].w);
                sh[4 * q] = __uint_as_float(pp[VEC / 4 + q].x); sh[4 * q + 1] = __uint_as_float(pp[VEC / 4 + q].y);
                sh[4 * q + 2] = __uint_as_float(pp[VEC / 4 + q].z); sh[4 * q + 3] = __uint_as_float(pp[VEC / 4 + q].w);
            }
        }
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            const int row = vrow + i * RPP;
            uint4 va = pa[i];
            if constexpr (PRE) {
                va = affine_vec<DT>(va, sc, sh, a.pre_act);
                if (pre_store && a_hm[i] && pkv < k_end && (BM % RPP == 0 || row < BM))
                    *(uint4 *)((T *)a.pre_y + (int64_t)(m0 + row) * a.Cin + pkv) = va;
            }
            if (BM % RPP == 0 || row < BM) *(uint4 *)(As + (buf * BM + row) * ROWB + vcol * 16) = va;
        }
        if constexpr (LOAD != LOAD_BT) {
#pragma unroll
            for (int i = 0; i < BV; ++i) {
                const int row = vrow + i * RPP;
                if (BN % RPP == 0 || row < BN) *(uint4 *)(Bs + (buf * BN + row) * ROWB + vcol * 16) = pb[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < BTV; ++i) {
                const int idx = tid + i * THREADS;
                const int kk = idx / NV, nv = idx - kk * NV;
                if (idx < BK * NV) {
                    const T *e = (const T *)&pb[i];
#pragma unroll
                    for (int q = 0; q < VEC; ++q) *(T *)(Bs + (buf * BN + nv * VEC + q) * ROWB + kk * (int)sizeof(T)) = e[q];
                }
            }
        }
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int lrow = lane & 31, lhalf = lane >> 5;

    auto compute = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < KV / 2; ++ks) {
            uint4 fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = *(const uint4 *)(As + (buf * BM + wm * (BM / WM) + i * 32 + lrow) * ROWB + ks * 32 + lhalf * 16);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[j] = *(const uint4 *)(Bs + (buf * BN + wn * (BN / WN) + j * 32 + lrow) * ROWB + ks * 32 + lhalf * 16);
            if constexpr (DT == DT_BF16) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[j]),
                                                                            __builtin_bit_cast(bf16x8, fa[i]), acc[i][j], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            const float av = __uint_as_float(e == 0 ? fa[i].x : e == 1 ? fa[i].y : e == 2 ? fa[i].z : fa[i].w);
                            const float bv = __uint_as_float(e == 0 ? fb[j].x : e == 1 ? fb[j].y : e == 2 ? fb[j].z : fb[j].w);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv, av, acc[i][j], 0, 0, 0);
                        }
            }
        }
    };

    // Pipeline: LDS buffer p holds block kb, register set p^1 holds block kb+1 (in flight), and the loads
    // of block kb+2 are issued into register set p before the MFMAs of block kb start.  Loads and LDS
    // stores in the loop body are unconditional (blocks past the end of the slice read as zeros and land in
    // a buffer nobody reads), which keeps the body branch-free and the outstanding-load counts exact.
    load_global(ra[0], rb[0], rp[0], rkv[0]);
    store_lds(0, ra[0], rb[0], rp[0], rkv[0]);
    load_global(ra[1], rb[1], rp[1], rkv[1]);
    __syncthreads();
    int kb = kb_lo;
    for (; kb + 1 < nkb; kb += 2) {             // whole pairs of blocks; a single loop exit keeps one accumulator set
        load_global(ra[0], rb[0], rp[0], rkv[0]);
        compute(0);
        store_lds(1, ra[1], rb[1], rp[1], rkv[1]);
        __syncthreads();
        load_global(ra[1], rb[1], rp[1], rkv[1]);
        compute(1);
        store_lds(0, ra[0], rb[0], rp[0], rkv[0]);
        __syncthreads();
    }
    if (kb < nkb) compute(0);                   // odd block count: the last block already sits in LDS buffer 0
    __syncthreads();                            // the epilogue reuses the tile buffers

    igemm_epilogue<DT, TM, TN>(a, acc, smem + wave * 4608, m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane, slice, y_off);
}

constexpr int DMA_PATCH = 32 * 36 * 4;          // igemm_dma_kernel: bytes of one wave's epilogue patch
constexpr bool dma_own_patch(int stage, int ns) { return stage < DMA_PATCH * ((4 + ns - 1) / ns); }      // whether it needs LDS beside the stages

// Epilogue of a 16x16 tile (fp32): the lane has channels n .. n + 3 of row m of the problem at y_off (a launch of one problem need not be
// the first: a chunk of one image of a batched product).
__device__ __forceinline__ void finish_16x16(const GemmArgs &a, const float __attribute__((ext_vector_type(4))) &acc, int m, int n, int64_t y_off)
{
    if (m >= a.m_hi || n >= a.n_hi) return;
    const int64_t o = (int64_t)m * a.y_row + n + y_off;
    float *y = (float *)a.y + o;
    const float *res = a.res ? (const float *)a.res + o : nullptr;
    if (n + 4 <= a.n_hi && a.y_row % 4 == 0 && a.n_lo % 4 == 0 && y_off % 4 == 0 && (((uintptr_t)a.y | (uintptr_t)a.res | (uintptr_t)a.bias) & 15) == 0) {
        const float4 b = a.bias ? *(const float4 *)(a.bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
        float v[4] = {__fmaf_rn(acc[0], a.alpha, b.x), __fmaf_rn(acc[1], a.alpha, b.y), __fmaf_rn(acc[2], a.alpha, b.z), __fmaf_rn(acc[3], a.alpha, b.w)};
        if (res) {
            const float4 r = *(const float4 *)res;
            v[0] = __fadd_rn(v[0], r.x); v[1] = __fadd_rn(v[1], r.y); v[2] = __fadd_rn(v[2], r.z); v[3] = __fadd_rn(v[3], r.w);
        }
        act_vec<4>(v, a.act);
        store_vec4(y, v);
    } else {
        for (int c = 0; c < 4; ++c) finish_one<DT_F32>(acc[c], a.alpha, a.bias, a.act, (const float *)a.res, (float *)a.y, o + c, n + c, a.n_hi);
    }
}

// ------------------------------------------------------------------------------------------------
// The same product with the global -> LDS leg done by the memory pipeline itself ("buffer_load ... lds", 16 bytes per
// lane on gfx950): tiles go straight from L2 / HBM into LDS without passing through registers, so many K blocks can be
// in flight at once (NS stages of LDS) at no register cost.  What bounds the register-staged kernel above is the
// latency of its single block of prefetch, not a throughput; here block kb + NS - 1 is requested before block kb is
// consumed.
//
// Layout.  One such load makes a wave write 64 x 16 bytes back to back, so tile rows are unpadded (KV x 16 bytes) and
// consecutive lanes fill consecutive 16-byte slots: thread t owns slot t of every pass of 256 slots (RPP = 256 / KV
// tile rows per pass).  Bank conflicts of the fragment reads are avoided by an XOR swizzle instead of padding: the
// 16-byte chunk with logical index q of tile row r sits in slot q ^ swz(r), swz(r) = (r / (256 / ROWB)) % KV, which the
// loading lane applies on the global side (it fetches the logical chunk that belongs into its slot).
//
// Order of additions per output element is the one of igemm_kernel (ascending 32-byte k groups, zero fill beyond the
// K range; a stage that lies wholly beyond K multiplies zeros), so both kernels produce the same bits.
//
// Synchronisation: the loads are counted by vmcnt.  At the end of step kb the wave waits until only the loads of the
// NS - 2 youngest blocks are outstanding (block kb + 1 has landed), and for its own fragment reads, then meets the
// others at a bare s_barrier.  The stages are separate __shared__ arrays so that the compiler can see that a load
// into one stage does not alias the reads of another (with one array it waits for vmcnt(0) before every read).
//
// MF is the edge of an MFMA tile.  16 (fp32 only: v_mfma_f32_16x16x4_f32) is for a launch's surplus tiles, see igemm_dma_kernel: lanes 0-15, 16-31,
// 32-47 and 48-63 then hold one k each of an MFMA's four, and take them from the 32-byte group such that they follow each other as in the
// 32x32 MFMAs (0, 4, 1, 5, 2, 6, 3, 7).
template <int DT, int BM, int BN, int WM, int WN, int KV, int NS, bool TAPS, int MF, typename Stage>
__device__ __forceinline__ void igemm_dma_tile(const GemmArgs &a, Stage stage_at, unsigned char *own_patch, int m0, int n0, int slice, int z)
{
    typedef typename El<DT>::T T;
    constexpr int VEC = El<DT>::VEC;
    constexpr int ESZ = (int)sizeof(T);
    constexpr int BK = KV * VEC;
    constexpr int ROWB = KV * 16;               // unpadded tile row
    constexpr int RPP = THREADS / KV;           // tile rows covered by one pass of all threads
    constexpr int TM = BM / WM / MF, TN = BN / WN / MF;
    constexpr int AV = BM / RPP, BV = BN / RPP; // loads per thread and block
    constexpr int STAGE = (BM + BN) * ROWB;     // of which a stage holds at least as many bytes
    constexpr int R256 = 256 / ROWB;            // tile rows per 256 bytes of LDS (one sweep over the 64 banks)
    constexpr int PATCH = DMA_PATCH;
    constexpr bool OWN_PATCH = dma_own_patch(STAGE, NS);
    static_assert((MF == 32 || (MF == 16 && DT == DT_F32 && TM == 1 && TN == 1)) && WM * WN == 4 && TM >= 1 && TN >= 1 && BM % RPP == 0 && BN % RPP == 0 && NS >= 3 && NS <= 8 && (KV == 4 || KV == 8), "tile shape");
    static_assert((NS - 2) * (AV + BV) < 64, "outstanding loads exceed the counter");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int zq = __builtin_amdgcn_readfirstlane(div_by(z, a.div_zh));
    const int zb = a.z_lo + zq, zh = z - zq * a.zh;
    const int64_t x_zoff = zb * a.x_zb + zh * a.x_zh, w_zoff = zb * a.w_zb + zh * a.w_zh;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc((const T *)a.x + x_zoff, a.x_bytes - x_zoff * ESZ);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc((const T *)a.w + w_zoff, a.w_bytes - w_zoff * ESZ);
    const int64_t y_off = zb * a.y_zb + zh * a.y_zh;

    const int HoWo = a.Ho * a.Wo;
    const unsigned x_img = (unsigned)a.x_img * ESZ, x_pix = (unsigned)a.x_pix * ESZ;         // bytes; offsets fit 32 bits
    const int vrow = tid / KV;                                  // tile row of this thread's slot in pass 0
    const int lcol = (tid % KV) ^ ((vrow / R256) % KV);         // logical chunk that belongs into the slot

    // per-thread A rows: byte offset of the window origin (or OOB) and one bit per tap, set where the tap reads nothing
    unsigned a_off[AV], a_bad[AV];
#pragma unroll
    for (int i = 0; i < AV; ++i) {
        const int m = m0 + vrow + i * RPP;
        const bool ok = m < a.m_hi;
        const int mm = ok ? m : a.m_lo;
        const int img = div_by(mm, a.div_howo), rem = mm - img * HoWo;
        const int oh = div_by(rem, a.div_wo), ow = rem - oh * a.Wo;
        const int ih0 = oh * a.stride - a.pad, iw0 = ow * a.stride - a.pad;
        const unsigned at = (unsigned)img * x_img + (unsigned)(ih0 * a.W + iw0) * x_pix;      // wraps below zero at the border
        a_off[i] = ok ? at : OOB;
        a_bad[i] = TAPS ? ~(ok ? taps_inside(ih0, iw0, a.H, a.W, a.kh, a.kw, a.tap_bits) : 0u) : 0u;
    }
    unsigned b_off[BV];
#pragma unroll
    for (int i = 0; i < BV; ++i) {
        const int n = n0 + vrow + i * RPP;
        b_off[i] = n < a.n_hi ? (unsigned)n * ((unsigned)a.w_row * ESZ) : OOB;
    }

    // K range of this slice, in blocks of BK (kb_per_slice counts 64-byte blocks)
    const int nkb_all = (a.K + BK - 1) / BK;
    const int per = a.kb_per_slice / (KV / 4);
    const int kb_lo = slice * per;
    const int nkb = min(nkb_all, kb_lo + per);
    const int k_end = min(a.K, nkb * BK);       // loads at or beyond k_end return zeros

    int kv = kb_lo * BK + lcol * VEC;
    int kr = 0, ksx = 0, kci = kv;
    if constexpr (TAPS) {
        const int tap = div_by(kv, a.div_cin);
        kci = kv - tap * a.Cin;
        kr = div_by(tap, a.div_kw);
        ksx = tap - kr * a.kw;
    }

    // Requests for the next K block (one block per step, ascending).  A block is AV + BV loads per thread; they are issued
    // one at a time (request_part) so that a step can spread them between its MFMA groups: the unit that moves global
    // data into LDS takes the loads of all four waves in turn, and a wave that queues several at once is held there
    // while its matrix core runs dry.
    const int wave_slot = wave * 1024;
    // What is masked gets an offset with the top bit set (OOB), by arithmetic: of selects the compiler makes branches with
    // loads in both arms, and since it cannot count loads across them it then waits for requests of the newest blocks.
    unsigned rq_bad = 0, rq_da = 0, rq_db = 0, rq_tap = 31u;
    auto request_begin = [&]() {
        rq_bad = ~(unsigned)((kv - k_end) >> 31) & OOB;
        rq_db = (unsigned)(kv * ESZ);
        if constexpr (TAPS) {
            rq_da = (unsigned)(kr * a.W + ksx) * x_pix + (unsigned)(kci * ESZ);
            rq_tap = (unsigned)(kr * a.kw + ksx) & 31u;                         // beyond K rq_bad masks whatever tap this is
        } else {
            rq_da = rq_db;
        }
    };
    auto request_part = [&](unsigned char *stage, int p) {                      // p in [0, AV + BV), a compile-time constant
        if (p < AV) {
            const int i = p;
            const unsigned bad = rq_bad | (TAPS ? (a_bad[i] >> rq_tap) << 31 : 0u);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GACER_LDS(stage + i * RPP * ROWB + wave_slot), 16,
                                                     (int)((a_off[i] + rq_da) | bad), 0, 0, 0);
        } else {
            const int i = p - AV;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, GACER_LDS(stage + (BM + i * RPP) * ROWB + wave_slot), 16,
                                                     (int)((b_off[i] + rq_db) | rq_bad), 0, 0, 0);
        }
    };
    auto request_end = [&]() {
        kv += BK;
        if constexpr (TAPS) {
            kci += BK;
            if (a.Cin >= BK) {                  // at most one tap boundary per block: select-only update
                const bool w1 = kci >= a.Cin;
                kci -= w1 ? a.Cin : 0;
                ksx += w1 ? 1 : 0;
                const bool w2 = ksx == a.kw;
                ksx = w2 ? 0 : ksx;
                kr += w2 ? 1 : 0;
            } else {
                const int tap = div_by(kv, a.div_cin);
                kci = kv - tap * a.Cin;
                kr = div_by(tap, a.div_kw);
                ksx = tap - kr * a.kw;
            }
        }
    };
    auto request = [&](unsigned char *stage) {                                  // a whole block at once (pipeline fill)
        request_begin();
#pragma unroll
        for (int p = 0; p < AV + BV; ++p) request_part(stage, p);
        request_end();
    };

    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typename std::conditional<MF == 32, f32x16, f32x4>::type acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < MF * MF / 64; ++e) acc[i][j][e] = 0.f;

    const int lrow = lane & (MF - 1), lhalf = MF == 32 ? lane >> 5 : (lane >> 4) & 1;
    const bool odd = MF == 16 && lane >= 32;
    // fragment reads: tile row lrow (+ a multiple of MF, which leaves the swizzle unchanged), logical chunk 2 g + lhalf
    const int frag_lo = (lhalf ^ ((lrow / R256) % KV)) * 16;
    const int a_row0 = (wm * (BM / WM) + lrow) * ROWB, b_row0 = (BM + wn * (BN / WN) + lrow) * ROWB;
    constexpr int G = KV / 2;                   // k groups (32 bytes of k) per block; group g lives in register set g & 1
    uint4 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[1][i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[1][j] = make_uint4(0u, 0u, 0u, 0u);
    auto fragments = [&](const unsigned char *stage, int g, int set) {
        const int col = frag_lo ^ (g * 32);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[set][i] = *(const uint4 *)(stage + a_row0 + i * 32 * ROWB + col);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[set][j] = *(const uint4 *)(stage + b_row0 + j * 32 * ROWB + col);
    };
    auto mfmas = [&](int set) {
        if constexpr (DT == DT_BF16) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[set][j]),
                                                                        __builtin_bit_cast(bf16x8, fa[set][i]), acc[i][j], 0, 0, 0);
        } else if constexpr (MF == 16) {
            const uint4 &va = fa[set][0], &vb = fb[set][0];
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(odd ? vb.y : vb.x), __uint_as_float(odd ? va.y : va.x), acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(odd ? vb.w : vb.z), __uint_as_float(odd ? va.w : va.z), acc[0][0], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const uint4 &va = fa[set][i], &vb = fb[set][j];
                        const float av = __uint_as_float(e == 0 ? va.x : e == 1 ? va.y : e == 2 ? va.z : va.w);
                        const float bv = __uint_as_float(e == 0 ? vb.x : e == 1 ? vb.y : e == 2 ? vb.z : vb.w);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv, av, acc[i][j], 0, 0, 0);
                    }
        }
    };

    // vmcnt(N) & lgkmcnt(0): the loads of all but the NS - 2 youngest blocks have landed, own LDS reads are done
    constexpr int PENDING = (NS - 2) * (AV + BV);
    constexpr int WAIT_NEXT = (PENDING & 15) | (7 << 4) | ((PENDING >> 4) << 14);
    constexpr int WAIT_ALL = (7 << 4);
    auto meet = [&](int imm_is_all) {
        if (imm_is_all) __builtin_amdgcn_s_waitcnt(WAIT_ALL); else __builtin_amdgcn_s_waitcnt(WAIT_NEXT);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // One step consumes block kb from `cur` and requests block kb + NS - 1 into the stage that block kb - 1 has left.
    // The step is rotated by one k group: the fragments of the last group of a block are in registers (set 1) when the
    // barrier is passed, and its MFMAs run first in the next step, covering the LDS latency of that step's first
    // fragments.  Slot 0 of a step is therefore the previous block's last group (before the first block: zeros, which
    // leave the accumulators at zero), slots 1 .. G - 1 are groups 0 .. G - 2 of this block.  Each slot issues the
    // fragment reads of the group after it and its share of the block's global requests, then its MFMAs; the
    // scheduling barriers keep that order in the generated code.  The chain of every accumulator still walks k upwards.
    constexpr int SCHED_ALU_MAY_CROSS = 0x2 | 0x4;       // vector and scalar ALU may move across; memory operations and MFMAs stay put
    auto step = [&](const unsigned char *cur, unsigned char *into) {
        request_begin();
#pragma unroll
        for (int slot = 0; slot < G; ++slot) {
            fragments(cur, slot, slot & 1);
#pragma unroll
            for (int p = slot * (AV + BV) / G; p < (slot + 1) * (AV + BV) / G; ++p) request_part(into, p);
            if (slot == G - 1) request_end();   // address arithmetic for the next block: free to mix with the MFMAs below
            __builtin_amdgcn_sched_barrier(SCHED_ALU_MAY_CROSS);
            mfmas((slot & 1) ^ 1);
            __builtin_amdgcn_sched_barrier(SCHED_ALU_MAY_CROSS);
        }
        meet(0);
    };

#pragma unroll
    for (int i = 0; i < NS - 1; ++i) request(stage_at(i));
    meet(0);                                    // block kb_lo has landed
    const int n_blocks = nkb - kb_lo;
    int done = 0;
    for (; done + NS <= n_blocks; done += NS) { // whole rounds over the stages; a single loop exit keeps one accumulator set
#pragma unroll
        for (int i = 0; i < NS; ++i) step(stage_at(i), stage_at((i + NS - 1) % NS));
    }
    const int rest = n_blocks - done;
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
        if (rest > i) step(stage_at(i), stage_at((i + NS - 1) % NS));
    mfmas(1);                                   // last group of the last block
    meet(1);                                    // trailing requests (all beyond K: zeros) have landed; the epilogue reuses the stages

    if constexpr (MF == 16) {
        finish_16x16(a, acc[0][0], m0 + wm * 16 + lrow, n0 + wn * 16 + (lane >> 4) * 4, y_off);
    } else {
        unsigned char *patch = OWN_PATCH ? own_patch + wave * PATCH : stage_at(wave % NS) + (wave / NS) * PATCH;
        igemm_epilogue<DT, TM, TN>(a, acc, patch, m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane, slice, y_off);
    }
}

// The launch.  `surplus` (fp32, 64x64 tiles, one slice): the last tiles, a.surplus of them, are computed as four 32x32 tiles each, by
// workgroups of their own at the end of the grid.  fp32 is bound by the matrix cores, so that a launch takes as long as the unit with
// the most tiles; 784 tiles on 256 units took as long as 1024 (151 us for 6272x512x2304), and take 132 us with the last 16 cut up.
template <int DT, int BM, int BN, int WM, int WN, int KV, int NS, bool TAPS>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(2 * NS * (BM + BN) * KV * 16 <= 160 * 1024 ? 2 : 1)))      // two workgroups per unit where LDS allows
void igemm_dma_kernel(GemmArgs a)
{
    constexpr int STAGE = (BM + BN) * KV * 16;
    constexpr bool OWN_PATCH = dma_own_patch(STAGE, NS);
    __shared__ __align__(1024) unsigned char st0[STAGE];
    __shared__ __align__(1024) unsigned char st1[STAGE];
    __shared__ __align__(1024) unsigned char st2[STAGE];
    __shared__ __align__(1024) unsigned char st3[NS > 3 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char st4[NS > 4 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char st5[NS > 5 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char st6[NS > 6 ? STAGE : 16];
    __shared__ __align__(1024) unsigned char st7[NS > 7 ? STAGE : 16];
    // the stages are separate arrays and always named by a compile-time index, so that the compiler can tell a stage
    // being filled from the one being read (it would otherwise wait for every outstanding load before each LDS read)
    auto stage_at = [&](int i) -> unsigned char * {
        return i == 0 ? st0 : i == 1 ? st1 : i == 2 ? st2 : i == 3 ? st3 : i == 4 ? st4 : i == 5 ? st5 : i == 6 ? st6 : st7;
    };
    __shared__ __align__(16) unsigned char own_patch[OWN_PATCH ? 4 * DMA_PATCH : 16];


    constexpr bool SURPLUS = DT == DT_F32 && BM == 64 && BN == 64;
    const int whole = SURPLUS ? (int)gridDim.x - 4 * a.surplus : (int)gridDim.x;
    const bool cut = SURPLUS && (int)blockIdx.x >= whole;
    const int part = cut ? xcd_contiguous((int)blockIdx.x - whole, 4 * a.surplus) : 0;
    const int tile = cut ? whole + (part >> 2) : xcd_contiguous((int)blockIdx.x, whole);
    const int by_m = div_by(tile, a.div_tiles_m), by_n = div_by(tile, a.div_tiles_n);
    const int tile_m = __builtin_amdgcn_readfirstlane(a.n_major ? tile - by_m * a.tiles_m : by_n);
    const int tile_n = __builtin_amdgcn_readfirstlane(a.n_major ? by_m : tile - by_n * a.tiles_n);
    const int m0 = a.m_lo + tile_m * BM, n0 = a.n_lo + tile_n * BN;
    if constexpr (SURPLUS) {
        if (cut) {
            const int m1 = m0 + (part >> 1 & 1) * 32, n1 = n0 + (part & 1) * 32;
            if (m1 < a.m_hi && n1 < a.n_hi) igemm_dma_tile<DT, 32, 32, 2, 2, KV, NS, TAPS, 16>(a, stage_at, own_patch, m1, n1, 0, 0);
            return;
        }
    }
    igemm_dma_tile<DT, BM, BN, WM, WN, KV, NS, TAPS, 32>(a, stage_at, own_patch, m0, n0, blockIdx.y, blockIdx.z);
}

// ------------------------------------------------------------------------------------------------
// Second pass of a split-K operator: out = act(alpha * (s0 + s1 + ... ) + bias + res), slices added in
// ascending order.  One thread per FV consecutive output channels of the launched sub-range (FV = 4 when
// the range and the pointers allow 16-byte accesses), coalesced along n.  Bound by the chain of one thread: arguments in one struct
// of its own, and slices, bias and residual requested at once, KS slices without a branch (those past the last read it again).
// Us per operator with its pass, before (sixteen conditional loads, the operator's whole argument block) / here, fp32: 8x1000x2048
// in eight slices 7.99 / 7.39, 32x1000x1280 in five 7.77 / 7.31, 147x512x4608 in three 14.24 / 13.74, 49x512x4608 10.40 / 9.99.
struct FinishArgs {
    const float *ws, *bias;
    const void *res;
    void *y;
    int64_t slice;             // elements of a slice
    int groups, Nl, m_lo, n_lo, y_row, last, act;      // threads that have outputs; last: the last slice
    float alpha;
    unsigned div_nl[2];
};

template <typename T, int FV, int KS>
__global__ __launch_bounds__(THREADS) void splitk_finish(FinishArgs a)
{
    const int i = (int)blockIdx.x * THREADS + (int)threadIdx.x;
    if (i >= a.groups) return;
    const int64_t idx = (int64_t)i * FV;
    const int mr = div_by((int)idx, a.div_nl);          // idx < 2^31: the launched sub-range holds fewer elements
    const int n = a.n_lo + ((int)idx - mr * a.Nl);
    const int64_t o = (int64_t)(a.m_lo + mr) * a.y_row + n;
    typedef typename std::conditional<FV == 4, float4, float>::type F;
    F p[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) p[q] = *(const F *)(a.ws + (int64_t)min(q, a.last) * a.slice + idx);
    float bv[FV], rv[FV];
#pragma unroll
    for (int e = 0; e < FV; ++e) bv[e] = rv[e] = 0.f;
    if (a.bias) {
#pragma unroll
        for (int e = 0; e < FV; ++e) bv[e] = a.bias[n + e];
    }
    if (a.res) {
#pragma unroll
        for (int e = 0; e < FV; ++e) rv[e] = load_in((const T *)a.res, o + e);
    }
    float v[FV];
#pragma unroll
    for (int e = 0; e < FV; ++e) v[e] = ((const float *)&p[0])[e];
#pragma unroll
    for (int q = 1; q < KS; ++q)
        if (q <= a.last) {
#pragma unroll
            for (int e = 0; e < FV; ++e) v[e] = __fadd_rn(v[e], ((const float *)&p[q])[e]);
        }
#pragma unroll
    for (int e = 0; e < FV; ++e) v[e] = __fmaf_rn(v[e], a.alpha, bv[e]);
    if (a.res) {
#pragma unroll
        for (int e = 0; e < FV; ++e) v[e] = __fadd_rn(v[e], rv[e]);
    }
    activate_n<FV>(v, a.act);
    if constexpr (FV == 4 && sizeof(T) == 4) {
        *(float4 *)((float *)a.y + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (FV == 4) {
        *(uint2 *)((unsigned short *)a.y + o) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    } else {
        store_out<T>((T *)a.y, o, v[0]);
    }
}

template <typename T, int FV>
static void go_finish(const GemmArgs &a, hipStream_t s)
{
    const int64_t total = (int64_t)(a.m_hi - a.m_lo) * (a.n_hi - a.n_lo);
    FinishArgs b;
    b.ws = a.ws; b.bias = a.bias; b.res = a.res; b.y = a.y;
    b.slice = total;
    b.groups = (int)(total / FV);
    b.Nl = a.n_hi - a.n_lo; b.m_lo = a.m_lo; b.n_lo = a.n_lo; b.y_row = (int)a.y_row; b.last = a.ksplit - 1; b.act = a.act;
    b.alpha = a.alpha;
    divisor(b.Nl, b.div_nl);
    const dim3 grid((unsigned)((b.groups + THREADS - 1) / THREADS)), block(THREADS);
    if (a.ksplit <= 2) GACER_LAUNCH((splitk_finish<T, FV, 2>), grid, block, 0, s, b);
    else if (a.ksplit <= 4) GACER_LAUNCH((splitk_finish<T, FV, 4>), grid, block, 0, s, b);
    else if (a.ksplit <= 8) GACER_LAUNCH((splitk_finish<T, FV, 8>), grid, block, 0, s, b);
    else GACER_LAUNCH((splitk_finish<T, FV, 16>), grid, block, 0, s, b);
}

template <typename T>
static void finish(const GemmArgs &a, hipStream_t s)
{
    const int Nl = a.n_hi - a.n_lo;
    const bool v4 = Nl % 4 == 0 && a.n_lo % 4 == 0 && a.y_row % 4 == 0 && (((uintptr_t)a.ws) & 15) == 0 && (((uintptr_t)a.y) & 15) == 0;
    if (v4) go_finish<T, 4>(a, s);
    else go_finish<T, 1>(a, s);
}

void launch_finish(const GemmArgs &a, hipStream_t s) { a.dtype == DT_BF16 ? finish<unsigned short>(a, s) : finish<float>(a, s); }

static void set_tiling(GemmArgs &b, int tiles_m, int tiles_n)
{
    b.tiles_m = tiles_m;
    b.tiles_n = tiles_n;
    divisor(tiles_m, b.div_tiles_m);
    divisor(tiles_n, b.div_tiles_n);
    divisor(b.zh, b.div_zh);
}
static void set_divisors(GemmArgs &b)
{
    divisor(b.Ho * b.Wo, b.div_howo);
    divisor(b.Wo, b.div_wo);
    divisor(b.Cin, b.div_cin);
    divisor(b.kw, b.div_kw);
    b.tap_bits = tap_rows(b.kh, b.kw);
}

// Tile numbering of a launch.  m-major numbering gives every XCD a band of output rows: A is fetched into one L2 only,
// B into every L2 that holds a band; n-major numbering is the mirror image.  Takes the order that moves fewer bytes
// into the L2s (late convolution layers have far more weights than activations, early ones the opposite).
int tile_order(const GemmArgs &a, int tiles_m, int tiles_n, int esz)
{
    const double Ml = a.m_hi - a.m_lo, Nl = a.n_hi - a.n_lo;
    const double A = Ml * a.stride * a.stride * (double)(a.K / (a.kh * a.kw)) * esz;     // input pixels behind the output rows
    const double B = Nl * (double)a.K * esz;
    const double m_major = A + (tiles_m < 8 ? tiles_m : 8) * B, n_major = B + (tiles_n < 8 ? tiles_n : 8) * A;
    return n_major < m_major ? 1 : 0;
}

// ------------------------------------------------------------------------------------------------
template <int DT, int BM, int BN, int WM, int WN, int KV>
static LaunchInfo go(const GemmArgs &a, hipStream_t s, bool dry, bool vec_ok, int phase)
{
    typedef typename El<DT>::T T;
    constexpr int ROWB = KV * 16 + 16;
    const int tiles_m = (a.m_hi - a.m_lo + BM - 1) / BM, tiles_n = (a.n_hi - a.n_lo + BN - 1) / BN;
    const int z = a.zb * a.zh;
    const int ks = a.b_trans ? 1 : a.ksplit;
    LaunchInfo li;
    li.workgroups = tiles_m * tiles_n * z * ks;
    li.threads = THREADS;
    li.lds_bytes = 2 * (BM + BN) * ROWB;
    const int by_lds = (160 * 1024) / li.lds_bytes;
    li.wg_per_cu = by_lds < 8 ? by_lds : 8;     // 8 wave slots per SIMD, one wave of each workgroup per SIMD
    static const std::string shape = std::string(DT == DT_BF16 ? "bf16_" : "f32_") + std::to_string(BM) + "x" + std::to_string(BN) +
                                     "x" + std::to_string(KV * El<DT>::VEC);
    static const std::string n_vec = "igemm_" + shape, n_bt = "igemm_bt_" + shape, n_gather = "igemm_gather_" + shape,
                             n_taps = "igemm_taps_" + shape, n_pre = "igemm_affine_" + shape;
    const bool taps = !(a.kh == 1 && a.kw == 1 && a.pad == 0);
    if (taps && a.kh * a.kw > 31) vec_ok = false;      // the tapped loader keeps one validity bit per tap in a 32-bit mask
    li.kernel = a.pre_scale ? n_pre.c_str() : a.b_trans ? n_bt.c_str() : (!vec_ok ? n_gather.c_str() : (taps ? n_taps.c_str() : n_vec.c_str()));
    li.phases = ks > 1 ? 2 : 1;
    if (phase == 2) li.kernel = "splitk_finish";
    if (dry || li.workgroups == 0) return li;
    dim3 grid(tiles_m * tiles_n, ks, z), block(THREADS);
    if (phase == 2) {
        if (ks > 1) finish<T>(a, s);
        return li;
    }
    GemmArgs b = a;
    b.n_major = tile_order(a, tiles_m, tiles_n, (int)sizeof(T));
    set_divisors(b);
    set_tiling(b, tiles_m, tiles_n);
    // the picker pairs a fused affine with 128-byte and a B stored [k][n] with 64-byte blocks only
    constexpr int LOAD_OTHER = KV == 8 ? LOAD_AFFINE : LOAD_BT;
    if (KV == 8 ? a.pre_scale != nullptr : a.b_trans != 0)
        GACER_LAUNCH((igemm_kernel<DT, BM, BN, WM, WN, KV, LOAD_OTHER>), grid, block, 0, s, b);
    else if (!vec_ok)
        GACER_LAUNCH((igemm_kernel<DT, BM, BN, WM, WN, KV, LOAD_GATHER>), grid, block, 0, s, b);
    else if (taps)
        GACER_LAUNCH((igemm_kernel<DT, BM, BN, WM, WN, KV, LOAD_TAPS>), grid, block, 0, s, b);
    else            // wide bf16 rows of more than 256 bytes are igemm_dma_kernel's: no loader of their own here, the one for windows takes them too
        GACER_LAUNCH((igemm_kernel<DT, BM, BN, WM, WN, KV, DT == DT_F32 || KV == 4 || BN == 32 ? LOAD_VEC : LOAD_TAPS>), grid, block, 0, s, b);
    if (ks > 1 && phase == 0) finish<T>(a, s);
    return li;
}

// How many of `tiles` 64x64 tiles (fp32, one slice) to cut into quarters: those beyond a multiple of the compute units, up to half of these (a quarter per
// unit and tile then still fits beside the others).  Up to 128 tiles, mostly chunks of decomposed operators, are cut altogether.
// Us whole / cut, by the tiles: chunks of 256 channels, K = 2048: 32 (512 rows) 35.7 / 20.4, 64 35.8 / 20.4, 100 35.9 / 28.2, 128 36.1 / 28.5, K = 144: 32 6.1 / 4.3,
// 64 6.2 / 4.5, 100 and 128 6.3 / 5.3; 272 (4352x256x512) 20.2 / 16.5, 288 (512x2304x768) 28.2 / 21.5, 320 (5120x256x144) 9.8 / 8.3,
// (5120x256x1152, 3x3) 41.4 / 32.4, 356 (5696x256x512) 20.4 / 19.5, 384 (512x3072x768, GELU) 30.6 / 26.6, 588 (9408x256x2304) 114 / 109, 784 (6272x512x2304)
// 151 / 132, 800 (12800x256x2048) 126 / 111, 1568 (25088x256x1152) 134 / 125, 3136 (100352x128x1152) 248 / 239; more than half of
// them: 132 (1352x384x1728) 34.2 / 38.1, 392 (25088x64x576) 24.5 / 26.5, 400 (1568x1024x512) 21.3 / 22.3.
static int surplus_tiles(int tiles)
{
    const int r = tiles % 256;
    return r <= 128 ? r : 0;
}

// launcher of igemm_dma_kernel (operands 16-byte aligned in every stride, B rows contiguous in k, at most 31 taps)
template <int DT, int BM, int BN, int WM, int WN, int KV, int NS>
static LaunchInfo go_dma(const GemmArgs &a, hipStream_t s, bool dry, bool vec_ok, int phase)
{
    typedef typename El<DT>::T T;
    constexpr int STAGE = (BM + BN) * KV * 16;
    const int tiles_m = (a.m_hi - a.m_lo + BM - 1) / BM, tiles_n = (a.n_hi - a.n_lo + BN - 1) / BN;
    const int z = a.zb * a.zh;
    const int ks = a.ksplit;
    const int surplus = DT == DT_F32 && z * ks == 1 ? surplus_tiles(tiles_m * tiles_n) : 0;
    LaunchInfo li;
    li.workgroups = tiles_m * tiles_n * z * ks + 3 * surplus;
    li.threads = THREADS;
    li.lds_bytes = NS * STAGE + (dma_own_patch(STAGE, NS) ? 4 * DMA_PATCH : 0);
    const int by_lds = (160 * 1024) / li.lds_bytes;
    li.wg_per_cu = by_lds < 8 ? by_lds : 8;
    static const std::string shape = std::string(DT == DT_BF16 ? "bf16_" : "f32_") + std::to_string(BM) + "x" + std::to_string(BN) +
                                     "x" + std::to_string(KV * El<DT>::VEC) + "s" + std::to_string(NS);
    static const std::string n_one = "igemm_dma_" + shape, n_taps = "igemm_dma_taps_" + shape;
    const bool taps = !(a.kh == 1 && a.kw == 1 && a.pad == 0);
    li.kernel = taps ? n_taps.c_str() : n_one.c_str();
    li.phases = ks > 1 ? 2 : 1;
    if (phase == 2) li.kernel = "splitk_finish";
    if (dry || li.workgroups == 0) return li;
    dim3 grid(tiles_m * tiles_n + 3 * surplus, ks, z), block(THREADS);
    if (phase == 2) {
        if (ks > 1) finish<T>(a, s);
        return li;
    }
    GemmArgs b = a;
    b.n_major = tile_order(a, tiles_m, tiles_n, (int)sizeof(T));
    set_divisors(b);
    set_tiling(b, tiles_m, tiles_n);
    b.surplus = surplus;
    if (taps) GACER_LAUNCH((igemm_dma_kernel<DT, BM, BN, WM, WN, KV, NS, true>), grid, block, 0, s, b);
    else GACER_LAUNCH((igemm_dma_kernel<DT, BM, BN, WM, WN, KV, NS, false>), grid, block, 0, s, b);
    if (ks > 1 && phase == 0) finish<T>(a, s);
    return li;
}

// Tile of igemm_dma_kernel in bf16.  Two things bound these launches: the bytes that a unit draws from its L2, which the stages receive
// at 105 to 115 bytes per ns (a 64x64 tile alone on its unit takes 0.2 us per 128 bytes of K; its 16 KB alone take 0.15 us, the matrix cores alone
// 0.05), and what a tile costs beside its K loop (1 us for 64x64, 4 for 128x128 with one workgroup per unit).  So: the
// largest tile of which about one per unit is left, counted in workgroups, and smaller ones the shorter K is.
// Us a launch in a chain, 64x64 / 128x64 / 128x128 / 256x128, by the workgroups of 128x64: 3136x256x1024 (100) 6.9 / 9.1 / 11.5 / 18.4, 12544x128x512
// (196) 6.4 / 6.3 / 8.6 / 12.3, 1568x1280x320 (260) 6.4 / 7.3 / 8.5 / 11.4, 50176x64x256 (392) 8.9 / 7.1 / 9.2 / 10.8, 12544x256x512 (392) 11.0 / 9.0 / 9.6 / 13.2,
// 3136x1024x256 with a residual (400) 9.3 / 7.8 / 8.7 / 12.0, 12544x512x128 with a residual (784) 11.8 / 9.3 / 10.3 / 11.4, 12544x512x256 (784) 12.6 / 11.5 / 10.7 / 11.6, 3136x2048x512 with a
// residual (800) 19.5 / 18.6 / 16.2 / 17.2, 12544x1024x256 with a residual (1568) 23.8 / 21.1 / 21.4 / 19.2; long K: 2048x768x768 (192) 7.9 / 8.4 / 10.4 / 15.8,
// 2048x768x3072 (192) 19.9 / 18.8 / 23.0 / 45.9, 4096x768x768 (384) 11.2 / 12.0 / 11.2 / 16.0, 4096x768x3072 (384) 31.5 / 30.3 / 25.0 / 45.7, 1024x3072x768 with a GELU
// (384) 13.0 / 14.7 / 17.8 / 29.0, 8192x768x3072 (768) 60.5 / 48.7 / 49.9 / 48.7, 8192x2304x768 (2304) 55.6 / 50.6 / 49.1 / 46.1; and 128x32 / 64x64 for N <= 32:
// 25088x32x1152 (3x3) 7.9 / 9.1, 50176x32x192 5.7 / 7.9.
// Where a launch has a few workgroups more than the units hold, us 64x64 / 128x64 (64-byte blocks of K) / 128x64 / 128x128, by the workgroups of 128x64:
// 66560x64x1024 (520) 24.7 / - / 28.5 / 32.4, 102400x64x1024 (800) 35.8 / - / 38.3 / 43.8, 66560x64x2048 (520) 48.5 / - / 53.9 / 60.4, 33856x128x1024 (530)
// 20.3 / - / 21.3 / 23.4, 16640x256x768 (520) 16.0 / - / 17.2 / 16.8, 6272x1024x1024 (784) 26.1 / - / 23.9 / 21.9, 2560x3072x3072 (960) 109 / - / 79.7 / 70.3;
// 66560x64x384 (520) 13.6 / 14.8 / 15.9 / -, 89600x64x384 (700) 17.3 / 16.1 / 17.9 / -, 140800x64x512 (1100) - / 28.7 / 30.5 / -; 33920x256x512 (1060) - / - / 21.3 / 21.9;
// 100352x64x2160 (784, 3x3) 59.7 / - / 54.0 / -.  Before (64x64 and 128x128 tiles staged through registers below 1.5 KB of K, fewer
// tiles to choose from above) 98 such shapes took 9 % longer, 12544x96x576 8.5, 25088x32x1152 11.1, 12544x256x512 11.5, 4096x768x3072 31.7.
static LaunchInfo pick_dma_bf16(const GemmArgs &a, hipStream_t s, bool dry, int phase)
{
    const int64_t M = a.m_hi - a.m_lo, N = a.n_hi - a.n_lo, z = (int64_t)a.zb * a.zh * a.ksplit, k_bytes = (int64_t)a.K * 2;
    const bool taps = !(a.kh == 1 && a.kw == 1 && a.pad == 0);
    auto wgs = [&](int bm, int bn) { return (M + bm - 1) / bm * ((N + bn - 1) / bn) * z; };
    if (N <= 32) return go_dma<DT_BF16, 128, 32, 4, 1, 8, 3>(a, s, dry, true, phase);
    const int64_t w = wgs(128, 64);
    // A GELU's epilogue (erf) takes as long as a kilobyte of K, and only other workgroups of the unit cover it: smaller tiles, or those of which more fit.
    // Us 64x64 / 128x64 (64-byte blocks) / 128x64 / 128x128, by the workgroups of 128x64: K = 256 384 (900x3072) 8.4 / 10.1 / 10.1 / 14.1, 480 12.1 / 10.7 / 10.6 / 14.5, 768
    // 14.2 / 13.1 / 17.1 / 16.4, 1152 18.7 / 20.6 / 23.9 / 26.7, 3072 43.6 / 37.5 / 46.5 / 44.9; K = 512 384 10.4 / 12.2 / 11.9 / 16.1, 512 15.2 / 13.8 / 12.9 / 17.0, 576 15.4 / 16.1 /
    // 19.3 / 18.3, 1008 22.5 / 21.9 / 22.0 / 21.8, 1152 24.6 / 26.2 / 28.9 / 31.7, 3072 57.8 / 53.6 / 64.1 / 57.4; K = 768 672 21.0 / 21.6 / 22.9 / 23.5, 816 26.0 / 27.3 / 25.7 /
    // 25.0, 1136 30.6 / 33.5 / 33.9 / 39.9, 1344 42.5 / 38.3 / 40.8 / 42.5; K = 2048 192 16.9 / 22.6 / 18.4 / 27.6, 576 36.8 / 45.4 / 40.8 / 40.5, 672 44.7 / 46.7 / 42.2 / 43.3.
    const bool gelu = !taps && a.act == ACT_GELU;
    if (gelu && k_bytes <= 1024) {
        if (w < 450 || (w > 1024 && w <= 1200)) return go_dma<DT_BF16, 64, 64, 2, 2, 8, 3>(a, s, dry, true, phase);
        if (w > 512 || k_bytes <= 512) return go_dma<DT_BF16, 128, 64, 2, 2, 4, 3>(a, s, dry, true, phase);
        return go_dma<DT_BF16, 128, 64, 2, 2, 8, 3>(a, s, dry, true, phase);
    }
    if (gelu && ((w > 512 && w <= (k_bytes <= 2048 ? 800 : k_bytes <= 3072 ? 700 : k_bytes <= 4096 ? 600 : 512)) || (w > 1024 && w <= 1200 && k_bytes <= 3072)))
        return go_dma<DT_BF16, 64, 64, 2, 2, 8, 3>(a, s, dry, true, phase);
    const bool wide = (N + 127) / 128 * 128 <= (N + 63) / 64 * 64;             // 128 columns waste no more than 64
    if (wide && k_bytes >= 512) {
        if (wgs(256, 128) >= 384) return go_dma<DT_BF16, 256, 128, 2, 2, 4, 3>(a, s, dry, true, phase);
        const int64_t w2 = wgs(128, 128);
        // two per unit; some more than these wait for a whole second wave of them
        if (k_bytes <= 1024 ? w2 >= 384 && (w2 <= 512 || w2 > 560 || k_bytes <= 576) : w2 > 256 && (taps || (w2 > 384 && w2 <= 512)))
            return go_dma<DT_BF16, 128, 128, 2, 2, 4, 4>(a, s, dry, true, phase);
        // one workgroup per unit: nothing covers the epilogue, so where that is long (erf) only with a long K (us 128x64 / here: 2688x1024x1024 14.7 / 20.3, x2048
        // 24.7 / 27.7, x3072 34.2 / 33.5, x4096 40.4 / 38.3)
        if (k_bytes >= (a.act == ACT_GELU ? 6144 : 1536) && w2 >= 160 && w2 <= 256) return go_dma<DT_BF16, 128, 128, 2, 2, 8, 3>(a, s, dry, true, phase);
    }
    if (k_bytes <= 512 ? w >= 300 : k_bytes <= 1024 && N <= 64 && w > 512) return go_dma<DT_BF16, 128, 64, 2, 2, 4, 3>(a, s, dry, true, phase);       // four per unit
    // two per unit, with the same wait; 64x64 tiles, of which there are three per unit, wait for less
    const bool spill = !taps && w > 512 && k_bytes > 1024 && w <= (k_bytes <= 2048 ? (N <= 64 ? 832 : 600) : N <= 64 ? 640 : 512);
    if (!spill && (k_bytes <= 1024 ? w >= 300 : w > 400 || (k_bytes >= 4096 && w >= (gelu ? 300 : 192)))) return go_dma<DT_BF16, 128, 64, 2, 2, 8, 3>(a, s, dry, true, phase);
    // alone on its unit with a long K a fourth stage pays (1024x768x768 7.0 -> 6.5); with more workgroups it costs one of them its place
    if (wgs(64, 64) <= 256 && k_bytes >= (taps ? 4096 : 1024)) return go_dma<DT_BF16, 64, 64, 2, 2, 8, 4>(a, s, dry, true, phase);
    return go_dma<DT_BF16, 64, 64, 2, 2, 8, 3>(a, s, dry, true, phase);
}

template <int DT>
static LaunchInfo pick(const GemmArgs &a, hipStream_t s, bool dry, int phase)
{
    constexpr int VEC = El<DT>::VEC;
    const bool vec_ok = (a.Cin % VEC == 0) && (a.x_pix % VEC == 0) && (a.x_img % VEC == 0) && (a.w_row % VEC == 0) &&
                        (a.x_zb % VEC == 0) && (a.x_zh % VEC == 0) && (a.w_zb % VEC == 0) && (a.w_zh % VEC == 0) &&
                        (((uintptr_t)a.x) % 16 == 0) && (((uintptr_t)a.w) % 16 == 0);
    const int M = a.m_hi - a.m_lo, N = a.n_hi - a.n_lo;
    const int64_t z = (int64_t)a.zb * a.zh * (a.b_trans ? 1 : a.ksplit);
    // Tile choice is free (it never changes the bits): narrowest N padding first, then the cheapest shape.
    auto waste = [&](int bn) { return (double)((N + bn - 1) / bn * bn) / (double)N; };
    int bn = 128;
    if (waste(64) < waste(bn) - 1e-9) bn = 64;
    if (waste(32) < waste(bn) - 1e-9) bn = 32;
    auto wgs = [&](int bm, int bnn) { return (int64_t)((M + bm - 1) / bm) * ((N + bnn - 1) / bnn) * z; };
    // Cost of a tile shape: workgroups landing on the busiest compute unit x outputs per workgroup / relative
    // efficiency of the shape.  Measured: bf16 gains from the 128x128 tile (fewer LDS reads per MFMA); fp32 MFMAs are slow
    // enough that all shapes are equal and only the fill counts, which is never worse with the 64x64 tile.
    // Fewer workgroups than compute units leaves units idle and hides no latency: penalised.
    auto cost = [&](int bm, int bnn, double eff) {
        const int64_t w = wgs(bm, bnn);
        return (double)((w + 255) / 256) * bm * bnn / eff * (w < 256 ? 1.1 : 1.0);
    };
    enum { T64x64, T128x128, T128x32 } shape = T64x64;
    if (bn < 64) shape = T128x32;
    else if (DT == DT_BF16 && bn == 128 && cost(128, 128, 1.0) < cost(64, 64, 0.8) * 0.999) shape = T128x128;
    // kernels staged through registers, with blocks of 128 (KV = 8) or 64 bytes of K
    auto staged = [&](auto kv, bool vec) {
        constexpr int KV = decltype(kv)::value;
        if constexpr (DT == DT_BF16)
            if (shape == T128x128) return go<DT, 128, 128, 2, 2, KV>(a, s, dry, vec, phase);
        if (shape == T64x64) return go<DT, 64, 64, 2, 2, KV>(a, s, dry, vec, phase);
        return go<DT, 128, 32, 4, 1, KV>(a, s, dry, vec, phase);
    };
    const std::integral_constant<int, 8> blocks128;
    const std::integral_constant<int, 4> blocks64;
    // fused per-channel affine: the A tile passes through registers (the executor fuses only 16-byte aligned, vector-multiple operands)
    if (a.pre_scale) return staged(blocks128, true);
    // The direct-to-LDS pipeline (igemm_dma_kernel) wins once the K loop is long enough to fill its stages: in bf16 from 256 bytes of K on
    // (windows, with their longer address code: 512), fp32 from 512 bytes (windows 1.5 KB): us on the register-staged kernel / here,
    // 25088x128x256 23.4 / 20.6, 392x1280x320 10.5 / 9.1, 1568x1024x256 14.3 / 14.0, 12544x512x128 24.7 / 24.8, 4704x256x256 13.4 / 10.3, below
    // 6272x576x96 13.5 / 13.7, 25088x256x64 16.9 / 17.1.
    const bool taps = !(a.kh == 1 && a.kw == 1 && a.pad == 0);
    const int64_t k_bytes = (int64_t)a.K * (int64_t)sizeof(typename El<DT>::T);
    if (vec_ok && !a.b_trans && (!taps || a.kh * a.kw <= 31)) {
        if constexpr (DT == DT_BF16) {
            // N <= 32: two of these workgroups fit a unit, three of the register-staged ones (six with 64-byte blocks).  Rows go where fewer waves of
            // workgroups are needed, here if both need as many; windows of up to 64 channels stay there where there are many.  Us there / here, by the
            // workgroups: rows of K = 128 784 (two halves) 19.0 / 20.5, 1568 15.1 / 17.8, 2809 23.5 / 27.3, K = 136 512 6.8 / 6.2, 600 7.7 / 8.2, 800 9.9 / 9.6, 1300
            // 15.7 / 16.8, K = 256 700 11.9 / 12.1, 1000 15.9 / 15.7, 2500 32.1 / 34.4; 3x3 of 32 channels 784 11.9 / 10.9, 1960 19.3 / 19.3, 2940 26.0 / 27.7, of
            // 64 1960 27.7 / 27.7, 2940 36.8 / 37.8, of 96 2940 53.2 / 50.1.
            const int64_t w = wgs(128, 32), there = k_bytes <= 256 ? 1536 : 768;
            const bool narrow = N <= 32 && (taps ? w > 2048 && k_bytes <= 1152 : (w + 511) / 512 > (w + there - 1) / there);
            if (k_bytes >= (taps ? 512 : 256) && !narrow) return pick_dma_bf16(a, s, dry, phase);
        } else {
            if (shape != T128x32 && k_bytes >= (taps ? 1536 : 512)) return go_dma<DT, 64, 64, 2, 2, 8, 3>(a, s, dry, vec_ok, phase);
        }
    }
    // short K, or the latency-bound gather loader (more waves per unit): 64-byte blocks
    if (a.b_trans || a.K <= 16 * VEC || !vec_ok) return staged(blocks64, vec_ok);
    return staged(blocks128, vec_ok);
}

LaunchInfo launch_igemm(const GemmArgs &a, hipStream_t s, bool dry, int phase)
{
    if (a.attn_scores) return launch_attention(a, s, dry);
    if (a.dw) return launch_expand_dw(a, *a.dw, s, dry);
    if (a.stem) return launch_stem(a, s, dry);
    if (a.halo) return launch_conv3(a, s, dry);
    if (a.kwaves) return launch_slices(a, s, dry, phase);
    if (rows_takes(a)) return launch_rows(a, s, dry || phase == 2);
    return a.dtype == DT_BF16 ? pick<DT_BF16>(a, s, dry, phase) : pick<DT_F32>(a, s, dry, phase);
}

}  // namespace gacer
