// K slices side by side in one workgroup: for products with few output tiles and a long K (late convolution layers, short
// token batches, classifiers).  Wave w of the workgroup owns slice w of the K range and a whole 32x32 output tile (fp32: 16x16 where
// there are few); the slice accumulators meet in LDS, are added in ascending order and go through the epilogue, so one launch does what a slice kernel
// plus a finishing pass over fp32 partial tiles in memory did.  Very long K (the first classifier layer of a VGG) is cut once
// more over the grid: workgroup row y owns slices y * S .. y * S + S - 1 and writes its sum to the workspace, splitk_finish
// adds those.  An output element is the sum of its slice chains in that fixed order, whatever part of the operator is launched.
//
// Waves share no operand (their K ranges are disjoint), so each has two LDS stages of its own and there is no barrier in the
// loop: a stage is one batch of 128 bytes of K for 32 + 32 rows, filled by eight direct-to-LDS loads of eight rows each,
// swizzled as in igemm_dma_kernel, read into fragments at once and refilled while the MFMAs of the batch run.
//
// What bounds it.  Long slices: the path from L2 into LDS, about 45 bytes per clock and unit (each wave computes the tile for its
// own K, so 64 rows are moved per 32x32 of output, twice what four waves sharing a 64x64 tile move), hence few tiles only; in
// fp32 the matrix cores from about 4 KB of K on.  Short slices, which is most launches: the length of one wave's chain of
// instructions.  A dependent kernel starts 1.0 us after its predecessor's last store, a dependent instruction takes 1.7 ns, and a
// slice of a few batches is one round trip to memory, so the code in front of the first load and behind the last MFMA is as long
// as the rest.  Hence: arguments in one compact block whose loads the compiler issues at once; byte offsets in 32 bits; rows
// beyond the launched range not masked (what they compute is not stored, and beyond the tensor the descriptor returns zeros);
// the K position in the scalar offset of the loads, so that rows of one pitch (SL_ROWS) need no vector arithmetic per batch; the
// K tail masked by one instruction per load; no requests beyond the slice, but for waves with fewer than two batches; bias and
// residual requested before the K loop; in fp32 two batches in flight, not one (see the fragments' type).  Us per launch in a chain of
// eight dependent ones, before these / with them: bf16 49x160x960 4.73 / 3.51, 144x768x768 4.71 / 3.52, 784x512x1024 7.45 / 5.55, 49x512x4608 9.09 / 7.77; fp32 49x160x960
// 8.66 / 7.30, 784x128x512 6.58 / 5.15, 784x512x2048 25.0 / 21.5, affine + 98x128x128 5.26 / 4.15.
#include <hip/hip_runtime.h>
#include <string>
#include "device_util.h"
#include "gemm_util.h"
#include "kernels.h"
#include "slices_geom.h"

namespace gacer {

// How A rows are addressed: one pitch for all rows; strided 1x1 (rows by image, row and column); taps of which a batch of 128 bytes
// never crosses one; any taps; one pitch with a fused per-channel affine operator in front.
enum { SL_ROWS, SL_STRIDED, SL_TAPS, SL_TAPS_ANY, SL_AFFINE };

struct SlicesArgs {
    const void *x, *w;
    const float *bias;
    const void *res;
    void *y;
    float *ws;
    unsigned x_bytes, w_bytes, bias_bytes, res_bytes;  // ranges of the buffer descriptors (0 where there is no bias or residual)
    unsigned x_pitch, w_pitch;     // bytes between input pixels, between weight rows
    int run, extra;                // tiles per XCD: the first `extra` XCDs have one more
    unsigned div_inner[2];         // tile number -> (outer, inner) tile index
    int inner, n_major;
    int m_lo, m_hi, n_lo, n_hi;
    int K, per, k_last;            // K elements, of which a wave has `per`; see slices_offset
    int y_row, act;
    float alpha;
    int split, vec_out;
    // SL_STRIDED, SL_TAPS, SL_TAPS_ANY
    int HoWo, Wo, H, W, kh, kw, stride, pad, Cin;
    unsigned x_img;                // bytes between images
    unsigned div_howo[2], div_wo[2], div_cin[2], div_kw[2];
    unsigned tap_rows;             // bit r * kw for every tap row r
    // SL_AFFINE
    const float *pre_scale, *pre_shift;
    void *pre_y;
    int pre_act;
};

template <int DT, int LOAD, int S, int PRE_MAX = 0, int TILE = 32>
__global__ __launch_bounds__(64 * S) void slices_kernel(SlicesArgs a)
{
    typedef typename El<DT>::T T;
    constexpr int VEC = El<DT>::VEC;
    constexpr int ESZ = (int)sizeof(T);
    constexpr int BE = 128 / ESZ;               // elements per batch and row
    constexpr int PL = TILE / 8;                // loads of A rows, and of B rows, per batch
    constexpr int HALF = TILE * 128, STAGE = 2 * HALF;                          // bytes of one wave's stage: A rows, then B rows
    constexpr bool T32 = TILE == 32;
    static_assert(T32 || (TILE == 16 && DT == DT_F32), "tile");
    constexpr bool PRE = LOAD == SL_AFFINE, TAPS = LOAD == SL_TAPS || LOAD == SL_TAPS_ANY, PITCH = LOAD == SL_ROWS || PRE;
    __shared__ __align__(1024) unsigned char st0[S * STAGE];
    __shared__ __align__(1024) unsigned char st1[S * STAGE];
    __shared__ __align__(16) float pre[PRE ? 2 * PRE_MAX : 4];                  // scale, shift

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = (int)blockIdx.x & 7;        // see xcd_contiguous
    const int tile = xcd * a.run + min(xcd, a.extra) + ((int)blockIdx.x >> 3);
    const int outer = div_by(tile, a.div_inner), inner = tile - outer * a.inner;
    const int m0 = a.m_lo + (a.n_major ? inner : outer) * TILE, n0 = a.n_lo + (a.n_major ? outer : inner) * TILE;
    const __amdgpu_buffer_rsrc_t xr = rsrc_of(a.x, a.x_bytes), wr = rsrc_of(a.w, a.w_bytes);

    // Load p of a stage fills rows 8 p .. 8 p + 7: lane l row 8 p + l / 8, slot l % 8, which holds logical chunk
    // (l % 8) ^ ((row / 2) % 8) -- two values per lane, by the parity of p
    const int c0 = (lane & 7) ^ (lane >> 4), row0 = lane >> 3;
    const int kl[2] = {c0 * VEC, (c0 ^ 4) * VEC};
    unsigned a_off[PL], a_bad[PL], b_off[PL];      // a_bad: one bit per tap, set where the tap reads nothing
#pragma unroll
    for (int p = 0; p < PL; ++p) {
        const unsigned kb = (unsigned)(kl[p & 1] * ESZ);
        b_off[p] = (unsigned)(n0 + row0) * a.w_pitch + (unsigned)p * 8u * a.w_pitch + kb;
        a_bad[p] = 0u;
        if constexpr (PITCH) {
            a_off[p] = (unsigned)(m0 + row0) * a.x_pitch + (unsigned)p * 8u * a.x_pitch + kb;
        } else {
            const int m = m0 + row0 + 8 * p;
            const int img = div_by(m, a.div_howo), rem = m - img * a.HoWo;
            const int oh = div_by(rem, a.div_wo), ow = rem - oh * a.Wo;
            const int ih0 = oh * a.stride - a.pad, iw0 = ow * a.stride - a.pad;
            a_off[p] = (unsigned)img * a.x_img + (unsigned)(ih0 * a.W + iw0) * a.x_pitch;        // wraps below zero at the border
            if (LOAD != SL_TAPS_ANY) a_off[p] += kb;
            if constexpr (TAPS) a_bad[p] = ~taps_inside(ih0, iw0, a.H, a.W, a.kh, a.kw, a.tap_rows);
        }
    }

    // K range of this wave, in elements; loads at or beyond k_end return zeros.  Only the range that holds the end of K can end
    // inside a batch.
    const int slice = (int)blockIdx.y * S + wave;
    const SlicesRange range = slices_range(a.K, a.per, slice);
    const int k_lo = range.k_lo, k_end = range.k_end;
    const int batches = (k_end - k_lo + BE - 1) / BE;
    unsigned tail[2];                           // OOB where the lane's elements of the last batch lie beyond k_end
#pragma unroll
    for (int h = 0; h < 2; ++h) tail[h] = k_lo + (batches - 1) * BE + kl[h] < k_end ? 0u : OOB;

    // position of the next batch; SL_TAPS: a batch never crosses a tap (128 bytes divide a tap's channels), so the tap is a scalar
    int kb = k_lo, tap = 0, ksx = 0, kci = 0;
    unsigned da = 0;                            // SL_TAPS: byte distance of the batch from the window's origin
    if constexpr (LOAD == SL_TAPS) {
        tap = div_by(k_lo, a.div_cin);
        kci = k_lo - tap * a.Cin;
        const int kr = div_by(tap, a.div_kw);
        ksx = tap - kr * a.kw;
        da = (unsigned)(kr * a.W + ksx) * a.x_pitch + (unsigned)(kci * ESZ);
    }
    auto request = [&](unsigned char *stage) {
        // What is masked gets the top bit (out of range) by arithmetic: of selects the compiler makes branches with loads in both
        // arms, cannot count across them and waits for loads of the newest batch too.
        unsigned bad[2];
        const int soff = slices_offset(kb, a.k_last, ESZ);
        if constexpr (PRE) {                    // requests run past the end of the slice, see below
#pragma unroll
            for (int h = 0; h < 2; ++h) bad[h] = ~(unsigned)((kb + kl[h] - k_end) >> 31) & OOB;
        } else {
            const unsigned last = kb + BE > k_end ? ~0u : 0u, beyond = kb >= k_end ? OOB : 0u;
#pragma unroll
            for (int h = 0; h < 2; ++h) bad[h] = (tail[h] & last) | beyond;
        }
        unsigned off[PL];
        if constexpr (LOAD == SL_TAPS) {
#pragma unroll
            for (int p = 0; p < PL; ++p) off[p] = (a_off[p] + da) | (a_bad[p] << (31 - tap) & OOB) | bad[p & 1];
        } else if constexpr (LOAD == SL_TAPS_ANY) {
            unsigned dl[2], tl[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = div_by(kb + kl[h], a.div_cin), ci = kb + kl[h] - t * a.Cin;
                const int r = div_by(t, a.div_kw), q = t - r * a.kw;
                dl[h] = (unsigned)(r * a.W + q) * a.x_pitch + (unsigned)(ci * ESZ);
                tl[h] = 31u - ((unsigned)t & 31u);
            }
#pragma unroll
            for (int p = 0; p < PL; ++p) off[p] = (a_off[p] + dl[p & 1]) | (a_bad[p] << tl[p & 1] & OOB) | bad[p & 1];
        } else {
#pragma unroll
            for (int p = 0; p < PL; ++p) off[p] = a_off[p] | bad[p & 1];
        }
#pragma unroll
        for (int p = 0; p < PL; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GACER_LDS(stage + p * 1024), 16, (int)off[p], TAPS ? 0 : soff, 0, 0);
#pragma unroll
        for (int p = 0; p < PL; ++p)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, GACER_LDS(stage + HALF + p * 1024), 16, (int)(b_off[p] | bad[p & 1]), soff, 0, 0);
        kb += BE;
        if constexpr (LOAD == SL_TAPS) {
            kci += BE;
            da += 128u;
            if (kci == a.Cin) {                 // next tap: next column, or the first column of the next row
                kci = 0;
                ++tap;
                ++ksx;
                da += a.x_pitch - (unsigned)(a.Cin * ESZ);
                if (ksx == a.kw) { ksx = 0; da += (unsigned)(a.W - a.kw) * a.x_pitch; }
            }
        }
    };

    // the four consecutive channels of one row that thread t of the first 256 (64) finishes: accumulator element e of lane l is row
    // (e/4)*8 + (l/32)*4 + e%4, column l%32 (16x16 tiles: row l/16*4 + e, column l%16); thread t owns element t / 16 of lanes 4 (t % 16)
    // .. + 3 and reads LDS contiguously
    const int e0 = tid >> 4, l0 = (tid & 15) * 4;
    const int m = m0 + (T32 ? (e0 >> 2) * 8 + (l0 >> 5) * 4 + (e0 & 3) : (l0 >> 4) * 4 + e0), n = n0 + (l0 & (TILE - 1));
    const bool inside = tid < TILE * TILE / 4 && m < a.m_hi && n < a.n_hi, n_vec = inside && a.vec_out && n + 4 <= a.n_hi;
    const unsigned o = (unsigned)m * (unsigned)a.y_row + (unsigned)n;
    typedef typename std::conditional<DT == DT_BF16, uint2, uint4>::type R;
    uint4 braw;
    R rraw;
    auto request_epilogue = [&]() {
        braw = buf_load16(rsrc_of(a.bias, a.bias_bytes), n_vec ? (unsigned)n * 4u : OOB);
        if constexpr (DT == DT_BF16) rraw = buf_load8(rsrc_of(a.res, a.res_bytes), n_vec ? o * 2u : OOB);
        else rraw = buf_load16(rsrc_of(a.res, a.res_bytes), n_vec ? o * 4u : OOB);
    };

    // fragments as native vectors: through uint4's members the fp32 ones become scalar loads that the compiler joins again without
    // knowing any more which stage they read, and waits for every outstanding request before them
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef typename std::conditional<DT == DT_BF16, bf16x8, f32x4>::type F;
    typename std::conditional<T32, f32x16, f32x4>::type acc;
    constexpr int NE = T32 ? 16 : 4;
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[e] = 0.f;
    // 16x16 tiles: a quarter of the wave has one k of an MFMA's four.  So that they follow each other as in the 32x32 MFMAs (0, 4, 1, 5, 2, 6, 3,
    // 7 of a 32-byte group), quarters 0 and 2 read the group's first chunk, 1 and 3 its second, the upper two its odd elements.
    const int lrow = lane & (TILE - 1), lhalf = T32 ? lane >> 5 : (lane >> 4) & 1;
    const bool odd = !T32 && lane >= 32;
    const int frag = lrow * 128, frag_lo = (lhalf ^ ((lrow >> 1) & 7)) * 16;
    constexpr int WAIT_BATCH = (2 * PL & 15) | (7 << 4) | (15 << 8);            // vmcnt: the older of the two batches in flight has landed
    constexpr int WAIT_LAST = (7 << 4) | (15 << 8);                             // vmcnt(0)
    constexpr int WAIT_LDS = 15 | (7 << 4) | (3 << 14);                         // lgkmcnt(0)
    // SL_AFFINE: the waves of channel 0 also store the transformed A, four stores per batch behind the batch's requests (the
    // other waves, and masked lanes, store out of range).  vmcnt counts them: four more may be outstanding
    // at every second batch, where a wait for eight would cost one memory latency (at the loop's entry there are no stores yet).
    // With that and the parameters requested together with the operands, DenseNet's 40 such products of 8 images take 299 us in
    // bf16, 378 before.  So that the counts hold, every step requests a batch, beyond the slice one of zeros.
    constexpr int WAIT_STORED = (2 * PL + 4) | (7 << 4) | (15 << 8);
    const __amdgpu_buffer_rsrc_t yr = rsrc_of(PRE ? a.pre_y : nullptr, PRE && n0 == 0 ? (unsigned)(a.m_hi * a.K) * ESZ : 0u);
    auto step = [&](unsigned char *stage, int k0, int wait, bool more) {
        if (wait == WAIT_STORED) __builtin_amdgcn_s_waitcnt(WAIT_STORED);
        else if (wait == WAIT_BATCH) __builtin_amdgcn_s_waitcnt(WAIT_BATCH);
        else __builtin_amdgcn_s_waitcnt(WAIT_LAST);
        asm volatile("" ::: "memory");
        F fa[4], fb[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            fa[g] = *(const F *)(stage + frag + (frag_lo ^ (g * 32)));
            fb[g] = *(const F *)(stage + HALF + frag + (frag_lo ^ (g * 32)));
        }
        // left alone, the scheduler reads fragments group by group between the MFMAs and issues the requests behind most of them
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            __builtin_amdgcn_s_waitcnt(WAIT_LDS);                               // the stage may be refilled
            asm volatile("" ::: "memory");
            request(stage);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (PRE) {                // the stand-alone operator's arithmetic, and its output tensor on the side
                const int kv = k0 + g * 2 * VEC + lhalf * VEC;
                float sc[VEC], sh[VEC];
#pragma unroll
                for (int q = 0; q < VEC; q += 4) {
                    const float4 s4 = *(const float4 *)(pre + kv + q), h4 = *(const float4 *)(pre + PRE_MAX + kv + q);
                    sc[q] = s4.x; sc[q + 1] = s4.y; sc[q + 2] = s4.z; sc[q + 3] = s4.w;
                    sh[q] = h4.x; sh[q + 1] = h4.y; sh[q + 2] = h4.z; sh[q + 3] = h4.w;
                }
                fa[g] = __builtin_bit_cast(F, affine_vec<DT>(__builtin_bit_cast(uint4, fa[g]), sc, sh, a.pre_act));
                const i32x4 v = __builtin_bit_cast(i32x4, fa[g]);
                const unsigned bad = (~(unsigned)(((m0 + lrow - a.m_hi) & (kv - k_end)) >> 31) & OOB) | (odd ? OOB : 0u);
                __builtin_amdgcn_raw_buffer_store_b128(v, yr, (int)((unsigned)((m0 + lrow) * a.K + kv) * ESZ | bad), 0, 0);
            }
            if constexpr (DT == DT_BF16) {
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], fb[g], acc, 0, 0, 0);
            } else if constexpr (!T32) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? fa[g][1] : fa[g][0], odd ? fb[g][1] : fb[g][0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? fa[g][3] : fa[g][2], odd ? fb[g][3] : fb[g][2], acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[g][e], fb[g][e], acc, 0, 0, 0);
            }
        }
    };

    unsigned char *w0 = st0 + wave * STAGE, *w1 = st1 + wave * STAGE;
    int b = 0;
    if constexpr (PRE) {                        // zeros beyond K: a zero element of B meets something finite
        const int pre_n = (a.K + BE - 1) / BE * BE;
        const __amdgpu_buffer_rsrc_t psr = rsrc_of(a.pre_scale, (unsigned)a.K * 4u), phr = rsrc_of(a.pre_shift, (unsigned)a.K * 4u);
        const int k0 = tid * 4;                 // the first 256 S channels are requested ahead of the operands: one memory latency
        const uint4 sc = buf_load16(psr, (unsigned)(k0 * 4)), sh = buf_load16(phr, (unsigned)(k0 * 4));
        asm volatile("" ::: "memory");
        request(w0);
        request(w1);
        if (k0 < pre_n) {
            *(uint4 *)(pre + k0) = sc;
            *(uint4 *)(pre + PRE_MAX + k0) = sh;
        }
        for (int k = k0 + 256 * S; k < pre_n; k += 256 * S) {
            *(uint4 *)(pre + k) = buf_load16(psr, (unsigned)(k * 4));
            *(uint4 *)(pre + PRE_MAX + k) = buf_load16(phr, (unsigned)(k * 4));
        }
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);   // parameters written; the requests stay in flight across the barrier
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        for (; b + 2 <= batches; b += 2) {
            step(w0, k_lo + b * BE, WAIT_BATCH, true);
            step(w1, k_lo + (b + 1) * BE, WAIT_STORED, true);
        }
        if (b < batches) step(w0, k_lo + b * BE, WAIT_BATCH, true);
        __builtin_amdgcn_s_waitcnt(WAIT_LAST);  // the requests beyond the slice have landed: `part` overlays the stage
        asm volatile("" ::: "memory");
        request_epilogue();
    } else {
        // both, whatever the number of batches: behind a branch the compiler no longer knows how many loads follow those of w0, and
        // waits for most of the second batch before it reads the first
        request(w0);
        request(w1);
        request_epilogue();
        for (; b + 4 <= batches; b += 2) {
            step(w0, 0, WAIT_BATCH, true);
            step(w1, 0, WAIT_BATCH, true);
        }
        if constexpr (DT == DT_F32 && T32) mfma_settle<DT>();
        const int rest = batches - b;           // 0 to 3; every batch but the last two requests the one after next
        if (rest == 3) {
            step(w0, 0, WAIT_BATCH, true);
            step(w1, 0, WAIT_BATCH, false);
            step(w0, 0, WAIT_LAST, false);
        } else if (rest == 2) {
            step(w0, 0, WAIT_BATCH, false);
            step(w1, 0, WAIT_LAST, false);
        } else if (rest == 1) {
            step(w0, 0, WAIT_LAST, false);
        } else {
            __builtin_amdgcn_s_waitcnt(WAIT_LAST);                              // an empty slice: its requests, all zeros, have landed
        }
    }

    // ---- sum over the slices and epilogue; each wave's accumulator goes into its own first stage ----
#pragma unroll
    for (int e = 0; e < NE; ++e) *(float *)(w0 + (e * 64 + lane) * 4) = acc[e];
    __syncthreads();
    if (!inside) return;
    const unsigned char *part = st0 + (e0 * 64 + l0) * 4;
    float4 s4 = *(const float4 *)part;
    float v[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
    for (int s = 1; s < S; ++s) {
        s4 = *(const float4 *)(part + s * STAGE);
        v[0] = __fadd_rn(v[0], s4.x); v[1] = __fadd_rn(v[1], s4.y); v[2] = __fadd_rn(v[2], s4.z); v[3] = __fadd_rn(v[3], s4.w);
    }
    T *yg = (T *)a.y;
    if (a.split) {
        const unsigned Nl = (unsigned)(a.n_hi - a.n_lo);
        float *q = a.ws + ((unsigned)blockIdx.y * (unsigned)(a.m_hi - a.m_lo) + (unsigned)(m - a.m_lo)) * Nl + (unsigned)(n - a.n_lo);
        if (n_vec) {
            *(float4 *)q = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            for (int c = 0; c < 4; ++c)
                if (n + c < a.n_hi) q[c] = v[c];
        }
    } else if (n_vec) {
        const float bv[4] = {__uint_as_float(braw.x), __uint_as_float(braw.y), __uint_as_float(braw.z), __uint_as_float(braw.w)};
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = __fmaf_rn(v[c], a.alpha, bv[c]);
        if (a.res) {
            float rv[4];
            load_vec4((const T *)&rraw, rv);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = __fadd_rn(v[c], rv[c]);
        }
        act_vec<4>(v, a.act);
        store_vec4(yg + o, v);
    } else {
        for (int c = 0; c < 4; ++c) finish_one<DT>(v[c], a.alpha, a.bias, a.act, (const T *)a.res, yg, o + c, n + c, a.n_hi);
    }
}

// S waves per workgroup (one K slice each), ksplit workgroups along K
template <int DT, int S, int TILE = 32>
static LaunchInfo go_slices(const GemmArgs &a, hipStream_t s, bool dry, int phase)
{
    typedef typename El<DT>::T T;
    constexpr int ESZ = (int)sizeof(T);
    const int tiles_m = (a.m_hi - a.m_lo + TILE - 1) / TILE, tiles_n = (a.n_hi - a.n_lo + TILE - 1) / TILE;
    LaunchInfo li;
    li.workgroups = tiles_m * tiles_n * a.ksplit;
    li.threads = 64 * S;
    // 16 KB of affine parameters beside the stages of four waves leave room for a second workgroup on the unit, which the rule for
    // four waves counts on where there are more tiles than units; 32 KB do not, and keep the workgroups of a smaller launch on units of
    // their own when other tenants fill some (ResNet-101, DenseNet-121 and MobileNetV3 of 8 images, bf16: round 1472 us, with 16
    // KB throughout 1523).  Affine + product, us, with 32 / 16 KB: fp32 3136x128x128 9.6 / 6.8, 3136x128x1000 28.5 /
    // 21.5, bf16 8.6 / 6.2 and 15.7 / 12.4.  (Sized at launch instead, the array costs bf16 up to 11 %: the compiler then no longer
    // knows that the loads into the stages do not fill it, and waits for them.)
    constexpr int PRE_SMALL = S == 4 ? SLICES_PRE_MAX / 2 : SLICES_PRE_MAX;
    const bool small = a.K <= PRE_SMALL && tiles_m * tiles_n * a.ksplit > 256;
    li.lds_bytes = S * 512 * TILE + (a.pre_scale ? 8 * (small ? PRE_SMALL : SLICES_PRE_MAX) : 0);
    li.wg_per_cu = (160 * 1024) / li.lds_bytes;
    static const std::string shape = std::string(DT == DT_BF16 ? "bf16_x" : "f32_x") + std::to_string(S) + (TILE == 16 ? "_16x16" : "");
    static const std::string n_one = "igemm_slices_" + shape, n_pre = "igemm_affine_slices_" + shape;
    li.kernel = phase == 2 ? "splitk_finish" : a.pre_scale ? n_pre.c_str() : n_one.c_str();
    li.phases = a.ksplit > 1 ? 2 : 1;
    if (dry || li.workgroups == 0) return li;
    if (phase != 2) {
        SlicesArgs b;
        b.x = a.x; b.w = a.w; b.bias = a.bias; b.res = a.res; b.y = a.y; b.ws = a.ws;
        auto range = [](int64_t bytes) { return (unsigned)(bytes < 0 ? 0 : bytes > 0x7FFFFFFF ? 0x7FFFFFFF : bytes); };
        b.split = a.ksplit > 1;
        b.x_bytes = range(a.x_bytes);
        b.w_bytes = range(a.w_bytes);
        b.bias_bytes = a.bias && !b.split ? (unsigned)a.n_hi * 4u : 0u;
        b.res_bytes = a.res && !b.split ? range(((int64_t)(a.m_hi - 1) * a.y_row + a.n_hi) * ESZ) : 0u;
        b.x_pitch = (unsigned)(a.x_pix * ESZ);
        b.w_pitch = (unsigned)(a.w_row * ESZ);
        b.run = tiles_m * tiles_n / 8;
        b.extra = tiles_m * tiles_n % 8;
        b.n_major = tile_order(a, tiles_m, tiles_n, ESZ);
        b.inner = b.n_major ? tiles_m : tiles_n;
        divisor(b.inner, b.div_inner);
        b.m_lo = a.m_lo; b.m_hi = a.m_hi; b.n_lo = a.n_lo; b.n_hi = a.n_hi;
        b.K = a.K;
        b.per = a.kb_per_wave * (64 / ESZ);
        b.k_last = slices_last(a.K, ESZ);
        b.y_row = (int)a.y_row;
        b.act = a.act;
        b.alpha = a.alpha;
        const int Nl = a.n_hi - a.n_lo;
        const uintptr_t AL = 4 * ESZ - 1;
        b.vec_out = b.split ? Nl % 4 == 0 && ((uintptr_t)a.ws & 15) == 0
                            : a.y_row % 4 == 0 && a.n_lo % 4 == 0 && ((uintptr_t)a.y & AL) == 0 && ((uintptr_t)a.res & AL) == 0 && ((uintptr_t)a.bias & 15) == 0;
        b.HoWo = a.Ho * a.Wo; b.Wo = a.Wo; b.H = a.H; b.W = a.W; b.kh = a.kh; b.kw = a.kw; b.stride = a.stride; b.pad = a.pad; b.Cin = a.Cin;
        b.x_img = (unsigned)(a.x_img * ESZ);
        divisor(b.HoWo, b.div_howo);
        divisor(b.Wo, b.div_wo);
        divisor(b.Cin, b.div_cin);
        divisor(b.kw, b.div_kw);
        b.tap_rows = tap_rows(a.kh, a.kw);
        b.pre_scale = a.pre_scale; b.pre_shift = a.pre_shift; b.pre_y = a.pre_y; b.pre_act = a.pre_act;
        const dim3 grid(tiles_m * tiles_n, a.ksplit), block(64 * S);
        const bool taps = !(a.kh == 1 && a.kw == 1 && a.pad == 0);
        // rows of one pitch: unit stride and no gap between images (a single image has none)
        const bool pitch = !taps && a.stride == 1 && a.x_img == (int64_t)a.Ho * a.Wo * a.x_pix;
        if (a.pre_scale && small) GACER_LAUNCH((slices_kernel<DT, SL_AFFINE, S, PRE_SMALL, TILE>), grid, block, 0, s, b);
        else if (a.pre_scale) GACER_LAUNCH((slices_kernel<DT, SL_AFFINE, S, SLICES_PRE_MAX, TILE>), grid, block, 0, s, b);
        else if (pitch) GACER_LAUNCH((slices_kernel<DT, SL_ROWS, S, 0, TILE>), grid, block, 0, s, b);
        else if (!taps) GACER_LAUNCH((slices_kernel<DT, SL_STRIDED, S, 0, TILE>), grid, block, 0, s, b);
        else if (a.Cin * ESZ % 128 == 0) GACER_LAUNCH((slices_kernel<DT, SL_TAPS, S, 0, TILE>), grid, block, 0, s, b);
        else GACER_LAUNCH((slices_kernel<DT, SL_TAPS_ANY, S, 0, TILE>), grid, block, 0, s, b);
    }
    if (a.ksplit > 1 && phase != 1) launch_finish(a, s);
    return li;
}

LaunchInfo launch_slices(const GemmArgs &a, hipStream_t s, bool dry, int phase)
{
    if (a.dtype == DT_BF16) return a.kwaves == 8 ? go_slices<DT_BF16, 8>(a, s, dry, phase) : go_slices<DT_BF16, 4>(a, s, dry, phase);
    // 16x16 tiles give the bits of 32x32 ones with a quarter of the matrix work per workgroup and half of its bytes, for twice the bytes per
    // output: up to two such workgroups per unit.  Us with 32x32 / 16x16, by the number of these: 125x32x1152 (16) 8.67 / 5.50, 1568x32x1152 (196)
    // 8.91 / 5.88, affine + 125x128x992 (64) 10.8 / 7.0, affine + 500x128x352 (256) 6.66 / 4.90, 392x160x960 (250) 7.60 / 5.15, 128x768x768 (384) 6.48 / 5.74,
    // 507x256x1152 (512) 9.01 / 8.49, 1568x96x576 (588) 5.70 / 6.53, 1875x128x1152 (944) 9.02 / 13.3.
    const int64_t t16 = (int64_t)((a.m_hi - a.m_lo + 15) / 16) * ((a.n_hi - a.n_lo + 15) / 16) * a.ksplit;
    // Beside a fused affine's parameters, eight waves leave room for one workgroup per unit: affine + 784x128x896 (392) 10.6 / 12.6.
    if (t16 <= (a.kwaves == 8 && a.pre_scale ? 256 : 512)) return a.kwaves == 8 ? go_slices<DT_F32, 8, 16>(a, s, dry, phase) : go_slices<DT_F32, 4, 16>(a, s, dry, phase);
    return a.kwaves == 8 ? go_slices<DT_F32, 8>(a, s, dry, phase) : go_slices<DT_F32, 4>(a, s, dry, phase);
}

}  // namespace gacer
