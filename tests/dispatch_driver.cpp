// Which kernel, and how many workgroups, the launchers of the built library choose (dry runs: nothing is launched, no GPU is needed).
// Exit code 0 = every check held.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include "../paper_2304_11745_amd/csrc/expand_geom.h"

using namespace gacer;

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); std::exit(1); } } while (0)

static LaunchInfo depthwise(int dtype, int n, int h, int w, int c, int k, int stride, int pad)
{
    StreamArgs a;
    std::memset(&a, 0, sizeof a);
    a.x = a.w = a.y = (void *)0x10000;           // aligned, never dereferenced
    a.dtype = dtype;
    a.N = n; a.H = h; a.W = w; a.C = c; a.k = k; a.stride = stride; a.pad = pad;
    a.Ho = (h + 2 * pad - k) / stride + 1; a.Wo = (w + 2 * pad - k) / stride + 1;
    a.n_hi = n; a.c_hi = c; a.x_pitch = a.y_pitch = c;
    return launch_dwconv(a, nullptr, true);
}

// A window position is a scalar offset of the tiled kernels' loads: none may pass the tensor and the pixels in front of it.
static void check_depthwise_windows()
{
    int left = 0, tiled = 0;
    for (int dtype : {DT_F32, DT_BF16})
        for (int k : {3, 5})
            for (int stride : {1, 2})
                for (int pad = 0; pad <= k; ++pad)
                    for (int n = 1; n <= 2; ++n)
                        for (int h = 1; h <= 9; ++h)
                            for (int w = 1; w <= 9; ++w)
                                for (int c : {8, 64, 40000, 400000}) {
                                    if (h + 2 * pad < k || w + 2 * pad < k) continue;
                                    const LaunchInfo li = depthwise(dtype, n, h, w, c, k, stride, pad);
                                    const int Ho = (h + 2 * pad - k) / stride + 1, Wo = (w + 2 * pad - k) / stride + 1;
                                    const long range = (long)n * h * w + pad * (w + 1);
                                    auto reach = [&](int th, int tw) { return (long)((th - 1) * stride + k - 1) * w + (tw - 1) * stride + k - 1; };
                                    auto wgs = [&](int th, int tw, int v) { return ((long)n * ((Ho + th - 1) / th) * ((Wo + tw - 1) / tw) * (c / v) + 255) / 256; };
                                    if (reach(1, 1) >= range) {
                                        CHECK(li.kernel == std::string(k == 5 ? "dwconv5x5" : "dwconv"));
                                        ++left;
                                        continue;
                                    }
                                    CHECK(li.kernel == std::string(k == 5 ? "dwconv5x5_tiled" : "dwconv3x3"));
                                    ++tiled;
                                    // some tile whose window fits makes this many workgroups
                                    bool ok = li.workgroups == wgs(1, 1, dtype == DT_BF16 ? 2 : 4);
                                    for (int tw = 1; tw <= 4; tw *= 2) ok = ok || (reach(2, tw) < range && li.workgroups == wgs(2, tw, 4));
                                    CHECK(ok);
                                }
    CHECK(left > 100 && tiled > 1000);
    CHECK(depthwise(DT_F32, 1, 1, 1, 64, 3, 1, 1).kernel == std::string("dwconv"));
    CHECK(depthwise(DT_BF16, 1, 2, 2, 64, 5, 1, 2).kernel == std::string("dwconv5x5"));
    CHECK(depthwise(DT_BF16, 2, 2, 2, 64, 3, 1, 1).kernel == std::string("dwconv3x3"));
}

// A product of M rows, N channels and K elements per row (or K input channels under a k x k window on an image of M positions).
static GemmArgs product(int dtype, int M, int N, int K, int k = 1)
{
    GemmArgs a;
    std::memset(&a, 0, sizeof a);
    a.x = a.w = a.y = (void *)0x10000;
    a.dtype = dtype;
    a.H = M; a.W = 1; a.Cin = K; a.Ho = M; a.Wo = 1;
    a.kh = a.kw = k; a.stride = 1; a.pad = k / 2; a.K = K * k * k;
    a.x_pix = K; a.x_img = (int64_t)M * K; a.w_row = a.K; a.y_row = N;
    a.m_hi = M; a.n_hi = N; a.alpha = 1.f;
    a.zb = a.zh = 1; a.ksplit = 1; a.kb_per_slice = 1 << 20;
    return a;
}

// The kernels that stage bf16 rows through registers have no loader for aligned single-tap rows of more than 256 bytes and more than 32 channels: none
// may come there.  Up to 32 channels the tiles' number decides.
static void check_bf16_rows()
{
    int dma = 0;
    for (int K = 8; K <= 4096; K += K < 256 ? 8 : 248)
        for (int M : {1, 31, 300, 5000, 70000})
            for (int N : {1, 32, 33, 64, 128, 200, 1000}) {
                const std::string name = launch_igemm(product(DT_BF16, M, N, K), nullptr, true).kernel;
                const bool is_dma = name.find("igemm_dma_bf16_") == 0, many = N <= 32 && M > 65536 && (K == 128 || M < 98304);
                CHECK(name.find("igemm_bf16_") != 0 || N <= 32 || name.rfind("x32") == name.size() - 3);
                CHECK((K * 2 >= 256 && !many) == is_dma);
                dma += is_dma;
            }
    CHECK(dma > 450);
    auto rows = [](int tiles, int K) { return std::string(launch_igemm(product(DT_BF16, tiles * 128, 32, K), nullptr, true).kernel); };
    for (int K : {136, 512}) {
        for (int tiles : {100, 512, 769, 1024}) CHECK(rows(tiles, K) == "igemm_dma_bf16_128x32x64s3");
        for (int tiles : {513, 768, 1025, 1600, 2500}) CHECK(rows(tiles, K) == "igemm_bf16_128x32x64");
    }
    CHECK(rows(512, 128) == "igemm_dma_bf16_128x32x64s3" && rows(513, 128) == "igemm_bf16_128x32x32" && rows(1024, 128) == "igemm_bf16_128x32x32");
    // windows of few channels, and 128x64 tiles that would begin a second wave on the units
    auto kernel = [](int M, int N, int K, int k) { return std::string(launch_igemm(product(DT_BF16, M, N, K, k), nullptr, true).kernel); };
    CHECK(kernel(2048 * 128, 32, 64, 3) == "igemm_dma_taps_bf16_128x32x64s3" && kernel(2049 * 128, 32, 64, 3) == "igemm_taps_bf16_128x32x64");
    CHECK(kernel(2049 * 128, 32, 72, 3) == "igemm_dma_taps_bf16_128x32x64s3");
    CHECK(kernel(512 * 128, 64, 1024, 1) == "igemm_dma_bf16_128x64x64s3" && kernel(513 * 128, 64, 1024, 1) == "igemm_dma_bf16_64x64x64s3");
    CHECK(kernel(832 * 128, 64, 1024, 1) == "igemm_dma_bf16_64x64x64s3" && kernel(833 * 128, 64, 1024, 1) == "igemm_dma_bf16_128x64x64s3");
    CHECK(kernel(384 * 64, 256, 2048, 1) == "igemm_dma_bf16_128x64x64s3" && kernel(386 * 64, 256, 2048, 1) == "igemm_dma_bf16_128x128x32s4");
    GemmArgs gelu = product(DT_BF16, 2688, 1024, 3072);
    gelu.act = ACT_GELU;
    CHECK(launch_igemm(gelu, nullptr, true).kernel == std::string("igemm_dma_bf16_128x128x64s3"));
    gelu = product(DT_BF16, 2688, 1024, 3064);
    CHECK(launch_igemm(gelu, nullptr, true).kernel == std::string("igemm_dma_bf16_128x128x64s3"));
    gelu.act = ACT_GELU;
    CHECK(launch_igemm(gelu, nullptr, true).kernel == std::string("igemm_dma_bf16_128x64x64s3"));
    auto with_gelu = [](int M, int N, int K) { GemmArgs a = product(DT_BF16, M, N, K); a.act = ACT_GELU; return std::string(launch_igemm(a, nullptr, true).kernel).substr(15); };
    CHECK(with_gelu(896, 3072, 256) == "64x64x64s3" && with_gelu(1280, 3072, 256) == "128x64x32s3" && with_gelu(3072, 3072, 256) == "64x64x64s3");
    CHECK(with_gelu(896, 3072, 512) == "64x64x64s3" && with_gelu(1280, 3072, 512) == "128x64x64s3" && with_gelu(1408, 3072, 512) == "128x64x32s3");
    CHECK(with_gelu(1280, 3072, 768) == "128x64x64s3" && with_gelu(1408, 3072, 768) == "64x64x64s3" && with_gelu(2048, 3072, 768) == "64x64x64s3" &&
          with_gelu(2176, 3072, 768) == "128x128x32s4" && with_gelu(3072, 3072, 768) == "64x64x64s3" && with_gelu(3328, 3072, 768) == "128x64x64s3");
    CHECK(with_gelu(512, 3072, 2048) == "64x64x64s3" && with_gelu(1536, 3072, 2048) == "64x64x64s3" && with_gelu(1664, 3072, 2048) == "128x64x64s3");
    CHECK(kernel(300 * 64, 256, 1024, 1) == "igemm_dma_bf16_64x64x64s3" && kernel(302 * 64, 256, 1024, 1) == "igemm_dma_bf16_128x64x64s3");
}

// fp32 launches of 64x64 tiles: as many tiles as lie beyond a multiple of 256, if at most 128, make four workgroups each, in launches of one
// problem (wherever in the batch it lies) and one slice of K.
static void check_surplus_tiles()
{
    for (int k : {1, 3})
        for (int rows : {1, 15, 16, 17, 31, 32, 33, 64, 65, 72, 96, 97, 128, 129, 200, 300})
            for (int N : {64, 120, 256})
                for (int z : {1, 2}) {
                    GemmArgs a = product(DT_F32, rows * 64 - 3, N, 260, k);
                    a.zb = z;
                    a.z_lo = rows % 2;
                    LaunchInfo li = launch_igemm(a, nullptr, true);
                    const int tiles = rows * ((N + 63) / 64), r = tiles % 256;
                    CHECK(std::string(li.kernel) == (k == 1 ? "igemm_dma_f32_64x64x32s3" : "igemm_dma_taps_f32_64x64x32s3"));
                    CHECK(li.workgroups == (z == 1 ? tiles + (r <= 128 ? 3 * r : 0) : 2 * tiles));
                    a.zb = 1;
                    a.ksplit = 2;
                    CHECK(launch_igemm(a, nullptr, true).workgroups == 2 * tiles);
                }
    // scores of one head, a chunk of one image of three
    for (int S : {64, 128, 256}) {
        GemmArgs a = product(DT_F32, S, S, 128);
        a.x_pix = a.w_row = 384; a.x_img = 0;
        a.x_zb = a.w_zb = (int64_t)S * 384; a.y_zb = (int64_t)S * S;
        a.z_lo = 1;
        CHECK(launch_igemm(a, nullptr, true).workgroups == 4 * (S / 64) * (S / 64));
    }
}

// A 3x3 convolution marked for conv3_kernel: images [b_lo, b_hi) and channels [n_lo, n_hi) of it.
static LaunchInfo staged(int images, int hw, int cin, int n_lo, int n_hi)
{
    GemmArgs a = product(DT_BF16, images * hw * hw, n_hi, cin, 3);
    a.H = a.W = a.Ho = a.Wo = hw;
    a.x_img = (int64_t)hw * hw * cin;
    a.x_bytes = images * a.x_img * 2;
    a.w_bytes = (int64_t)n_hi * a.K * 2;
    a.n_lo = n_lo;
    a.halo = 1;
    return launch_igemm(a, nullptr, true);
}

// Tiles of conv3_kernel on either side of its lines.
static void check_staged_tiles()
{
    struct { int images, hw, cin, n; const char *kernel; int wgs; } cases[] = {
        {8, 28, 128, 128, "conv3_bf16_64x64", 196}, {16, 28, 128, 128, "conv3_bf16_128x64", 196}, {20, 14, 512, 256, "conv3_bf16_64x64", 248},
        {21, 14, 512, 256, "conv3_bf16_128x64", 132}, {10, 56, 64, 32, "conv3_bf16_128x64", 245}, {5, 56, 64, 32, "conv3_bf16_64x64", 245},
        {20, 56, 64, 64, "conv3_bf16_128x64", 490}, {21, 56, 64, 64, "conv3_bf16_256x64", 258}, {20, 14, 512, 512, "conv3_bf16_128x64", 248},
        {21, 14, 512, 512, "conv3_bf16_256x64s3", 136}, {42, 14, 512, 512, "conv3_bf16_256x64", 264}, {40, 56, 64, 64, "conv3_bf16_256x64", 490}, {32, 56, 256, 256, "conv3_bf16_256x128", 784}};
    for (auto &c : cases) {
        const LaunchInfo li = staged(c.images, c.hw, c.cin, 0, c.n);
        CHECK(li.kernel == std::string(c.kernel));
        CHECK(li.workgroups == c.wgs);
        CHECK(li.lds_bytes <= 160 * 1024 && li.wg_per_cu == 160 * 1024 / li.lds_bytes);
    }
}

// A pointwise product and the depthwise convolution behind it as one launch: pairs on either side of what expand_dw_takes allows.
static void check_pointwise_depthwise_pairs()
{
    struct { int n, hw, c, co, k, stride; bool one; } cases[] = {
        {8, 28, 40, 240, 3, 1, true}, {16, 28, 40, 240, 3, 1, false}, {4, 28, 160, 480, 3, 1, false}, {8, 14, 192, 768, 3, 1, false}, {32, 7, 160, 960, 3, 1, true},
        {1, 112, 16, 96, 3, 2, true}, {8, 112, 16, 96, 3, 2, false}, {8, 14, 112, 672, 5, 1, true}, {9, 14, 112, 136, 5, 2, true}, {8, 28, 40, 120, 5, 1, true},
        {16, 28, 40, 120, 5, 1, false}, {8, 28, 80, 160, 5, 1, false}, {32, 7, 256, 256, 5, 1, false}, {64, 3, 160, 960, 5, 1, false}, {1, 56, 24, 72, 5, 1, false}};
    for (auto &c : cases) {
        const GemmArgs g = product(DT_BF16, c.n * c.hw * c.hw, c.co, c.c);
        StreamArgs d;
        std::memset(&d, 0, sizeof d);
        d.dtype = DT_BF16;
        d.N = d.n_hi = c.n; d.H = d.W = c.hw; d.C = d.c_hi = c.co; d.k = c.k; d.stride = c.stride; d.pad = c.k / 2;
        d.Ho = d.Wo = (c.hw + 2 * d.pad - c.k) / c.stride + 1;
        if (expand_dw_takes(g, d) != c.one) std::fprintf(stderr, "%d images %dx%d %d->%d %dx%d\n", c.n, c.hw, c.hw, c.c, c.co, c.k, c.k);
        CHECK(expand_dw_takes(g, d) == c.one);
    }
}

// 16x16 tiles of K slices in fp32: as many as the units hold at once.
static void check_small_tiles()
{
    for (int affine = 0; affine < 2; ++affine)
        for (int waves : {4, 8})
            for (int tiles : {1, 256, 257, 512, 513}) {
                GemmArgs a = product(DT_F32, tiles * 16, 16, 1024);
                a.kwaves = waves; a.kb_per_wave = 64 / waves;
                if (affine) a.pre_scale = a.pre_shift = (const float *)0x10000;
                const std::string name = launch_igemm(a, nullptr, true).kernel;
                CHECK((name.find("_16x16") != std::string::npos) == (tiles <= (affine && waves == 8 ? 256 : 512)));
            }
}

int main()
{
    check_pointwise_depthwise_pairs();
    check_small_tiles();
    check_staged_tiles();
    check_depthwise_windows();
    check_bf16_rows();
    check_surplus_tiles();
    std::printf("dispatch driver: all checks held\n");
    return 0;
}
