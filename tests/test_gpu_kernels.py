"""Single kernels at the sizes where they can go wrong (tile edges, remainders, both ends of the range a dispatch rule gives
them): every operator against the oracle evaluated on the operator's own inputs, every decomposition bit-exact."""
import numpy as np
import pytest

from parity import TOL_ONE_OP, rel_err

pytestmark = pytest.mark.gpu


def check(tenants, expect, splits=(), expect_split=()):
    """Runs the tenants unsplit, compares every operator with the oracle, checks that the kernels named in `expect` (prefixes)
    ran, and that the decompositions in `splits` ((axis, factor) applied wherever legal) reproduce every output bit, with the
    kernels in `expect_split` among those that ran.  Returns the names of the kernels that ran unsplit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import forward as F
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    data = [G.materialise(t, 411, i << 20) for i, t in enumerate(tenants)]
    sess = harness.Session(tenants, data)
    sess.poison_outputs()
    sess.run(B.GACER_MODE_SEQUENTIAL, 1)
    for i, (t, (_, params)) in enumerate(zip(tenants, data)):
        got = [sess.tensor(i, k) for k in range(len(t.tensors))]
        for k, op in enumerate(t.ops):
            e = rel_err(got[op.out], F.run_op(t, k, got, params))
            assert e <= TOL_ONE_OP[t.dtype], f"{t.name} op {k} ({op.kind}): rel err {e}"
    base = [[sess.tensor_bytes(i, op.out) for op in t.ops] for i, t in enumerate(tenants)]
    ran = {r["kernel"] for r in sess.trace(B.GACER_MODE_SEQUENTIAL, 1)}
    for prefix in expect:
        assert any(k.startswith(prefix) for k in ran), f"{prefix} did not run: {sorted(ran)}"
    ran_split = set()
    for axis, factor in splits:
        sess.set_plan(sess.uniform_splits(axis, factor), [])
        sess.poison_outputs()
        sess.run(B.GACER_MODE_PLAN, 1)
        for i, t in enumerate(tenants):
            for k, op in enumerate(t.ops):
                assert sess.tensor_bytes(i, op.out) == base[i][k], f"{axis} x{factor}: {t.name} op {k} differs"
        if expect_split:
            ran_split |= {r["kernel"] for r in sess.trace(B.GACER_MODE_PLAN, 1)}
    assert ran_split >= set(expect_split), sorted(ran_split)
    sess.close()
    return ran


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_k_slices_inside_a_workgroup(dtype):
    """slices_kernel: one row and one channel, one past a 32-wide tile, K that ends inside a 128-byte batch, taps that a batch
    crosses and taps it does not, four and eight waves, 512 tiles (once with taps on a channel window), K cut over the grid as
    well, a fused affine."""
    from synth import graphs as G
    specs = [  # batch, hw, cin, [(cout, k, stride, pad, act, residual)]
        (1, 1, 512, [(1, 1, 1, 0, "none", False)]),
        (3, 11, 72, [(33, 1, 1, 0, "relu", False), (40, 1, 1, 0, "none", False), (40, 3, 1, 1, "relu6", True), (65, 3, 2, 1, "gelu", False)]),
        (2, 9, 128, [(31, 3, 1, 1, "hswish", False)]),
        (2, 14, 64, [(64, 3, 1, 1, "relu", False), (64, 3, 1, 1, "none", True)]),
        (1, 64, 128, [(128, 1, 1, 0, "relu", False)]),          # 512 tiles of 32x32
        (5, 13, 256, [(288, 1, 1, 0, "relu", False)]),          # 243 tiles, then 297
        (5, 13, 256, [(352, 1, 1, 0, "relu", False)]),
    ]
    tenants = []
    for i, (batch, hw, cin, layers) in enumerate(specs):
        b = G._B(f"slices{i}", dtype, batch)
        x = y = b.tensor(batch, cin, hw, hw)
        for cout, k, stride, pad, act, res in layers:
            y = b.conv(y, cout, k, stride, pad, act, res=y if res else -1)
        tenants.append(b.done(x, y))
    b = G._B("window", dtype, 1)                    # 512 tiles, taps, an input that is a channel window
    x, wide = b.tensor(1, 64, 64, 64), b.tensor(1, 192, 64, 64)
    y = b.conv(x, 64, 1, 1, 0, "relu", out=b.view(wide, 64, 64))
    tenants.append(b.done(x, b.conv(y, 128, 3, 1, 1, "none")))
    b = G._B("long_rows", dtype, 7)
    x = b.tensor(7, 128, 7, 7)
    tenants.append(b.done(x, b.gemm(x, 26, "relu", flatten=True)))
    b = G._B("affine", dtype, 3)
    x = b.tensor(3, 136, 5, 5)
    y = b.conv(b.affine(x, "relu"), 40, 1, 1, 0, "relu")
    tenants.append(b.done(x, y))
    names = {"f32": ["igemm_slices_f32_x4", "igemm_slices_f32_x8", "igemm_affine_slices_f32", "splitk_finish"],
             "bf16": ["igemm_slices_bf16_x4", "igemm_slices_bf16_x8", "igemm_affine_slices_bf16", "splitk_finish"]}
    check(tenants, names[dtype], [("batch", 2), ("cout", 2), ("cout", 8)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_k_slices_addressing(dtype):
    """The ways slices_kernel addresses its rows: one pitch, strided 1x1 (rows that end inside an image), a padded 1x1 (its border
    rows read nothing), windows with more padding than kernel, one input pixel per window row; slices of no, one, two, three, four
    and five batches, the last one ending inside a batch; a residual with a channel count that is no multiple of four."""
    from synth import graphs as G
    e = 64 if dtype == "bf16" else 32                # elements of a batch
    tenants = []
    for i, (batch, hw, cin, cout, k, stride, pad, res) in enumerate([
            (3, 9, 2 * e, 40, 1, 2, 0, False), (2, 7, 4 * e - 8, 33, 1, 3, 0, False), (2, 6, 3 * e, 36, 1, 1, 1, False), (2, 5, e, 40, 3, 1, 4, False),
            (3, 7, 72, 32, 3, 2, 3, False), (2, 1, 4 * e, 33, 3, 1, 1, False), (3, 5, 3 * e + 8, 3 * e + 8, 1, 1, 0, True),
            (3, 5, 7 * e + 8, 70, 1, 1, 0, False), (3, 5, 11 * e + 8, 33, 1, 1, 0, False), (1, 9, 16 * e, 36, 1, 1, 0, False), (1, 9, 20 * e - 8, 36, 1, 1, 0, False),
            (1, 9, 36 * e - 8, 36, 1, 1, 0, False)]):             # eight waves, five batches each, in either type
        b = G._B(f"rows{i}", dtype, batch)
        x = b.tensor(batch, cin, hw, hw)
        tenants.append(b.done(x, b.conv(x, cout, k, stride, pad, "relu", res=x if res else -1)))
    ran = check(tenants, [f"igemm_slices_{dtype}_x4"], [("batch", 2), ("cout", 2), ("cout", 8)])
    assert all(n.startswith("igemm_slices") or n == "splitk_finish" for n in ran), ran


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_k_slices_of_one_row(dtype):
    """slices_kernel where a descriptor holds a single row of K, of input or of weights, and waves have one batch of it or none: the
    squeeze layers of a channel gate for one image, one channel, a 3x3 window on one pixel, a fused affine."""
    from synth import graphs as G
    tenants = []
    for i, (batch, hw, cin, cout, k, affine) in enumerate([(1, 1, 72, 24, 1, False), (1, 1, 120, 32, 1, False), (1, 1, 168, 42, 1, False), (1, 1, 240, 64, 1, False),
                                                           (1, 1, 672, 168, 1, False), (1, 1, 120, 1, 1, False), (3, 5, 120, 1, 1, False), (1, 1, 24, 1, 3, False),
                                                           (1, 1, 136, 33, 1, True), (2, 3, 264, 1, 1, True)]):
        if dtype == "bf16" and cin == 72:
            cin = 104                                # shorter rows are rowgemm_kernel's
        b = G._B(f"row{i}", dtype, batch)
        x = y = b.tensor(batch, cin, hw, hw)
        if affine:
            y = b.affine(x, "relu")
        tenants.append(b.done(x, b.conv(y, cout, k, 1, k // 2, "relu")))
    ran = check(tenants, [f"igemm_slices_{dtype}_x4", f"igemm_affine_slices_{dtype}_x4"], [("cout", 2)])
    assert all("slices" in n for n in ran), ran


def test_long_k_with_few_tiles_in_fp32():
    """K cut over the grid beside the slices of a workgroup (one, three, five and eight workgroup rows along K, the last row with
    fewer batches than the others), and the shapes with 65 to 128 tiles that the tiled kernels with their own cut of K take."""
    from synth import graphs as G
    ran = {}
    for rows, cout, cin, k in [(8, 1000, 2048, 1), (7, 999, 1284, 1), (169, 256, 256, 3), (147, 500, 520, 3), (300, 72, 1244, 1), (416, 256, 256, 3), (405, 250, 2308, 1)]:
        b = G._B(f"few{rows}", "f32", 1)
        x = b.tensor(1, cin, rows if k == 1 else {169: 13, 147: 21, 416: 26}[rows], 1 if k == 1 else {169: 13, 147: 7, 416: 16}[rows])
        ran[rows] = check([b.done(x, b.conv(x, cout, k, 1, k // 2, "relu"))], [], [("cout", 2), ("cout", 8)])
    sliced = {r: any(n.startswith("igemm_slices_f32_x8") for n in names) for r, names in ran.items()}
    assert sliced == {8: True, 7: True, 169: True, 147: True, 300: True, 416: False, 405: False}, ran
    assert {r for r, names in ran.items() if "splitk_finish" in names} == {8, 7, 169, 147, 416, 405}, ran
    assert any(n.startswith("igemm_dma_taps_f32_64x64") for n in ran[416]) and any(n.startswith("igemm_dma_f32_64x64") for n in ran[405]), ran


def test_k_slices_on_small_tiles_in_fp32():
    """16x16 tiles (up to 512 of them) and 32x32 ones give the same bits: whole operators on either side of the line, whose halves and eighths lie
    below it; rows, strided rows, windows, a fused affine with a remainder of rows and channels, K cut over the grid."""
    from synth import graphs as G
    tenants = []
    for i, (batch, h, w, cin, cout, k, stride, affine, res) in enumerate([
            (1, 17, 15, 132, 33, 1, 1, False, True), (2, 9, 9, 260, 70, 1, 2, False, False), (3, 5, 5, 128, 32, 3, 1, False, False), (2, 13, 11, 40, 47, 3, 1, False, True),
            (3, 5, 7, 612, 120, 1, 1, True, False), (1, 7, 7, 100, 31, 1, 1, True, False), (1, 33, 31, 128, 144, 1, 1, False, False), (4, 16, 16, 96, 140, 3, 1, False, False),
            (4, 23, 11, 200, 132, 1, 1, True, False), (1, 1, 1, 2048, 1000, 1, 1, False, False), (2, 7, 7, 2052, 250, 1, 1, False, True), (8, 1, 1, 4096, 2050, 1, 1, False, False)]):
        b = G._B(f"small{i}", "f32", batch)
        x = b.tensor(batch, cin, h, w)
        r = b.conv(x, cout, 1, stride, 0, "none") if res else -1
        tenants.append(b.done(x, b.conv(b.affine(x, "relu") if affine else x, cout, k, stride, k // 2, "relu", res=r)))
    small = {"igemm_slices_f32_x4_16x16", "igemm_slices_f32_x8_16x16", "igemm_affine_slices_f32_x4_16x16", "igemm_affine_slices_f32_x8_16x16"}
    ran = check(tenants, [], [("batch", 2), ("cout", 2), ("cout", 8)], ["igemm_slices_f32_x4_16x16", "igemm_slices_f32_x8_16x16"])
    assert ran == small | {"igemm_slices_f32_x4", "igemm_slices_f32_x8", "igemm_affine_slices_f32_x4", "splitk_finish"}, sorted(ran)


def test_number_of_tiles_for_k_slices_in_fp32():
    """Either side of each limit on the 32x32 tiles (512, 1024) and on the batches of K they ask for (72), and of the 64x64 tiles (128) from which on a long K
    stays on slices; halves and eighths of the channels give the bits of the whole operator."""
    from synth import graphs as G
    for rows, cout, cin, sliced in [(3270, 130, 2276, True), (3270, 130, 2272, False), (1010, 1000, 2308, True), (1030, 1000, 2308, False),
                                    (1000, 500, 2564, True), (960, 500, 2564, False)]:
        b = G._B(f"limit{rows}", "f32", 1)
        x = b.tensor(1, cin, rows, 1)
        names = check([b.done(x, b.conv(x, cout, 1, 1, 0, "relu"))], [], [("cout", 2), ("cout", 8)])
        assert any(n.startswith("igemm_slices_f32_x4") for n in names) == sliced, (rows, cout, cin, names)


def test_finishing_pass_of_every_number_of_slices():
    """splitk_finish for two, three, four, five and eight slices in fp32, whole vectors and channel counts or chunks that are none, with
    and without a residual and an activation."""
    from synth import graphs as G
    tenants = []
    for i, (batch, hw, cin, cout, k, act) in enumerate([(8, 1, 4096, 512, 1, "relu"), (3, 7, 512, 512, 3, "none"), (1, 13, 256, 256, 3, "relu6"),
                                                        (8, 1, 2048, 1001, 1, "gelu"), (8, 1, 2048, 1000, 1, "none"), (2, 7, 512, 510, 3, "hswish"),
                                                        (2, 7, 1536, 1000, 1, "relu")]):
        b = G._B(f"finish{i}", "f32", batch)
        x = b.tensor(batch, cin, hw, hw)
        tenants.append(b.done(x, b.conv(x, cout, k, 1, k // 2, act, res=x if cin == cout else -1)))
    check(tenants, ["splitk_finish"], [("batch", 2), ("cout", 8)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_affine_with_many_channels_in_front_of_k_slices(dtype):
    """The fused affine form of slices_kernel with several batches of K per wave (its stores counted by the waits), K that ends
    inside a batch, four and eight waves, more channels than one pass over the parameters copies, K cut over the grid, the most
    channels it takes.  Batch and channel chunks un-fuse the pairs: their outputs, the affine tensor among them, keep every bit."""
    from synth import graphs as G
    tenants = []
    for i, (batch, hw, cin, cout) in enumerate([(3, 5, 1000, 40), (2, 7, 1160, 33), (2, 6, 2056, 65), (2, 5, 4096, 40), (5, 40, 600, 64), (2, 34, 2056, 136)]):
        b = G._B(f"pre{i}", dtype, batch)
        x = b.tensor(batch, cin, hw, hw)
        tenants.append(b.done(x, b.conv(b.affine(x, ["relu", "relu6", "none"][i % 3]), cout, 1, 1, 0, "relu")))
    check(tenants, [f"igemm_affine_slices_{dtype}_x4", f"igemm_affine_slices_{dtype}_x8"], [("batch", 2), ("cout", 2)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_stems_and_odd_channel_counts(dtype):
    """stem_kernel: runs of one chunk and of many, odd and even chunk counts, odd strides (runs that start on an odd element in
    bf16), image rows of odd length, output rows shorter and longer than a 128-position tile, windows wider than the padding,
    1 / 33 / 65 channels, a residual."""
    from synth import graphs as G
    specs = [  # batch, h, cin, [(cout, k, stride, pad, act, residual)]
        (2, 33, 3, [(64, 7, 2, 3, "relu", False)]),
        (1, 150, 3, [(65, 3, 1, 1, "relu", False)]),
        (3, 35, 3, [(16, 3, 2, 1, "hswish", False)]),
        (1, 67, 3, [(33, 11, 4, 2, "none", False)]),
        (2, 9, 5, [(5, 5, 1, 2, "relu6", True), (7, 1, 1, 0, "none", False), (1, 2, 1, 0, "gelu", False)]),
        (2, 8, 1, [(3, 3, 1, 1, "none", False), (13, 3, 1, 0, "relu", False), (40, 4, 3, 2, "none", False)]),
        (1, 4, 3, [(8, 3, 1, 1, "none", False)]),
    ]
    tenants = []
    for i, (batch, hw, cin, layers) in enumerate(specs):
        b = G._B(f"stem{i}", dtype, batch)
        x = y = b.tensor(batch, cin, hw, hw)
        for cout, k, stride, pad, act, res in layers:
            y = b.conv(y, cout, k, stride, pad, act, res=y if res else -1)
        tenants.append(b.done(x, y))
    check(tenants, [f"stem_{dtype}"], [("batch", 2), ("cout", 2), ("cout", 8)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_stems_whose_workgroups_walk_several_tiles(dtype):
    """stem_kernel with about 1200 tiles for at most 1024 workgroups, an image that is no whole number of tiles and of odd row
    length (strips at the ends of the tensor alternate with others, chunks start at other images than the first): 64 and 32
    channels per workgroup, whole groups and remainders, even and odd strides; weights and strip of more than 64 KB."""
    from synth import graphs as G
    tenants = []
    for i, (batch, h, w, cout, k, stride, pad, act) in enumerate([
            (12, 113, 113, 64, 3, 1, 1, "relu"), (12, 113, 113, 65, 3, 1, 1, "relu6"), (12, 113, 113, 24, 3, 1, 1, "gelu"),
            (12, 227, 227, 33, 7, 2, 3, "none"), (2, 37, 500, 32, 7, 2, 3, "hswish")]):
        b = G._B(f"walk{i}", dtype, batch)
        x = b.tensor(batch, 3, h, w)
        tenants.append(b.done(x, b.conv(x, cout, k, stride, pad, act)))
    ran = check(tenants, [], [("batch", 2), ("cout", 2)])
    assert ran == {f"stem_{dtype}"}, ran


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_direct_to_lds_pipeline(dtype):
    """igemm_dma_kernel: ragged M, N and K, channels that are no multiple of a K block (a block crosses taps) and that are, strides,
    5x5 taps, a residual, one tap, every tile shape."""
    from synth import graphs as G
    specs = [  # batch, h, w, cin, cout, k, stride, pad, act, residual
        (3, 45, 37, 40, 100, 5, 1, 2, "relu", False), (2, 61, 59, 120, 120, 3, 1, 1, "relu6", True), (3, 91, 83, 96, 124, 3, 2, 1, "none", False),
        (1, 80, 53, 1000, 250, 1, 1, 0, "gelu", False), (1, 63, 1, 2056, 8248, 1, 1, 0, "none", False), (1, 112, 112, 776, 1000, 1, 1, 0, "hswish", False),
        (2, 95, 79, 160, 250, 3, 1, 1, "relu", False), (4, 95, 79, 88, 250, 3, 1, 1, "none", False), (3, 40, 37, 240, 120, 3, 1, 1, "relu", False),
    ]
    tenants = []
    for i, (batch, h, w, cin, cout, k, stride, pad, act, res) in enumerate(specs):
        b = G._B(f"dma{i}", dtype, batch)
        x = b.tensor(batch, cin, h, w)
        tenants.append(b.done(x, b.conv(x, cout, k, stride, pad, act, res=x if res else -1)))
    ran = check(tenants, [], [("batch", 2), ("cout", 2)])
    names = {"f32": ["f32_64x64x32s3", "taps_f32_64x64x32s3"],
             "bf16": ["bf16_64x64x64s3", "bf16_64x64x64s4", "bf16_256x128x32s3", "taps_bf16_64x64x64s3", "taps_bf16_64x64x64s4", "taps_bf16_128x128x64s3", "taps_bf16_128x128x32s4"]}
    assert ran == {"igemm_dma_" + n for n in names[dtype]}, sorted(ran)


@pytest.mark.parametrize("name,spec", [
    ("128x32x64s3", (3, 81, 83, 144, 27, 1, 1, "none", True)), ("taps_128x32x64s3", (3, 81, 83, 72, 30, 3, 1, "relu6", False)),
    ("128x64x32s3", (1, 131, 127, 136, 200, 1, 1, "relu", True)), ("taps_128x64x32s3", (4, 113, 111, 64, 58, 2, 1, "none", True)),
    ("128x64x64s3", (1, 131, 127, 328, 136, 1, 1, "hswish", True)), ("taps_128x64x64s3", (2, 113, 111, 40, 130, 3, 1, "relu", False)),
    ("128x128x32s4", (2, 161, 155, 256, 122, 1, 1, "none", False)), ("64x64x64s4", (1, 130, 8, 1032, 520, 1, 1, "gelu", False))])
def test_direct_to_lds_tiles_of_short_k(name, spec):
    """The bf16 tiles of igemm_dma_kernel that short rows and narrow outputs take: ragged rows, channels (no multiple of a vector or of four) and K."""
    from synth import graphs as G
    batch, h, w, cin, cout, k, stride, act, res = spec
    b = G._B("tile", "bf16", batch)
    x = b.tensor(batch, cin, h, w)
    y = b.conv(x, cout, k, stride, k // 2, "none") if res else -1
    ran = check([b.done(x, b.conv(x, cout, k, stride, k // 2, act, res=y))], [], [("batch", 2), ("cout", 2), ("cout", 8)])
    assert ran == {"igemm_dma_" + ("taps_bf16_" + name[5:] if name.startswith("taps_") else "bf16_" + name)}, sorted(ran)


@pytest.mark.parametrize("spec", [(1, 139, 30, 132, 250, 1, 1, "relu6", True), (3, 39, 37, 44, 250, 3, 1, "relu", False), (1, 139, 30, 132, 251, 1, 1, "none", True),
                                  (4, 113, 59, 392, 190, 1, 2, "hswish", False), (5, 40, 27, 60, 247, 3, 1, "gelu", True)])
def test_surplus_tiles_in_quarters(spec):
    """fp32 launches with some tiles more than a multiple of the units: the last ones in quarters, ragged rows and channels (quarters that lie
    outside, vectors that reach over the end), chunks that are cut up altogether.  Each of those tiles makes four workgroups."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    batch, h, w, cin, cout, k, stride, act, res = spec
    b = G._B("surplus", "f32", batch)
    x = b.tensor(batch, cin, h, w)
    y = b.conv(x, cout, 1, stride, 0, "none") if res else -1
    t = b.done(x, b.conv(x, cout, k, stride, k // 2, act, res=y))
    n, c, ho, wo = t.tensors[t.output]
    tiles = ((n * ho * wo + 63) // 64) * ((c + 63) // 64)
    assert tiles > 256 and 0 < tiles % 256 <= 128
    check([t], ["igemm_dma"], [("batch", 2), ("cout", 2), ("cout", 8)])
    sess = harness.Session([t], [G.materialise(t, 411, 0)])
    last = sess.trace(B.GACER_MODE_SEQUENTIAL, 1)[-1]
    sess.close()
    assert last["kernel"].endswith("f32_64x64x32s3") and last["workgroups"] == tiles + 3 * (tiles % 256), (last, tiles)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("keys", [64, 72, 120, 256])
@pytest.mark.parametrize("head", [128, 192])
def test_attention_of_one_head(dtype, keys, head):
    """Products of one head, in chunks of three, two and one image: a launch of a single problem that is not the first one.  Key counts
    that fill the last 64x64 tile, half of it, and less."""
    from synth import graphs as G
    b = G._B("one_head", dtype, 5)
    x = b.tensor(5, 3 * head, keys, 1)
    check([b.done(x, b.attention(x, 1))], [], [("batch", 2), ("batch", 4)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_non_finite_inputs_reach_their_windows_only(dtype):
    """Infinities and NaN in the input make exactly the outputs non-finite whose window holds one (padding, tails of K and of tiles
    and the neighbours in memory are zeros times something finite); all other outputs are as without them."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import forward as F
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    specs = [  # batch, cin, h, w, cout, k, stride, pad, groups
        (2, 3, 37, 41, 64, 7, 2, 3, 1), (2, 3, 33, 35, 40, 3, 1, 1, 1), (2, 72, 9, 11, 40, 3, 1, 1, 1), (2, 64, 9, 9, 33, 3, 1, 1, 1),
        (3, 200, 5, 5, 70, 1, 1, 0, 1), (16, 64, 56, 56, 64, 3, 1, 1, 1), (2, 88, 61, 59, 70, 3, 1, 1, 1), (3, 40, 40, 40, 96, 1, 1, 0, 1),
        (2, 24, 9, 9, 24, 5, 1, 2, 24), (70, 48, 9, 9, 48, 5, 1, 2, 48),
    ]
    tenants, data, clean, bad = [], [], [], []
    for i, (batch, cin, h, w, cout, k, stride, pad, groups) in enumerate(specs):
        b = G._B(f"nonfinite{i}", dtype, batch)
        x = b.tensor(batch, cin, h, w)
        tenants.append(b.done(x, b.conv(x, cout, k, stride, pad, "none", groups=groups)))
        xv, params = G.materialise(tenants[-1], 77, i << 20)
        mark = np.zeros(xv.shape, bool)
        for (n, c, r, q), v in {(0, 0, 0, 0): np.nan, (0, cin - 1, h - 1, w - 1): np.inf, (batch - 1, cin - 1, h - 1, w - 1): -np.inf,
                                (batch // 2, cin // 2, h // 2, w // 2): np.nan}.items():
            mark[n, c, r, q] = True
        clean.append(np.where(mark, np.float32(0), xv))
        xv = np.where(mark, np.float32(np.nan), xv)
        xv[0, cin - 1, h - 1, w - 1], xv[batch - 1, cin - 1, h - 1, w - 1] = np.inf, -np.inf
        data.append((xv, params))
        ones = torch.ones((cout, cin // groups, k, k))
        bad.append(torch.nn.functional.conv2d(torch.from_numpy(mark.astype(np.float32)), ones, stride=stride, padding=pad, groups=groups).numpy() > 0)
    sess = harness.Session(tenants, data)
    sess.poison_outputs()
    sess.run(B.GACER_MODE_SEQUENTIAL, 1)
    for i, t in enumerate(tenants):
        got = sess.output(i)
        assert np.array_equal(~np.isfinite(got), bad[i]), f"{t.name}: non-finite outputs elsewhere"
        ref = F.run_op(t, 0, [clean[i], None], data[i][1])
        e = rel_err(np.where(bad[i], 0, got), np.where(bad[i], 0, ref))
        assert e <= TOL_ONE_OP[dtype], f"{t.name}: rel err {e}"
    sess.close()


def test_input_staged_once_for_nine_taps():
    """conv3_kernel: images narrower and wider than a column strip, a last strip that is narrower, rows shorter than a tile by
    far, a tile that ends inside an image row, the three tile shapes with remainders (chunks take smaller tiles than the whole
    operator), a residual, one and several pairs of channel blocks, an input that is a channel window of a wider tensor."""
    from synth import graphs as G
    specs = [  # batch, h, w, cin, [(cout, act, residual)]
        (16, 56, 56, 64, [(64, "relu", False), (64, "relu", True)]),
        (2, 131, 113, 64, [(136, "hswish", False)]),
        (1, 191, 251, 128, [(65, "relu6", False)]),
        (67, 29, 13, 128, [(250, "gelu", False)]),
        (61, 53, 5, 64, [(130, "none", False)]),
        (15, 101, 37, 64, [(250, "hswish", False)]),
    ]
    tenants = []
    for i, (batch, h, w, cin, layers) in enumerate(specs):
        b = G._B(f"halo{i}", "bf16", batch)
        x = y = b.tensor(batch, cin, h, w)
        for cout, act, res in layers:
            y = b.conv(y, cout, 3, 1, 1, act, res=y if res else -1)
        tenants.append(b.done(x, y))
    b = G._B("window", "bf16", 15)
    x, wide = b.tensor(15, 64, 55, 57), b.tensor(15, 192, 55, 57)
    y = b.conv(x, 64, 3, 1, 1, "relu", out=b.view(wide, 64, 64))
    tenants.append(b.done(x, b.conv(y, 64, 3, 1, 1, "none")))
    check(tenants, ["conv3_bf16_256x64", "conv3_bf16_256x128"], [("batch", 2), ("cout", 2), ("cout", 8)], ["conv3_bf16_128x64", "conv3_bf16_256x64"])


@pytest.mark.parametrize("tile,spec", [("128x64", (4, 61, 59, 64, 120, "relu", True)), ("128x64", (16, 27, 29, 64, 130, "hswish", False)), ("256x64s3", (4, 57, 53, 256, 250, "none", False)),
                                       ("256x64", (12, 57, 53, 256, 120, "relu", True))])
def test_staged_3x3_with_three_weight_stages(tile, spec):
    """conv3_kernel with few tiles: 128 positions, and 256 where K is long, both with three stages of weights, and 256 with two where there are more
    than one per unit; ragged images and channels."""
    from synth import graphs as G
    batch, h, w, cin, cout, act, res = spec
    b = G._B("staged", "bf16", batch)
    x = b.tensor(batch, cin, h, w)
    y = b.conv(x, cout, 1, 1, 0, "none") if res else -1
    ran = check([b.done(x, b.conv(x, cout, 3, 1, 1, act, res=y))], [], [("batch", 2), ("cout", 2)])
    assert [n for n in ran if n.startswith("conv3")] == ["conv3_bf16_" + tile]


@pytest.mark.parametrize("spec", [(3, 61, 59, 64, 250, "relu", True), (16, 29, 27, 64, 130, "none", False), (5, 57, 113, 128, 64, "hswish", True), (30, 5, 100, 192, 70, "relu6", False)])
def test_staged_3x3_in_chunks_of_few_tiles(spec):
    """conv3_kernel on 64x64 tiles, for chunks of an operator that leave half of the units empty on larger ones: two strips of columns, images that
    end inside a tile, ragged channels; every chunk has the bits of the whole."""
    from synth import graphs as G
    batch, h, w, cin, cout, act, res = spec
    b = G._B("chunks", "bf16", batch)
    x = b.tensor(batch, cin, h, w)
    y = b.conv(x, cout, 1, 1, 0, "none") if res else -1
    t = b.done(x, b.conv(x, cout, 3, 1, 1, act, res=y))
    ran = check([t], ["conv3_bf16_128x64"], [("batch", 2), ("cout", 2), ("cout", 8)], ["conv3_bf16_64x64"])
    assert "conv3_bf16_64x64" not in ran


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_with_short_k(dtype):
    """rowgemm_kernel: every number of 32-byte k groups, K that fills half a group, one column of tiles, two and more, four side by
    side (bf16, more than 6000 tiles), rows and channels that end inside a tile, strided rows, a residual, an output that is a channel
    window; chunks of channels that start inside a vector."""
    from synth import graphs as G
    v = 8 if dtype == "bf16" else 4                  # elements of a vector
    specs = [  # batch, h, w, cin, cout, stride, act, residual
        (1, 401, 97, v, 33, 1, "relu", False), (3, 113, 131, 2 * v, 2 * v, 1, "none", True), (1, 211, 193, 3 * v, 70, 1, "gelu", False), (2, 159, 131, 4 * v, 30, 1, "relu6", False),
        (1, 223, 191, 6 * v, 101, 1, "none", False), (1, 203, 211, 7 * v, 64, 1, "hswish", False), (3, 207, 215, 9 * v, 40, 2, "relu", False), (2, 131, 127, 12 * v, 12 * v, 1, "relu", True),
        (2, 181, 183, 5 * v, 42, 1, "none", False), (1, 9, 7, 5 * v, 20, 1, "relu", False), (1, 1, 1, 2 * v, 7, 1, "none", False),
    ]
    if dtype == "bf16":
        specs += [(1, 241, 203, 16, 97, 1, "relu6", False), (1, 227, 223, 24, 128, 1, "none", False), (1, 241, 211, 40, 100, 1, "relu", False), (2, 157, 131, 64, 160, 1, "none", False), (1, 227, 225, 88, 100, 1, "relu", False), (1, 143, 199, 256, 264, 1, "none", False)]
    tenants = []
    for i, (batch, h, w, cin, cout, stride, act, res) in enumerate(specs):
        b = G._B(f"rows{i}", dtype, batch)
        x = b.tensor(batch, cin, h, w)
        if cin == 256:                               # a residual behind four columns side by side
            x = b.conv(x, 64, 1, 1, 0, "relu")
            y = b.conv(x, cout, 1, 1, 0, "none")
            tenants.append(b.done(0, b.conv(x, cout, 1, 1, 0, "relu", res=y)))
            continue
        tenants.append(b.done(x, b.conv(x, cout, 1, stride, 0, act, res=x if res else -1)))
    b = G._B("window", dtype, 2)
    x, wide = b.tensor(2, 3 * v, 151, 149), b.tensor(2, 96, 151, 149)
    y = b.conv(x, 32, 1, 1, 0, "relu", out=b.view(wide, 40, 32))
    tenants.append(b.done(x, y))
    check(tenants, [f"rowgemm_{dtype}_x32", f"rowgemm_{dtype}_x64"] + (["rowgemm_bf16_x128"] if dtype == "bf16" else []), [("batch", 2), ("cout", 2), ("cout", 8)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tiles_finished_in_registers(dtype):
    """The epilogue of the tiled kernels at channel counts that are no multiple of a vector or of four, with and without a residual,
    one and several tiles per wave; chunks whose channels start inside a vector; attention products of several images."""
    from synth import graphs as G
    specs = [  # batch, h, w, cin, cout, k, act, residual
        (2, 61, 59, 48, 48, 3, "relu", True), (2, 67, 59, 40, 42, 3, "hswish", True), (1, 131, 127, 200, 200, 1, "relu6", True), (3, 75, 71, 136, 133, 1, "none", True),
        (2, 95, 79, 160, 250, 3, "relu", True), (1, 112, 112, 776, 999, 1, "gelu", False), (2, 113, 111, 136, 27, 1, "relu", True), (1, 150, 149, 104, 130, 1, "relu", False),
        (1, 130, 129, 104, 122, 1, "relu", True), (2, 113, 111, 24, 58, 3, "relu6", True),
    ]
    tenants = []
    for i, (batch, h, w, cin, cout, k, act, res) in enumerate(specs):
        b = G._B(f"tiles{i}", dtype, batch)
        x = b.tensor(batch, cin, h, w)
        y = b.conv(x, cout, k, 1, k // 2, "none") if res else -1
        tenants.append(b.done(x, b.conv(x, cout, k, 1, k // 2, act, res=y)))
    tenants.append(G.small_bert(dtype, 3))
    check(tenants, [f"igemm_dma_{dtype}", f"igemm_{dtype}_64x64", f"igemm_taps_{dtype}", f"igemm_bt_{dtype}"], [("batch", 2), ("cout", 2), ("cout", 8)])


@pytest.mark.parametrize("batch,keys,hidden", [(2, 72, 128), (3, 8, 64), (2, 24, 192), (1, 128, 128), (2, 120, 64), (1, 32, 64), (2, 104, 128)])
def test_attention_as_one_launch(batch, keys, hidden):
    """Scores, softmax and context of an attention in one launch: key counts that are no multiple of a query tile, of a k group or of
    the lanes of a row, both ends of its range; every operator against the oracle, every tensor with the bits of the three launches.
    Decomposing one of the three, or a sync edge inside the triple, brings the three launches back; batch and channel chunks elsewhere
    and edges at its ends do not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    t = G._bert("attention", "bf16", batch, keys, 2, hidden, hidden // 64, 96)
    other = G._bert("longer", "bf16", 2, 136, 1, 64, 1, 96)     # stays three launches, and so do 16 features per head
    check([t, other, G.small_bert("bf16", 2)], ["attention_bf16", "softmax", "igemm_bt_bf16"], [("batch", 2)] if batch > 1 else [])
    sess = harness.Session([t, other], [G.materialise(x, 411, i << 20) for i, x in enumerate([t, other])])

    def snapshot():
        sess.poison_outputs()
        sess.run(B.GACER_MODE_PLAN, 2)
        return [sess.tensor_bytes(0, op.out) for op in t.ops]

    def fused():
        return [r["op"] for r in sess.trace(B.GACER_MODE_PLAN, 1) if r["kernel"] == "attention_bf16"]
    qk = [i for i, op in enumerate(t.ops) if op.kind == "bgemm_qk"]
    want, launches = snapshot(), sess.launch_count()
    assert fused() == qk
    sess.set_fuse_affine(False)
    assert snapshot() == want and fused() == [] and sess.launch_count() == launches == len(t.ops) + len(other.ops)
    sess.set_fuse_affine(True)
    for syncs, left in [([(0, qk[0], 1, 3)], qk[1:]), ([(0, qk[0] + 1, 1, 3)], qk[1:]), ([(1, 2, 0, qk[1] + 1)], qk[:1]), ([(1, 2, 0, qk[1] + 2)], qk[:1]),
                        ([(1, 2, 0, qk[1]), (0, qk[0] + 2, 1, 3)], qk), ([(0, qk[0] + 2, 1, 3, 1)], qk[1:])]:
        sess.set_plan([(0, 0, "batch", 1)], syncs)
        assert fused() == left, syncs
        assert snapshot() == want, syncs
    if batch > 1:
        for k in range(3):
            sess.set_plan([(0, qk[1] + k, "batch", 2), (0, qk[0] - 1, "cout", 2)], [])
            assert fused() == qk[:1] and snapshot() == want, k
    sess.close()


def test_attention_whose_context_lies_where_the_scores_were():
    """A caller that uses buffers again: in the first layer the context over the scores, which nothing reads any more, in the second a
    softmax in place.  Outputs are those of tensors with memory of their own; the first layer goes back to three launches, the second does
    not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    t = G._bert("attention", "bf16", 4, 120, 2, 128, 2, 96)
    sess = harness.Session([t], [G.materialise(t, 411, 0)])
    qk = [i for i, op in enumerate(t.ops) if op.kind == "bgemm_qk"]

    def run():
        sess.run(B.GACER_MODE_SEQUENTIAL, 2)
        return sess.tensor_bytes(0, t.output), [r["op"] for r in sess.trace(B.GACER_MODE_SEQUENTIAL, 1) if r["kernel"] == "attention_bf16"]
    want, fused = run()
    assert fused == qk
    tensors = sess._descs[0].tensors
    for q, (tensor, over, left) in ((qk[0], (t.ops[qk[0] + 2].out, t.ops[qk[0]].out, qk[1:])), (qk[1], (t.ops[qk[1] + 1].out, t.ops[qk[1]].out, qk[1:]))):
        assert sess.acts[0][tensor].numel() <= sess.acts[0][over].numel()
        tensors[tensor].dptr = tensors[over].dptr
        sess.poison_outputs()
        B.check(sess.ctx, B.gacer_load_tenants(sess.ctx, sess._descs, 1))
        got, fused = run()
        assert got == want and fused == left, q
    sess.close()


# batch, h, w, cin, c, window, stride, activations: bands that end inside the image, one band, images of one row or column, channels that end
# inside a block of 32, K of half a 32-byte group, of one block and of several, cut into slices (few tiles) or not (many)
EXPAND = [(1, 28, 28, 32, 192, 3, 1, "relu6", "relu6"), (2, 27, 23, 24, 40, 3, 2, "relu", "none"), (3, 14, 13, 64, 72, 3, 1, "none", "relu"), (1, 14, 14, 96, 576, 3, 2, "relu6", "relu6"),
          (2, 7, 7, 160, 960, 3, 1, "hswish", "hswish"), (9, 14, 14, 112, 136, 5, 2, "gelu", "relu"), (5, 9, 11, 48, 56, 5, 1, "relu", "gelu"), (2, 1, 28, 40, 32, 3, 1, "relu", "relu"),
          (2, 28, 1, 40, 32, 3, 2, "relu", "relu"), (1, 56, 55, 8, 96, 3, 1, "relu6", "relu6"), (1, 97, 113, 16, 24, 3, 2, "relu", "relu6"), (1, 2, 2, 16, 8, 5, 1, "relu", "none"),
          (40, 7, 7, 160, 200, 3, 1, "relu", "relu"), (1, 1, 1, 264, 64, 3, 2, "relu", "relu"), (33, 13, 15, 104, 96, 3, 2, "relu6", "none")]


@pytest.mark.parametrize("spec", EXPAND, ids=lambda s: "x".join(map(str, s[:7])))
def test_pointwise_and_depthwise_as_one_launch(spec):
    """expand_dw_kernel against the oracle and, every tensor, against the two launches; decomposing either operator or a sync edge between
    them brings the two launches back, other edges do not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    batch, h, w, cin, c, k, stride, act1, act2 = spec
    tenants = []
    for i in range(2):
        b = G._B(f"expand{i}", "bf16", batch)
        x, wide = b.tensor(batch, 8, h, w), b.tensor(batch, cin + 16, h, w)
        y = b.conv(x, cin, 1, 1, 0, "none", out=b.view(wide, 8, cin)) if i else b.conv(x, cin, 1, 1, 0, "none")       # a window as input
        y = b.conv(b.conv(y, c, 1, 1, 0, act1), c, k, stride, k // 2, act2, groups=c)
        tenants.append(b.done(x, b.conv(y, 16, 1, 1, 0, "relu")))
    check(tenants, ["expand_dw_bf16"], [("batch", 2), ("cout", 2)] if batch > 1 else [("cout", 2)])
    sess = harness.Session(tenants, [G.materialise(t, 411, i << 20) for i, t in enumerate(tenants)])

    def snapshot():
        sess.poison_outputs()
        sess.run(B.GACER_MODE_PLAN, 2)
        return [sess.tensor_bytes(i, op.out) for i, t in enumerate(tenants) for op in t.ops]

    def fused():
        return sorted((r["tenant"], r["op"]) for r in sess.trace(B.GACER_MODE_PLAN, 1) if r["kernel"].startswith("expand_dw_bf16"))
    want = snapshot()
    assert fused() == [(0, 1), (1, 1)] and sess.launch_count() == 8
    sess.set_fuse_affine(False)
    assert snapshot() == want and fused() == [] and sess.launch_count() == 8
    sess.set_fuse_affine(True)
    for syncs, left in [([(0, 1, 1, 3)], [(1, 1)]), ([(0, 0, 1, 2)], [(0, 1)]), ([(0, 2, 1, 3, 1)], [(1, 1)]), ([(0, 2, 1, 1), (0, 0, 1, 3)], [(0, 1), (1, 1)])]:
        sess.set_plan([], syncs)
        assert fused() == left and snapshot() == want, syncs
    for op in (1, 2):
        sess.set_plan([(0, op, "cout", 2), (1, 0, "cout", 2)], [])
        assert fused() == [(1, 1)] and snapshot() == want, op
    sess.close()


def test_pointwise_and_depthwise_over_a_buffer_that_is_used_again():
    """The depthwise result where the pointwise operator's input was: two launches, and the outputs of tensors with memory of their own."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    b = G._B("turn", "bf16", 2)
    x = b.tensor(2, 8, 14, 14)
    first = b.conv(x, 64, 1, 1, 0, "none")
    y = b.conv(b.conv(first, 64, 1, 1, 0, "relu"), 64, 3, 1, 1, "relu", groups=64)
    t = b.done(x, b.conv(y, 16, 1, 1, 0, "relu"))
    sess = harness.Session([t], [G.materialise(t, 411, 0)])

    def run():
        sess.run(B.GACER_MODE_SEQUENTIAL, 2)
        return sess.tensor_bytes(0, t.output), any(r["kernel"].startswith("expand_dw") for r in sess.trace(B.GACER_MODE_SEQUENTIAL, 1))
    want, fused = run()
    assert fused
    sess._descs[0].tensors[y].dptr = sess._descs[0].tensors[first].dptr
    sess.poison_outputs()
    B.check(sess.ctx, B.gacer_load_tenants(sess.ctx, sess._descs, 1))
    got, fused = run()
    assert got == want and not fused
    sess.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_depthwise_output_tiles(dtype):
    """Every output tile of the depthwise kernel (from one output per thread to 2 x 4, chosen by the number of outputs), 3x3 and 5x5,
    strides 1 and 2: rows and columns that end inside a tile, images one pixel wide, padding wider than the kernel reaches, a
    residual.  Chunks run on other tiles than the whole, chunks of channels that are no multiple of four on the generic kernels."""
    from synth import graphs as G
    specs = [  # batch, h, w, c, k, stride, pad, act, residual
        (2, 13, 11, 36, 3, 1, 1, "relu6", True), (1, 9, 1, 8, 3, 2, 1, "none", False), (2, 7, 5, 12, 3, 1, 4, "relu", False), (2, 8, 9, 20, 5, 2, 5, "gelu", False),
        (3, 47, 47, 64, 3, 1, 1, "none", True), (7, 45, 47, 64, 3, 1, 1, "hswish", True), (5, 95, 99, 64, 3, 1, 0, "relu6", False), (9, 45, 47, 68, 3, 1, 1, "relu", True),
        (6, 47, 45, 64, 3, 2, 1, "relu", False), (15, 47, 47, 64, 3, 2, 1, "none", False), (45, 47, 45, 64, 3, 2, 1, "relu6", False),
        (3, 47, 47, 64, 5, 1, 2, "relu", True), (7, 45, 47, 64, 5, 1, 2, "none", True), (11, 45, 47, 64, 5, 1, 2, "relu6", True),
        (9, 47, 45, 64, 5, 2, 2, "none", False), (15, 47, 47, 64, 5, 2, 2, "relu", False), (31, 47, 45, 64, 5, 2, 2, "hswish", False),
        (1, 12, 13, 20, 5, 1, 2, "relu6", True), (12, 47, 45, 64, 5, 2, 2, "none", False),
    ]
    tenants = []
    for i, (batch, h, w, c, k, stride, pad, act, res) in enumerate(specs):
        b = G._B(f"dwt{i}", dtype, batch)
        x = b.tensor(batch, c, h, w)
        tenants.append(b.done(x, b.conv(x, c, k, stride, pad, act, groups=c, res=x if res else -1)))
    ran = check(tenants, [], [("batch", 2), ("cout", 2)])
    assert ran == {"dwconv3x3", "dwconv5x5_tiled"}, sorted(ran)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_depthwise_windows_larger_than_the_tensor(dtype):
    """One image smaller than its window runs on the generic kernels; two of them, or one that just holds the window of one output, on
    the tiled ones."""
    from synth import graphs as G
    tenants = []
    for i, (batch, h, w, c, k, stride, pad) in enumerate([(1, 1, 1, 40, 3, 1, 1), (1, 2, 2, 40, 5, 1, 2), (1, 1, 1, 24, 5, 2, 2), (1, 1, 3, 12, 3, 1, 1),
                                                          (1, 3, 1, 12, 5, 1, 2), (1, 2, 2, 40, 3, 1, 1), (2, 1, 1, 40, 3, 1, 1), (1, 3, 3, 40, 5, 2, 2)]):
        b = G._B(f"tiny{i}", dtype, batch)
        x = b.tensor(batch, c, h, w)
        tenants.append(b.done(x, b.conv(x, c, k, stride, pad, "relu6", groups=c)))
    ran = check(tenants, [], [("cout", 2)])
    assert ran == {"dwconv", "dwconv5x5", "dwconv3x3", "dwconv5x5_tiled"}, sorted(ran)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pools_and_norms_read_up_front(dtype):
    """Pooling windows of 2 and 3 (maximum with and without padding, mean, images smaller than the window) and the
    ones left to the tap by tap kernel (5, ragged channels); global means around the 16 and 64 positions a wavefront has in flight,
    with a remainder of channels; layer normalisation of one to four vectors per lane with and without a remainder and a residual;
    softmax rows of every lane group."""
    from synth import graphs as G
    tenants = []

    def one(name, batch, shape, op):
        b = G._B(name, dtype, batch)
        x = b.tensor(batch, *shape)
        tenants.append(b.done(x, op(b, x)))
    for i, (batch, c, h, w, k, stride, pad) in enumerate([(2, 24, 13, 11, 3, 2, 1), (3, 40, 9, 7, 3, 1, 1), (1, 8, 1, 2, 3, 1, 1), (2, 16, 8, 9, 2, 2, 0),
                                                          (2, 16, 6, 5, 2, 1, 1), (2, 16, 9, 9, 5, 2, 2), (2, 11, 9, 8, 3, 2, 0)]):
        one(f"max{i}", batch, (c, h, w), lambda b, x: b.maxpool(x, k, stride, pad))
    for i, (c, h, k, stride) in enumerate([(24, 9, 2, 2), (16, 10, 3, 1), (9, 7, 3, 2)]):
        one(f"mean{i}", 2, (c, h, h + 1), lambda b, x: b.avgpool(x, k, stride))
    for i, (c, h, w) in enumerate([(65, 1, 1), (130, 8, 8), (72, 5, 13), (64, 16, 16), (20, 15, 17), (33, 25, 31)]):
        one(f"gap{i}", 3, (c, h, w), lambda b, x: b.gavgpool(x))
    for i, (c, rows) in enumerate([(8, 5), (256, 3), (512, 6), (520, 7), (768, 9), (1024, 2), (1032, 5), (2048, 3), (2056, 2), (13, 4)]):
        one(f"ln{i}", 2, (c, rows, 1), lambda b, x: b.layernorm(x, x if i % 2 else -1))
    for i, c in enumerate([8, 16, 24, 64, 120, 256, 512, 7]):
        one(f"sm{i}", 2, (c, 9, 1), lambda b, x: b.softmax(x))
    check(tenants, ["maxpool", "gavgpool", "layernorm", "softmax"], [("batch", 2)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_depthwise_5x5(dtype):
    """The tiled 5x5 kernel: output rows shorter than a tile, one past it, strides 1 and 2, padding 0 to 2, a residual; ragged channel
    ranges and stride 3 on the one-vector kernel.  Chunks of what is tiled as a whole run on either."""
    from synth import graphs as G
    specs = [  # batch, hw, c, stride, pad, act, residual
        (3, 7, 24, 1, 2, "hswish", True), (2, 14, 40, 2, 2, "relu", False), (1, 5, 8, 1, 0, "none", False), (2, 9, 12, 2, 1, "relu6", False),
        (2, 13, 9, 1, 2, "none", False), (1, 11, 16, 3, 2, "relu", False),
        (70, 9, 48, 1, 2, "hswish", True), (23, 25, 72, 2, 2, "relu", False), (31, 19, 40, 1, 0, "none", False), (45, 30, 36, 2, 1, "relu6", False),
        (190, 3, 160, 1, 2, "none", False),
    ]
    tenants = []
    for i, (batch, hw, c, stride, pad, act, res) in enumerate(specs):
        b = G._B(f"dw{i}", dtype, batch)
        x = b.tensor(batch, c, hw, hw)
        tenants.append(b.done(x, b.conv(x, c, 5, stride, pad, act, groups=c, res=x if res else -1)))
    ran = check(tenants, ["dwconv5x5_tiled"], [("batch", 2), ("cout", 2), ("cout", 8)])
    assert "dwconv5x5" in ran, sorted(ran)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_affine_in_front_of_a_product_around_channel_windows(dtype):
    """Affine + ReLU that writes a channel window of a wider tensor, read by a 1x1 convolution: the neighbouring channels,
    written by another operator, keep their contents.  One that reads a window whose rows do not start at whole vectors."""
    from synth import graphs as G
    tenants = []
    for i, (batch, hw, cout) in enumerate([(2, 5, 40), (3, 40, 64)]):           # a window read at a pitch that is no whole vector
        b = G._B(f"rows{i}", dtype, batch)
        x, wide = b.tensor(batch, 24, hw, hw), b.tensor(batch, 21, hw, hw)
        y = b.affine(b.conv(x, 16, 3, 1, 1, "none", out=b.view(wide, 0, 16)), "relu")
        tenants.append(b.done(x, b.conv(y, cout, 1, 1, 0, "relu")))
    for i, (batch, hw, cout) in enumerate([(2, 5, 40), (3, 40, 64), (1, 64, 136)]):          # K slices, one and several tiles per unit
        b = G._B(f"pair{i}", dtype, batch)
        x, wide = b.tensor(batch, 24, hw, hw), b.tensor(batch, 64, hw, hw)
        b.conv(x, 16, 1, 1, 0, "none", out=b.view(wide, 24, 16))
        y, mid = b.conv(x, 16, 3, 1, 1, "relu"), b.view(wide, 8, 16)
        b.t.ops.append(G.Op("affine", y, mid, scale=b.param((16,), "uniform"), shift=b.param((16,), "uniform"), cin=16, cout=16, act="relu"))
        tenants.append(b.done(x, b.conv(mid, cout, 1, 1, 0, "relu")))
    check(tenants, ["eltwise"], [("batch", 2), ("cout", 2)])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_affine_pair_over_buffers_that_are_used_again(dtype):
    """Two buffers in turn: an affine in place, and a product that writes where the affine's input was.  Outputs are those of tensors with
    memory of their own, the pairs are issued one by one."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_11745_amd import binding as B
    from paper_2304_11745_amd import harness
    from synth import graphs as G
    tenants = []
    for i, (batch, hw, c) in enumerate([(2, 9, 136), (3, 40, 64)]):
        b = G._B(f"turn{i}", dtype, batch)
        x = b.tensor(batch, 24, hw, hw)
        y = b.conv(x, c, 3, 1, 1, "none")
        tenants.append(b.done(x, b.conv(b.affine(y, "relu"), c, 1, 1, 0, "relu")))
    sess = harness.Session(tenants, [G.materialise(t, 411, i << 20) for i, t in enumerate(tenants)])

    def run():
        sess.run(B.GACER_MODE_SEQUENTIAL, 2)
        return [sess.tensor_bytes(i, t.output) for i, t in enumerate(tenants)], sess.launch_count(B.GACER_MODE_SEQUENTIAL)
    want, launches = run()
    assert launches == 4
    assert tenants[0].output == tenants[1].output
    for tensor, over in ((tenants[0].output, tenants[0].ops[0].out), (tenants[0].ops[1].out, tenants[0].ops[0].out)):
        at = [sess._descs[i].tensors[tensor].dptr for i in range(2)]
        for i in range(2):
            sess._descs[i].tensors[tensor].dptr = sess._descs[i].tensors[over].dptr
        sess.poison_outputs()
        B.check(sess.ctx, B.gacer_load_tenants(sess.ctx, sess._descs, 2))
        sess.run(B.GACER_MODE_SEQUENTIAL, 2)
        assert sess.launch_count(B.GACER_MODE_SEQUENTIAL) == 6
        assert [sess.tensor_bytes(i, over if tensor == t.output else t.output) for i, t in enumerate(tenants)] == want, (tensor, over)
        for i in range(2):
            sess._descs[i].tensors[tensor].dptr = at[i]
    sess.close()
