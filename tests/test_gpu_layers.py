"""Per-kernel GPU parity against the CPU oracle on small seeded shapes that span
several tiles and ragged tails (odd sizes, stride 2, padding edges, channel
counts that are not multiples of the tile)."""
import numpy as np
import pytest

from workloads import gen, zoo

pytestmark = pytest.mark.gpu

BF16_TOL = 1e-2   # relative L2 vs the fp32-activation oracle (mode F)
F32_TOL = 1e-4




def _run_case(model, seed, batch, act_dtype=None, tol=None, bias_std=0.1, kernels=()):
    """kernels: (launch name with tile, problems) pairs the schedule has to hold."""
    from tests import harness
    model.shapes()
    blob = gen.make_blob(model, seed, bias_std=bias_std)
    x = gen.make_input(seed + 1, batch, model.in_c, model.in_h, model.in_w, "normal", model.dtype)
    g = harness.GpuDag([(model, blob, act_dtype)], batch)
    try:
        have = [(L.kernel, L.n_problems) for L in g.dag.launches()]
        for name, n in kernels:
            assert sum(k for h, k in have if h == name) == n, (name, n, have)
        y = g.run(x)[0]
    finally:
        g.close()
    wide = (model.dtype == "f32") or act_dtype == "f32"
    ref_f = harness.oracle_nhwc(model, blob, x, False)
    assert y.shape == ref_f.shape
    assert np.isfinite(y).all()
    e = harness.rel_l2(y, ref_f)
    lim = tol if tol is not None else (F32_TOL if wide else BF16_TOL)
    assert e <= lim, f"rel L2 {e} > {lim}"
    if not wide:
        ref_s = harness.oracle_nhwc(model, blob, x, True)
        assert harness.rel_l2(y, ref_s) <= 2e-3
        ex = harness.elem_excess(y, ref_s, harness.ELEM_C_BF16)
    else:
        ex = harness.elem_excess(y, ref_f, harness.ELEM_C_F32)
    assert ex <= 1.0, f"an element is {ex:.2f}x its bound away from the oracle"
    return e


CONV_CASES = [  # cin, cout, k, stride, pad, H, W, batch
    (3, 16, 3, 1, 1, 32, 32, 1), (3, 64, 7, 2, 3, 37, 41, 2), (16, 24, 1, 1, 0, 17, 19, 3), (24, 144, 1, 1, 0, 28, 28, 2),
    (64, 64, 3, 1, 1, 14, 14, 2), (32, 160, 3, 2, 1, 15, 15, 3), (128, 256, 3, 2, 1, 9, 9, 2), (72, 40, 3, 1, 0, 11, 13, 1),
    (256, 512, 1, 2, 0, 14, 14, 2), (8, 8, 3, 1, 1, 5, 5, 1), (320, 1280, 1, 1, 0, 7, 7, 2), (64, 192, 3, 1, 1, 56, 56, 1),
    (3, 64, 11, 4, 2, 67, 71, 2), (64, 192, 5, 1, 2, 27, 27, 2), (16, 32, 15, 1, 7, 19, 17, 1),   # large kernels (up to 15x15)
]


@pytest.mark.parametrize("case", CONV_CASES)
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_conv_relu(case, mode):
    cin, cout, k, s, p, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("c", dtype, cin, h, w)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU)
    _run_case(m, 100 + cin + cout, b, act_dtype="f32" if mode == "bf16_wide" else None)


KWAVE_CASES = [  # cin, cout, k, stride, pad, H, W, batch, tile
    (64, 64, 3, 1, 1, 56, 56, 4, "64x64x4"),          # 196 tiles of 64x64, the last one whole
    (12, 70, 3, 1, 1, 61, 53, 3, "64x64x4"),          # ragged rows and columns, Cop % 4 != 0, a step that spans three taps
    (4, 128, 1, 1, 0, 80, 81, 2, "64x64x4"),          # a reduction of one piece
    (3, 64, 5, 2, 2, 161, 157, 4, "64x64x4 scalar"),  # element-wise fetch (3 channels)
    (5, 33, 3, 1, 1, 8, 4, 1, "32x32x8 scalar"),      # element-wise fetch: exactly one tile of rows, one column past one tile
    (36, 31, 3, 2, 1, 9, 11, 1, "32x32x8"),           # ragged, a tail of 4 elements in the last step, Cop % 4 != 0
    (32, 32, 1, 1, 0, 33, 1, 1, "32x32x8"),           # one step for eight waves, one row past a tile
    (512, 36, 3, 1, 1, 7, 7, 3, "32x32x8"),           # 144 steps over eight waves
]


@pytest.mark.parametrize("case", KWAVE_CASES)
def test_conv_f32_shared_reduction(case):
    """fp32 convolutions with the reduction shared by the waves of a workgroup, at the edges of the tiles and of the
    reduction steps, with a residual; held to 2 sqrt(K) fp32 roundings of the oracle's (the serial sum's typical error
    and this kernel's, which is smaller)."""
    cin, cout, k, s, p, h, w, b, tile = case
    m = zoo.Model("c", "f32", cin, h, w)
    a = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU, residual=a)
    _run_case(m, 900 + cin + cout, b, tol=2.0 * (cin * k * k) ** 0.5 * 2.0 ** -23, kernels=[("conv_kwave " + tile, 2)])


# (with 16 x 16 pixels x 32 channels a workgroup: ragged pixel and channel blocks, channel counts that 4 and 8 do not divide, strides, a
# patch wider than the image's padding, one and two input channels)
@pytest.mark.parametrize("case", [(3, 64, 3, 1, 1, 101, 97, 4), (3, 70, 7, 2, 3, 229, 221, 4), (1, 36, 5, 2, 2, 263, 255, 4), (2, 39, 3, 2, 0, 250, 203, 8)])
def test_conv_f32_patch_of_few_channels(case):
    """fp32 convolutions of one to three channels over an input patch in LDS, with a residual; the bound of the shared reduction."""
    cin, cout, k, s, p, h, w, b = case
    m = zoo.Model("c", "f32", cin, h, w)
    a = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.HARDSWISH, residual=a)
    _run_case(m, 940 + cin + cout, b, tol=2.0 * (cin * k * k) ** 0.5 * 2.0 ** -23, kernels=[("conv_rgb", 2)])


def test_conv_f32_few_channel_siblings():
    """Sibling layers of two, three, one and three channels, 3x3 stride 2 on 224 x 224: held like the above."""
    m = zoo.Model("c", "f32", 3, 224, 224)
    sides = [m.add(zoo.CONV, -1, cin=3, cout=c, k=1, stride=1, pad=0, act=zoo.NONE) for c in (2, 3, 1, 3)]
    wide = [m.add(zoo.CONV, a, cin=c, cout=32, k=3, stride=2, pad=1, act=zoo.RELU) for a, c in zip(sides, (2, 3, 1, 3))]
    t = wide[0]
    for w in wide[1:]:
        t = m.add(zoo.CONCAT, t, residual=w)
    _run_case(m, 950, 4, tol=2.0 * ((9 * 3) ** 0.5 + 3 ** 0.5) * 2.0 ** -23, kernels=[("conv_rgb", 4)])   # (the roundings of both layers)


@pytest.mark.parametrize("cin, k, kw", [(1, 2, 0), (1, 7, 1), (2, 2, 1), (1, 3, 0), (3, 3, 0), (3, 1, 7)])
def test_conv_f32_few_channels_loses_nothing_to_a_serial_sum(cin, k, kw):
    """The distance from 64 bits is no larger than that of one fused multiply-add after another, the longest order any kernel has (both of
    2 x 64 x 80 x 80 elements: the two distances' own scatter is below 0.5 %)."""
    m = zoo.Model("c", "f32", cin, 80 + k - 1, 80 + (kw or k) - 1)
    m.add(zoo.CONV, -1, cin=cin, cout=64, k=k, kw=kw, stride=1, pad=0, act=zoo.NONE)
    m.add(zoo.MAXPOOL, 0, k=1, stride=1, pad=0)
    m.shapes()
    blob = gen.make_blob(m, 61, bias_std=0.1)
    x = gen.make_input(62, 16, cin, m.in_h, m.in_w, "normal", "f32")
    from tests import harness
    g = harness.GpuDag([(m, blob, None)], 16)
    try:
        assert "conv_rgb" in [L.kernel for L in g.dag.launches()]
        y = g.run(x)[0][:2].reshape(2, 80, 80, 64)
    finally:
        g.close()
    L = m.layers[0]
    w = blob[L.w_off:L.w_off + 4 * 64 * cin * k * (kw or k)].view(np.float32).reshape(64, cin, k, kw or k).astype(np.float64)
    b = blob[L.b_off:L.b_off + 256].view(np.float32).astype(np.float64)
    exact, serial = np.zeros((2, 80, 80, 64)), np.zeros((2, 80, 80, 64), np.float32)
    for r in range(k):
        for s in range(kw or k):
            for c in range(cin):
                p = x[:2, c, r:r + 80, s:s + 80, None].astype(np.float64) * w[:, c, r, s]   # (exact: two 24-bit factors)
                exact += p
                serial = (serial + p).astype(np.float32)
    exact, serial = exact + b, (serial + b).astype(np.float32)
    assert np.linalg.norm(y - exact) <= 1.005 * np.linalg.norm(serial - exact)


@pytest.mark.parametrize("case", [(64, 40, 3, 1, 1, 61, 57, 4, "64x64x4"), (3, 64, 7, 2, 3, 161, 157, 4, "rgb"), (5, 64, 7, 2, 3, 161, 157, 4, "64x64x4 scalar"),
                                  (5, 33, 3, 1, 1, 9, 11, 1, "32x32x8 scalar"), (36, 31, 5, 2, 2, 9, 11, 1, "32x32x8")])
def test_conv_f32_weights_that_are_not_finite(case):
    """Infinite and NaN weights reach the outputs whose window holds their tap, and no output at the border where the tap
    lies outside the image; every other value meets the bound of the finite case."""
    from tests import harness
    cin, cout, k, s, p, h, w, b, tile = case
    m = zoo.Model("c", "f32", cin, h, w)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    m.shapes()
    blob = gen.make_blob(m, 71)
    wt = blob[m.layers[0].w_off:m.layers[0].w_off + 4 * cout * cin * k * k].view(np.float32).reshape(cout, cin, k, k)
    for o, value in ((1, np.inf), (2, -np.inf), (cout - 1, np.nan)):
        wt[o, cin - 1, 0, 0] = value      # outside the image in the first row and the first column
    wt[3, 0, k - 1, k - 1] = np.inf       # ... in the last ones
    x = gen.make_input(72, b, cin, h, w, "normal", "f32")
    g = harness.GpuDag([(m, blob, None)], b)
    try:
        assert ("conv_rgb" if tile == "rgb" else "conv_kwave " + tile) in [L.kernel for L in g.dag.launches()]
        y = g.run(x)[0]
    finally:
        g.close()
    ref = harness.oracle_nhwc(m, blob, x, False)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
    assert np.array_equal(y[np.isinf(y)], ref[np.isinf(ref)])
    border = ref.reshape(b, m.layers[0].out_h, m.layers[0].out_w, cout)[:, 0, :, 1]
    assert np.isfinite(border).all()
    finite = np.isfinite(ref)
    assert harness.rel_l2(y[finite], ref[finite]) <= 2.0 * (cin * k * k) ** 0.5 * 2.0 ** -23


@pytest.mark.parametrize("case", [(1, 8, 3, 1, 1, 61, 57, 5), (3, 3, 1, 1, 0, 97, 89, 3), (5, 7, 3, 2, 1, 301, 199, 5), (8, 8, 1, 1, 0, 67, 129, 4), (2, 1, 2, 2, 0, 131, 67, 9)])
def test_conv_f32_of_few_products(case):
    """fp32 convolutions of few channels and products, one thread per output element, with a residual; held like the above."""
    cin, cout, k, s, p, h, w, b = case
    m = zoo.Model("c", "f32", cin, h, w)
    a = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU, residual=a)
    _run_case(m, 930 + cin + cout, b, tol=2.0 * (cin * k * k) ** 0.5 * 2.0 ** -23, kernels=[("conv_direct", 2)])


def test_conv_f32_beyond_the_shared_reduction():
    """2^24 output rows, one more than the shared-reduction kernel decodes: the element-wise kernel, held like the above."""
    m = zoo.Model("c", "f32", 1, 4096, 4096)
    m.add(zoo.CONV, -1, cin=1, cout=1, k=3, stride=1, pad=1, act=zoo.RELU)
    _run_case(m, 911, 1, tol=2.0 * 9 ** 0.5 * 2.0 ** -23, kernels=[("conv_direct", 1)])


@pytest.mark.parametrize("case", [(128, 40, 3, 1, 1, 8, 4, 1),    # exactly one tile of rows, 18 steps over eight waves, a ragged column tile
                                  (120, 31, 3, 2, 1, 13, 11, 1),  # rows padded to 32 elements: the last step is half a step; padding channels
                                  (1024, 32, 1, 1, 0, 11, 3, 1),  # 16 steps, one row past a tile
                                  (512, 512, 3, 1, 1, 7, 7, 3),   # many column tiles, 72 steps
                                  (64, 128, 5, 1, 0, 36, 36, 4)]) # 64 tiles of rows: the end of the range
def test_conv_bf16_shared_reduction(case):
    """bf16 convolutions of few tiles and a long reduction: with a residual, and stored inside a concatenation."""
    cin, cout, k, s, p, h, w, b = case
    m = zoo.Model("c", "bf16", cin, h, w)
    e = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    r = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU, residual=e)
    c = m.add(zoo.CONV, -1, cin=cin, cout=24, k=k, stride=s, pad=p, act=zoo.HARDSWISH)
    q = m.add(zoo.CONCAT, c, residual=r)
    m.add(zoo.CONV, q, cin=24 + cout, cout=32, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 970 + cin + cout, b, kernels=[("conv_kwave 32x32x8", 1), ("conv_kwave 64x64x8", 2)] if h == 36 else [("conv_kwave 32x32x8", 3)])   # (the last case: two problems share a launch)


@pytest.mark.parametrize("case", [(512, 512, 3, 1, 1, 7, 7, 16, 3),    # whole tiles of columns, ragged rows
                                  (1024, 120, 1, 1, 0, 31, 1, 24, 16), # ragged rows and columns, 16 steps: two per wave
                                  (120, 248, 3, 2, 1, 13, 11, 9, 16),  # a step that spans two taps, a last step of half its length
                                  (2048, 512, 1, 1, 0, 5, 5, 5, 16)])  # weights larger than the input
def test_shared_reduction_in_large_launches_keeps_its_bits(case):
    """One member has 32x32 tiles, a launch of many members 64x64 ones: the same bits, a residual included."""
    from tests import harness
    cin, cout, k, s, p, h, w, b, members = case
    m = zoo.Model("c", "bf16", cin, h, w)
    e = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.NONE)
    r = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.HARDSWISH, residual=e)
    m.add(zoo.MAXPOOL, r, k=1, stride=1, pad=0)
    m.shapes()
    blob = gen.make_blob(m, 81)
    x = gen.make_input(82, b, cin, h, w, "normal", "bf16")
    outs = []
    for n, kernel in ((1, "conv_kwave 32x32x8"), (members, "conv_kwave 64x64x8")):
        g = harness.GpuDag([(m, blob, None)] * n, b)
        try:
            assert sum(L.n_problems for L in g.dag.launches() if L.kernel == kernel) == 2 * n, [L.kernel for L in g.dag.launches()]
            outs.append(g.run(x))
        finally:
            g.close()
    assert all(np.array_equal(y, outs[0][0]) for y in outs[1])
    harness.check_against_oracle("shared reduction", m, blob, None, x, outs[0][0], rows=[0, b - 1])


PATCH_CASES = [  # cin, cout, groups, H, W, batch, tile
    (128, 32, 1, 90, 91, 8, "256x32"),           # the widest image of the 256-row patches, a ragged last tile, two runs of 64 channels
    (64, 64, 1, 56, 56, 21, "256x64"),           # one run of 64 channels
    (192, 72, 1, 41, 37, 22, "256x64"),          # three runs, a ragged column tile
    (64, 520, 1, 57, 45, 11, "512x128"),         # a ragged column tile
    (128, 136, 1, 57, 45, 26, "512x128"),        # two runs of 64 channels, ragged rows and columns
    (64, 264, 1, 19, 140, 17, "512x128"),        # an image wider than the 256-row patches hold
    (256, 256, 32, 41, 67, 6, "256x64 diag"),    # groups of 8: diagonal blocks
    (256, 256, 32, 27, 220, 3, "512x64 diag"),   # the same, 512 rows
    (256, 256, 4, 1, 91, 181, "256x64"),         # groups of 64, images of one row
]


@pytest.mark.parametrize("case", PATCH_CASES)
def test_conv_patch(case):
    """3x3 stride-1 convolutions from an input patch in LDS: with a residual, and stored inside a concatenation."""
    cin, cout, groups, h, w, b, tile = case
    m = zoo.Model("c", "bf16", cin, h, w)
    conv = dict(cin=cin, cout=cout, k=3, stride=1, pad=1, groups=groups)
    e = m.add(zoo.CONV, -1, act=zoo.NONE, **conv)
    s = m.add(zoo.CONV, -1, cin=cin, cout=8, k=1, stride=1, pad=0, act=zoo.NONE)
    r = m.add(zoo.CONV, -1, act=zoo.HARDSWISH if tile == "256x32" else zoo.RELU6, residual=e, **conv)
    q = m.add(zoo.CONCAT, s, residual=r)
    m.add(zoo.CONV, q, cin=8 + cout, cout=8, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 990 + cin + cout + groups, b, kernels=[("conv_patch " + tile, 2)])


def _same_bits(m, few, many, kernel_few, kernel_many, x=None, blob=None):
    """The first images of a batch, run in a handle for `few` and in one for `many` images, asserting each one's kernel."""
    from tests import harness
    m.shapes()
    blob = gen.make_blob(m, 61) if blob is None else blob
    x = gen.make_input(62, many, m.in_c, m.in_h, m.in_w, "normal", m.dtype) if x is None else x
    ys = []
    for b, kernel in ((few, kernel_few), (many, kernel_many)):
        g = harness.GpuDag([(m, blob, None)], b)
        try:
            assert kernel in [L.kernel for L in g.dag.launches()], (kernel, [L.kernel for L in g.dag.launches()])
            ys.append(g.run(x[:b])[0][:few])
        finally:
            g.close()
    assert np.array_equal(ys[0], ys[1], equal_nan=True)
    return x, blob, ys[0]


@pytest.mark.parametrize("case", [(64, 32, 1, 23, 29, 5, 70, "conv_mfma_64x64", "256x32"),
                                  (128, 136, 1, 57, 45, 3, 26, "conv_mfma_64x64", "512x128"),
                                  (192, 72, 1, 41, 37, 7, 22, "conv_mfma_64x64", "256x64"),
                                  (256, 256, 32, 21, 35, 2, 24, "conv_mfma_64x64", "256x64 diag"),
                                  (256, 256, 32, 7, 220, 1, 12, "conv_mfma_64x64", "512x64 diag"),
                                  (256, 256, 4, 21, 35, 2, 24, "conv_mfma_64x64", "256x64")])
def test_conv_patch_has_the_bits_of_the_tile_kernel(case):
    """The planner takes the patch kernel by the size of a launch: an image's bits must not depend on it."""
    cin, cout, groups, h, w, few, many, small, tile = case
    m = zoo.Model("c", "bf16", cin, h, w)
    a = m.add(zoo.CONV, -1, cin=cin, cout=cout, k=3, stride=1, pad=1, groups=groups, act=zoo.NONE)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    assert np.isfinite(_same_bits(m, few, many, small, "conv_patch " + tile)[2]).all()


def _bits_and_parity(m, act_dtype, few, many, seed=71, kernel=None, n=1):
    """The first images of a batch of `many`, n of whose launches are issued to `kernel`, have the bits that a batch of `few`, none of whose are,
    gives them, and meet the oracle."""
    from tests import harness
    m.shapes()
    blob = gen.make_blob(m, seed, bias_std=0.1)
    x = gen.make_input(seed + 1, many, m.in_c, m.in_h, m.in_w, "normal", m.dtype)
    g = harness.GpuDag([(m, blob, act_dtype)], many)
    try:
        if kernel:
            names = {b: [L.name.decode() for L in g.dag.launches(b)] for b in (few, many)}
            assert names[many].count(kernel) == n and kernel not in names[few], names
        large, small = g.run(x)[0], g.run(x[:few])[0]
    finally:
        g.close()
    assert np.isfinite(large).all() and np.array_equal(large[:few], small)
    wide = act_dtype == "f32"
    last = x[-1:]   # (the ragged end of the launch)
    ref = harness.oracle_nhwc(m, blob, last, not wide)
    assert harness.rel_l2(large[-1:], ref) <= (F32_TOL if wide else 2e-3)
    assert harness.elem_excess(large[-1:], ref, harness.ELEM_C_F32 if wide else harness.ELEM_C_BF16) <= 1.0


# Rows of 61 x 53 pixels: 6 images are 607 blocks of 32 (the last of 6 rows), 12 are 1213, 16 1617, 21 2122, 31 3133, 41 4143; one image is 102, too
# few for any form.  `streams`: of the three layers (8 -> cin, cin -> cout, cout -> cin with the first as residual) so many do.
@pytest.mark.parametrize("cin, cout, act_dtype, many, streams", [(8, 8, None, 12, 3), (40, 40, None, 12, 3), (72, 24, None, 12, 2), (64, 128, None, 12, 2), (128, 40, None, 21, 2),
                                                                 (200, 104, None, 41, 2), (328, 24, None, 31, 2), (16, 64, "f32", 21, 3), (24, 72, "f32", 12, 2), (40, 8, "f32", 12, 2),
                                                                 (104, 32, "f32", 21, 2), (184, 96, "f32", 16, 2)])
def test_pointwise_rows_that_stream(cin, cout, act_dtype, many, streams):
    """Many rows and a short reduction stream through waves of their own; one image keeps the tile kernel: the same bits.
    Partial pieces and blocks of columns, a residual, every activation the kernel has."""
    m = zoo.Model("c", "bf16", 8, 61, 53)
    e = m.add(zoo.CONV, -1, cin=8, cout=cin, k=1, stride=1, pad=0, act=zoo.RELU6)
    a = m.add(zoo.CONV, e, cin=cin, cout=cout, k=1, stride=1, pad=0, act=zoo.HARDSWISH)
    a = m.add(zoo.CONV, a, cin=cout, cout=cin if cin <= 128 else 16, k=1, stride=1, pad=0, act=zoo.RELU, residual=e if cin <= 128 else zoo.NO_RESIDUAL)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    _bits_and_parity(m, act_dtype, 1, many, kernel="conv_stream", n=streams)


@pytest.mark.parametrize("cout, stride, pad, act_dtype", [(16, 2, 1, "f32"), (40, 1, 0, "f32"), (104, 2, 0, "f32"), (24, 2, 1, None), (64, 1, 1, "f32"), (128, 2, 1, None), (40, 1, 1, None)])
def test_first_layers_that_stream(cout, stride, pad, act_dtype):
    """3x3 convolutions over the model input gather their rows tap by tap: ragged blocks of rows and columns, windows over every border."""
    m = zoo.Model("c", "bf16", 3, 123 if stride == 2 else 61, 107 if stride == 2 else 53)
    a = m.add(zoo.CONV, -1, cin=3, cout=cout, k=3, stride=stride, pad=pad, act=zoo.HARDSWISH if cout == 16 else zoo.RELU6)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    _bits_and_parity(m, act_dtype, 1, 6, kernel="conv_stream")


@pytest.mark.parametrize("h, w, c, pad, act_dtype, many", [(61, 53, 160, 1, None, 12), (61, 53, 160, 1, None, 16), (60, 50, 136, 0, None, 24), (61, 53, 160, 1, "f32", 12), (60, 50, 136, 0, "f32", 18), (33, 30, 248, 1, "f32", 24)])
def test_depthwise_two_rows_per_thread(h, w, c, pad, act_dtype, many):
    """3x3 stride-1 depthwise layers of 384 workgroups or more (bf16 rows 512) compute two rows per thread; one image keeps one row: the same bits."""
    m = zoo.Model("c", "bf16", 8, h, w)
    a = m.add(zoo.CONV, -1, cin=8, cout=c, k=1, stride=1, pad=0, act=zoo.RELU)
    a = m.add(zoo.DWCONV, a, cin=c, cout=c, k=3, stride=1, pad=pad, act=zoo.HARDSWISH if c == 160 else zoo.RELU6)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    _bits_and_parity(m, act_dtype, 1, many, kernel="dwconv_rows", n=1 if act_dtype or many > 12 else 0)


# 21 images: 2122 blocks of 32 rows, resident weights; 6 images: 607, 152 workgroups with the weights in a ring (440 channels are seven pieces); other
# activations than ReLU keep the tile, and `n` counts the plain layers that stream
@pytest.mark.parametrize("first, grow, act, many, kernel, n", [(64, 32, zoo.RELU, 21, "conv_stream", 5), (40, 24, zoo.RELU6, 16, "conv_stream", 3), (128, 72, zoo.NONE, 16, "conv_stream", 1),
                                                               (64, 32, zoo.RELU, 6, "conv_long", 2), (136, 40, zoo.RELU, 6, "conv_long", 2), (200, 56, zoo.RELU, 6, "conv_long", 2),
                                                               (440, 72, zoo.RELU, 6, "conv_long", 2)])
def test_dense_layers_that_stream(first, grow, act, many, kernel, n):
    """Dense layers whose rows stream: an affine stage on the way in, the input a prefix of a concatenation's tensor."""
    m = zoo.Model("c", "bf16", 8, 61, 53)
    t = m.add(zoo.CONV, -1, cin=8, cout=first, k=1, stride=1, pad=0, act=zoo.RELU)
    c = first
    for _ in range(2):
        a = m.add(zoo.DWCONV, t, cin=c, cout=c, k=1, stride=1, pad=0, act=act)
        a = m.add(zoo.CONV, a, cin=c, cout=128, k=1, stride=1, pad=0, act=zoo.RELU)
        a = m.add(zoo.CONV, a, cin=128, cout=grow, k=1, stride=1, pad=0, act=zoo.NONE)
        t = m.add(zoo.CONCAT, t, residual=a)
        c += grow
    m.add(zoo.MAXPOOL, t, k=1, stride=1, pad=0)
    _bits_and_parity(m, None, 1, many, kernel=kernel, n=n)


def _streaming_model(kind, side=61):
    m = zoo.Model("c", "bf16", 3 if kind == "first" else 8, side, 53)
    if kind == "first":
        a = m.add(zoo.CONV, -1, cin=3, cout=24, k=3, stride=1, pad=1, act=zoo.HARDSWISH)
    else:
        a = m.add(zoo.CONV, -1, cin=8, cout=72, k=1, stride=1, pad=0, act=zoo.SILU)
        if kind == "affine":
            a = m.add(zoo.DWCONV, a, cin=72, cout=72, k=1, stride=1, pad=0, act=zoo.RELU)
        a = m.add(zoo.CONV, a, cin=72, cout=128 if kind == "affine" else 24, k=1, stride=1, pad=0, act=zoo.NONE)
    m.add(zoo.AVGPOOL, a, k=1, stride=1, pad=0)   # (a maximum would drop NaN)
    return m.shapes()


@pytest.mark.parametrize("kind, act_dtype, batch, kernel", [("plain", None, 12, "conv_stream"), ("plain", "f32", 16, "conv_stream"), ("affine", None, 6, "conv_long"), ("affine", None, 21, "conv_stream"),
                                                            ("first", None, 6, "conv_stream"), ("first", "f32", 6, "conv_stream")])
def test_streaming_keeps_what_is_not_finite(kind, act_dtype, batch, kernel):
    """Infinite and NaN inputs, weights and biases: every image has the bits (NaN where it is NaN) of a pass of one, which keeps the tile kernel."""
    from tests import harness
    m = _streaming_model(kind)
    blob = gen.make_blob(m, 83, bias_std=0.1)
    last = m.layers[-2]
    k = last.k * last.k * last.cin
    w = blob[last.w_off:last.w_off + 2 * last.cout * k].view(np.uint16).reshape(last.cout, k)
    w[1, 0], w[2, k - 1], w[3, k // 2] = 0x7F80, 0xFF80, 0x7FC0   # inf, -inf, NaN
    blob[last.b_off:last.b_off + 4 * last.cout].view(np.float32)[4:7] = np.inf, -np.inf, np.nan
    x = gen.make_input(84, batch, m.in_c, 61, 53, "normal", "bf16")
    x[0, 0, 0, 0], x[1, 1, 60, 52], x[-1, 2, 60, 0], x[-1, 0, 30, 26] = np.inf, np.nan, -np.inf, np.inf
    g = harness.GpuDag([(m, blob, act_dtype)], batch)
    try:
        assert kernel in [L.name.decode() for L in g.dag.launches(batch)] and kernel not in [L.name.decode() for L in g.dag.launches(1)]
        large = g.run(x)[0]
        ones = np.concatenate([g.run(x[i:i + 1])[0] for i in (0, 1, 2, batch - 1)])
    finally:
        g.close()
    assert np.isnan(large).any() and np.isinf(large).any() and np.isfinite(large).any()
    assert np.array_equal(large[[0, 1, 2, batch - 1]], ones, equal_nan=True)


@pytest.mark.parametrize("kind, act_dtype, kernel", [("plain", None, "conv_stream"), ("plain", "f32", "conv_stream"), ("affine", None, "conv_stream"), ("first", None, "conv_stream"), ("long", None, "conv_long")])
def test_streaming_launches_of_ragged_members(kind, act_dtype, kernel):
    """Five members share a streaming launch with batches of their own, one of them none: every member has the bits of a DAG of its own, one image at a time."""
    import torch
    import paper_2410_21120_amd as fi
    from tests import harness
    m = _streaming_model("affine" if kind == "long" else kind)
    batches = {"plain": [9, 0, 1, 5, 14], "affine": [17, 0, 1, 6, 9], "first": [3, 0, 1, 1, 2], "long": [3, 0, 1, 1, 2]}[kind]
    B, blobs = max(batches), [gen.make_blob(m, 90 + i, bias_std=0.1) for i in range(len(batches))]
    xs = [gen.make_input(95 + i, B, m.in_c, 61, 53, "normal", "bf16") for i in range(len(batches))]
    made = [fi.make_spec(m, b.ctypes.data, b.nbytes, act_dtype=act_dtype) for b in blobs]
    dag = fi.Dag([s for s, _ in made], B, fi.TorchAllocators("cuda:0"), keepalive=(blobs, [k for _, k in made]), per_member_inputs=True, serial_lanes=True)
    stream = torch.cuda.current_stream().cuda_stream
    dag.load(stream)
    try:
        assert kernel in [L.name.decode() for L in dag.launches(-(-sum(batches) // len(batches)))]   # (as many blocks in all)
        n = m.layers[-1].cout * 61 * 53
        ins = [torch.from_numpy(gen.to_nhwc_storage(x, "bf16").view(np.int16)).cuda() for x in xs]
        outs = [torch.full((B, n), -7.0, dtype=torch.float32, device="cuda:0") for _ in batches]
        for _ in range(2):
            dag.run_batches([t.data_ptr() for t in ins], batches, [o.data_ptr() for o in outs], stream)
        torch.cuda.synchronize()
        got = [o.cpu().numpy() for o in outs]
    finally:
        dag.unload()
        dag.destroy()
    for i, b in enumerate(batches):
        assert np.all(got[i][b:] == -7.0), i
        g = harness.GpuDag([(m, blobs[i], act_dtype)], 1)
        try:
            for j in sorted({0, b // 2, b - 1}) if b else ():
                assert np.array_equal(got[i][j], g.run(xs[i][j:j + 1])[0][0]), (i, j)
        finally:
            g.close()


@pytest.mark.parametrize("features, batch", [(1000, 4), (1001, 33), (7, 1)])
def test_fc_f32_shared_reduction(features, batch):
    """fp32 fully connected layers over a flattened map (a reduction of 3 x 2 x 50 elements: not a whole step)."""
    m = zoo.Model("c", "f32", 50, 3, 2)
    a = m.add(zoo.CONV, -1, cin=50, cout=50, k=1, stride=1, pad=0, act=zoo.RELU)
    m.add(zoo.FC, a, cin=50 * 6, cout=features)
    _run_case(m, 950 + features, batch, tol=2.0 * 350 ** 0.5 * 2.0 ** -23)


@pytest.mark.parametrize("cin, k, stride", [(64, 3, 1), (128, 5, 2), (72, 3, 1)])
def test_conv_256x64_tile_has_the_bits_of_the_small_tile(cin, k, stride):
    """Images wider than a patch: the 256x64 tile walks 64-channel runs with a loop of its own, other channel strides with the common one."""
    m = zoo.Model("c", "bf16", cin, 131 if stride == 1 else 263, 125 if stride == 1 else 251)
    a = m.add(zoo.CONV, -1, cin=cin, cout=64, k=k, stride=stride, pad=k // 2, act=zoo.NONE)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    assert np.isfinite(_same_bits(m, 1, 5, "conv_mfma_64x64", "conv_mfma_256x64")[2]).all()


@pytest.mark.parametrize("case", [(32, 21, 35, 2, 24, "conv_mfma_64x64", "conv_patch 256x64 diag"), (32, 7, 220, 1, 12, "conv_mfma_64x64", "conv_patch 512x64 diag"),
                                  (8, 21, 35, 12, 24, "conv_mfma_128x64", "conv_patch 256x64 diag"), (16, 29, 110, 10, 20, "conv_mfma_128x64", "conv_mfma_256x64")])
def test_grouped_conv_activations_that_are_not_finite(case):
    """Groups of at most 32 channels: an infinite or NaN activation reaches the 32 output channels of its block and no others,
    whichever kernel the size of the launch asks for."""
    groups, h, w, few, many, small, large = case
    m = zoo.Model("c", "bf16", 256, h, w)
    a = m.add(zoo.CONV, -1, cin=256, cout=256, k=3, stride=2 if "mfma" in large else 1, pad=1, groups=groups, act=zoo.NONE)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    x = gen.make_input(62, many, 256, h, w, "normal", "bf16")
    x[0, 5, 2, 3], x[0, 70, 4, 30], x[0, 255, h - 1, w - 1] = np.inf, np.nan, -np.inf
    y = _same_bits(m, few, many, small, large, x=x)[2].reshape(few, -1, 8, 32)
    hit = ~np.isfinite(y[0]).all(axis=(0, 2))
    assert hit.tolist() == [True, False, True, False, False, False, False, True] and np.isfinite(y[1:]).all()


def test_long_reductions_in_small_launches_keep_their_bits():
    """ResNet-50's last stage in isolation, a 3x3 over 512 channels and a 1x1 over 2048 at 7x7: one member at batch 32 has
    64x64 tiles; at batch 96 the 3x3 reads from a patch; eight members at batch 32 take the patch and, for the 1x1, the 128x128 tile
    with three reduction tiles in flight (52 workgroups each).  A member's images must come out with the same bits (the
    reduction order depends on none of these), and meet the oracle."""
    from tests import harness
    m = zoo.Model("stage4", "bf16", 512, 7, 7)
    a = m.add(zoo.CONV, -1, cin=512, cout=512, k=3, stride=1, pad=1, act=zoo.RELU)
    a = m.add(zoo.CONV, a, cin=512, cout=2048, k=1, stride=1, pad=0, act=zoo.RELU)
    a = m.add(zoo.CONV, a, cin=2048, cout=512, k=1, stride=1, pad=0, act=zoo.RELU)
    m.add(zoo.CONV, a, cin=512, cout=24, k=1, stride=1, pad=0, act=zoo.NONE)
    m.shapes()
    blob = gen.make_blob(m, 777)
    x = gen.make_input(778, 96, 512, 7, 7, "normal", "bf16")
    outs = {}
    for members, batch, kernels in ((1, 32, ["conv_mfma_64x64"] * 3), (1, 96, ["conv_patch 256x64"]), (1, 31, ["conv_mfma_64x64"] * 3),
                                    (8, 32, ["conv_patch 256x64", "conv_mfma_128x128 deep"]),
                                    (8, 31, ["conv_patch 256x64", "conv_mfma_128x128 deep"])):   # (31: ragged last tiles)
        g = harness.GpuDag([(m, blob, None)] * members, batch)
        try:
            have = [L.kernel for L in g.dag.launches()]
            assert all(have.count(k) >= kernels.count(k) for k in kernels), have
            outs[members, batch] = g.run(x[:batch])
        finally:
            g.close()
    first = outs[1, 96][0]
    assert np.isfinite(first).all()
    for (members, batch), ys in outs.items():
        assert all(np.array_equal(y, first[:batch]) for y in ys), (members, batch)
    harness.check_against_oracle("last-stage layers, deep prefetch", m, blob, None, x[:32], outs[8, 32][0], rows=[0, 7, 31])


@pytest.mark.parametrize("case", [(128, 128, 3, 1, 1, 127, 129, 4),   # 256x128 tile: long reduction, ragged last tile
                                  (64, 64, 3, 1, 1, 127, 129, 4),     # 256x64 tile: narrow, long reduction
                                  (256, 128, 1, 1, 0, 127, 129, 4)])  # 128x128 tile, pointwise prologue
def test_conv_large_tiles_bf16(case):
    """Shapes large enough (>= 256 workgroups) for the planner to pick the 256-row tiles."""
    import paper_2410_21120_amd as fi
    from tests import harness
    cin, cout, k, s, p, h, w, b = case
    m = zoo.Model("t", "bf16", cin, h, w)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU)
    m.shapes()
    blob = gen.make_blob(m, 300 + cin)
    g = harness.GpuDag([(m, blob, None)], b)
    try:
        names = [L.name.decode() for L in g.dag.launches()]
    finally:
        g.close()
    want = "conv_mfma_256x128" if (cin, cout) == (128, 128) else "conv_mfma_256x64" if cin == 64 else "conv_mfma_128x128"
    assert want in names, names
    _run_case(m, 300 + cin, b)


@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
@pytest.mark.parametrize("act", [zoo.NONE, zoo.RELU, zoo.RELU6])
def test_conv_residual_and_activation(mode, act):
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("r", dtype, 16, 13, 13)
    a = m.add(zoo.CONV, -1, cin=16, cout=40, k=3, stride=1, pad=1, act=zoo.RELU)
    b = m.add(zoo.CONV, a, cin=40, cout=40, k=1, stride=1, pad=0, act=zoo.NONE)
    m.add(zoo.CONV, b, cin=40, cout=40, k=3, stride=1, pad=1, act=act, residual=a)
    _run_case(m, 7, 2, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(32, 3, 1, 1, 20, 20, 2), (96, 3, 2, 1, 15, 17, 2), (144, 3, 1, 1, 7, 7, 3), (24, 3, 2, 1, 9, 9, 1),
                                  (72, 5, 2, 2, 21, 19, 2), (120, 5, 1, 2, 14, 14, 2)])
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_depthwise(case, mode):
    c, k, s, p, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("d", dtype, c, h, w)
    m.add(zoo.DWCONV, -1, cin=c, cout=c, k=k, stride=s, pad=p, act=zoo.RELU6)
    _run_case(m, 200 + c, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(64, 3, 2, 1, 23, 23, 2), (16, 2, 2, 0, 32, 32, 1), (24, 2, 2, 0, 15, 17, 3)])
@pytest.mark.parametrize("mode", ["bf16", "f32"])
def test_maxpool_exact(case, mode):
    """Pooling moves values without arithmetic: the result is bit-exact."""
    from tests import harness
    c, k, s, p, h, w, b = case
    m = zoo.Model("p", mode, c, h, w)
    m.add(zoo.MAXPOOL, -1, k=k, stride=s, pad=p)
    m.shapes()
    blob = np.zeros(64, np.uint8)
    x = -np.abs(gen.make_input(3, b, c, h, w, "normal", mode)) - 1.0  # all negative: padding must not win
    if mode == "bf16":
        x = gen.bf16_to_f32(gen.bf16_bits(x)).reshape(x.shape)
    g = harness.GpuDag([(m, blob)], b)
    try:
        y = g.run(x)[0]
    finally:
        g.close()
    assert np.array_equal(y, harness.oracle_nhwc(m, blob, x, False))


@pytest.mark.parametrize("case", [(64, 1, 9, 11, 2), (24, 1, 5, 2, 3), (40, 0, 7, 6, 1), (192, 1, 28, 28, 4), (8, 1, 1, 1, 2), (16, 1, 3, 13, 1)])  # C, pad, H, W, batch
def test_maxpool_3x3_stride1_inside_the_arena_is_exact(case):
    """The 3x3 stride-1 max pool of an Inception branch (bf16 tensors between other nodes: four outputs per thread),
    widths that are not multiples of four, with and without padding, all-negative inputs so that padding must not win."""
    from tests import harness
    c, p, h, w, b = case
    m = zoo.Model("p3", "bf16", c, h, w)
    a = m.add(zoo.MAXPOOL, -1, k=1, stride=1, pad=0)
    a = m.add(zoo.MAXPOOL, a, k=3, stride=1, pad=p)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    m.shapes()
    blob = np.zeros(64, np.uint8)
    x = -np.abs(gen.make_input(4 + c, b, c, h, w, "normal", "bf16")) - 1.0
    x = gen.bf16_to_f32(gen.bf16_bits(x)).reshape(x.shape)
    g = harness.GpuDag([(m, blob)], b)
    try:
        y = g.run(x)[0]
        names = [L.name.decode() for L in g.dag.launches()]
    finally:
        g.close()
    assert names.count("maxpool") == 3
    assert np.array_equal(y, harness.oracle_nhwc(m, blob, x, False))


@pytest.mark.parametrize("case", [(128, 128, 1, 7, 1, 3, 17, 17, 2), (128, 192, 7, 1, 1, 3, 17, 17, 2), (384, 384, 1, 3, 1, 1, 8, 8, 2),
                                  (384, 384, 3, 1, 1, 1, 8, 8, 2), (24, 40, 3, 1, 2, 1, 15, 13, 1), (3, 16, 1, 5, 1, 2, 20, 21, 2),
                                  (16, 16, 5, 2, 2, 2, 19, 18, 1)])   # cin, cout, kh, kw, stride, pad, H, W, batch
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_rectangular_kernels(case, mode):
    """1 x n, n x 1 and other rectangular kernels; padding only along the dimensions the kernel extends over."""
    cin, cout, kh, kw, s, p, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("rect", dtype, cin, h, w)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=kh, kw=kw, stride=s, pad=p, act=zoo.RELU)
    _run_case(m, 1500 + cin + kh * 16 + kw, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(128, 128, 32, 3, 1, 1, 14, 14, 2), (64, 96, 4, 3, 2, 1, 15, 17, 2), (48, 48, 48, 3, 1, 1, 9, 9, 1),
                                  (32, 64, 2, 1, 1, 0, 12, 12, 3), (256, 256, 32, 3, 2, 1, 28, 28, 1),
                                  # channel strides that whole reduction tiles divide: a column tile walks its own groups' channels only.
                                  # One group per 64-channel tile; two groups per tile; groups wider than a tile (tiles straddle them);
                                  # the 256-row and the 128-row tile; a 1x1 and a 5x5 filter
                                  (192, 192, 3, 3, 1, 1, 13, 11, 2), (256, 128, 4, 3, 2, 1, 14, 14, 2), (128, 320, 2, 3, 1, 1, 9, 10, 2),
                                  (128, 128, 32, 3, 1, 1, 56, 56, 24), (128, 128, 32, 3, 1, 1, 32, 32, 16), (256, 192, 8, 1, 1, 0, 12, 12, 2),
                                  (64, 128, 2, 5, 1, 2, 11, 11, 1)])  # cin, cout, groups, k, stride, pad, H, W, batch
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_grouped_conv(case, mode):
    """Grouped convolution (each output channel sees its own group of input channels), up to one group per channel."""
    cin, cout, groups, k, s, p, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("gc", dtype, cin, h, w)
    m.add(zoo.CONV, -1, cin=cin, cout=cout, k=k, stride=s, pad=p, act=zoo.RELU, groups=groups)
    _run_case(m, 700 + cin + groups, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(16, 24, 13, 15), (8, 8, 6, 6), (20, 12, 9, 7), (64, 64, 28, 28)])   # channels of the two sources, H, W
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_concat_of_two_branches(case, mode):
    """Concatenation followed by a convolution that mixes all channels: vector path (first source a multiple
    of 8 channels) and element path (20 + 12), padded channel strides on both sides."""
    ca, cb, h, w = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("cat", dtype, 8, h, w)
    a = m.add(zoo.CONV, -1, cin=8, cout=ca, k=1, stride=1, pad=0, act=zoo.RELU)
    b = m.add(zoo.CONV, -1, cin=8, cout=cb, k=3, stride=1, pad=1, act=zoo.RELU)
    c = m.add(zoo.CONCAT, a, residual=b)
    m.add(zoo.CONV, c, cin=ca + cb, cout=10, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 500 + ca + cb, 2, act_dtype="f32" if mode == "bf16_wide" else None)


def test_concat_as_output_node_is_exact():
    """A concat that is the member's output copies values: the fp32 result equals the oracle's exactly in
    storage-rounding mode (both sides hold the same bf16 values)."""
    from tests import harness
    m = zoo.Model("cat_out", "bf16", 8, 8, 10)
    a = m.add(zoo.MAXPOOL, -1, k=3, stride=2, pad=0, ceil=True)
    b = m.add(zoo.MAXPOOL, -1, k=2, stride=2, pad=0, ceil=True)
    m.add(zoo.CONCAT, a, residual=b)
    m.shapes()
    blob = np.zeros(64, np.uint8)   # no weighted node
    x = gen.make_input(3, 2, 8, 8, 10, "normal", "bf16")
    g = harness.GpuDag([(m, blob, None)], 2)
    try:
        y = g.run(x)[0]
    finally:
        g.close()
    assert np.array_equal(y, harness.oracle_nhwc(m, blob, x, True))


@pytest.mark.parametrize("case", [(64, 3, 2, 0, 23, 24, 2), (16, 3, 2, 0, 8, 8, 1), (24, 3, 1, 1, 14, 14, 2), (40, 2, 2, 0, 7, 9, 3), (8, 2, 2, 1, 5, 5, 1)])
@pytest.mark.parametrize("mode", ["bf16", "f32"])
def test_maxpool_ceil_mode_exact(case, mode):
    """Pooling whose size rounds up: windows hang over the far edge; those taps never win (all-negative input)."""
    from tests import harness
    c, k, s, p, h, w, b = case
    m = zoo.Model("pc", mode, c, h, w)
    m.add(zoo.MAXPOOL, -1, k=k, stride=s, pad=p, ceil=True)
    m.shapes()
    blob = np.zeros(64, np.uint8)   # no weighted node
    x = -np.abs(gen.make_input(3, b, c, h, w, "normal", mode)) - 0.5
    if mode == "bf16":
        x = gen.bf16_to_f32(gen.bf16_bits(x)).reshape(x.shape)
    g = harness.GpuDag([(m, blob, None)], b)
    try:
        y = g.run(x)[0]
    finally:
        g.close()
    ref = harness.oracle_nhwc(m, blob, x, False)
    assert y.shape == ref.shape and np.array_equal(y, ref)


@pytest.mark.parametrize("case", [(64, 2, 2, 0, 28, 28, 2), (24, 3, 1, 1, 9, 11, 2), (40, 3, 2, 1, 15, 14, 1), (8, 5, 1, 2, 7, 7, 3),
                                  (192, 3, 1, 1, 17, 17, 3), (16, 3, 1, 0, 6, 5, 2)])
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_avgpool_between_convs(case, mode):
    """Window average pooling (divisor = window area, zero padding counted) between two convolutions."""
    c, k, s, p, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("ap", dtype, 8, h, w)
    a = m.add(zoo.CONV, -1, cin=8, cout=c, k=1, stride=1, pad=0, act=zoo.RELU)
    a = m.add(zoo.AVGPOOL, a, k=k, stride=s, pad=p)
    m.add(zoo.CONV, a, cin=c, cout=12, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 900 + c + k, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("act", [zoo.HARDSWISH, zoo.HARDSIGMOID, zoo.SILU, zoo.SIGMOID])
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_smooth_activations_in_every_epilogue(act, mode):
    """Hard-swish, hard-sigmoid, SiLU and sigmoid after an MFMA / direct convolution, a split-K convolution
    (finished by the reduce kernel), a depthwise convolution and a small-batch FC."""
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("acts", dtype, 16, 12, 12)
    a = m.add(zoo.CONV, -1, cin=16, cout=40, k=3, stride=1, pad=1, act=act)
    a = m.add(zoo.DWCONV, a, cin=40, cout=40, k=3, stride=2, pad=1, act=act)
    a = m.add(zoo.CONV, a, cin=40, cout=64, k=3, stride=1, pad=1, act=act)      # 6x6 outputs, K = 360: split-K at this size
    a = m.add(zoo.GAP, a)
    m.add(zoo.FC, a, cin=64, cout=20, act=act)
    _run_case(m, 1100, 2, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(64, 16, 9, 11, 2), (24, 8, 7, 7, 3), (120, 32, 14, 14, 1)])   # channels, squeeze width, H, W, batch
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_squeeze_excite_block(case, mode):
    """global average -> FC (ReLU) -> FC (hard sigmoid) -> per-channel scaling of the block's tensor -> 1x1 projection."""
    c, sq, h, w, b = case
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("se", dtype, 8, h, w)
    x = m.add(zoo.CONV, -1, cin=8, cout=c, k=1, stride=1, pad=0, act=zoo.HARDSWISH)
    g = m.add(zoo.GAP, x)
    g = m.add(zoo.FC, g, cin=c, cout=sq, act=zoo.RELU)
    g = m.add(zoo.FC, g, cin=sq, cout=c, act=zoo.HARDSIGMOID)
    y = m.add(zoo.MUL, x, residual=g)
    m.add(zoo.CONV, y, cin=c, cout=16, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 1200 + c, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_slice_branch_concat_shuffle_unit(mode):
    """One ShuffleNet-V2-style unit: half of the channels kept, the other half through 1x1 -> depthwise -> 1x1,
    concatenated and shuffled in two groups; odd half-width (29) so the element paths with ragged padding run."""
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("shuf", dtype, 8, 10, 9)
    x = m.add(zoo.CONV, -1, cin=8, cout=58, k=1, stride=1, pad=0, act=zoo.RELU)
    a = m.add(zoo.SLICE, x, first=0, cout=29)
    b = m.add(zoo.SLICE, x, first=29, cout=29)
    b = m.add(zoo.CONV, b, cin=29, cout=29, k=1, stride=1, pad=0, act=zoo.RELU)
    b = m.add(zoo.DWCONV, b, cin=29, cout=29, k=3, stride=1, pad=1, act=zoo.NONE)
    y = m.add(zoo.CONCAT, a, residual=b)
    y = m.add(zoo.SHUFFLE, y, groups=2)
    m.add(zoo.CONV, y, cin=58, cout=12, k=1, stride=1, pad=0, act=zoo.NONE)
    _run_case(m, 1300, 2, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(16, 8, 3, 9, 7, 2), (64, 32, 4, 28, 28, 4), (24, 16, 2, 5, 5, 1)])   # first width, growth, layers, H, W, batch
@pytest.mark.parametrize("mode", ["bf16", "bf16_wide"])
def test_dense_block_concatenations(case, mode):
    """A DenseNet-style block: every layer normalises (per-channel affine + ReLU) everything concatenated so far and appends
    `growth` new channels.  With bf16 activations the new channels are written straight into the block's final tensor and
    the affine nodes read its prefixes with that tensor's channel stride; with fp32 activations every concatenation copies."""
    c0, growth, layers, h, w, b = case
    m = zoo.Model("dense", "bf16", 8, h, w)
    t = m.add(zoo.CONV, -1, cin=8, cout=c0, k=3, stride=1, pad=1, act=zoo.RELU)
    c = c0
    for _ in range(layers):
        a = m.add(zoo.DWCONV, t, cin=c, cout=c, k=1, stride=1, pad=0, act=zoo.RELU)
        a = m.add(zoo.CONV, a, cin=c, cout=4 * growth, k=1, stride=1, pad=0, act=zoo.RELU)
        a = m.add(zoo.CONV, a, cin=4 * growth, cout=growth, k=3, stride=1, pad=1, act=zoo.NONE)
        t = m.add(zoo.CONCAT, t, residual=a)
        c += growth
    t = m.add(zoo.DWCONV, t, cin=c, cout=c, k=3, stride=2, pad=1, act=zoo.RELU)
    t = m.add(zoo.GAP, t)
    m.add(zoo.FC, t, cin=c, cout=10)
    _run_case(m, 1700 + c0, b, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("mode", ["bf16", "bf16_wide"])
def test_reduction_module_concatenations(mode):
    """An Inception-style reduction module: a strided convolution, a two-convolution branch, a strided max pool and an
    average pool of the same input, joined by nested concatenations (pool outputs and convolution outputs side by side in
    one tensor), then read by a dense convolution."""
    m = zoo.Model("red", "bf16", 8, 17, 15)
    x = m.add(zoo.CONV, -1, cin=8, cout=48, k=1, stride=1, pad=0, act=zoo.RELU)
    b1 = m.add(zoo.CONV, x, cin=48, cout=40, k=3, stride=2, pad=0, act=zoo.RELU)
    b2 = m.add(zoo.CONV, x, cin=48, cout=16, k=1, stride=1, pad=0, act=zoo.RELU)
    b2 = m.add(zoo.CONV, b2, cin=16, cout=24, k=3, stride=2, pad=0, act=zoo.RELU)
    b3 = m.add(zoo.MAXPOOL, x, k=3, stride=2, pad=0)
    b4 = m.add(zoo.AVGPOOL, x, k=3, stride=2, pad=0)
    y = m.add(zoo.CONCAT, b1, residual=b2)
    y = m.add(zoo.CONCAT, y, residual=b3)
    y = m.add(zoo.CONCAT, y, residual=b4)
    m.add(zoo.CONV, y, cin=160, cout=12, k=3, stride=1, pad=1, act=zoo.NONE)
    _run_case(m, 1800, 3, act_dtype="f32" if mode == "bf16_wide" else None)


@pytest.mark.parametrize("case", [(64, 16, 24, 2), (64, 8, 20, 4), (48, 0, 48, 3), (120, 56, 64, 2), (24, 0, 24, 3), (64, 32, 32, 1)])  # C, first, width, shuffle groups
def test_slice_and_shuffle_inside_the_arena_are_exact(case):
    """Channel slices at vector-aligned and unaligned offsets, widths that do and do not fill whole 8-channel vectors,
    shuffles in 1..4 groups, all between other nodes (bf16 tensors in the arena: the 8-channel form of the gather):
    values only move, so the result equals the oracle's bit for bit."""
    from tests import harness
    c, first, width, groups = case
    m = zoo.Model("gath", "bf16", c, 6, 5)
    a = m.add(zoo.MAXPOOL, -1, k=1, stride=1, pad=0)
    a = m.add(zoo.SLICE, a, first=first, cout=width)
    a = m.add(zoo.SHUFFLE, a, groups=groups)
    m.add(zoo.MAXPOOL, a, k=1, stride=1, pad=0)
    m.shapes()
    x = gen.make_input(5 + c, 3, c, 6, 5, "normal", "bf16")
    blob = np.zeros(64, np.uint8)
    g = harness.GpuDag([(m, blob, None)], 3)
    try:
        y = g.run(x)[0]
    finally:
        g.close()
    assert np.array_equal(y, harness.oracle_nhwc(m, blob, x, True))


def test_shuffle_as_output_node_is_exact():
    from tests import harness
    m = zoo.Model("shuf_out", "bf16", 24, 5, 7)
    a = m.add(zoo.MAXPOOL, -1, k=1, stride=1, pad=0)
    a = m.add(zoo.SLICE, a, first=6, cout=12)
    m.add(zoo.SHUFFLE, a, groups=4)
    m.shapes()
    x = gen.make_input(3, 2, 24, 5, 7, "normal", "bf16")
    blob = np.zeros(64, np.uint8)
    g = harness.GpuDag([(m, blob, None)], 2)
    try:
        y = g.run(x)[0]
    finally:
        g.close()
    assert np.array_equal(y, harness.oracle_nhwc(m, blob, x, True))


@pytest.mark.parametrize("mode", ["bf16", "bf16_wide", "f32"])
def test_gap_fc_softmax_chain(mode):
    dtype = "f32" if mode == "f32" else "bf16"
    m = zoo.Model("g", dtype, 24, 7, 9)
    a = m.add(zoo.GAP, -1)
    a = m.add(zoo.FC, a, cin=24, cout=50, act=zoo.RELU)
    a = m.add(zoo.FC, a, cin=50, cout=10)
    m.add(zoo.SOFTMAX, a)
    e = _run_case(m, 31, 5, act_dtype="f32" if mode == "bf16_wide" else None)
    assert e < 5e-3


def test_fc_on_spatial_input_bf16():
    """FC over a flattened C,H,W tensor (the 25088-input layer shape, scaled down)."""
    m = zoo.Model("f", "bf16", 40, 7, 7)
    m.add(zoo.FC, -1, cin=40 * 49, cout=130, act=zoo.RELU)
    _run_case(m, 5, 8)


@pytest.mark.parametrize("mode", ["bf16", "bf16_wide"])
@pytest.mark.parametrize("batch", [33, 70])
def test_fc_batches_above_32_and_residual(batch, mode):
    """The FC kernel takes 32 images per pass: batches that need two and three passes (the last one ragged), a
    feature count that is not a multiple of 32, and an FC that adds a residual."""
    m = zoo.Model("f", "bf16", 24, 5, 3)
    a = m.add(zoo.FC, -1, cin=24 * 15, cout=77, act=zoo.RELU)
    b = m.add(zoo.FC, a, cin=77, cout=77, act=zoo.NONE)
    c = m.add(zoo.FC, b, cin=77, cout=77, act=zoo.RELU, residual=a)
    m.add(zoo.FC, c, cin=77, cout=1000)
    _run_case(m, 77, batch, act_dtype="f32" if mode == "bf16_wide" else None)


def test_batch_smaller_than_max_batch():
    from tests import harness
    m = zoo.resnet18(hw=64)
    blob = gen.make_blob(m, 1000)
    x = gen.make_input(7, 4, 3, 64, 64, "normal", "bf16")
    g = harness.GpuDag([(m, blob)], 4)
    try:
        full = g.run(x)[0]
        part = g.run(x[:3])[0]
        one = g.run(x[2:3])[0]
    finally:
        g.close()
    assert np.array_equal(full[:3], part) and np.array_equal(full[2:3], one)
