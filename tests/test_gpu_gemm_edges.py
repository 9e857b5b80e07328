"""The tile kernels of gemm.hip and gemm_bf16_128.hip at the sizes where they can go wrong, against
the oracle, per element: edges of tiles and k-tiles, rows that are no multiple
of a 16-byte unit or shorter than one, operands at the very end of an
allocation; and the fp32 split at values it does not hold for."""

import numpy as np
import pytest
import torch

import oracle
from paper_1603_04467_amd import tfdense as T
from tests.parity import product_bound, to_f64
from tests.test_gpu_ops import DEV, _check_elementwise, _run_gemm
from tests import test_gpu_ops as ops

pytestmark = pytest.mark.gpu

# tile configurations of both types: 256 wide, 128 x 128, 64 x 64 with k split
# over wave groups, 64 x 64
TILES = [1, 3, 2, 4]
# one element; one below, at and above a tile edge and a k-tile (16 or 32
# fp32, 64 16-bit values); k of one k-tile per wave group and one less; units
# broken in m, n and k
SIZES = [(1, 1, 1), (64, 64, 16), (63, 65, 33), (129, 127, 64), (255, 257, 15), (260, 136, 65), (130, 3, 191),
         (2, 200, 256), (5, 6, 257), (257, 72, 320)]


@pytest.mark.parametrize("din,dout", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
@pytest.mark.parametrize("tile", TILES)
def test_tile_edges(tile, layout, din, dout):
    for n, (size, extra) in enumerate((s, e) for s in SIZES for e in (0, 3)):
        m, nn, k = size
        epi = ("none", "bias", "bias_relu")[n % 3]
        got, want, pre, D = _run_gemm(m, nn, k, layout, din, dout, epi, seed=n, ld_extra=extra, tile=tile)
        _check_elementwise(got, ops._LAST["a"], ops._LAST["b"], layout == "TN", layout == "NT", ops._LAST["bias"], epi,
                           dout, f"tile {tile} {layout} {din}->{dout} {size} ld+{extra}")


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
@pytest.mark.parametrize("tile", TILES)
def test_integers_exact(tile, layout, dt):
    """Small integers: every product and sum is exact, so every k is summed once and every value lands in its place."""
    rng = np.random.default_rng([tile, len(layout), dt == torch.float32])
    for m, n, k in [(300, 263, 1000), (70, 90, 449)]:
        a = rng.integers(-3, 4, size=(m, k)).astype(np.float64)
        b = rng.integers(-3, 4, size=(k, n)).astype(np.float64)
        ad = torch.from_numpy(a.T.copy() if layout == "TN" else a).to(DEV, dt)
        bd = torch.from_numpy(b.T.copy() if layout == "NT" else b).to(DEV, dt)
        c = torch.full((m, n), float("nan"), dtype=torch.float32, device=DEV)
        with T.tuning(gemm_tile=tile):
            T.tfd_matmul(ad, bd, c, transpose_a=layout == "TN", transpose_b=layout == "NT")
        assert np.array_equal(to_f64(c), a @ b)


@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
@pytest.mark.parametrize("tile", TILES)
def test_f32_values_outside_the_split(tile, layout):
    """Infinities, NaN, values that round up to infinity in 16 bits and values
    below the split's range: each output that has such an operand is what the
    fp32 product gives, every other one keeps its bound."""
    m, n, k = 300, 280, 70
    rng = np.random.default_rng(7)
    a = rng.standard_normal((m, k)).astype(np.float32)
    b = rng.standard_normal((k, n)).astype(np.float32)
    a[3, 5] = np.inf
    a[40, 69] = -np.inf
    a[130, 0] = np.nan
    b[2, 77] = np.inf
    a[200, 9] = np.float32(3.4e38)           # rounds up to infinity in 16 bits
    b[9, :] *= np.float32(2.0 ** -20)
    a[250, :] *= np.float32(2.0 ** -112)     # a third plane below the smallest 16-bit step
    a[299, :] *= np.float32(2.0 ** -120)
    b[:, 270] *= np.float32(2.0 ** -105)
    a[7, :] = 0.0                            # zeros are not tiny
    ad = torch.from_numpy(a.T.copy() if layout == "TN" else a).to(DEV)
    bd = torch.from_numpy(b.T.copy() if layout == "NT" else b).to(DEV)
    c = torch.full((m, n), 7.0, device=DEV)
    with T.tuning(gemm_tile=tile):
        T.tfd_matmul(ad, bd, c, transpose_a=layout == "TN", transpose_b=layout == "NT")
    got = c.cpu().numpy().astype(np.float64)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        want = a64 @ b64
        terms = np.abs(a64) @ np.abs(b64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf]) and not np.any(np.isinf(got[~inf]))
    ok = np.isfinite(want) & (terms > 2.0 ** -120)   # below, fp32 products are subnormal themselves
    bound = product_bound(np.where(ok, terms, 0.0), k, np.where(ok, got, 0.0), "f32")
    assert np.all(np.abs(got - want)[ok] <= bound[ok])
    # the tiny rows are in the bound's range, not skipped
    assert ok[250, :70].all() and np.any(got[250, :70] != 0)


def _small_beside_large(m, n, k, layout, tile, small_in_a):
    """Values below 2^-109, whose low bits (below 2^-140: all of them) no 16-bit plane holds, in outputs of ordinary
    size: beside factors of 2^19 to 2^100, in the last k too. Each output keeps the fp32 product's bound, and NaN
    stays in its row. m rows of small values, n columns of large ones; the product as it is or transposed."""
    rng = np.random.default_rng([tile, small_in_a, m, n, k])
    small = rng.standard_normal((m, k)).astype(np.float32)
    large = rng.standard_normal((k, n)).astype(np.float32)
    tiny = [3 % m, 140 % m, m - 1]
    for row, e in zip(tiny, (-120, -126, -140)):
        small[row] *= np.float32(2.0 ** e)
    zero, nan = [r for r in range(m) if r not in tiny][:2] if m > 4 else (None, None)
    if zero is not None:
        small[zero] = 0.0
        small[zero, k - 1] = np.float32(2.0 ** -140)  # one value alone, exactly 0 in the planes times 2^19
        small[nan, 4] = np.nan
    large[:, 0] *= np.float32(2.0 ** 60)
    if n > 1:
        large[:, n // 2] *= np.float32(2.0 ** 100)
    if n > 2:
        large[:, n - 1] = np.float32(2.0 ** 19) * np.where(large[:, n - 1] > 0, np.float32(1.5), np.float32(1.0))
    a, b = (small, large) if small_in_a else (large.T.copy(), small.T.copy())
    ad = torch.from_numpy(a.T.copy() if layout == "TN" else a).to(DEV)
    bd = torch.from_numpy(b.T.copy() if layout == "NT" else b).to(DEV)
    c = torch.full((a.shape[0], b.shape[1]), 7.0, device=DEV)
    with T.tuning(gemm_tile=tile):
        T.tfd_matmul(ad, bd, c, transpose_a=layout == "TN", transpose_b=layout == "NT")
    got = c.cpu().numpy().astype(np.float64)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    want, terms = a64 @ b64, np.abs(a64) @ np.abs(b64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = np.isfinite(want) & (terms > 2.0 ** -122)   # below, fp32 products are subnormal themselves
    view = ok if small_in_a else ok.T
    assert view[tiny[0], 0] and view[tiny, n // 2].all()
    if n > 2 and zero is not None:
        assert view[[*tiny, zero], n - 1].all()
    bound = product_bound(np.where(ok, terms, 0.0), k, np.where(ok, got, 0.0), "f32")
    assert np.all(np.abs(np.where(ok, got - want, 0.0)) <= bound)


@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
@pytest.mark.parametrize("tile", [0, *TILES])
def test_f32_small_operands_beside_large_ones(tile, layout):
    for m, n, k in [(300, 280, 70), (264, 272, 160)]:  # with and without k-tiles and units loaded apart
        for small_in_a in (True, False):
            _small_beside_large(m, n, k, layout, tile, small_in_a)


@pytest.mark.parametrize("layout", ["NN", "TN"])
def test_f32_small_operands_in_rows_shorter_than_a_unit(layout):
    """The kernel that loads every k-tile element by element sums again as the others do."""
    for k in (5, 70):
        _small_beside_large(300, 2, k, layout, 4, layout == "NN")  # NN: b is k x 2; TN: a is k x 2


@pytest.mark.parametrize("tile", [0, *TILES])
def test_f32_largest_omitted_products(tile):
    """Operands whose omitted plane products are as large as they get (0.97 * 2^-24 of x y, of one sign)."""
    x = np.float32(1.0 + 2.0 ** -8 - 2.0 ** -17 - 2.0 ** -23)
    for k in (1, 16, 300):
        a, b = torch.full((130, k), float(x), device=DEV), torch.full((k, 70), float(x), device=DEV)
        c = torch.empty(130, 70, device=DEV)
        with T.tuning(gemm_tile=tile):
            T.tfd_matmul(a, b, c)
        got, want = to_f64(c), np.full((130, 70), k * float(x) ** 2)
        assert np.all(np.abs(got - want) <= product_bound(want, k, got, "f32")), k


def test_operands_at_the_end_of_an_allocation():
    """An operand whose last row ends where its storage ends, m/n-contiguous with broken units: the last k-tile is the
    one loaded element by element, and only elements of the operand are read (a value past it would change integers)."""
    for dt in (torch.float32, torch.bfloat16):
        for k in (16, 64, 96, 130):
            rng = np.random.default_rng(k)
            a = rng.integers(-3, 4, size=(k, 67)).astype(np.float64)
            b = rng.integers(-3, 4, size=(k, 45)).astype(np.float64)
            # NaN right behind each operand
            buf = torch.full((k * 67 + 16,), float("nan"), dtype=dt, device=DEV)
            buf2 = torch.full((k * 45 + 16,), float("nan"), dtype=dt, device=DEV)
            ad = buf[:k * 67].view(k, 67)
            bd = buf2[:k * 45].view(k, 45)
            ad.copy_(torch.from_numpy(a))
            bd.copy_(torch.from_numpy(b))
            for tile in TILES:
                c = torch.full((67, 45), float("nan"), device=DEV)
                with T.tuning(gemm_tile=tile):
                    T.tfd_matmul(ad, bd, c, transpose_a=True)
                assert np.array_equal(to_f64(c), a.T @ b), (dt, k, tile)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
@pytest.mark.parametrize("din,dout", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
def test_empty_sum(din, dout, layout, tile):
    """k = 0 (the weight gradient of an empty batch): C = epilogue(0) bit for bit, in every call that multiplies,
    whatever the workgroups before have left in LDS."""
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16}
    ta, tb = layout == "TN", layout == "NT"
    nan = torch.full((512, 512), float("nan"), dtype=tdt[din], device=DEV)
    scratch = torch.empty(512, 512, dtype=tdt[dout], device=DEV)
    with T.tuning(gemm_tile=4):
        T.tfd_matmul(nan, nan, scratch)  # every stage of its workgroups holds NaN
    for m, n in [(3, 5), (264, 136), (600, 512)]:
        a = torch.empty((0, m) if ta else (m, 0), dtype=tdt[din], device=DEV)
        b = torch.empty((n, 0) if tb else (0, n), dtype=tdt[din], device=DEV)
        kw = dict(transpose_a=ta, transpose_b=tb)
        bias = torch.linspace(-1.0, 1.0, n, device=DEV)
        new = lambda dt=dout: torch.full((m, n), float("nan"), dtype=tdt[dt], device=DEV)  # noqa: E731
        y = bias.to(tdt[dout]).expand(m, n)
        relu = torch.where(y > 0, y, torch.zeros_like(y))
        with T.tuning(gemm_tile=tile):
            for epi, want in [("none", torch.zeros_like(y)), ("bias", y), ("bias_relu", relu)]:
                c = new()
                T.tfd_matmul(a, b, c, bias=None if epi == "none" else bias, epilogue=epi, **kw)
                assert torch.equal(c, want) and not torch.signbit(c[want == 0]).any(), (epi, m, n)
            if din != dout:
                continue
            feats = torch.randn(m, n, device=DEV).to(tdt[din])
            mask, want_mask = T.new_relu_mask(m, n, DEV), T.new_relu_mask(m, n, DEV)
            c = new()
            T.tfd_matmul_relu_mask(a, b, bias, c, mask, **kw)
            T.tfd_relu_mask(relu.contiguous(), want_mask)
            assert torch.equal(c, relu) and torch.equal(mask, want_mask), (m, n)
            for call, arg in [(T.tfd_matmul_relu_grad_bias_add_grad, feats),
                              (T.tfd_matmul_relu_mask_grad_bias_add_grad, mask)]:
                bp, db = new(), torch.full((n,), float("nan"), device=DEV)
                call(a, b, arg, bp, db, **kw)
                assert not bp.any() and not db.any(), (call, m, n)
            out, grad, db = new(), new(), torch.full((n,), float("nan"), device=DEV)
            loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
            T.tfd_matmul_l2_loss_grad(a, b, bias, out, feats, grad, loss, db, **kw)
            want_grad, want_loss = new(), torch.zeros(1, dtype=torch.float64, device=DEV)
            T.tfd_l2_loss_grad(y.contiguous(), feats, want_grad, want_loss)
            assert torch.equal(out, y) and torch.equal(grad, want_grad) and torch.equal(loss, want_loss), (m, n)
            want_db = want_grad.double().sum(0)  # m values in some order
            assert ((db - want_db).abs() <= 2 * m * 2.0 ** -24 * want_grad.double().abs().sum(0)).all(), (m, n)


@pytest.mark.parametrize("tile", [0, *TILES, 8])
@pytest.mark.parametrize("din,dout", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("side", ["m", "n"])
def test_more_tiles_than_a_grid_of_their_threads(side, din, dout, tile):
    """2^30 rows or columns: one workgroup per tile would need 2^32 threads or more on the smaller tiles."""
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16}
    long = 2 ** 30
    x = torch.arange(512, device=DEV, dtype=torch.float32).to(tdt[din]).repeat(long // 512).view(long, 1)  # exact
    two, bias = torch.full((1, 1), 2.0, dtype=tdt[din], device=DEV), None
    c = torch.full((long, 1) if side == "m" else (1, long), float("nan"), dtype=tdt[dout], device=DEV)
    with T.tuning(gemm_tile=tile):
        if side == "m":
            T.tfd_matmul(x, two, c, transpose_b=True)
        else:
            bias = torch.arange(2 ** 20, device=DEV, dtype=torch.float32).remainder_(2).repeat(long // 2 ** 20)
            T.tfd_matmul(two, x.view(1, long), c, bias=bias, epilogue="bias")
    for part in range(0, long, 2 ** 28):
        cut = slice(part, part + 2 ** 28)
        want = 2.0 * x.view(-1)[cut].float()
        if bias is not None:
            want += bias[cut]
        assert torch.equal(c.view(-1)[cut], want.to(tdt[dout])), part


# gemm_bf16_128.hip takes whole 16-byte units: one of them; one unit below, at
# and above a tile edge and a k-tile, fewer k-tiles than stages; with two stages
# (more than 256 tiles); 256 x 128 tiles (10 k-tiles, more than 256 square ones)
SIZES128 = [(8, 8, 8), (128, 128, 64), (120, 136, 72), (136, 120, 56), (264, 248, 136), (128, 256, 200), (256, 8, 264),
            (2104, 2200, 72), (2176, 2056, 584)]


@pytest.mark.parametrize("dout", ["bf16", "f32"])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_tiles128_edges(layout, dout):
    for n, (m, nn, k) in enumerate(SIZES128):
        epi = ("none", "bias", "bias_relu")[n % 3]
        m -= 3 if layout != "TN" else 0  # (TN: rows of 16-byte units along m)
        got, want, pre, D = _run_gemm(m, nn, k, layout, "bf16", dout, epi, seed=n, ld_extra=8 * (n % 2), tile=7)
        _check_elementwise(got, ops._LAST["a"], ops._LAST["b"], layout == "TN", layout == "NT", ops._LAST["bias"], epi,
                           dout, f"128 {layout} {dout} {(m, nn, k)}")


# taken by 128 x 128 tiles in four stages, in two, and by 256 x 128 tiles
@pytest.mark.parametrize("size", [(1800, 2040, 1000), (3000, 2504, 328), (2176, 2056, 1288), (2048, 4096, 576)])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_tiles128_fused_epilogues(size, layout):
    """Every fused epilogue stores the plain call's bits, put through the separate call."""
    m, n, k = size
    ta, tb = layout == "TN", layout == "NT"
    g = torch.Generator(device=DEV).manual_seed(m + n + k)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    a, b, feats, target = rnd(*((k, m) if ta else (m, k))), rnd(*((n, k) if tb else (k, n))), rnd(m, n), rnd(m, n)
    bias = torch.randn(n, generator=g, device=DEV)
    kw = dict(transpose_a=ta, transpose_b=tb)
    new = lambda: torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)  # noqa: E731
    db = lambda: torch.full((n,), float("nan"), device=DEV)  # noqa: E731
    mask, want_mask = T.new_relu_mask(m, n, DEV), T.new_relu_mask(m, n, DEV)

    plain, forced = new(), new()
    T.tfd_matmul(a, b, plain, **kw)
    with T.tuning(gemm_tile=7):
        T.tfd_matmul(a, b, forced, **kw)
    assert torch.equal(plain, forced), "another kernel took the problem"

    c, want = new(), new()
    T.tfd_matmul_relu_mask(a, b, bias, c, mask, **kw)
    T.tfd_matmul(a, b, want, bias=bias, epilogue="bias_relu", **kw)
    T.tfd_relu_mask(want, want_mask)
    assert torch.equal(c, want) and torch.equal(mask, want_mask)

    # column sums: n32 values in another order, each sum within 2 rows 2^-24 of the sum of magnitudes
    def sums_ok(got, ref):
        slack = ref.double().abs().sum(0) * (2 * m * 2.0 ** -24)
        return bool(((got.double() - ref.double().sum(0)).abs() <= slack).all())

    want_bp, want_db = new(), db()
    T.tfd_relu_grad_bias_add_grad(plain, feats, want_bp, want_db)
    bp, d = new(), db()
    T.tfd_matmul_relu_grad_bias_add_grad(a, b, feats, bp, d, **kw)
    assert torch.equal(bp, want_bp) and sums_ok(d, bp)
    T.tfd_relu_mask(feats, mask)
    bp, d = new(), db()
    T.tfd_matmul_relu_mask_grad_bias_add_grad(a, b, mask, bp, d, **kw)
    assert torch.equal(bp, want_bp) and sums_ok(d, bp)

    out, grad, want_grad, d = new(), new(), new(), db()
    loss, want_loss = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
    T.tfd_matmul_l2_loss_grad(a, b, bias, out, target, grad, loss, d, **kw)
    T.tfd_matmul(a, b, want, bias=bias, epilogue="bias", **kw)
    T.tfd_l2_loss_grad(want, target, want_grad, want_loss)
    assert torch.equal(out, want) and torch.equal(grad, want_grad) and sums_ok(d, grad)
    assert abs(loss.item() - want_loss.item()) <= m * n * 2.0 ** -52 * want_loss.item()


@pytest.mark.parametrize("size", [(2048, 1792, 128), (8448, 768, 128), (1792, 3584, 128), (1800, 1024, 64)])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_fused_epilogues_beside_64_wide_plain_tiles(size, layout):
    """Sizes whose plain call runs on 64 x 64 tiles and whose fused calls on 128 x 128 ones: the same bits."""
    with T.tuning(gemm_tile=4):
        m, n, k = size
        g = torch.Generator(device=DEV).manual_seed(5)
        a = torch.randn(*((k, m) if layout == "TN" else (m, k)), generator=g, device=DEV).to(torch.bfloat16)
        b = torch.randn(*((n, k) if layout == "NT" else (k, n)), generator=g, device=DEV).to(torch.bfloat16)
        kw = dict(transpose_a=layout == "TN", transpose_b=layout == "NT")
        c64 = T.tfd_matmul(a, b, torch.empty(m, n, dtype=torch.bfloat16, device=DEV), **kw)
    c = T.tfd_matmul(a, b, torch.empty(m, n, dtype=torch.bfloat16, device=DEV), **kw)
    assert torch.equal(c, c64)
    test_tiles128_fused_epilogues(size, layout)
