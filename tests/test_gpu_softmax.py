"""Parity of the softmax cross-entropy cost head (tfd_softmax_cross_entropy_grad)
with the oracle's definition, element by element.

Error model of the kernel (fp32 arithmetic, row maximum m subtracted): each
exp(z - m) carries the rounding of z - m (at most |z - m| 2^-24 relative
after exp) and a few ulp of its own; the row sum adds at most
(cols / 64 + 6) ulp (a strided sum per lane, then a 64-lane butterfly); the
reciprocal and the product one ulp each. So |p_gpu - p| is bounded by
K 2^-24 p with K = cols / 64 + 2 max|z - m| + 16, and the subtraction of one
adds at most 2^-24. A 16-bit gradient adds its own rounding (2^-8 |G|
relative). Each row's loss term is log(s) + m - z_y with m and z_y exact in
float64, so it is off by at most the error of log(s): (K + 4 |log s| + 4)
2^-24 per row.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1603_04467_amd import tfdense as T
from paper_1603_04467_amd.workloads import to_bf16_bits
from tests.parity import to_f64

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _logits(rng, rows, cols, dt, scale):
    a = (rng.standard_normal((rows, cols)) * scale).astype(np.float32)
    if dt == "bf16":
        bits = to_bf16_bits(a)
        return oracle.bf16_bits_to_f64(bits), torch.from_numpy(bits.view(np.int16).copy()).view(torch.bfloat16).to(DEV)
    return a.astype(np.float64), torch.from_numpy(a).to(DEV)


def _run(z, labels):
    g = torch.full_like(z, float("nan"))
    loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
    T.tfd_softmax_cross_entropy_grad(z, labels, g, loss)
    torch.cuda.synchronize()
    return g, loss


def _bounds(z_h, dt):
    rows, cols = z_h.shape
    spread = float(np.max(z_h.max(axis=1) - z_h.min(axis=1))) if z_h.size else 0.0
    K = cols / 64 + 2 * spread + 16
    p = oracle.softmax(z_h)
    return K, p


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 10), (256, 10), (100, 1000), (64, 4096), (7, 32768),
                                       (1029, 65)])
@pytest.mark.parametrize("scale", [1.0, 30.0])
def test_softmax_xent_matches_oracle(dt, rows, cols, scale):
    rng = np.random.default_rng([rows, cols, int(scale), dt == "bf16"])
    z_h, z = _logits(rng, rows, cols, dt, scale)
    y = rng.integers(0, cols, size=rows, dtype=np.int32)
    g, loss = _run(z, torch.from_numpy(y).to(DEV))
    g_want, l_want = oracle.softmax_cross_entropy_grad(z_h, y, grad_dtype="f64")
    K, p = _bounds(z_h, dt)
    allowed = K * 2.0 ** -24 * p + 2.0 ** -24
    if dt == "bf16":
        allowed = allowed + 2.0 ** -8 * np.abs(g_want)
    err = np.abs(to_f64(g) - g_want)
    assert np.all(np.isfinite(to_f64(g)))
    bad = err > allowed
    assert not np.any(bad), f"gradient: {int(bad.sum())} elements outside the bound, max|err| {err.max():.3e}"
    # rows of the gradient sum to zero up to the same rounding
    lse = np.log(np.sum(np.exp(z_h - z_h.max(axis=1, keepdims=True)), axis=1))
    allowed_loss = float(np.sum(K + 4 * np.abs(lse) + 4)) * 2.0 ** -24
    assert abs(loss.item() - l_want) <= allowed_loss, (loss.item(), l_want, allowed_loss)


def test_softmax_xent_one_class_and_uniform_rows_exact():
    # a single class: p = 1, G = 0, loss = 0 exactly
    z = torch.randn(5, 1, device=DEV)
    g, loss = _run(z, torch.zeros(5, dtype=torch.int32, device=DEV))
    assert torch.equal(g, torch.zeros_like(g)) and loss.item() == 0.0
    # equal logits over a power-of-two class count: p = 2^-e exactly
    z = torch.full((3, 256), 2.5, device=DEV)
    labels = torch.tensor([0, 100, 255], dtype=torch.int32, device=DEV)
    g, loss = _run(z, labels)
    want = torch.full_like(z, 1.0 / 256)
    want[torch.arange(3), labels.long()] -= 1.0
    assert torch.equal(g, want)
    assert abs(loss.item() - 3 * np.log(256.0)) <= 3 * 8 * 2.0 ** -23


def test_softmax_xent_empty_batch_writes_zero_loss():
    z = torch.empty(0, 10, device=DEV)
    g, loss = _run(z, torch.empty(0, dtype=torch.int32, device=DEV))
    assert loss.item() == 0.0


def test_softmax_xent_label_out_of_range_gives_nan_loss():
    rng = np.random.default_rng(7)
    z_h, z = _logits(rng, 4, 12, "f32", 1.0)
    y = np.array([3, 12, -1, 0], dtype=np.int32)
    g, loss = _run(z, torch.from_numpy(y).to(DEV))
    assert np.isnan(loss.item())
    p = oracle.softmax(z_h)
    gh = to_f64(g)
    K, _ = _bounds(z_h, "f32")
    # the two bad rows are p itself; the good rows are p - onehot
    for r in (1, 2):
        assert np.all(np.abs(gh[r] - p[r]) <= K * 2.0 ** -24 * p[r])
    g_want, _ = oracle.softmax_cross_entropy_grad(z_h[[0, 3]], y[[0, 3]], grad_dtype="f64")
    assert np.all(np.abs(gh[[0, 3]] - g_want) <= K * 2.0 ** -24 * p[[0, 3]] + 2.0 ** -24)


def test_softmax_xent_is_deterministic():
    rng = np.random.default_rng(11)
    _, z = _logits(rng, 4099, 1000, "f32", 3.0)
    y = torch.from_numpy(rng.integers(0, 1000, size=4099, dtype=np.int32)).to(DEV)
    g1, l1 = _run(z, y)
    g2, l2 = _run(z, y)
    assert torch.equal(g1, g2) and torch.equal(l1, l2)


def test_softmax_xent_rejects_bad_arguments():
    z = torch.zeros(4, 3, device=DEV)
    y = torch.zeros(4, dtype=torch.int32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    with pytest.raises(T.TfdError):
        T.tfd_softmax_cross_entropy_grad(z, y, z, loss)          # grad aliases the logits
    with pytest.raises(T.TfdError):
        T.tfd_softmax_cross_entropy_grad(torch.zeros(4, 0, device=DEV), y, torch.zeros(4, 0, device=DEV), loss)
    with pytest.raises(T.TfdError):
        T.tfd_softmax_cross_entropy_grad(z, y, torch.empty_like(z), loss, workspace=torch.empty(0, dtype=torch.uint8,
                                                                                               device=DEV))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
# around the wavefront-per-row limit (512), whole and broken 16-byte chunks at
# both ends of a row, the largest rows a block of 256 and of 1024 threads holds
# in each type, and rows beyond that
@pytest.mark.parametrize("cols", [512, 513, 1031, 2048, 8191, 16384, 16391, 32760, 65528, 65551])
@pytest.mark.parametrize("shift", [0, 1])
def test_softmax_xent_row_per_block(dt, cols, shift):
    rows, rng = 5, np.random.default_rng([cols, shift, dt == "bf16"])
    z_h, z = _logits(rng, rows, cols, dt, 4.0)
    y = rng.integers(0, cols, size=rows, dtype=np.int32)
    y[0], y[1] = 0, cols - 1
    # shift: rows that start one element past a 16-byte boundary, the gradient's one further (another alignment)
    buf = torch.empty(rows * cols + 2 * shift, dtype=z.dtype, device=DEV)
    zs = buf[shift:shift + rows * cols].view(rows, cols)
    zs.copy_(z)
    for gshift in sorted({shift, 2 * shift}):
        out = torch.full((rows * cols + 2 * shift,), float("nan"), dtype=z.dtype, device=DEV)
        g = out[gshift:gshift + rows * cols].view(rows, cols)
        loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
        T.tfd_softmax_cross_entropy_grad(zs, torch.from_numpy(y).to(DEV), g, loss)
        g_want, l_want = oracle.softmax_cross_entropy_grad(z_h, y, grad_dtype="f64")
        K, p = _bounds(z_h, dt)
        allowed = K * 2.0 ** -24 * p + 2.0 ** -24
        if dt == "bf16":
            allowed = allowed + 2.0 ** -8 * np.abs(g_want)
        err = np.abs(to_f64(g) - g_want)
        assert np.all(err <= allowed), float(err.max())
        lse = np.log(np.sum(np.exp(z_h - z_h.max(axis=1, keepdims=True)), axis=1))
        assert abs(loss.item() - l_want) <= float(np.sum(K + 4 * np.abs(lse) + 4)) * 2.0 ** -24


def test_softmax_xent_more_rows_than_a_grid_of_row_blocks():
    """2^24 + 3 rows of 520 16-bit columns: a block per row would need more than 2^32 threads."""
    rows, cols = 2 ** 24 + 3, 520
    z = torch.zeros(rows, cols, dtype=torch.bfloat16, device=DEV)
    z[::4096, 7] = 4.0
    y = (torch.arange(rows, device=DEV) % cols).to(torch.int32)
    g = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device=DEV)
    loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
    T.tfd_softmax_cross_entropy_grad(z, y, g, loss)
    at = [0, 1, 4096, 2 ** 23 + 5, 2 ** 24 - 1, 2 ** 24, 2 ** 24 + 2]
    z_h = to_f64(z[at])
    want, _ = oracle.softmax_cross_entropy_grad(z_h, y[at].cpu().numpy(), grad_dtype="f64")
    assert np.all(np.abs(to_f64(g[at]) - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -22)
    part = g.view(-1)[::997]  # of every second row
    assert not (part != part).any()
    peaked = (rows + 4095) // 4096
    hit = int(((torch.arange(0, rows, 4096, device=DEV) % cols) == 7).sum())
    want_loss = (rows - peaked) * np.log(cols) + peaked * np.log(cols - 1 + np.exp(4.0)) - 4.0 * hit
    assert abs(loss.item() - want_loss) <= 1e-6 * want_loss


@pytest.mark.parametrize("rows", [1, 4, 5, 11, 600])
@pytest.mark.parametrize("dt,cols", [("f32", 10), ("f32", 513), ("bf16", 1031), ("bf16", 32768), ("f32", 65551)])
def test_softmax_xent_workspace_of_8_bytes_per_four_rows(dt, cols, rows):
    """The workspace that the query asks for, 8 bytes for every four rows, is enough for every kernel, which stays
    inside it; with 8 bytes per row the gradient is the same."""
    need = T.tfd_softmax_xent_workspace_size(rows)
    assert need == 8 * ((rows + 3) // 4)
    rng = np.random.default_rng([rows, cols])
    z_h, z = _logits(rng, rows, cols, dt, 4.0)
    y = rng.integers(0, cols, size=rows, dtype=np.int32)
    got = []
    for nbytes in (need, 8 * rows):
        buf = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
        g = torch.full_like(z, float("nan"))
        loss = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
        T.tfd_softmax_cross_entropy_grad(z, torch.from_numpy(y).to(DEV), g, loss, workspace=buf[:nbytes])
        assert bool((buf[nbytes:] == 0x5A).all())
        got.append((g, loss.item()))
    assert torch.equal(got[0][0], got[1][0])
    _, want = oracle.softmax_cross_entropy_grad(z_h, y, grad_dtype="f64")
    for _, loss in got:
        assert abs(loss - want) <= 1e-6 * want
