"""MLP inference on split operands at the edges of its tiles: inputs and hidden
units that are no multiple of 32 or 16, batches with a remainder, filters that
share their rows among work-groups, and values that are not finite.  Bound:
FP32 rounding of every term and partial sum (2^-24 each, m + h + 8 of them in a
chain) of the magnitudes summed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    return pkg


def _forward(w, x, m, h):
    """FP64 predictions of one filter and the magnitude its terms sum to."""
    w, x = w.astype(np.float64), x.astype(np.float64)
    w1, b1, w2, b2 = w[: h * m].reshape(m, h), w[h * m: h * m + h], w[h * m + h: h * m + 2 * h], w[-1]
    with np.errstate(invalid="ignore", over="ignore"):
        out = np.fmax(x @ w1 + b1, 0.0) @ w2 + b2  # a NaN unit counts as 0, as in the kernels
        mag = (np.abs(x) @ np.abs(w1) + np.abs(b1)) @ np.abs(w2) + np.abs(b2)
    return out, mag


def _draw(F, m, h, nq, seed):
    g = np.random.default_rng(seed)
    w = g.uniform(-1, 1, (F, h * m + 2 * h + 1)).astype(np.float32) / np.float32(np.sqrt(m))
    return w, g.standard_normal((nq, m)).astype(np.float32)


@pytest.mark.parametrize("F,m,h,nq", [(1, 4, 4, 1), (3, 36, 20, 33), (2, 32, 256, 65), (2, 256, 256, 500),
                                      (300, 96, 96, 65), (2, 228, 144, 31), (3, 160, 200, 17), (2, 64, 64, 257),
                                      (1100, 32, 16, 3), (2, 128, 252, 40), (4, 256, 64, 50), (2, 192, 160, 33)])
def test_split_inference_at_tile_edges(F, m, h, nq):
    pkg = _pkg()
    w, x = _draw(F, m, h, nq, F + m + h)
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in range(0, F, max(1, F // 7)):
        want, mag = _forward(w[f], x, m, h)
        assert np.all(np.abs(got[:, f] - want) <= (m + h + 8) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("m,h", [(256, 256), (96, 96)])
def test_split_inference_with_values_that_are_not_finite(m, h):
    pkg = _pkg()
    w, x = _draw(3, m, h, 70, 5)
    x[3, 7], x[40, 1] = np.nan, np.inf
    x[66, 2] = 3.4e38       # finite, but a bf16 part would round it to infinity
    w[1, 11] = np.inf       # input 0, hidden unit 11
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in range(3):
        want, mag = _forward(w[f], x, m, h)
        fin = np.isfinite(want) & np.isfinite(mag) & (mag < 1e37)
        assert np.all(np.abs(got[fin, f] - want[fin]) <= (m + h + 8) * 2.0 ** -24 * mag[fin])
        rest = ~fin & (mag > 1e39)  # infinite in FP32 too
        assert np.array_equal(np.isfinite(got[rest, f]), np.isfinite(want[rest]) & (np.abs(want[rest]) < 3.4e38))
    assert got[3, 0] == w[0, -1]  # every hidden unit a NaN: the output bias alone


@pytest.mark.parametrize("F,m,h,nq", [(800, 4, 4, 1), (500, 36, 20, 33), (260, 32, 256, 129), (260, 256, 256, 97),
                                      (780, 228, 144, 31), (780, 160, 200, 17), (400, 128, 252, 64), (260, 256, 64, 100),
                                      (769, 192, 160, 32), (768, 192, 160, 32)])
def test_split_inference_of_many_filters(F, m, h, nq):
    """As above with the filters it takes for the work to be worth the split (the last two: either side of it)."""
    test_split_inference_at_tile_edges(F, m, h, nq)


@pytest.mark.parametrize("m,h", [(256, 256), (96, 96)])
def test_many_filters_with_values_that_are_not_finite(m, h):
    pkg = _pkg()
    F = 300
    w, x = _draw(F, m, h, 97, 5)
    x[3, 7], x[40, 1] = np.nan, np.inf
    x[66, 2] = 3.4e38       # finite, but a bf16 part would round it to infinity
    w[1, 11] = np.inf       # input 0, hidden unit 11
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in (0, 1, 2, F - 1):
        want, mag = _forward(w[f], x, m, h)
        fin = np.isfinite(want) & np.isfinite(mag) & (mag < 1e37)
        assert np.all(np.abs(got[fin, f] - want[fin]) <= (m + h + 8) * 2.0 ** -24 * mag[fin])
        rest = ~fin & (mag > 1e39)  # infinite in FP32 too
        assert np.array_equal(np.isfinite(got[rest, f]), np.isfinite(want[rest]) & (np.abs(want[rest]) < 3.4e38))
    assert got[3, 0] == w[0, -1]  # every hidden unit a NaN: the output bias alone


@pytest.mark.parametrize("m,h", [(256, 256), (96, 96)])
@pytest.mark.parametrize("ex,ew,eo", [(0, 0, 0), (58, -58, 0), (60, -60, 0), (105, -105, 0), (120, -120, 0), (-105, 105, 0),
                                      (-120, 120, 0), (0, -112, 112), (0, -122, 122), (-122, 0, 122), (58, 58, -60),
                                      (-60, -60, 120)])
def test_operands_at_the_ends_of_the_range(m, h, ex, ew, eo):
    """Inputs, first and output weights times 2^ex, 2^ew and 2^eo: FP32 accuracy
    as long as FP32's own sums are in range, whatever a bf16 part can hold."""
    pkg = _pkg()
    F = 300
    w, x = _draw(F, m, h, 97, 7)
    w[:, : m * h] *= np.float32(2.0 ** ew)
    w[:, m * h: m * h + h] = 0
    w[:, m * h + h: -1] *= np.float32(2.0 ** eo)
    w[:, -1] = 0
    x *= np.float32(2.0 ** ex)
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in (0, 7, F - 1):
        want, mag = _forward(w[f], x, m, h)
        assert np.all(np.abs(got[:, f] - want) <= (m + h + 8) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("m,h", [(256, 256), (96, 96)])
def test_finite_operands_whose_products_overflow(m, h):
    """Every term positive and beyond the largest float: infinity, not what
    +inf and -inf of its parts would leave."""
    pkg = _pkg()
    F = 300
    w, x = _draw(F, m, h, 97, 8)
    w, x = np.abs(w), np.abs(x)
    w[:, : m * h] = (w[:, : m * h] + np.float32(0.01)) * np.float32(1e25)
    y = (x + np.float32(0.01)) * np.float32(1e25)
    y[1::2] = x[1::2]  # rows in range between them
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(y).cuda()).cpu().numpy()
    assert np.all(np.isposinf(got[0::2]))
    for f in (0, 7, F - 1):
        want, mag = _forward(w[f], y[1::2], m, h)
        assert np.all(np.abs(got[1::2, f] - want) <= (m + h + 8) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("F,m,h,nq", [(300, 256, 256, 2000), (260, 240, 64, 1999), (300, 96, 96, 4001), (257, 32, 64, 3000)])
def test_filters_that_share_their_rows_among_work_groups(F, m, h, nq):
    """Batches enough that a filter's are dealt to several work-groups, the last
    of them with a remainder, rows that are not finite among them."""
    pkg = _pkg()
    w, x = _draw(F, m, h, nq, F + nq)
    odd = [0, 47, 48, nq // 2, nq - 1]
    x[odd[0], 1], x[odd[1], 0], x[odd[2]], x[odd[3], 3], x[odd[4], 2] = np.nan, np.inf, np.nan, -np.inf, np.nan
    got = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    fine = np.setdiff1d(np.arange(nq), odd)
    for f in (0, 1, F // 2, F - 1):
        want, mag = _forward(w[f], x, m, h)
        assert np.all(np.abs(got[fine, f] - want[fine]) <= (m + h + 8) * 2.0 ** -24 * mag[fine])
        assert got[48, f] == w[f, -1]  # every hidden unit a NaN: the output bias alone
