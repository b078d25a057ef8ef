"""CNN inference on split operands at the edges of its tiles: channels that are
no multiple of 16 or 32, positions past a tile, shapes the split kernel leaves
to the plain one, filters that share their queries among work-groups, and
values that are not finite.  Bound: FP32 rounding (2^-24) of every term and
partial sum in a chain of 3 + 3C + m + C + 8 over the magnitudes summed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as W

pytestmark = pytest.mark.gpu


def _pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    return pkg


def _forward(w, x, C):
    """FP64 predictions of one filter for x [nq, m], and the magnitude summed."""
    w = w.astype(np.float64)
    w1, b1 = w[: 3 * C].reshape(C, 3), w[3 * C: 4 * C]
    w2, b2 = w[4 * C: 4 * C + 3 * C * C].reshape(C, C, 3), w[4 * C + 3 * C * C: 5 * C + 3 * C * C]
    w3, b3 = w[5 * C + 3 * C * C: 6 * C + 3 * C * C], w[-1]
    out, mag = [], []
    with np.errstate(invalid="ignore", over="ignore"):
        for row in x.astype(np.float64):
            xp = np.pad(row, 1)
            taps = np.stack([xp[:-2], xp[1:-1], xp[2:]])
            h = np.pad(np.fmax(w1 @ taps + b1[:, None], 0.0), ((0, 0), (1, 1)))
            hm = np.pad(np.abs(w1) @ np.abs(taps) + np.abs(b1)[:, None], ((0, 0), (1, 1)))
            m = len(row)
            z = sum(w2[:, :, t] @ h[:, t:t + m] for t in range(3)) + b2[:, None]
            zm = sum(np.abs(w2[:, :, t]) @ hm[:, t:t + m] for t in range(3)) + np.abs(b2)[:, None]
            out.append(w3 @ np.fmax(z, 0.0).mean(axis=1) + b3)
            mag.append(np.abs(w3) @ zm.mean(axis=1) + np.abs(b3))
    return np.array(out), np.array(mag)


@pytest.mark.parametrize("F,m,C,nq", [(1, 4, 4, 1), (2, 20, 36, 3), (2, 96, 96, 7), (2, 16, 100, 5), (2, 48, 68, 4),
                                      (300, 8, 12, 9), (1, 256, 16, 6), (1, 256, 64, 3), (1, 300, 4, 2),
                                      (2, 36, 64, 33)])
def test_split_cnn_inference_at_tile_edges(F, m, C, nq):
    pkg = _pkg()
    w = W.cnn_weights(F, C, seed=F + m + C, out_bias=0.5)
    x = np.random.default_rng(m).standard_normal((nq, m)).astype(np.float32)
    got = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, C, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in range(0, F, max(1, F // 5)):
        want, mag = _forward(w[f], x, C)
        assert np.all(np.abs(got[:, f] - want) <= (4 * C + m + 11) * 2.0 ** -24 * mag)


def test_split_cnn_inference_with_values_that_are_not_finite():
    pkg = _pkg()
    m, C, nq = 40, 20, 12
    w = W.cnn_weights(3, C, seed=4)
    w[1, 4 * C + 5] = np.inf     # a second-layer weight
    x = np.random.default_rng(6).standard_normal((nq, m)).astype(np.float32)
    x[3, 5], x[7, 0] = np.nan, np.inf
    got = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, C, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in range(3):
        want, mag = _forward(w[f], x, C)
        fin = np.isfinite(want) & np.isfinite(mag)
        assert fin.sum() >= (9 if f != 1 else 0)
        assert np.all(np.abs(got[fin, f] - want[fin]) <= (4 * C + m + 11) * 2.0 ** -24 * mag[fin])
        assert np.array_equal(np.isfinite(got[:, f]), np.isfinite(want))


@pytest.mark.parametrize("m,C", [(40, 20), (96, 96)])
@pytest.mark.parametrize("ea,ew,eo", [(0, 0, 0), (58, -58, 0), (105, -105, 0), (118, -118, 0), (-105, 105, 0), (-118, 118, 0),
                                      (0, -122, 122), (-122, 0, 122)])
def test_operands_at_the_ends_of_the_range(m, C, ea, ew, eo):
    """The first layer, the second and the readout times 2^ea, 2^ew and 2^eo:
    FP32 accuracy, whatever a bf16 part can hold."""
    pkg = _pkg()
    w = W.cnn_weights(2, C, seed=9)
    w[:, : 4 * C] *= np.float32(2.0 ** ea)
    w[:, 4 * C: 4 * C + 3 * C * C] *= np.float32(2.0 ** ew)
    w[:, 4 * C + 3 * C * C: 5 * C + 3 * C * C] = 0
    w[:, 5 * C + 3 * C * C: -1] *= np.float32(2.0 ** eo)
    w[:, -1] = 0
    x = np.random.default_rng(m).standard_normal((7, m)).astype(np.float32)
    got = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, C, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in range(2):
        want, mag = _forward(w[f], x, C)
        assert np.all(np.abs(got[:, f] - want) <= (4 * C + m + 11) * 2.0 ** -24 * mag)


def test_finite_operands_whose_products_overflow():
    pkg = _pkg()
    m, C = 40, 20
    w = np.abs(W.cnn_weights(2, C, seed=10)) + np.float32(0.01)
    w[:, : 4 * C] *= np.float32(1e25)
    w[:, 4 * C: 4 * C + 3 * C * C] *= np.float32(1e25)
    x = np.abs(np.random.default_rng(1).standard_normal((7, m))).astype(np.float32) + np.float32(0.01)
    got = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, C, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.all(np.isposinf(got))


@pytest.mark.parametrize("F,m,C", [(257, 64, 64), (520, 96, 32), (600, 128, 32), (1030, 40, 20), (1030, 96, 16),
                                   (2050, 256, 8), (4100, 16, 4)])
@pytest.mark.parametrize("nq", [1, 5])
def test_split_cnn_inference_with_more_filters_than_cus(F, m, C, nq):
    """Work-groups of fewer wavefronts, with one and two sets of planes."""
    pkg = _pkg()
    w = W.cnn_weights(F, C, seed=F + C, out_bias=0.5)
    x = np.random.default_rng(m).standard_normal((nq, m)).astype(np.float32)
    got = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, C, torch.from_numpy(x).cuda()).cpu().numpy()
    for f in (0, 1, F // 2, F - 1):
        want, mag = _forward(w[f], x, C)
        assert np.all(np.abs(got[:, f] - want) <= (4 * C + m + 11) * 2.0 ** -24 * mag)
