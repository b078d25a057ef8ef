"""One SGD step of the MLP filters on FP32 matrix cores at the edges of its
tiles: one and sixteen input tiles, an odd number of them (the rows' 16-byte
pieces do not divide evenly), hidden units that fill part of the wavefronts,
batches of one row to all 64, and rows that do not start at 16 bytes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,h,batch,shift", [(16, 16, 1, 0), (48, 32, 64, 0), (240, 256, 33, 0), (256, 16, 64, 1),
                                             (256, 256, 64, 3), (112, 240, 5, 2)])
def test_step_matches_fp64_gradient(m, h, batch, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    F, lr = 3, 0.05
    w = W.mlp_weights(F, m, h, seed=m + h)
    rng = np.random.default_rng(m * h + batch)
    x = rng.standard_normal((F, batch, m)).astype(np.float32)
    y = rng.uniform(1, 4, (F, batch)).astype(np.float32)
    buf = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")
    xt = buf[shift:shift + x.size].view(F, batch, m)  # shift floats past a 16-byte boundary
    xt.copy_(torch.from_numpy(x))
    wt = torch.from_numpy(w.copy()).cuda()
    loss = pkg.mlp_sgd_step(wt, m, h, xt, torch.from_numpy(y).cuda(), lr).cpu().numpy()
    got = wt.cpu().numpy().astype(np.float64)
    for f in range(F):
        l64, g = O.mlp_mse_grad(w[f].astype(np.float64), x[f], y[f].astype(np.float64), m, h)
        assert abs(loss[f] - l64) <= 1e-5 * l64
        step_got, step_want = got[f] - w[f], -lr * g
        # FP32 sums of the gradient, and the rounding of each updated weight
        assert np.all(np.abs(step_got - step_want) <= 1e-4 * np.abs(step_want).max() + 2.0 ** -23 * np.abs(w[f]))
