"""CNN SGD on the matrix cores at the edges of its tiles: one to six channel
tiles, weight-gradient tiles shared among wavefronts or several per wavefront,
four, two and one example at a time with a remainder, shapes left to the plain
kernel.  The step must equal the FP64 gradient step: FP32 rounding (2^-24) of
chains of at most 3C + m + B terms, forward and backward, on gradients measured
against their largest entry, as in the other SGD tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    return pkg


@pytest.mark.parametrize("F,m,C,B", [(2, 4, 4, 1), (2, 96, 32, 7), (1, 96, 96, 3), (1, 100, 48, 5), (2, 16, 20, 6),
                                     (1, 32, 64, 4), (1, 256, 16, 3), (1, 192, 64, 2), (1, 132, 84, 2), (3, 8, 12, 33)])
def test_cnn_sgd_step_at_tile_edges(F, m, C, B):
    pkg = _pkg()
    lr = 0.05
    w = W.cnn_weights(F, C, seed=7)
    rng = np.random.default_rng(8)
    x = rng.standard_normal((F, B, m)).astype(np.float32)
    y = rng.uniform(1, 4, (F, B)).astype(np.float32)
    wt = torch.from_numpy(w.copy()).cuda()
    loss = pkg.cnn_sgd_step(wt, m, C, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), lr).cpu().numpy()
    got = wt.cpu().numpy().astype(np.float64)
    for f in range(F):
        l64, g = O.cnn_mse_grad(w[f].astype(np.float64), x[f], y[f].astype(np.float64), C)
        assert abs(loss[f] - l64) <= 1e-5 * l64
        step_got, step_want = got[f] - w[f], -lr * g
        # the stored weights round the step to 2^-24 of their own size
        assert np.all(np.abs(step_got - step_want) <= 1e-4 * np.abs(step_want).max() + 2.0 ** -23 * np.abs(w[f]))


def test_cnn_steps_in_a_row_and_alone_agree():
    """A filter's step does not depend on the other filters of the call, and
    repeated steps are deterministic."""
    pkg = _pkg()
    F, m, C, B = 3, 48, 20, 9
    w = torch.from_numpy(W.cnn_weights(F, C, seed=3)).cuda()
    g = torch.Generator(device="cuda").manual_seed(4)
    x, y = torch.randn((F, B, m), generator=g, device="cuda"), torch.rand((F, B), generator=g, device="cuda") * 4
    runs = []
    for _ in range(2):
        wt = w.clone()
        for _ in range(5):
            pkg.cnn_sgd_step(wt, m, C, x, y, 0.02)
        runs.append(wt.cpu())
    assert torch.equal(runs[0], runs[1])
    for f in range(F):
        wt = w[f:f + 1].clone()
        for _ in range(5):
            pkg.cnn_sgd_step(wt, m, C, x[f:f + 1].contiguous(), y[f:f + 1].contiguous(), 0.02)
        assert torch.equal(wt[0].cpu(), runs[0][f])


@pytest.mark.parametrize("F,m,C,B", [(128, 96, 32, 32), (16, 132, 84, 4)])
def test_cnn_step_is_done_on_return(F, m, C, B):
    """Both kernels' calls return with the step's results on the device."""
    pkg = _pkg()
    w = torch.from_numpy(W.cnn_weights(F, C, seed=3)).cuda()
    x, y = torch.randn((F, B, m), device="cuda"), torch.rand((F, B), device="cuda")
    pkg.cnn_sgd_step(w, m, C, x, y, 0.02)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(3):
            pkg.cnn_sgd_step(w, m, C, x, y, 0.02)
            assert stream.query()


def test_cnn_step_in_a_captured_graph():
    """The matrix-core step may be captured; each replay is one more step."""
    pkg = _pkg()
    F, m, C, B = 5, 48, 16, 8
    w = torch.from_numpy(W.cnn_weights(F, C, seed=3)).cuda()
    x, y = torch.randn((F, B, m), device="cuda"), torch.rand((F, B), device="cuda")
    want = w.clone()
    pkg.cnn_sgd_step(want, m, C, x, y, 0.02)
    graph, held = torch.cuda.CUDAGraph(), w.clone()
    with torch.cuda.graph(graph):
        pkg.cnn_sgd_step(held, m, C, x, y, 0.02)
    assert torch.equal(held, w)
    for _ in range(4):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(held, want)
        pkg.cnn_sgd_step(want, m, C, x, y, 0.02)


def test_cnn_training_allocates_no_gradients_it_does_not_use():
    """Training on the matrix cores keeps the weights and the best ones, and no
    third array of their size."""
    pkg = _pkg()
    sizes = []

    class Counted(dict):
        def __setitem__(self, ptr, nbytes):
            sizes.append(nbytes)
            super().__setitem__(ptr, nbytes)

    alloc = pkg.TorchAllocator()
    alloc.live = Counted()
    ix = pkg.Index(allocator=alloc).build(torch.from_numpy(W.random_walk(2000, 32, seed=1)).cuda(), leaf_capacity=100,
                                          n_segments=8)
    F, C = ix.info()["n_leaves"], 16
    sizes.clear()
    ix.train_filters(n_global=60, n_local=10, max_epochs=2, seed=3, arch="cnn", hidden=C, th_override=0.0)
    assert ix.info()["n_filters"] == F
    assert sizes.count(4 * F * (3 * C * C + 6 * C + 1)) == 2
