"""Training steps of few rows: the gradient of up to 16 rows in one small
work-group, more in tiles, against the oracle around the line; and the time of
a one-row step."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair  # noqa: E402

import paper_1703_04789_amd as sp  # noqa: E402
import workloads as W  # noqa: E402
from oracle import precond as pre  # noqa: E402

pytestmark = pytest.mark.gpu


def _fp32(p):
    return {k: np.asarray(np.asarray(v, np.float32), np.float64) if np.ndim(v) else float(np.float32(v)) for k, v in p.items()}


@pytest.mark.parametrize("hidden", [1, 63, 64, 65, 200, 256])
@pytest.mark.parametrize("rows", [1, 3, 4, 5, 15, 16, 17, 64])
def test_steps_of_few_rows(hidden, rows):
    # tolerances as for the other training tests: loss 1e-9 relative, FP32
    # weights 2e-7
    p = W.mlp_init(hidden, 21)
    m = sp.MLP(p)
    rng = np.random.default_rng(22)
    F = rng.standard_normal((rows, 5)).astype(np.float32)
    Y = rng.standard_normal(rows).astype(np.float32)
    Fd, Yd = torch.tensor(F, device="cuda"), torch.tensor(Y, device="cuda")
    ref, state = _fp32(p), {}
    for _ in range(2):
        loss = m.train_step(Fd, Yd, 1e-3)
        lref, g = pre.loss_and_grads(ref, F.astype(np.float64), Y.astype(np.float64))
        assert abs(loss - lref) < 1e-9 * lref
        ref = _fp32(pre.adam_step(ref, g, state, 1e-3))
        got = m.params()
        for k in ("W1", "b1", "w2", "b2"):
            assert np.abs(np.asarray(got[k], np.float64) - ref[k]).max() < 2e-7, k


@pytest.mark.parametrize("batch", [3, 16, 17])
def test_interleaved_batches_of_few_rows(batch):
    # batch b takes rows b, b + nb, ..: strided rows in either form.  An FP32
    # weight may round the other way in each of the nb steps
    wl = W.hubbard_small()
    gpu = make_pair(wl.L, wl.N, wl.twoM, wl.D, wl.twoS, wl.G, U=wl.U, seed=wl.seed, oracle=False)[1]
    p = W.mlp_init(64, 5)
    rec = sp.MLP(p, capacity=400)
    gpu.set_precond(record=rec)
    gpu.sweep(1, max_sub=32, max_iter=64)
    F, Y = (a.astype(np.float64) for a in rec.dataset())
    rows = len(Y)
    nb = -(-rows // batch)
    assert rows > 2 * batch
    losses = rec.train(1, batch, 1e-3)
    ref, state, want = _fp32(p), {}, []
    for b in range(nb):
        loss, g = pre.loss_and_grads(ref, F[b::nb], Y[b::nb])
        want.append(loss)
        ref = _fp32(pre.adam_step(ref, g, state, 1e-3))
    assert abs(losses[0] - np.mean(want)) < 1e-6 * np.mean(want)
    got = rec.params()
    for k in ("W1", "b1", "w2", "b2"):
        assert np.abs(np.asarray(got[k], np.float64) - ref[k]).max() < 2e-7 * nb, k


def _usec(m, rows):
    F, Y = torch.randn(rows, 5, device="cuda"), torch.randn(rows, device="cuda")
    best = float("inf")
    for _ in range(200):
        torch.cuda.synchronize()
        t = time.perf_counter()
        m.train_step(F, Y, 1e-6)
        best = min(best, 1e6 * (time.perf_counter() - t))
    return best


def test_a_row_costs_less_than_tiles_of_them():
    # launches and the wait for the loss are the same for both; the kernels of
    # a step in tiles take 16 us, those of one row should take half of it
    m = sp.MLP(W.mlp_init(256, 1))
    one, many = _usec(m, 1), _usec(m, 1000)
    print(f"[train] 1 row {one:.1f} us, 1000 rows {many:.1f} us", flush=True)
    assert one < 0.85 * many
