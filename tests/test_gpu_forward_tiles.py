"""The model's outputs at the row counts where its tiles grow, and that their
time does not jump there."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1703_04789_amd as sp  # noqa: E402
import workloads as W  # noqa: E402
from oracle import precond as pre  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [16384, 16385, 32768, 32769, 49152, 49153, 65537])
def test_outputs_at_the_edges_of_the_tiles(rows):
    # FP32 outputs of FP64 sums
    p = W.mlp_init(200, 31)
    F = np.random.default_rng(32).standard_normal((rows, 5)).astype(np.float32)
    y = sp.MLP(p).forward(torch.tensor(F, device="cuda")).cpu().numpy()
    want = pre.forward({k: np.asarray(np.asarray(v, np.float32), np.float64) for k, v in p.items()}, F.astype(np.float64))
    assert np.abs(y - want).max() < 1e-6 * np.abs(want).max()


def _usec(m, rows, calls=40):
    F = torch.randn(rows, 5, device="cuda")
    for _ in range(3):
        m.forward(F)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):  # the calls without their launches
        for _ in range(calls):
            m.forward(F)
    best = float("inf")
    for _ in range(10):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / calls)
    return best


def test_one_row_more_does_not_add_a_quarter():
    m = sp.MLP(W.mlp_init(256, 1))
    a, b = _usec(m, 16384), _usec(m, 16385)
    print(f"[forward] 16384 rows {a:.2f} us, 16385 rows {b:.2f} us", flush=True)
    assert b < 1.12 * a
