"""Products and environment updates recorded into a graph by the caller: a
replay reads the environments as they are then, and calls made between the
replays are not disturbed by them."""
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair  # noqa: E402

import numpy as np  # noqa: E402
import paper_1703_04789_amd as sp  # noqa: E402
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _state(stream, K=8, D=24, G=3, precision="fp64"):
    # dense integrals: the MPO is mixed into the environments at every inner site
    tab = W.make_block_table(K, K, 0, D)
    return sp.SPMPS(tab, W.random_blocks(tab, 3), sp.mpo_abinitio(*W.abinitio_integrals(K, 4)), 0, G,
                    stream=stream.cuda_stream, precision=precision)


def _vectors(gpu, k, seed):
    x = torch.tensor(np.random.default_rng(seed).standard_normal(gpu.site_size(k)), device="cuda")
    return x, torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))


def _capture(stream, f):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        f()
    return g


def _replay(g, stream):
    with torch.cuda.stream(stream):
        g.replay()
    torch.cuda.synchronize()


def _eager(gpu, k, x):
    y, ny = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    torch.cuda.synchronize()
    gpu.heff_apply(k, x, y, ny)
    torch.cuda.synchronize()
    return y, ny


@pytest.mark.parametrize("plan", ["as chosen", "block products"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("warm", [False, True])
def test_replayed_products_read_the_environments_of_the_moment(plan, precision, warm):
    print(f"[case] graph replay {plan} {precision} warm={warm}", flush=True)
    s = torch.cuda.Stream()
    k, a, b = 4, _state(s, precision=precision), _state(s, precision=precision)
    for h in (a, b):
        if plan == "block products":
            h.set_heff_plan(k, 0)
        for j in range(1, k):
            h.env_update(j, +1)
    x, y, ny = _vectors(a, k, 1)
    if warm:
        _eager(a, k, x)
    g = _capture(s, lambda: a.heff_apply_noalloc(k, x, y, ny))
    # an eager call between the recording and the first replay
    want = _eager(b, k, x)
    for u, v in zip(_eager(a, k, x), want):
        assert torch.equal(u, v)
    rng = np.random.default_rng(2)
    for step in range(3):
        _replay(g, s)
        assert torch.equal(y, want[0]) and torch.equal(ny, want[1]), step
        for u, v in zip(_eager(a, k, x), want):  # the replay leaves eager calls alone
            assert torch.equal(u, v), step
        # another right environment, then another left one
        q, d = ((k + 1, -1), (k - 1, +1))[step % 2]
        t = rng.standard_normal(a.site_size(q)) / np.sqrt(a.site_size(q))
        for h in (a, b):
            h.set_site(q, t)
            h.env_update(q, d)
        y.fill_(float("nan"))
        ny.fill_(float("nan"))
        want = _eager(b, k, x)
    _replay(g, s)
    assert torch.equal(y, want[0]) and torch.equal(ny, want[1])


def test_replays_leave_products_at_other_sites_alone():
    s = torch.cuda.Stream()
    k, a, b = 4, _state(s), _state(s)
    for h in (a, b):
        for j in range(1, k):
            h.env_update(j, +1)
    x, y, ny = _vectors(a, k, 1)
    g = _capture(s, lambda: a.heff_apply_noalloc(k, x, y, ny))
    for h in (a, b):  # the centre moves on
        h.env_update(k, +1)
    x2 = _vectors(a, k + 1, 3)[0]
    want = _eager(b, k + 1, x2)
    for _ in range(3):
        for u, v in zip(_eager(a, k + 1, x2), want):
            assert torch.equal(u, v)
        _replay(g, s)


def test_replayed_environment_updates():
    # a graph of one left update and the product after it, against eager calls
    s = torch.cuda.Stream()
    k, a, b = 4, _state(s), _state(s)
    for h in (a, b):
        for j in range(1, k - 1):
            h.env_update(j, +1)
    x, y, ny = _vectors(a, k, 1)

    def body():
        a.env_update(k - 1, +1)
        a.heff_apply_noalloc(k, x, y, ny)
        a.heff_apply_noalloc(k, y, x2, ny2)

    x2, ny2 = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    g = _capture(s, body)
    rng = np.random.default_rng(4)
    for step in range(3):
        t = rng.standard_normal(a.site_size(k - 1)) / np.sqrt(a.site_size(k - 1))
        for h in (a, b):
            h.set_site(k - 1, t)
        _replay(g, s)
        b.env_update(k - 1, +1)
        want = _eager(b, k, x)
        assert torch.equal(y, want[0]) and torch.equal(ny, want[1]), step
        want2 = _eager(b, k, want[0])
        assert torch.equal(x2, want2[0]) and torch.equal(ny2, want2[1]), step
