"""Diagonals of H_eff and N_eff in one launch (few terms) and in three (many):
against the oracle on both sides of the line, at sectors of one tile and more,
and their times at the smallest states, where launches are all there is."""
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair, rel_err  # noqa: E402

import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _diag(h, k):
    dh, dn = (torch.full((h.site_size(k),), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
    h.heff_diag(k, dh, dn)
    torch.cuda.synchronize()
    return dh.cpu().numpy(), dn.cpu().numpy()


# (sites, D, G, ab-initio, path): units of the widest block 3 G (Hubbard) on
# both sides of 80, sectors of 1 to 36 states, wide MPOs whose outer sites
# have few terms and whose centre has many, the plain path
CASES = [(4, 1, 1, False, "tiled"), (8, 300, 3, False, "tiled"), (6, 20, 26, False, "tiled"), (6, 20, 27, False, "tiled"),
         (6, 12, 4, True, "tiled"), (5, 24, 11, True, "tiled"), (6, 20, 26, False, "plain"), (6, 12, 4, True, "plain")]


@pytest.mark.parametrize("case", CASES)
def test_diagonals_of_every_site(case):
    K, D, G, ab, path = case
    kw = dict(op="abinitio", integrals=W.abinitio_integrals(K, 4)) if ab else {}
    tab, gpu, orc = make_pair(K, K - K % 2, 0, D, 0, G, seed=3, path=path, **kw)
    for k in range(1, K + 1):
        if k > 1:
            gpu.env_update(k - 1, +1)
            orc.update_left(k - 1)
        # FP64 sums of at most some thousand terms of one magnitude
        for got, want in zip(_diag(gpu, k), orc.heff_diag(k)):
            assert rel_err(got, orc.mps.site_packed(k, want)) < 1e-11, k


def _usec(f, reps=40):
    for _ in range(5):
        f()
    best = float("inf")
    for _ in range(8):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(reps):
            f()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / reps)
    return best


def test_diagonals_of_few_terms_are_one_launch():
    # a call of three dependent launches costs more than two of one launch
    gpu = make_pair(8, 8, 0, 16, 0, 5, oracle=False)[1]
    n = gpu.site_size(4)
    for k in range(1, 4):
        gpu.env_update(k, +1)
    x = torch.ones(n, dtype=torch.float64, device="cuda")
    dh, dn = torch.empty_like(x), torch.empty_like(x)
    one = _usec(lambda: x.add_(1.0))
    d = _usec(lambda: gpu.heff_diag(4, dh, dn))
    print(f"[diag] {d:.1f} us, one elementwise launch {one:.1f} us", flush=True)
    assert d < 1.8 * one
