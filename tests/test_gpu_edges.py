"""Kernels and dispatch branches at the sizes where they can go wrong (tile
edges, remainders, split reductions), against the FP64 oracle.

Tolerance 1e-11 relative, as for the other single contractions: FP64 sums of
at most some ten thousand terms of one magnitude."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair, rel_err  # noqa: E402

import paper_1703_04789_amd as sp  # noqa: E402
import workloads as W  # noqa: E402
from oracle import precond as pre  # noqa: E402

pytestmark = pytest.mark.gpu


def _left(gpu, orc, k):
    for j in range(1, k):
        gpu.env_update(j, +1)
        orc.update_left(j)


def _pair(K, D, G, twoM=0, twoS=0, N=None, seed=3, **kw):
    ab = kw.pop("abinitio", False)
    if ab:
        kw.update(op="abinitio", integrals=W.abinitio_integrals(K, 4))
    return make_pair(K, K - K % 2 if N is None else N, twoM, D, twoS, G, seed=seed, **kw)


# (sites, D, G, site, ab-initio): sectors of 36 states (two 32-wide tiles, the
# second narrow), sectors of one state, and more than 256 (g, row) units per
# tile, so that the parts of a tile are summed
DIAG = [(8, 300, 3, 4, False), (8, 300, 3, 5, False), (6, 12, 24, 3, True), (6, 12, 24, 4, True), (5, 40, 40, 3, True),
        (4, 1, 2, 2, False)]


@pytest.mark.parametrize("case", DIAG)
def test_diagonal_tiles_and_parts(case):
    K, D, G, k, ab = case
    tab, gpu, orc = _pair(K, D, G, abinitio=ab)
    _left(gpu, orc, k)
    n = gpu.site_size(k)
    dh, dn = (torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
    gpu.heff_diag(k, dh, dn)
    torch.cuda.synchronize()
    ref_h, ref_n = (orc.mps.site_packed(k, v) for v in orc.heff_diag(k))
    assert rel_err(dh.cpu().numpy(), ref_h) < 1e-11
    assert rel_err(dn.cpu().numpy(), ref_n) < 1e-11


# (sites, D, G, site, ab-initio, precision): particle-number blocks of 252
# states (two tiles of columns), of 70 (odd remainders in every direction), of
# one; channels cut into several parts; every arithmetic and both tile widths
CHAIN = [(10, 1000, 2, 5, False, "fp64"), (8, 300, 3, 4, False, "fp64"), (8, 300, 3, 5, False, "fp32"),
         (8, 37, 5, 6, False, "bf16x3"), (4, 1, 2, 2, False, "fp64"), (6, 60, 3, 3, True, "fp64"),
         (6, 60, 3, 4, True, "fp32"), (7, 100, 2, 4, True, "bf16x3"), (8, 90, 2, 5, True, "bf16x3")]
# FP64 as above; the reduced precisions as for their other products
TOL = {"fp64": 1e-11, "fp32": 1e-5, "bf16x3": 1e-4}


@pytest.mark.parametrize("case", CHAIN)
def test_chained_products_at_tile_edges(case):
    K, D, G, k, ab, prec = case
    tab, gpu, orc = _pair(K, D, G, abinitio=ab, precision=prec)
    for j in range(1, k):  # unit left environments stay in the FP32 range
        orc.mps.left_orthonormalize(j)
        orc.update_left(j)
    # the oracle's tensors on both sides: the right-canonical form of random
    # square sectors is conditioned like their QR (1e-10 at D = 1000)
    for j in range(1, K + 1):
        gpu.set_site(j, orc.mps.site_packed(j))
    for j in range(1, k):
        gpu.env_update(j, +1)
    for j in range(K, k, -1):
        gpu.env_update(j, -1)
    rng = np.random.default_rng(5)
    n = gpu.site_size(k)
    for plan in ("as chosen", "block products"):
        if plan != "as chosen":
            gpu.set_heff_plan(k, 0)
        x = rng.standard_normal(n)
        y_ref, ny_ref = orc.heff(k, orc.mps.dense_site(k, x))
        xd = torch.tensor(x, device="cuda")
        y, ny = (torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
        gpu.heff_apply(k, xd, y, ny)
        torch.cuda.synchronize()
        assert rel_err(y.cpu().numpy(), orc.mps.site_packed(k, y_ref)) < TOL[prec], plan
        assert rel_err(ny.cpu().numpy(), orc.mps.site_packed(k, ny_ref)) < TOL[prec], plan


@pytest.mark.parametrize("ab", [False, True])
def test_right_updates_after_moved_sites(ab):
    # the right environments rebuilt from changed tensors, then H_eff x at the
    # far left: sites of every width down to the boundary
    tab, gpu, orc = _pair(7, 45, 3, abinitio=ab)
    rng = np.random.default_rng(6)
    for k in range(7, 1, -1):
        a = rng.standard_normal(gpu.site_size(k)) / np.sqrt(gpu.site_size(k))
        gpu.set_site(k, a)
        orc.mps.A[k - 1] = orc.mps.dense_site(k, a)
        gpu.env_update(k, -1)
        orc.update_right(k)
    n = gpu.site_size(1)
    x = rng.standard_normal(n)
    y_ref, ny_ref = orc.heff(1, orc.mps.dense_site(1, x))
    xd = torch.tensor(x, device="cuda")
    y, ny = torch.empty_like(xd), torch.empty_like(xd)
    gpu.heff_apply(1, xd, y, ny)
    torch.cuda.synchronize()
    assert rel_err(y.cpu().numpy(), orc.mps.site_packed(1, y_ref)) < 1e-11
    assert rel_err(ny.cpu().numpy(), orc.mps.site_packed(1, ny_ref)) < 1e-11


def test_premixed_environments_of_several_lds_tiles():
    # K = 14: more environment blocks of one shape than a tile of sources
    # holds; against the plain path (the oracle's dense MPO is too large)
    K, D, G = 14, 12, 2
    ig = W.abinitio_integrals(K, 4)
    a, b = (make_pair(K, K, 0, D, 0, G, seed=3, op="abinitio", integrals=ig, oracle=False, path=p)[1]
            for p in ("tiled", "plain"))
    rng = np.random.default_rng(7)
    for k in range(1, K + 1):
        x = torch.tensor(rng.standard_normal(a.site_size(k)), device="cuda")
        out = []
        for h in (a, b):
            y, ny = torch.empty_like(x), torch.empty_like(x)
            h.heff_apply(k, x, y, ny)
            out.append((y, ny))
        torch.cuda.synchronize()
        for u, v in zip(*out):
            assert rel_err(u.cpu().numpy(), v.cpu().numpy()) < 1e-11, k
        for h in (a, b):
            if k < K:
                h.env_update(k, +1)


@pytest.mark.parametrize("hidden", [1, 64, 65, 128, 129, 256])
@pytest.mark.parametrize("rows", [1, 63, 65, 257, 16385])
def test_model_training_at_tile_edges(hidden, rows):
    # two Adam steps and a forward pass; tolerances as for the other training
    # tests (loss 1e-9 relative, FP32 weights 2e-7, FP32 outputs 1e-6)
    p = W.mlp_init(hidden, 11)
    m = sp.MLP(p)
    rng = np.random.default_rng(12)
    F = rng.standard_normal((rows, 5)).astype(np.float32)
    Y = rng.standard_normal(rows).astype(np.float32)
    Fd, Yd = torch.tensor(F, device="cuda"), torch.tensor(Y, device="cuda")
    ref = {k: np.asarray(np.asarray(v, np.float32), np.float64) if np.ndim(v) else float(np.float32(v)) for k, v in p.items()}
    state = {}
    for _ in range(2):
        loss = m.train_step(Fd, Yd, 1e-3)
        lref, g = pre.loss_and_grads(ref, F.astype(np.float64), Y.astype(np.float64))
        assert abs(loss - lref) < 1e-9 * lref
        ref = pre.adam_step(ref, g, state, 1e-3)
        ref = {k: np.asarray(np.asarray(v, np.float32), np.float64) if np.ndim(v) else float(np.float32(v))
               for k, v in ref.items()}
        got = m.params()
        for k in ("W1", "b1", "w2", "b2"):
            assert np.abs(np.asarray(got[k], np.float64) - ref[k]).max() < 2e-7, k
    y = m.forward(Fd).cpu().numpy()
    want = pre.forward({k: np.asarray(v, np.float64) for k, v in got.items()}, F.astype(np.float64))
    assert np.abs(y - want).max() < 1e-6 * np.abs(want).max()


@pytest.mark.parametrize("K,D", [(8, 16), (8, 64), (10, 200), (16, 256), (16, 480), (16, 700)])
def test_gauge_moves_at_register_tile_edges(K, D):
    # sectors of 1 to more than 64 columns and 1 to more than 256 rows (odd
    # remainders of 16 on the way): the right-canonical form of random tensors.
    # Single tensors are conditioned like their QR; their orthonormality and
    # the centre, which collects every R, are not
    tab, gpu, orc = _pair(K, D, 2)
    for k in range(2, K + 1):
        a = orc.mps.dense_site(k, gpu.get_site(k))  # (sigma, left, right)
        m = np.tensordot(a, a, axes=([0, 2], [0, 2]))
        assert np.abs(m - np.eye(len(m))).max() < 1e-11, k
    assert rel_err(gpu.get_site(1), orc.mps.site_packed(1)) < 1e-11
