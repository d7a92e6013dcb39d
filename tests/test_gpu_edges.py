"""Kernels and dispatch branches at the sizes where they can go wrong (tile
edges, remainders, split reductions), against the FP64 oracle.

Tolerance 1e-11 relative, as for the other single contractions: FP64 sums of
at most some ten thousand terms of one magnitude."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair, rel_err  # noqa: E402

import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _left(gpu, orc, k):
    for j in range(1, k):
        gpu.env_update(j, +1)
        orc.update_left(j)


def _pair(K, D, G, twoM=0, twoS=0, N=None, seed=3, **kw):
    ab = kw.pop("abinitio", False)
    if ab:
        kw.update(op="abinitio", integrals=W.abinitio_integrals(K, 4))
    return make_pair(K, K if N is None else N, twoM, D, twoS, G, seed=seed, **kw)


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
