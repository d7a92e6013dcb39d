"""sp_heff_profile: the mixing of the left environment is a phase of its own
wherever there is one, whatever the site's plan."""
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair  # noqa: E402

import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["abinitio", "hubbard"])
def test_mixing_is_timed_apart_from_the_products(op):
    K = 6
    gpu = make_pair(K, K, 0, 16, 0, 3, op=op, integrals=W.abinitio_integrals(K, 4), oracle=False)[1]
    seen = set()
    for k in range(1, K + 1):
        for plan in ("as chosen", "block products"):
            if plan == "block products":
                gpu.set_heff_plan(k, 0)
            fused = gpu.heff_plan(k)[0] > 0
            x = torch.ones(gpu.site_size(k), dtype=torch.float64, device="cuda")
            y, ny = torch.empty_like(x), torch.empty_like(x)
            mix = gpu.heff_profile(k, x, y, ny, reps=2)["premix_once"]
            assert (mix["ms"] > 0) == (mix["flops"] > 0), (k, plan, mix)
            seen.add((fused, mix["flops"] > 0))
        if k < K:
            gpu.env_update(k, +1)
    assert {(True, True), (False, True)} <= seen if op == "abinitio" else {m for _, m in seen} == {False}
