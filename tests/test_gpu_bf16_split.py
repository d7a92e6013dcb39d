"""The split of FP64 operands into two bf16 values (SP_BF16X3), value by value:
a chain of doubly occupied and empty sites has site tensors of one element and
environments of one value, so N_eff x is x L R times the sum of the quadrature
coefficients.  With two of the three factors 1 it is the split of the third,
hi + lo, exactly: both fit an FP32 accumulator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1703_04789_amd as sp  # noqa: E402
from det_states import product_state  # noqa: E402

pytestmark = pytest.mark.gpu


def _bf16(v):
    """Nearest bf16 of FP32 values, ties to even."""
    u = np.float32(v).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def _split(v):
    hi = _bf16(v).astype(np.float64)
    return hi + _bf16(np.float32(v - hi)).astype(np.float64)


def _near_ties(n, seed):
    # bf16 value + residue half-way between two bf16 values + what FP32 drops
    # of the whole (2^-28) but keeps of the residue
    rng = np.random.default_rng(seed)
    hi = 1.0 + rng.integers(0, 127, n) / 128.0
    res = 2.0 ** -rng.integers(10, 13, n) * (1.0 + (2 * rng.integers(0, 128, n) + 1) / 256.0)
    v = hi + rng.choice([-1.0, 1.0], n) * res + rng.choice([-1.0, 1.0], n) * 2.0 ** -28
    f = np.float32(v).astype(np.float64)
    assert np.any(_split(v) != _split(f))  # rounding to FP32 first changes the split
    return v


def _handle():
    # sites 1 and 3 doubly occupied, 2 and 4 empty
    occ = [(p, s) for p in (0, 2) for s in (0, 1)]
    tab, blocks = product_state([(1.0, occ)], 4, 4)
    gpu = sp.SPMPS(tab, blocks, sp.mpo_identity(4), 0, 4, precision="bf16x3")
    for k in range(1, 5):
        assert gpu.site_size(k) == 1 and gpu.set_heff_plan(k, 0) == 0
    return gpu


def _neff(gpu, k, x):
    xd = torch.tensor([x], dtype=torch.float64, device="cuda")
    y, ny = torch.empty_like(xd), torch.empty_like(xd)
    gpu.heff_apply(k, xd, y, ny)
    torch.cuda.synchronize()
    return float(y[0]), float(ny[0])


@pytest.mark.parametrize("operand", ["site vector", "left environment", "right environment"])
def test_split_of_values_near_ties(operand):
    print(f"[case] bf16 split, {operand}", flush=True)
    gpu, k = _handle(), 2
    gpu.env_update(1, +1)
    one = _neff(gpu, k, 1.0)
    assert one[0] == one[1] and abs(one[0] - 1.0) < 1e-12
    for v in _near_ties(40, 9):
        if operand == "site vector":
            got, val = _neff(gpu, k, v), v
        else:  # the environment of a one-element tensor a is a a
            a = np.sqrt(v)
            val = a * a
            q, d = (1, +1) if operand == "left environment" else (3, -1)
            gpu.set_site(q, np.array([a]))
            gpu.env_update(q, d)
            got = _neff(gpu, k, 1.0)
        want = _split(np.array([val]))[0] * one[0]
        # FP64 sums of four equal terms around an exact split
        assert abs(got[0] - want) < 1e-12 * abs(want), (operand, val.hex())
        assert abs(got[1] - want) < 1e-12 * abs(want), (operand, val.hex())
