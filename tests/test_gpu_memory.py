"""Device memory of a tiled state: its environments, and around them only what
its launches use."""
import pytest

torch = pytest.importorskip("torch")

from gpu_util import make_pair  # noqa: E402

pytestmark = pytest.mark.gpu


def _used(f):
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    h = f()
    torch.cuda.synchronize()
    return h, free - torch.cuda.mem_get_info()[0]


def _env_bytes(h):
    """Bytes of the environments of every bond, from the product's minimal
    bytes: both environments, x, and the partial outputs of every point."""
    out = []
    for k in range(1, h.L + 1):
        n = h.site_size(k)
        x = torch.ones(n, dtype=torch.float64, device="cuda")
        y, ny = torch.empty_like(x), torch.empty_like(x)
        both = h.heff_profile(k, x, y, ny, reps=1)["fused_heff"]["bytes"] - 8.0 * (n + 2 * h.G * n)
        out.append(both - out[-1] if out else both - 8.0 * h.G)  # the boundary: 1 x 1, every channel or one
        if k < h.L:
            h.env_update(k, +1)
    return out


def test_a_quadrature_point_of_a_tiled_state_is_its_environments_and_little_else():
    # the lists are the same for every number of points, so that two states of
    # one table differ by what 27 points hold
    L, D = 32, 256
    make_pair(L, L, 0, 16, 0, 2, oracle=False)[1].close()  # the library's own arrays
    used, env = [], []
    for G in (9, 36):
        h, n = _used(lambda: make_pair(L, L, 0, D, 0, G, oracle=False)[1])
        used.append(n)
        env.append(_env_bytes(h))
        h.close()
    more, e = used[1] - used[0], [b - a for a, b in zip(*env)]
    # scratch per point, against the 6 channels of the largest environment: two
    # rotated states of the site vector (a third), two partial outputs (a
    # quarter each), the gathered diagonals.  The intermediates of the plain
    # path's passes are 8 times that environment and more
    print(f"[memory] {more / 2**20:.0f} MiB, environments {sum(e) / 2**20:.0f}, the largest {max(e) / 2**20:.0f}", flush=True)
    assert sum(e) < more < sum(e) + 2 * max(e)
