"""GPU tests of the PM force's sort, assignment and interpolation at the edges
of their tiles and windows, against the FP64 oracle."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tests.test_gpu_pm import check, pp  # noqa: E402,F401  (the oracle comparison, the fixture)


def params(L, n_mesh):
    rs = 1.25 * L / n_mesh
    return W.BoxParams(L=L, rs=rs, rcut=min(4.5 * rs, 0.45 * L), eps=0.0)


# sort tiles of 4096 particles; windows of 64; one, two and three passes (6 to
# 23 bits of cell number); fewer and more particles than cells
@pytest.mark.parametrize("n,n_mesh", [(1, 4), (63, 4), (64, 5), (65, 12), (4095, 16), (4096, 13), (4097, 33),
                                      (20481, 8), (9000, 162)])
def test_pm_tiles_and_windows(pp, n, n_mesh):  # noqa: F811
    rng = np.random.default_rng(n + n_mesh)
    L = 20.0
    pos = W.mixture(rng, n, L, 0.5, 1 + n // 300)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    if n > 1:
        check(pp, pos, mass, params(L, n_mesh), n_mesh)
    else:
        acc = pp.PMPlan(params(L, n_mesh), n_mesh).accel(torch.as_tensor(pos).cuda(), torch.as_tensor(mass).cuda())
        assert torch.isfinite(acc).all()


@pytest.mark.parametrize("n,at", [(64, 0.0), (1000, 7.3), (5000, 19.99)])
def test_pm_particles_in_one_cell(pp, n, at):  # noqa: F811
    """All particles but one in one cell: one run over many windows."""
    rng = np.random.default_rng(n)
    L, n_mesh = 20.0, 16
    d = L / n_mesh
    cell = np.floor(at / d) * d
    pos = cell + rng.random((3, n)) * d * 0.999
    pos[:, n // 2] = [3.1, 12.7, 0.4]
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    # the forces inside the cell nearly cancel: the FP32 results are held
    # against the largest force
    from oracle import pm as opm
    p = params(L, n_mesh)
    ref = opm.pm_accel(pos, mass.astype(np.float64), p, n_mesh)
    acc = pp.PMPlan(p, n_mesh).accel(torch.as_tensor(pos).cuda(), torch.as_tensor(mass).cuda()).cpu().numpy()
    assert np.abs(acc - ref).max() <= 1e-6 * np.abs(ref).max()
