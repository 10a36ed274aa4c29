"""Absorbing grids at the edge of the workspace budget.  Tall depth-only grids
need least without the streaming kernel's table of the side columns; a budget that
is enough for one step per launch runs them so, with the same bits, and what does
not fit at all is refused."""
import numpy as np
import pytest

import synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# nx, nz: bytes that the solve of 40 steps asked for when all such grids ran one step per
# launch (with the table the streaming kernel asks for 12 kB and 75 kB more)
NEED = {(8, 8192): 34501592, (64, 20000): 84133816}


def _case(nx, nz, nsteps):
    from paper_1502_07873_amd.query import device_medium, grid_tuple
    med = synthetic.random_layers_medium(np.random.default_rng(1), nz, 10.0, 2)
    g = synthetic.Grid(nx, nz, 10.0, synthetic.cfl_dt(10.0, med.vp_max()), nsteps, bc="absorbing")
    return grid_tuple(g), device_medium(med.kind, med.rho, med.lam, med.mu)


def _forward(budget, grid, medium, rec):
    from paper_1502_07873_amd import Context
    th = np.array([[35.0, 45.0, 0.02, 15.0, 1e13, 2e13, 1e13]])
    out = torch.full((grid[4] + 1, len(rec), 2), float("nan"), device="cuda")
    with Context(0, budget) as c:
        c.forward_solve_batch([grid], [medium], th, [rec], [out])
        torch.cuda.synchronize()
        return out.cpu().numpy(), c.get_option("last_variant")


@pytest.mark.parametrize("nx,nz", list(NEED))
def test_least_budget_of_tall_grids(nx, nz):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    grid, medium = _case(nx, nz, 40)
    rec = np.array([1, 3, nx - 2], dtype=np.int32)
    print(f"[gpu case] absorbing {nx}x{nz} at {NEED[nx, nz]} bytes", flush=True)
    tight, vt = _forward(NEED[nx, nz], grid, medium, rec)
    roomy, vr = _forward(1 << 30, grid, medium, rec)
    assert vr == 28 and vt != 28
    assert np.array_equal(tight, roomy)
    assert np.max(np.abs(roomy)) > 0


@pytest.mark.parametrize("nx,nz", [(8, 8192), (101, 76)])
def test_too_small_is_refused(nx, nz):
    # tiled and resident
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1502_07873_amd import eigseis
    grid, medium = _case(nx, nz, 40)
    with pytest.raises(eigseis.EigError, match="budget"):
        _forward(4096, grid, medium, np.array([1], dtype=np.int32))
