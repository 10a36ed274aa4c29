"""The streaming kernels (several leapfrog steps per launch with the strips'
rows in registers) at the edges of their tiles: strips of 128 and 64 columns
that end on, before and past a grid's last column, chunks of one row and of
the whole depth, step counts around the steps per launch, forcing windows at
every side.  Bitwise equal to the one-step kernel of the medium, whose traces
the oracle checks elsewhere and here on one solve per grid."""
import numpy as np
import pytest

import synthetic
from oracle import elastic
from _compare import check_receivers

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TRACE_TOL = 1e-4


def _thetas(g, n, rng):
    h = g.h
    lo = np.array([3.01 * h, 2.01 * h, 0.02, 12.0, 1e13, 1e13, 1e13])
    hi = np.array([(g.nx - 4.01) * h, (g.nz - 4.01) * h, 0.05, 20.0, 1e14, 1e14, 1e14])
    th = lo + (hi - lo) * rng.random((n, 7))
    th[0, :2] = lo[:2]
    th[-1, :2] = hi[:2]
    return th


def _run(variant, grid, medium, th, rec):
    from paper_1502_07873_amd import Context
    from paper_1502_07873_amd.query import device_medium, grid_tuple
    n = len(th)
    dm = device_medium(medium.kind, medium.rho, medium.lam, medium.mu)
    out = torch.full((n, grid.nsteps + 1, len(rec), 2), float("nan"), device="cuda")
    with Context(0, 8 << 30) as c:
        c.set_option("stencil_variant", variant)
        c.forward_solve_batch([grid_tuple(grid)] * n, [dm] * n, th, [rec] * n,
                              list(out.unbind(0)))
        torch.cuda.synchronize()
        assert c.get_option("last_variant") == variant
    return out.cpu().numpy()


# nx: one narrow strip, its end and one past it, a wide one's end and one past
# it, two wide, wide and narrow; nz: one row per chunk up to several chunks.
# `solves`: few (narrow strips, short chunks) or enough waves for wide strips
# and long chunks (400: several rounds of the chip)
@pytest.mark.parametrize("kind,variant,base", [("layered", 23, 0), ("layered", 26, 0),
                                               ("nodal", 24, 6), ("nodal", 27, 6)])
@pytest.mark.parametrize("nx,nz,solves", [(8, 8, 2), (64, 9, 3), (65, 17, 3), (121, 24, 3),
                                          (128, 25, 3), (129, 33, 2), (176, 40, 2), (177, 16, 2),
                                          (240, 18, 400), (129, 50, 400), (241, 10, 2)])
def test_strips_and_chunks(kind, variant, base, nx, nz, solves):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(nx * 100 + nz)
    h = 10.0
    med = (synthetic.random_layers_medium(rng, nz, h, 2) if kind == "layered" else
           synthetic.nodal_perturbed_medium(rng, nz, nx, h, nlayers=2, corr_len=40.0))
    rec = np.unique(np.r_[1, 55, 56, 57, 63, 64, 119, 120, 127, 128, nx - 2])
    rec = rec[rec <= nx - 2].astype(np.int32)
    for nsteps in (1, 7, 8, 9, 48) if solves < 100 else (49,):
        g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), nsteps)
        th = _thetas(g, solves, rng)
        print(f"[gpu case] stream {kind} variant {variant} {nx}x{nz}x{nsteps}, {solves} solves",
              flush=True)
        a, b = _run(variant, g, med, th, rec), _run(base, g, med, th, rec)
        assert np.array_equal(a, b), nsteps
        if nsteps >= 48:
            ref = elastic.forward(g, med, th[0], rec)
            assert np.max(np.abs(ref)) > 0
            check_receivers(a[0], ref, TRACE_TOL, what=f"{kind} {nx}x{nz}")


# absorbing edges: both sides in one strip, a lane's first or second node on the
# right side, sides in different strips, narrow and wide, a last row of its own
@pytest.mark.parametrize("nx,nz,solves", [(8, 8, 2), (64, 9, 3), (65, 17, 3), (128, 25, 3),
                                          (129, 33, 2), (168, 24, 2), (169, 41, 2), (200, 18, 400),
                                          (201, 50, 400), (129, 49, 400)])
def test_absorbing_strips_and_chunks(nx, nz, solves):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(nx * 100 + nz)
    h = 10.0
    med = synthetic.random_layers_medium(rng, nz, h, 2)
    rec = np.unique(np.r_[1, 2, 55, 56, 57, 63, 64, 127, 128, nx - 3, nx - 2])
    rec = rec[rec <= nx - 2].astype(np.int32)
    for nsteps in (1, 5, 6, 7, 48) if solves < 100 else (49,):
        g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), nsteps, bc="absorbing")
        th = _thetas(g, solves, rng)
        print(f"[gpu case] absorbing stream {nx}x{nz}x{nsteps}, {solves} solves", flush=True)
        a, b = _run(28, g, med, th, rec), _run(1, g, med, th, rec)
        assert np.array_equal(a, b), nsteps
        if nsteps >= 48:
            ref = elastic.forward(g, med, th[0], rec)
            assert np.max(np.abs(ref)) > 0
            check_receivers(a[0], ref, TRACE_TOL, what=f"absorbing {nx}x{nz}")
