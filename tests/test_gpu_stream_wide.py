"""Streaming kernels with strips of 128 columns, two per lane, and long runs.

A call with few solves is cut into strips of 64 columns whatever its width (a
launch of less than half the device's waves takes as long as one of them), so wide
strips need many solves; "last_strip" says which were run.  With 128 - 2 K columns
from strip to strip a grid has an inner strip (neither side in it) from 241
columns on at K = 8 and from 245 at K = 6; up to 128 columns both sides lie in one.
Bitwise equal to the one-step kernel of the medium, and one solve to the oracle."""
import numpy as np
import pytest

import synthetic
from oracle import elastic
from _compare import check_receivers
from test_gpu_stream import TRACE_TOL, _thetas

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(variant, grid, medium, th, rec):
    """Traces and the strip width of the last launch."""
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
        strip = c.get_option("last_strip")
    return out.cpu().numpy(), strip


def _medium(kind, rng, nx, nz, h):
    if kind == "nodal":
        return synthetic.nodal_perturbed_medium(rng, nz, nx, h, nlayers=2, corr_len=40.0)
    return synthetic.random_layers_medium(rng, nz, h, 2)


# one strip with both sides (66: column nx-1 in a lane's second node, 127: in its
# first), two strips (a narrow last one at 129 and 176, wide at 200), three and
# four with one and two inner ones; one chunk of rows or several (nz = 50 at 300)
WIDE = [(66, 20, 600), (127, 50, 600), (128, 20, 600), (129, 20, 1500), (200, 50, 300),
        (241, 20, 600), (245, 20, 600), (260, 50, 600), (361, 50, 300)]


@pytest.mark.parametrize("kind,bc,variant,base", [("layered", "rigid", 23, 0),
                                                  ("nodal", "rigid", 24, 6),
                                                  ("layered", "absorbing", 28, 1)])
@pytest.mark.parametrize("nx,nz,solves", WIDE)
def test_wide_strips(kind, bc, variant, base, nx, nz, solves):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(nx * 100 + nz)
    h = 10.0
    med = _medium(kind, rng, nx, nz, h)
    rec = np.unique(np.r_[1, 2, 63, 64, 111, 112, 115, 116, 119, 120, 127, 128, 129, 231, 232,
                          239, 240, nx // 2, nx - 3, nx - 2])
    rec = rec[rec <= nx - 2].astype(np.int32)
    g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), 49, bc=bc)
    th = _thetas(g, solves, rng)
    print(f"[gpu case] wide strips, {kind} {bc} {nx}x{nz}, {solves} solves", flush=True)
    a, strip = _run(variant, g, med, th, rec)
    assert strip == 128
    b, _ = _run(base, g, med, th, rec)
    assert np.array_equal(a, b)
    ref = elastic.forward(g, med, th[0], rec)
    assert np.max(np.abs(ref)) > 0
    check_receivers(a[0], ref, TRACE_TOL, what=f"{kind} {bc} {nx}x{nz}")


# the kernels of small launches (tile in LDS, 26 and 27) and the streaming ones over
# several hundred steps: every step count mod 8, which covers mod 4 and, from 331
# on, mod 6
@pytest.mark.parametrize("kind,variants,base,nx,nz", [("layered", (23, 26), 0, 201, 83),
                                                      ("nodal", (24, 27), 6, 300, 97)])
def test_long_runs(kind, variants, base, nx, nz):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(41)
    h = 10.0
    med = _medium(kind, rng, nx, nz, h)
    rec = np.array([1, 50, 63, 64, 127, 128, 129, nx - 2], dtype=np.int32)
    for nsteps in range(331, 339):
        g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), nsteps)
        th = synthetic.draw_uniform(np.random.default_rng(43), *synthetic.prior_box(g), 3)
        th[:, 2] = 0.1
        print(f"[gpu case] long runs, {kind} {nx}x{nz}x{nsteps}", flush=True)
        b, _ = _run(base, g, med, th, rec)
        for v in variants:
            a, _ = _run(v, g, med, th, rec)
            assert np.array_equal(a, b), (v, nsteps)
        if nsteps == 337:
            ref = elastic.forward(g, med, th[1], rec)
            assert np.max(np.abs(ref)) > 1.0
            check_receivers(b[1], ref, TRACE_TOL, what=f"{kind} {nx}x{nz}")
