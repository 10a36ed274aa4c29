"""Resident depth-only grids at the edges of their kernels' classes against the
tiled kernels, bit for bit: one and two columns per lane, the side columns in a
lane's first or second node, fewer rows than waves, full and uneven bands, the
most rows a wave keeps in registers and one more, grids too wide for one strip;
forward solves (all of a kind in one launch, too) and dual solves."""
import numpy as np
import pytest

import synthetic
from oracle import elastic
from _compare import check_receivers
from test_gpu_resident import TRACE_TOL, _ctx, _dev_medium, _forward, _say
from test_gpu_stream import _thetas

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GRIDS = {
    "rigid": [(8, 8), (20, 16), (66, 17), (66, 18), (64, 97), (65, 98), (40, 161), (40, 162),
              (67, 40), (130, 33), (100, 97), (90, 98), (131, 20), (126, 66)],
    "absorbing": [(8, 8), (64, 16), (64, 97), (63, 98), (40, 161), (40, 162), (65, 18), (66, 33),
                  (128, 34), (127, 66), (101, 76), (90, 98), (129, 20)],
}


def _spec(bc, nx, nz, rng):
    h = 10.0
    med = synthetic.random_layers_medium(rng, nz, h, 2)
    g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), int(rng.integers(120, 150)), bc=bc)
    rec = np.unique(np.r_[1, 2, nx // 2, 63, 64, 65, nx - 3, nx - 2])
    return g, med, rec[rec <= nx - 2].astype(np.int32)


@pytest.mark.parametrize("bc", ["rigid", "absorbing"])
def test_band_shapes(bc):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(53)
    spec = [_spec(bc, nx, nz, rng) for nx, nz in GRIDS[bc]]
    th = np.concatenate([_thetas(g, 3, rng)[1:2] for g, _, _ in spec])
    th[:, 1] = np.minimum(th[:, 1], 12 * 10.0)   # near enough to the surface to reach it
    outs = {}
    for res in (True, False):
        c = _ctx(res)
        _say(f"resident bands, {bc}: {len(spec)} grids in one call, resident={res}")
        outs[res] = _forward(c, spec, th)
        if res:  # and each by itself, in the kernel of its own class
            for s in range(len(spec)):
                _say(f"resident bands, {bc}: {GRIDS[bc][s]}")
                one = _forward(c, spec[s:s + 1], th[s:s + 1])
                assert np.array_equal(one[0], outs[True][s]), GRIDS[bc][s]
        c.close()
    for s, (g, m, rec) in enumerate(spec):
        assert np.array_equal(outs[True][s], outs[False][s]), GRIDS[bc][s]
        ref = elastic.forward(g, m, th[s], rec)
        assert np.max(np.abs(ref)) > 0
        check_receivers(outs[True][s], ref, TRACE_TOL, what=f"{bc} {GRIDS[bc][s]}")


@pytest.mark.parametrize("nx,nz", [(48, 44), (66, 60), (90, 41), (91, 40), (140, 40)])
def test_dual_solves(nx, nz):
    # receiver forces injected at the surface, the source window recorded
    from paper_1502_07873_amd import make_prior
    from paper_1502_07873_amd.query import grid_tuple
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(nx)
    h = 16.0
    med = synthetic.random_layers_medium(rng, nz, h, 2)
    g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), 200)
    lo, hi = synthetic.prior_box(g)
    th = synthetic.draw_uniform(rng, lo, hi, 2)
    rec = synthetic.equispaced_receivers(nx, 7)
    noise = rng.standard_normal((2, g.nsteps + 1, len(rec), 2)).astype(np.float32)
    dm = _dev_medium(med)
    _say(f"resident dual solves {nx}x{nz}")
    got = {}
    for res in (True, False):
        c = _ctx(res)
        H1 = torch.empty((2, 7, 7), dtype=torch.float64, device="cuda")
        H2 = torch.empty_like(H1)
        val = torch.empty(2, dtype=torch.float64, device="cuda")
        eig = torch.empty(1, dtype=torch.float64, device="cuda")
        st = torch.empty(2, dtype=torch.int32, device="cuda")
        hat = c.theorem3_eig([grid_tuple(g)] * 2, [dm] * 2, th, [rec] * 2,
                             [torch.as_tensor(n, device="cuda") for n in noise], 0.05,
                             make_prior(lo, hi), np.full(2, 0.5), H1, H2, val, eig, st, iters=2)
        torch.cuda.synchronize()
        got[res] = (np.asarray(hat), H1.cpu().numpy(), H2.cpu().numpy(), val.cpu().numpy())
        c.close()
    assert np.max(np.abs(got[True][2])) > 0
    for a, b in zip(got[True], got[False]):
        assert np.array_equal(a, b, equal_nan=True)
