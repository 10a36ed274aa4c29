"""A forced stencil variant runs wherever it can, whatever the options that choose
among the others say: the streaming kernel for absorbing edges (28) under every
steps-per-launch and edge-kernel setting, and what it does not cover (rigid edges,
nodal media) as if it were not forced.  The fields are the same bits throughout."""
import numpy as np
import pytest

import synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(kind, bc, variant, tb, fused):
    from paper_1502_07873_amd import Context
    from paper_1502_07873_amd.query import device_medium, grid_tuple
    rng = np.random.default_rng(17)
    nx, nz, h = 160, 90, 10.0
    med = (synthetic.random_layers_medium(rng, nz, h, 2) if kind == "layered" else
           synthetic.nodal_perturbed_medium(rng, nz, nx, h, nlayers=2, corr_len=40.0))
    g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), 50, bc=bc)
    dm = device_medium(med.kind, med.rho, med.lam, med.mu)
    rec = np.array([1, 40, 80, 158], dtype=np.int32)
    th = np.array([[400.0, 60.0, 0.02, 15.0, 1e13, 2e13, 1e13],
                   [1520.0, 75.0, 0.03, 12.0, 3e13, 1e13, 1e13]])
    out = torch.full((2, g.nsteps + 1, len(rec), 2), float("nan"), device="cuda")
    with Context(0, 1 << 30) as c:
        c.set_option("stencil_variant", variant)
        c.set_option("temporal_blocking", tb)
        c.set_option("fused_edges", fused)
        c.set_option("resident", 0)
        c.forward_solve_batch([grid_tuple(g)] * 2, [dm] * 2, th, [rec] * 2, list(out.unbind(0)))
        torch.cuda.synchronize()
        return out.cpu().numpy(), c.get_option("last_variant")


@pytest.mark.parametrize("tb,fused", [(0, 1), (2, 1), (3, 1), (4, 1), (4, 0), (2, 0)])
def test_forced_absorbing_stream(tb, fused):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"[gpu case] forced 28, temporal_blocking {tb}, fused_edges {fused}", flush=True)
    ref, v = _run("layered", "absorbing", 1, 0, 1)
    assert v == 1 and np.max(np.abs(ref)) > 0
    got, v = _run("layered", "absorbing", 28, tb, fused)
    assert v == 28
    assert np.array_equal(got, ref)
    for kind, bc in (("layered", "rigid"), ("nodal", "absorbing"), ("nodal", "rigid")):
        (a, va), (b, vb) = (_run(kind, bc, 28, tb, fused), _run(kind, bc, -1, tb, fused))
        assert va != 28 and np.array_equal(a, b), (kind, bc)
