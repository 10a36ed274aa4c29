"""The launch statistics: eig_ctx_stencil_stats counts launches in units of at most
four steps, the option "stencil_launches" as they are made, and the batch calls
and the serving engine count the same work alike."""
import numpy as np
import pytest

import synthetic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

STEPS = {23: 8, 24: 6, 26: 4, 27: 4, 11: 2, 6: 1}


def _case(kind, nsteps, n):
    from paper_1502_07873_amd.query import device_medium, grid_tuple
    rng = np.random.default_rng(31)
    nx, nz, h = 150, 90, 10.0
    med = (synthetic.random_layers_medium(rng, nz, h, 2) if kind == "layered" else
           synthetic.nodal_perturbed_medium(rng, nz, nx, h, nlayers=2, corr_len=40.0))
    g = synthetic.Grid(nx, nz, h, synthetic.cfl_dt(h, med.vp_max()), nsteps)
    lo, hi = synthetic.prior_box(g)
    th = synthetic.draw_uniform(rng, lo, hi, n)
    return (grid_tuple(g), device_medium(med.kind, med.rho, med.lam, med.mu), th,
            np.array([20, 75, 130], dtype=np.int32), lo, hi)


@pytest.mark.parametrize("variant", list(STEPS))
@pytest.mark.parametrize("nsteps", [6, 61])
def test_batch_and_engine_count_alike(variant, nsteps):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1502_07873_amd import Context, make_prior
    from paper_1502_07873_amd.eigseis import Server
    n = 3
    kind = "nodal" if variant in (24, 27, 6) else "layered"
    grid, med, th, rec, lo, hi = _case(kind, nsteps, n)
    k = STEPS[variant]
    launches, units = -(-nsteps // k), -(-nsteps // min(k, 4))
    f64 = dict(dtype=torch.float64, device="cuda")
    print(f"[gpu case] launch counts of variant {variant}, {nsteps} steps", flush=True)
    with Context(0, 1 << 30) as c:
        c.set_option("stencil_variant", variant)
        c.set_option("wave_cache_bytes", 0)
        c.set_option("resident", 0)
        H = torch.empty((n, 7, 7), **f64)
        c.stencil_stats(reset=True)
        assert c.get_option("stencil_launches") == 0
        for run in range(3):   # the third replays a captured graph
            c.jacobian_fd([grid] * n, [med] * n, th, [rec] * n, 1.0, H)
        torch.cuda.synchronize()
        assert c.get_option("last_variant") == variant
        assert c.get_option("stencil_launches") == 3 * launches
        st = c.stencil_stats(reset=True)
        assert st["launches"] == 3 * units
        assert st["updates"] == 3 * 15 * n * grid[0] * grid[1] * nsteps
        assert c.get_option("stencil_launches") == 0
        H2, dkl, eig = torch.empty((n, 7, 7), **f64), torch.empty(n, **f64), torch.empty(1, **f64)
        srv = Server(c, 1 << 30, 16)
        q = srv.submit(grid, med, th, rec, make_prior(lo, hi), np.full(n, 1 / n), H2, dkl, eig, 1.0)
        for _ in range(40):
            srv.step(5)
            torch.cuda.synchronize()
            if srv.poll(q):
                break
        assert srv.pending() == (0, 0)
        srv.close()
        assert c.get_option("stencil_launches") == launches
        assert c.stencil_stats(reset=True)["launches"] == units
        assert np.array_equal(H.cpu().numpy(), H2.cpu().numpy())
