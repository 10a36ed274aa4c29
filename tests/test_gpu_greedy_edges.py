"""The greedy search at the edges of its launch shapes: sample counts around a
wavefront, 256 and the 1024 of a block (one launch per step up to there, three
above), few candidates (no room for second copies of the sums: three launches),
room or none for the packed Hessians, subsets of the parameters, more steps than candidates."""
import numpy as np
import pytest
import torch

from oracle import laplace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,C,act", [
    (1, 3, 127), (1, 12, 127), (2, 1, 127), (2, 40, 127), (63, 9, 127), (64, 10, 5), (65, 5, 127),
    (256, 9, 2), (257, 300, 38), (1023, 11, 119), (1024, 12, 127), (1025, 12, 127),
    (1300, 2, 63)])
def test_greedy_launch_shapes(S, C, act):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1502_07873_amd import Context, make_prior
    rng = np.random.default_rng(S * 1000 + C)
    G = rng.standard_normal((S, C, 7, 12)) * (0.5 + rng.random((1, C, 1, 1)))
    scale = 10.0 ** np.array([-2, -2, 2, 1, -6, -6, -6])
    H = (G @ G.transpose(0, 1, 3, 2) + np.eye(7)) * np.outer(scale, scale)
    if C > 4:
        H[:, C - 1] = H[:, 1]          # a tie at every step
        H[S // 2, 3] = -H[S // 2, 3]   # not positive definite: NaN until others outweigh it
    w = rng.uniform(-0.2, 1.5, S)
    w /= w.sum()
    ix = [j for j in range(7) if (act >> j) & 1]
    lo, hi = -np.ones(7), np.linspace(1.0, 2.0, 7)
    K = C + 1 if C <= 3 else 6
    print(f"[gpu case] greedy S={S} C={C} act={act} K={K}", flush=True)
    Hd = torch.as_tensor(H, device="cuda")
    runs = []
    # with and without room for the packed Hessians
    for budget in (1 << 30, 8 * (S * (C + 49 + 8) + C) + 2048):
        order = torch.full((K,), -7, dtype=torch.int32, device="cuda")
        curve = torch.full((K,), -7.0, dtype=torch.float64, device="cuda")
        with Context(0, budget) as ctx:
            ctx.design_greedy(Hd, make_prior(lo, hi, active=ix), w, K, order, curve,
                              theta=np.zeros((S, 7)))
            torch.cuda.synchronize()
        runs.append((order.cpu().numpy(), curve.cpu().numpy()))
    order, curve = runs[0]
    assert np.array_equal(order, runs[1][0])
    assert np.array_equal(curve, runs[1][1], equal_nan=True)
    prior = laplace.uniform_prior(lo[ix], hi[ix])
    Hs = H[:, :, ix][:, :, :, ix]
    base, chosen = np.zeros((S, len(ix), len(ix))), []
    for k in range(K):
        vals = laplace.greedy_step_values(Hs, base, np.zeros((S, 7)), w, prior)
        vals[chosen] = np.nan
        if np.isnan(vals).all():
            assert order[k] == -1 and np.isnan(curve[k])
            continue
        c = int(order[k])
        # FP64 on scaled Hessians of condition below 1e4, sums of at most 1300
        # terms: some 1e-12
        tol = 1e-9 * max(1.0, np.nanmax(np.abs(vals)))
        assert vals[c] >= np.nanmax(vals) - tol and abs(curve[k] - vals[c]) <= tol, (k, c)
        assert C <= 4 or c != C - 1 or 1 in chosen
        chosen.append(c)
        base = base + Hs[:, c]
