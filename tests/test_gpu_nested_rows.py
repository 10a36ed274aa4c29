"""The nested estimator's blocks of 16, 32 and 64 outer rows at their edges and
where one gives way to the next, against the FP64 oracle; a row's log ratio does
not depend on how many rows its block takes."""
import numpy as np
import pytest

from oracle import nested

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(go, noise, gi, sigma):
    from paper_1502_07873_amd import Context
    lr = torch.empty(len(go), dtype=torch.float64, device="cuda")
    eig = torch.empty(1, dtype=torch.float64, device="cuda")
    with Context(0, 4 << 30) as c:
        dev = [torch.as_tensor(a, device="cuda") for a in (go, noise, gi)]
        c.nested_mc_eig(dev[0], dev[1], dev[2], sigma, lr, eig)
        torch.cuda.synchronize()
    return lr.cpu().numpy(), float(eig.cpu()[0])


# 300 inner samples are one range, so nouter / 16 waves decide
@pytest.mark.parametrize("nouter,nobs", [(1, 5), (15, 16), (16, 17), (17, 33), (8128, 20),
                                         (8160, 20), (8161, 20), (16320, 20), (16321, 20)])
def test_row_blocks(nouter, nobs):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    rng = np.random.default_rng(nouter + nobs)
    sigma, ninner = 0.02, 300
    A = rng.standard_normal((nobs, 4)) * 0.2
    go = (rng.standard_normal((nouter, 4)) @ A.T).astype(np.float32)
    gi = (rng.standard_normal((ninner, 4)) @ A.T).astype(np.float32)
    noise = rng.standard_normal((nouter, nobs)).astype(np.float32)
    print(f"[gpu case] nested rows {nouter} x {ninner} x {nobs}", flush=True)
    lr, eig = _run(go, noise, gi, sigma)
    pick = np.unique(np.r_[0, nouter // 2, np.arange(max(0, nouter - 40), nouter)])
    ref = nested.log_ratios(go[pick].astype(np.float64), noise[pick].astype(np.float64),
                            gi.astype(np.float64), sigma)
    # FP32 exponentials of 3e-6 relative, as the estimator's other tests allow
    assert np.max(np.abs(lr[pick] - ref)) <= 1e-5
    assert abs(eig - lr.mean()) <= 1e-9 * max(1.0, np.abs(lr).max())
    part, _ = _run(go[pick], noise[pick], gi, sigma)
    assert np.array_equal(part, lr[pick])
