"""Hessians near the ends of the FP64 range: the scaled factorisation does not
depend on the parameters' units, down to subnormal entries.  The matrices are
small integers times powers of two, so scaling them is exact and the log-det of
the scaled one is that of the integers plus the scales' logarithms."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# Cholesky of a 7 x 7 matrix of condition below 1e3 in FP64: below 1e-12; the
# scales add at most 14 * 533 log 2 = 5200 nats, rounded a few times: 1e-11
TOL = 1e-10
EXPONENTS = {"unit": [0] * 7, "low": [-500] * 7, "product just normal": [-511] * 7,
             "product subnormal": [-515] * 7, "entries subnormal": [-532] * 7,
             "lowest and unit": [0, -533, 0, -533, 0, 0, -533],
             "high": [500] * 7, "high and lowest": [500, -533, 0, 500, -533, -480, -481]}


def _matrices(rng, shape):
    G = rng.integers(-3, 4, shape + (7, 9)).astype(np.float64)
    return G @ np.swapaxes(G, -1, -2) + 7 * np.eye(7)


@pytest.mark.parametrize("name", list(EXPONENTS))
@pytest.mark.parametrize("act", [range(7), (1, 3, 4)])
def test_logdet_over_the_range(name, act):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1502_07873_amd import Context, make_prior
    rng = np.random.default_rng(11)
    act = list(act)
    n, S, C, K = len(act), 70, 12, 4
    e = np.array(EXPONENTS[name])
    unit = np.ldexp(1.0, e)
    A = _matrices(rng, (S, C))
    assert np.array_equal(A * unit[:, None] / unit[:, None], A)
    H = (A * unit[:, None]) * unit
    scale_log = 2 * np.log(2.0) * e[act].sum()
    lo, hi = -np.ones(7), np.linspace(1.0, 2.0, 7)
    lp = -np.log(hi - lo)[act].sum()

    def dkl(M):
        ld = np.linalg.slogdet(M[..., act, :][..., act])[1] + scale_log
        return -0.5 * (n * np.log(2 * np.pi) - ld) - 0.5 * n - lp

    print(f"[gpu case] log-det over the range: {name}, {n} parameters", flush=True)
    pr = make_prior(lo, hi, active=act)
    w = np.full(S, 1.0 / S)
    Hd = torch.as_tensor(H, device="cuda")
    mask = np.zeros((2, C), dtype=np.uint8)
    mask[0, [1, 4]] = mask[1, [0, 2, 5, 7]] = 1
    f64 = dict(dtype=torch.float64, device="cuda")
    got, logdet, eig, de = (torch.empty(k, **f64) for k in (S, S, 1, 2))
    st = torch.empty(S, dtype=torch.int32, device="cuda")
    order = torch.empty(K, dtype=torch.int32, device="cuda")
    curve = torch.empty(K, **f64)
    with Context(0, 1 << 30) as ctx:
        ctx.laplace_eig(Hd[:, 0].contiguous(), pr, w, got, eig, logdet=logdet, status=st)
        ctx.design_eval(Hd, torch.as_tensor(mask, device="cuda"), pr, w, de)
        ctx.design_greedy(Hd, pr, w, K, order, curve)
        torch.cuda.synchronize()
    assert int(st.abs().sum()) == 0
    assert np.max(np.abs(got.cpu().numpy() - dkl(A[:, 0]))) <= TOL
    for d in range(2):
        assert abs(float(de[d]) - w @ dkl(A[:, mask[d] > 0].sum(1))) <= TOL
    base = np.zeros((S, 7, 7))
    for k, c in enumerate(order.cpu().numpy()):
        vals = np.array([w @ dkl(base + A[:, q]) for q in range(C)])
        assert abs(float(curve[k]) - vals[c]) <= TOL
        base += A[:, c]
