"""GPU unbiased pion correlators at the ends of the FP64 range: the pairs that the estimator drops (a source with
itself, pieces of one noise vector) may overflow without a trace in the result.  One source and its solution
are scaled so that its own product is infinite and every product with another source is finite; the
oracle's operators at unit scale, weighted by the powers of two, are exact but for rounding (1e-12)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UP, DOWN = 2.0**520, 2.0**-260  # |O_aa| ~ 2^1040 overflows, O_ab O_ba ~ 2^520


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def fields(dims, n, seed):
    X, Y, Z, T = dims
    v = np.random.default_rng(seed).standard_normal((2, n, T, Z, Y, X, 4, 3, 2))
    return v[0, ..., 0] + 1j * v[0, ..., 1], v[1, ..., 0] + 1j * v[1, ..., 1]


def correlate(Op, Om, scale, keep):
    """sum_t0 sum_ab keep s_a^2 s_b^2 Op[t0 + dt]_ab Om[t0]_ba in units of UP^2 DOWN^2."""
    with np.errstate(over="ignore"):
        w = np.where(keep, np.multiply.outer(scale / UP, scale / DOWN) ** 2, 0.0)
    return np.array([np.sum(w * np.roll(Op, -dt, 0) * Om.transpose(0, 2, 1)) for dt in range(Op.shape[0])])


@pytest.mark.parametrize("dims,n", [((2, 2, 2, 4), 5), ((2, 2, 2, 16), 9), ((2, 2, 2, 18), 6), ((4, 2, 2, 66), 3)])
@pytest.mark.parametrize("big", [0, -1])
def test_infinite_diagonal(ctx, orc, dims, n, big):
    print(f"[gpu] pion range {dims} n {n}", flush=True)
    eta, X = fields(dims, n, 3 + n)
    scale = np.full(n, DOWN)
    scale[big] = UP
    O = orc.stochastic_operators(eta, X)
    s = scale.reshape(-1, 1, 1, 1, 1, 1, 1)
    got, Og = ctx.contract_pion_2pt(eta * s, X * s)
    assert not np.isfinite(Og[:, big, big]).any()
    want = correlate(O, O, scale, ~np.eye(n, dtype=bool)) / (dims[3] * n * (n - 1))
    assert np.linalg.norm(got / (UP * DOWN) ** 2 - want) / np.linalg.norm(want) <= 1e-12


@pytest.mark.parametrize("dims,nv,scheme", [((2, 4, 2, 4), 3, 0), ((2, 2, 2, 18), 2, 2)])
def test_infinite_pairs_of_one_noise_vector(ctx, orc, dims, nv, scheme):
    print(f"[gpu] momentum range {dims} scheme {scheme}", flush=True)
    src = orc.dilute(fields(dims, nv, 8)[0], scheme)
    n = src.shape[0]
    sol = fields(dims, n, 9)[1]
    vector = np.arange(n) // (n // nv)
    scale = np.where(vector == 1, UP, DOWN)
    s = scale.reshape(-1, 1, 1, 1, 1, 1, 1)
    p = (1, 0, 1)
    got = ctx.contract_pion_mom_dev(dev(src * s), dev(sol * s), n, dims, [p], scheme=scheme)[0]
    Op, Om = orc.stochastic_operators_mom(src, sol, p), orc.stochastic_operators_mom(src, sol, [-q for q in p])
    want = correlate(Op, Om, scale, vector[:, None] != vector[None, :]) / (dims[3] * nv * (nv - 1))
    assert np.linalg.norm(got / (UP * DOWN) ** 2 - want) / np.linalg.norm(want) <= 1e-12
