"""GPU contractions at the sizes where their tiles, chunks and batches end, against the oracle: source
counts around the 16-wide matrix tiles and the 64-wide row blocks, time extents around the 16 and 64
separations of a correlator block and past one, more momenta than a batch holds (repeated and aliased
ones among them), and the largest and smallest pi-pi groups.  FP64 sums of at most 2e5 products: 1e-12
relative is three orders above their rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RTOL = 1e-12


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def fields(dims, n, seed):
    X, Y, Z, T = dims
    rng = np.random.default_rng(seed)
    v = rng.standard_normal((2, n, T, Z, Y, X, 4, 3, 2))
    return v[0, ..., 0] + 1j * v[0, ..., 1], v[1, ..., 0] + 1j * v[1, ..., 1]


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


@pytest.fixture(scope="module")
def orc():
    import oracle

    return oracle


@pytest.mark.parametrize("dims,n", [((2, 2, 2, 2), 1), ((4, 2, 2, 4), 16), ((2, 2, 2, 16), 17), ((2, 2, 2, 18), 33),
                                    ((2, 2, 2, 64), 5), ((2, 2, 2, 66), 3), ((2, 2, 2, 130), 2), ((4, 2, 6, 4), 48),
                                    ((4, 4, 2, 4), 49), ((2, 2, 2, 4), 64), ((2, 2, 2, 4), 65), ((2, 2, 2, 2), 130)])
def test_pion_and_operators(ctx, orc, dims, n):
    from paper_1405_4524_amd import a2a

    print(f"[gpu] pion {dims} n {n}", flush=True)
    eta, X = fields(dims, n, n)
    corr, O = ctx.contract_pion_2pt(eta, X, mode=a2a.PION_ALL_PAIRS)
    want = orc.stochastic_operators(eta, X)
    assert rel(O, want) <= RTOL
    T = dims[3]
    full = np.array([np.sum(np.roll(want, -dt, 0) * want.transpose(0, 2, 1)) for dt in range(T)]) / (T * n * n)
    assert rel(corr, full) <= RTOL
    if n > 1:
        corr, _ = ctx.contract_pion_2pt(eta, X)
        assert rel(corr, orc.pion_from_O(want)) <= RTOL


@pytest.mark.parametrize("dims,n", [((2, 2, 2, 2), 4), ((2, 2, 4, 18), 12), ((2, 2, 2, 34), 20), ((2, 2, 2, 6), 128)])
def test_pipi(ctx, orc, dims, n):
    print(f"[gpu] pipi {dims} n {n}", flush=True)
    eta, X = fields(dims, n, 7 + n)
    d, v, p = ctx.contract_pipi_2pt(eta, X, want_pion=True)
    dw, vw = orc.contract_pipi(eta, X)
    assert rel(d, dw) <= RTOL and rel(v, vw) <= RTOL
    assert rel(p, orc.pion_from_O(orc.stochastic_operators(eta, X))) <= RTOL


@pytest.mark.parametrize("scheme,dims,nv", [(0, (4, 2, 6, 4), 5), (0, (2, 4, 2, 18), 19), (1, (4, 2, 2, 6), 3),
                                            (1, (2, 6, 2, 4), 17), (2, (4, 2, 6, 4), 2), (2, (2, 2, 2, 18), 3),
                                            (3, (6, 2, 2, 4), 3), (3, (2, 2, 4, 2), 9)])
@pytest.mark.parametrize("nmom", [1, 18])
def test_momenta(ctx, orc, scheme, dims, nv, nmom):
    import torch

    print(f"[gpu] momenta scheme {scheme} {dims} nv {nv} nmom {nmom}", flush=True)
    noise, _ = fields(dims, nv, 11 + nv)
    src = orc.dilute(noise, scheme)
    n = src.shape[0]
    _, sol = fields(dims, n, 13 + nv)
    moms = [(1, 0, 1)] if nmom == 1 else [(a, b, c) for a in (0, 1, -1) for b in (0, 1, 5) for c in (0, -3)]
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()  # noqa: E731
    got = ctx.contract_pion_mom_dev(dev(src), dev(sol), n, dims, moms, scheme=scheme)
    for m in range(0, len(moms), 5):
        assert rel(got[m], orc.pion_mom(src, sol, moms[m], n // nv)) <= RTOL, moms[m]
