"""GPU momentum-projected pions of spin-colour grouped sources that are not zero outside their own component
(smeared after dilution, say): the sums run over all of a source, against the oracle's.  One entry at
either end of the sources, or everything; a NaN outside the component reaches the result.  FP64 sums of at
most 2e5 products: 1e-12 relative, as for diluted sources."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MOMS = [(0, 0, 0), (1, 0, 1)]


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def sources(orc, dims, nv, scheme, seed):
    X, Y, Z, T = dims
    rng = np.random.default_rng(seed)
    v = rng.standard_normal((2, nv, T, Z, Y, X, 4, 3))
    src = orc.dilute(v[0] + 1j * v[1], scheme)
    w = rng.standard_normal((2,) + src.shape)
    return src, w[0] + 1j * w[1]


def spoil(src, scheme, where, value):
    """Entries outside the component (source k: component k % 12), of time-diluted pieces on their timeslice."""
    n, T = src.shape[:2]
    if where == "all":
        mask = np.ones(src.shape, bool)
        for k in range(n):
            if scheme == 3:
                mask[k] = False
                mask[k, k // 12 % T] = True
            mask[k, ..., k % 12 // 3, k % 3] = False
        src[mask] = value * np.random.default_rng(3).standard_normal(mask.sum())
    elif where == "first":
        src[0, 0, 0, 0, 0, 0, 1] = value
    else:
        src[-1, -1, -1, -1, -1, 3, 1] = value


@pytest.mark.parametrize("scheme,dims,nv", [(2, (4, 2, 6, 4), 2), (2, (2, 2, 2, 18), 3), (3, (6, 2, 2, 4), 3)])
@pytest.mark.parametrize("where", ["first", "last", "all"])
@pytest.mark.parametrize("mode", [0, 3])
def test_sources_with_other_components(ctx, orc, scheme, dims, nv, where, mode):
    print(f"[gpu] support scheme {scheme} {dims} {where}", flush=True)
    src, sol = sources(orc, dims, nv, scheme, 5 + nv)
    n = src.shape[0]
    spoil(src, scheme, where, 0.7)
    got = ctx.contract_pion_mom_dev(dev(src), dev(sol), n, dims, MOMS, scheme=scheme, mode=mode)
    for m, p in enumerate(MOMS):
        want = orc.pion_mom(src, sol, p, n // nv, mode)
        assert np.linalg.norm(got[m] - want) / np.linalg.norm(want) <= 1e-12, m


@pytest.mark.parametrize("scheme,dims", [(2, (2, 2, 2, 4)), (3, (2, 4, 2, 2))])
@pytest.mark.parametrize("where", ["first", "last"])
def test_nan_outside_the_component(ctx, orc, scheme, dims, where):
    print(f"[gpu] support nan scheme {scheme} {where}", flush=True)
    src, sol = sources(orc, dims, 2, scheme, 4)
    spoil(src, scheme, where, np.nan)
    got = ctx.contract_pion_mom_dev(dev(src), dev(sol), src.shape[0], dims, MOMS, scheme=scheme)
    assert np.isnan(got).all()
