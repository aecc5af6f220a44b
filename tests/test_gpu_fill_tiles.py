"""GPU outer-product fill and its contraction where their tiles change: the stored product on both sides of
1024 rows (16 x 16 and 32 x 32 tiles a wave), the contraction from one tile a wave to many, source counts
around the K step of 4 and the two register sets of 8.  Oracle: plain products on the host; on the larger
timeslices the Gram-matrix form, whose products are other ones.  FP64 sums of up to 1e10 products
in other orders: 1e-13 relative for S, 1e-12 for the correlators, as for the smaller sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


def fields(dims, n, seed):
    import torch

    X, Y, Z, T = dims
    gen = torch.Generator("cuda").manual_seed(seed)
    return [torch.randn((n, T, Z, Y, X, 4, 3, 2), dtype=torch.float64, device="cuda", generator=gen) for _ in range(4)]


def host(t):
    return t.cpu().numpy().view(np.complex128)[..., 0]


@pytest.mark.parametrize("dims", [(4, 4, 4, 2), (2, 6, 6, 2), (4, 4, 6, 2)])  # 768, 864 and 1152 rows
@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 13])
def test_fill(ctx, orc, dims, n):
    import torch

    print(f"[gpu] fill {dims} n={n}", flush=True)
    src, sol, _, _ = fields(dims, n, n)
    M = 12 * dims[0] * dims[1] * dims[2]
    S = torch.empty((M, M, 2), dtype=torch.float64, device="cuda")
    for dagger in (False, True):
        ctx.fill_propagator_dev(sol, src, n, dims, 1, 0, S, dagger=dagger)
        want = orc.fill_propagator(host(src), host(sol), 1, 0, dagger=dagger)
        assert np.linalg.norm(host(S) - want) / np.linalg.norm(want) < 1e-13, dagger


@pytest.mark.parametrize("dims,n", [((2, 2, 2, 2), 5), ((2, 2, 4, 4), 3), ((4, 4, 6, 2), 9), ((8, 8, 6, 3 * 2), 4)])
def test_contraction(ctx, orc, dims, n):
    print(f"[gpu] fill contraction {dims} n={n}", flush=True)
    src1, sol1, src2, sol2 = fields(dims, n, 20 + n)
    got = ctx.contract_fill_2pt_dev(sol1, src1, sol2, src2, n, dims, 1)
    want = orc.contract_fill(*(host(f) for f in (src1, sol1, src2, sol2)), 1) if dims[0] < 8 else \
        ctx.contract_fill_2pt_dev(sol1, src1, sol2, src2, n, dims, 1, method="gram")
    assert np.linalg.norm(got - want) / np.linalg.norm(want) < 1e-12


@pytest.mark.parametrize("dims", [(16, 16, 16, 2), (24, 24, 24, 2)])
def test_contraction_of_a_large_timeslice_in_little_memory(dims):
    """Partials of one per 64 x 64 entries at the most: 19 MB at 16^3x2 and 215 MB at 24^3x2."""
    from paper_1405_4524_amd import a2a

    n, M = 3, 12 * dims[0] * dims[1] * dims[2]
    print(f"[gpu] fill contraction {dims} n={n}", flush=True)
    src1, sol1, src2, sol2 = fields(dims, n, 31)
    with a2a.Context(0) as c:
        c.set_option("hbm_budget", c.mem_in_use() + 16 * dims[3] * ((M + 63) // 64) ** 2 + (1 << 16))
        got = c.contract_fill_2pt_dev(sol1, src1, sol2, src2, n, dims, 0)
        c.set_option("hbm_budget", 1 << 33)
        want = c.contract_fill_2pt_dev(sol1, src1, sol2, src2, n, dims, 0, method="gram")
    assert np.linalg.norm(got - want) / np.linalg.norm(want) < 1e-12
