"""GPU test of which inner layout the sources past the last whole tile of 16 take: fewer than 12 stay per
slot, with the per-thread stencil's FP32 intermediates and FP64 sums, whatever the lattice; 12 and more fill
a tile of their own.  Each layout's operator gives a source the same bits whatever it shares a call with, so
the outputs name the layout."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


# 512, 8192 and 147456 sites: the blocks of the matrix-core stencil come in 16, 16 and 4 parts
@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 8, 8, 16), (16, 16, 16, 36)])
@pytest.mark.parametrize("prec", [2, 3])
def test_layout_of_the_remainder(ctx, dims, prec):
    import torch

    from paper_1405_4524_amd import a2a, inputs

    X, Y, Z, T = dims
    print(f"[gpu] remainder {dims} prec {prec}", flush=True)
    U = torch.from_numpy(inputs.gauge_field(dims, 0.3, 7)).cuda()
    g = ctx.load_gauge_dev(U, dims, -1)
    c = ctx.load_clover(g, 1.2)
    psi = torch.empty((32, T, Z, Y, X, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.z2_noise_dev(dims, 5, 0, 32, psi)

    def schur(v):
        out = torch.empty_like(v)
        ctx.dslash_clover_dev(c, 0.125, v, out, v.shape[0], op=a2a.OP_SCHUR, prec=prec)
        return out

    ctx.set_option("interleave", 0)
    slot = schur(psi)
    ctx.set_option("interleave", 1)
    tile = schur(psi)
    assert not torch.equal(slot[16:17], tile[16:17])  # the two layouts round differently
    for r in (1, 4, 8, 9, 11, 12, 15):
        got = schur(psi[:16 + r].contiguous())
        assert torch.equal(got[:16], tile[:16]), r
        assert torch.equal(got[16:], (slot if r < 12 else tile)[16:16 + r]), r
    ctx.unload(g)


@pytest.mark.parametrize("dims,n", [((8, 8, 8, 16), 20), ((16, 16, 16, 36), 22)])
def test_solve_with_both_layouts(ctx, dims, n):
    """Whole tiles and per-slot sources in one solve: every source meets the tolerance, by the FP64
    residual of the operator applied to the returned solution."""
    import torch

    from paper_1405_4524_amd import a2a, inputs

    X, Y, Z, T = dims
    print(f"[gpu] solve {dims} n {n}", flush=True)
    g = ctx.load_gauge_dev(torch.from_numpy(inputs.gauge_field(dims, 0.3, 9)).cuda(), dims, -1)
    c = ctx.load_clover(g, 1.2)
    eta = torch.empty((n, T, Z, Y, X, 4, 3, 2), dtype=torch.float64, device="cuda")
    ctx.z2_noise_dev(dims, 6, 0, n, eta)
    sol, back = torch.empty_like(eta), torch.empty_like(eta)
    info, rc = ctx.solve_propagators_dev(c, eta, sol, n, 0.125, 1.2, tol=1e-10, prec=a2a.F16_F32)
    assert rc == 0
    ctx.dslash_clover_dev(c, 0.125, sol, back, n, op=a2a.OP_FULL_D, prec=a2a.F64)
    for i in range(n):
        res = ((back[i] - eta[i]).norm() / eta[i].norm()).item()
        assert res <= 1.01e-10 and abs(res - info[i]["true_rel_residual"]) <= 1e-12, (i, res, info[i])
    ctx.unload(g)
