"""GPU pion correlators of more sources than the pair sum has blocks for, and of as many as one block per patch
could not be launched for.  sum_ab O(t1)_ab O(t0)_ba = tr[(X0 E1^dag) (g5 X1 E0^dag g5)] needs matrices of the
96 components of a 2^3 timeslice alone.  Sums of up to 2e9 products of random signs, in FP64 over partial
sums: 1e-12 relative is three orders above their rounding."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1405_4524_amd import a2a

    with a2a.Context(0) as c:
        yield c


def expected(src, sol, T):
    import torch

    n = src.shape[0]
    E, X = (torch.view_as_complex(v).reshape(n, T, -1).permute(1, 2, 0).contiguous() for v in (src, sol))  # [T][K][n]
    g5 = torch.tensor([1.0] * 6 + [-1.0] * 6, dtype=torch.float64, device="cuda").repeat(X.shape[1] // 12)
    XE = [[X[a] @ E[b].conj().T.contiguous() for b in range(T)] for a in range(T)]
    diag = (E.conj() * g5[None, :, None] * X).sum(1)  # [T][n]
    out = []
    for dt in range(T):
        s = 0
        for t0 in range(T):
            t1 = (t0 + dt) % T
            full = ((XE[t0][t1] * g5[:, None]) * (g5[:, None] * XE[t1][t0]).T).sum()
            s = s + full - (diag[t1] * diag[t0]).sum()
        out.append(s / (T * n * (n - 1.0)))
    return torch.stack(out).cpu().numpy()


@pytest.mark.parametrize("T,n", [(2, 2046), (2, 2056), (18, 1024), (18, 1031), (2, 32776)])
def test_many_sources(ctx, T, n):
    import numpy as np
    import torch

    dims = (2, 2, 2, T)
    print(f"[gpu] pion {dims} n {n}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    src, sol = (torch.randn((n, T, 2, 2, 2, 4, 3, 2), dtype=torch.float64, device="cuda", generator=gen) for _ in range(2))
    got, _ = ctx.contract_pion_2pt_dev(src, sol, n, dims)
    want = expected(src, sol, T)
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 1e-12
    ctx.trim()
