"""GPU test: the reduction buffer holds what the slots at work can store: one partial (32 bytes) per 256 sites for
per-slot sources, for 64 slots at the least, whatever parts the matrix-core stencil would cut the sites in."""
import pytest

from paper_1405_4524_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,parts", [(0, 16, 1), (1, 16, 1), (2, 4, 1), (3, 11, 1), (2, 16, 16)])
def test_partials_of_the_layout(prec, n, parts):
    from paper_1405_4524_amd import a2a

    dims = (8, 8, 8, 16)  # 4096 sites a parity: 16 blocks of 256
    with a2a.Context(0) as c:
        before = c.mem_in_use()
        g = c.load_gauge(inputs.gauge_field(dims, 0.3, 5), -1)
        cl = c.load_clover(g, 1.2)
        c.dslash_clover(cl, 0.12, inputs.z2_noise(dims, n, seed=3), op=a2a.OP_SCHUR, prec=prec)
        c.unload(g)
        assert c.mem_in_use() - before == 64 * 16 * parts * 32
