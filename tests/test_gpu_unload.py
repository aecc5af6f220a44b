"""GPU test: a clover field's device memory, the matrix-core stencil's blocks of its operators included,
is returned when the field or its gauge field is unloaded."""
import pytest

from paper_1405_4524_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_unload_returns_the_memory(prec):
    from paper_1405_4524_amd import a2a

    dims = (4, 4, 4, 8)
    c = a2a.Context(0)
    try:
        U = inputs.gauge_field(dims, 0.3, 5)
        psi = inputs.z2_noise(dims, 16, seed=3)
        seen = []
        for unload_clover in (True, True, False):  # the first round also allocates the context's own buffers
            g = c.load_gauge(U, -1)
            cl = c.load_clover(g, 1.2)
            c.dslash_clover(cl, 0.12, psi, op=a2a.OP_SCHUR, prec=prec)
            if unload_clover:
                c.unload(cl)
            c.unload(g)
            seen.append(c.mem_in_use())
        assert seen[1] == seen[0] and seen[2] == seen[0], seen
    finally:
        c.finalize()
