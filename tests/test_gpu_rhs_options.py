"""GPU test: the RHS widths of the per-thread stencils can be set, given back to the library's choice (0, the
default), and are refused otherwise; a source's operator output does not depend on them."""
import numpy as np
import pytest

from paper_1405_4524_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("option,widths", [("rhs_block", (1, 2, 4)), ("rhs_block64", (1, 2))])
def test_default_can_be_restored(option, widths):
    from paper_1405_4524_amd import a2a

    dims = (4, 4, 4, 6)
    eta = inputs.z2_noise(dims, 3, seed=8)
    with a2a.Context(0) as c:
        cl = c.load_clover(c.load_gauge(inputs.gauge_field(dims, 0.3, 2), -1), 1.1)

        def results():
            for x in c.solve_propagators(cl, eta, 0.12, 1.1, prec=a2a.F16_F32)[1]:
                assert x["converged"]
            return [c.dslash_clover(cl, 0.12, eta, op=a2a.OP_SCHUR, prec=p) for p in (a2a.F64, a2a.F32, a2a.F16_F32)]

        want = results()
        for w in widths + (0,):
            c.set_option(option, w)
            assert all(np.array_equal(a, b) for a, b in zip(results(), want)), w
        for bad in (-1, 0.5, 3, 8):
            with pytest.raises(a2a.A2AError):
                c.set_option(option, bad)
        assert all(np.array_equal(a, b) for a, b in zip(results(), want))
