"""GPU test: a contraction that fails half way leaves nothing of its own on the stream, so that the caller's arrays
are free when it returns.  The memory-filling test hook queues long fills of the buffers that a call gets
before the one that the budget refuses."""
import pytest

pytestmark = pytest.mark.gpu

DIMS, N = (2, 2, 2, 4), 4096
O = 16 * 4 * N * N  # bytes of one [T][n][n] matrix, 1 GiB


@pytest.mark.parametrize("call", ["pion", "gram", "mixed", "momenta"])
def test_stream_is_idle_after_an_error(call):
    import torch

    from paper_1405_4524_amd import a2a

    print(f"[gpu] failed {call}", flush=True)
    f = torch.zeros((N, 4, 2, 2, 2, 4, 3, 2), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    run, fits = {
        "pion": (lambda c: c.contract_pion_2pt_dev(f, f, N, DIMS), O),
        "gram": (lambda c: c.contract_fill_2pt_dev(f, f, f, f, N, DIMS, 0, method="gram"), O),
        "mixed": (lambda c: c.contract_pipi_mixed_dev(f, 0, f, f, N, f, f, N, DIMS), O),
        "momenta": (lambda c: c.contract_pion_mom_dev(f, f, N, DIMS, [(1, 0, 0)]), O),  # p = -p here
    }[call]
    with a2a.Context(0, stream=stream.cuda_stream) as c:
        c.set_option("poison_memory", 1)
        c.set_option("hbm_budget", c.mem_in_use() + fits + 16 * N)  # O, but not what comes after it
        with pytest.raises(a2a.A2AError):
            run(c)
        assert stream.query()
