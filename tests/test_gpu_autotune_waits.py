"""tlb_autotune returns when the grid's stream is idle, whether or not it had heights to choose
from: grids with tiles, small grids without, and the variants of one height."""
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, flags", [((24, 80), 0), ((24, 80), 8), ((24, 80), 32),
                                          ((331, 258), 0)])
def test_autotune_waits_for_the_stream(torch_cuda, shape, flags):
    from paper_1904_10070_amd import TorusGrid
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0,
                                  flags=flags)
    g = TorusGrid(p.with_(dt=0.1 * inputs.stable_dt(p)), precision=32)
    g.set_state(*inputs.random_state(p, seed=3))
    x = torch_cuda.ones(4096, 4096, device="cuda")
    y = torch_cuda.empty_like(x)
    torch_cuda.mm(x, x, out=y)
    torch_cuda.cuda.synchronize()
    with torch_cuda.cuda.stream(g.stream):
        for _ in range(60):
            torch_cuda.mm(x, x, out=y)
    assert not g.stream.query()  # tens of milliseconds of work
    assert g.autotune() in (4, 8, 16)
    assert g.stream.query()
    g.close()
