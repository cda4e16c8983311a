"""The tile heights over 40 steps (a race between the halo copies of neighbouring tiles, or between a
tile's wavefronts, would spread), on grids of more row segments than the small-grid kernel takes, so
that every height is a kernel of its own; rows with and without 16-byte copies, ragged in both
directions.  Autotuned batches of small grids, which always run tiles, are compared with the grids
alone, which do not."""
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


def make(shape, precision):
    from paper_1904_10070_amd import TorusGrid
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0)
    g = TorusGrid(p.with_(dt=0.25 * inputs.stable_dt(p)), precision=precision)
    g.set_state(*inputs.random_state(p, seed=3))
    return g


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("shape", [(331, 258), (435, 200), (331, 255)])
def test_heights_agree_over_many_steps(torch_cuda, shape, precision):
    out = []
    for rows in (4, 8, 16):
        g = make(shape, precision)
        g.set_tile_rows(rows)
        g.step(40)
        out.append(g.get_state())
        g.close()
    for f, phi in out[1:]:
        assert torch_cuda.equal(f, out[0][0]) and torch_cuda.equal(phi, out[0][1])


@pytest.mark.parametrize("precision", [64, 32])
def test_small_grid_alone_and_as_tiles_over_many_steps(torch_cuda, precision):
    from paper_1904_10070_amd import TorusBatch
    alone, batched = make((52, 200), precision), make((52, 200), precision)
    batch = TorusBatch([batched])
    alone.step(40)
    batch.step(40)
    torch_cuda.cuda.synchronize()
    for a, b in zip(alone.get_state(), batched.get_state()):
        assert torch_cuda.equal(a, b)
    batch.close()
    alone.close()
    batched.close()
