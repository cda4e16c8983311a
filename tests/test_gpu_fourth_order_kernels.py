"""The fourth-order Cahn-Hilliard variant on the small-grid and the tile kernel, bit for bit.  It is
not available in batches, so the two are compared through a plane (flat limit) whose state repeats
along phi: twice the columns and twice R keep the spacing, and every coefficient changes by a power of
two.  The single plane is below the small-grid kernel's limit, the double one above it."""
import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


def run(p, precision, state, density, steps):
    from paper_1904_10070_amd import TorusGrid
    g = TorusGrid(p, precision=precision)
    phi, n, ut, up = state
    g.set_state(phi, density * n, ut, up)
    g.step(steps)
    out = g.get_state()
    g.close()
    return out


# 16-byte copies of the tile kernel and, with 382 or 255 columns, 4-byte ones
@pytest.mark.parametrize("precision, density, shape", [(64, 1.0, (320, 128)), (64, 1.0, (160, 255)),
                                                       (32, 1.0, (320, 256)), (32, 1.0, (210, 382)),
                                                       (32, 20.0, (320, 256))])
@pytest.mark.parametrize("flags", [33, 35])  # flat plane, without and with frozen advection
def test_kernels_agree(torch_cuda, precision, density, shape, flags):
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0,
                                  flags=flags)
    p = p.with_(dt=0.1 * inputs.stable_dt(p))
    state = inputs.random_state(p, seed=6)
    double = p.with_(R=2.0 * p.R, n_phi=2 * p.n_phi)
    small = run(p, precision, state, density, 6)
    tiles = run(double, precision, [np.concatenate([x, x], axis=1) for x in state], density, 6)
    for a, b in zip(small, tiles):
        for half in (b[..., :shape[1]], b[..., shape[1]:]):
            assert torch_cuda.equal(a, half), float((a - half).abs().max())
