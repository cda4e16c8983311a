"""The WENO-5 variant, whose face values are shared between neighbouring nodes and wavefronts, at
sides shorter than a stencil and at the edges of its tiles, against the oracle: FP64 to 1e-12 of the
largest value, as in the other parity tests, FP32 to 1e-5 after 4 steps (12 stages of about 20
dependent operations that round to 6e-8), also with a reference density other than one."""
import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (8, 64), (9, 65), (15, 63), (17, 132), (40, 260)])
@pytest.mark.parametrize("precision, density, tol", [(64, 1.0, 1e-12), (32, 1.0, 1e-5),
                                                     (32, 20.0, 1e-5)])
def test_weno5_of_any_size(torch_cuda, shape, precision, density, tol):
    from paper_1904_10070_amd import TorusGrid
    from oracle import ref
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0,
                                  flags=8)
    p = p.with_(dt=0.25 * inputs.stable_dt(p))
    phi, n, ut, up = inputs.random_state(p, seed=5)
    g = TorusGrid(p, precision=precision)
    g.set_state(phi, density * n, ut, up)
    g.step(4)
    f, ph = (x.double().cpu().numpy() for x in g.get_state())
    o = ref.RefGrid(**p.as_dict())
    o.set_state(phi, density * n, ut, up)
    o.step(4)
    f_ref, phi_ref = o.get_state()
    ef = np.abs(f - f_ref).max() / np.abs(f_ref).max()
    ep = np.abs(ph - phi_ref).max() / np.abs(phi_ref).max()
    print(shape, precision, density, f"{ef:.1e} {ep:.1e}", flush=True)
    assert ef <= tol and ep <= tol
    g.close()
