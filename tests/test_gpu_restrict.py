"""tlb_restrict at the edges of its 64-node segments, for the factors with and without a kernel of
their own, on coarse grids of one row or column, against oracle/cnn_ref.py.  Bars: the sums have
k + 1 terms in each direction (k <= 32), all in FP64: (2 k + 4) 1.1e-16 < 1e-14 relative to the
largest value; FP32 adds the rounding of the stored values, 2e-7 as in the other tests."""
import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coarse, k", [((3, 1), 2), ((1, 63), 4), ((4, 64), 4), ((2, 65), 8),
                                       ((5, 130), 6), ((6, 129), 2), ((1, 1), 32), ((2, 66), 32)])
@pytest.mark.parametrize("precision", [32, 64])
def test_restrict_of_any_size(torch_cuda, coarse, k, precision):
    from paper_1904_10070_amd import TorusGrid
    from paper_1904_10070_amd.binding import restrict
    from oracle import cnn_ref as C
    shape = (coarse[0] * k, coarse[1] * k)
    pf = inputs.TorusParams(1.0, 2.5, shape[0], shape[1], 0.5, 2e-3, 0.05, 0.3, 1e-6)
    fine = TorusGrid(pf, precision)
    small = TorusGrid(pf.with_(n_theta=coarse[0], n_phi=coarse[1]), precision)
    f, phi = inputs.random_populations(*shape, seed=k)
    fine.set_state(phi, f=f)
    restrict(fine, small)
    fc, phic = (x.double().cpu().numpy() for x in small.get_state())
    f_ref, phi_ref = C.restrict_state(f, phi, k, 1.0, 2.5)
    tol = 1e-14 if precision == 64 else 2e-7
    ef = np.abs(fc - f_ref).max() / np.abs(f_ref).max()
    ep = np.abs(phic - phi_ref).max() / np.abs(phi_ref).max()
    print(coarse, k, precision, f"{ef:.1e} {ep:.1e}", flush=True)
    assert ef <= tol and ep <= tol
    fine.close()
    small.close()
