"""tlb_get_state of FP32 grids: planes that are and are not a multiple of four values, output
pointers that are and are not 16-byte aligned, and each output alone, against the stored
deviations read back (f + n_ref w_i w_j, one rounding: 1 ulp of f < 1.2e-7 n_ref)."""
import ctypes

import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (8, 64), (31, 33), (33, 124)])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("want", ["both", "f", "phi"])
def test_get_state_of_any_size_and_alignment(torch_cuda, shape, offset, want):
    torch = torch_cuda
    from paper_1904_10070_amd import TorusGrid
    p = inputs.TorusParams(1.0, 2.5, shape[0], shape[1], 0.5, 2e-3, 0.05, 0.3, 1e-6)
    g = TorusGrid(p, precision=32)
    f, phi = inputs.random_populations(*shape, seed=3)
    g.set_state(phi, f=20.0 * f)
    plane = shape[0] * shape[1]
    out_f = torch.full((16 * plane + 8,), 7.0, device="cuda")
    out_phi = torch.full((plane + 8,), 7.0, device="cuda")
    ptr = lambda t, on: ctypes.c_void_p(t.data_ptr() + 4 * offset) if on else None  # noqa: E731
    rc = g.lib.tlb_get_state(g._h, ptr(out_f, want != "phi"), ptr(out_phi, want != "f"))
    assert rc == 0
    torch.cuda.synchronize()
    # n_ref: the mean density, to two digits, is what full minus stored populations sum to
    v = np.array([3.0 - 6.0 ** 0.5, 3.0 + 6.0 ** 0.5, 3.0 + 6.0 ** 0.5, 3.0 - 6.0 ** 0.5]) / 12.0
    w = np.outer(v, v).reshape(16, 1)
    stored = g.f[0].double().cpu().numpy().reshape(16, plane)
    n_ref = float(np.round((20.0 * f).reshape(16, plane).sum(0) - stored.sum(0), 0).mean())
    got_f = out_f.double().cpu().numpy()
    got_phi = out_phi.double().cpu().numpy()
    if want != "phi":
        err = np.abs(got_f[offset:offset + 16 * plane].reshape(16, plane) - (stored + n_ref * w)).max()
        assert err <= 1.2e-7 * n_ref, (err, n_ref)
        assert np.all(got_f[:offset] == 7.0) and np.all(got_f[offset + 16 * plane:] == 7.0)
    else:
        assert np.all(got_f == 7.0)
    if want != "f":
        assert np.array_equal(got_phi[offset:offset + plane],
                              phi.astype(np.float32).astype(np.float64).reshape(-1))
        assert np.all(got_phi[:offset] == 7.0) and np.all(got_phi[offset + plane:] == 7.0)
    else:
        assert np.all(got_phi == 7.0)
    g.close()
