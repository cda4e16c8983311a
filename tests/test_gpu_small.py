"""The small-grid stage kernel against the tile kernel and the oracle.  A batch always runs tiles, so
a grid stepped alone and in a batch compares the two: bit for bit, on sides shorter than a stencil,
ragged row segments, and either side of the size where grids change from one kernel to the other.
Above that size, the tile heights agree bit for bit and the fourth-order Cahn-Hilliard variant
(not available in batches) agrees with the oracle: FP64 to 1e-12, as in the other parity tests; FP32
to 1e-5 of the largest value after 4 steps (each stage rounds to 6e-8, 12 stages of about 20
dependent operations)."""
import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


def make(p, precision, density=1.0, seed=3):
    from paper_1904_10070_amd import TorusGrid
    g = TorusGrid(p, precision=precision)
    phi, n, ut, up = inputs.random_state(p, seed=seed)
    g.set_state(phi, density * n, ut, up)
    return g


def params(shape, flags=0):
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0,
                                  flags=flags)
    return p.with_(dt=0.25 * inputs.stable_dt(p))


@pytest.mark.parametrize("shape", [(1, 1), (2, 1), (1, 2), (2, 3), (3, 5), (7, 2), (5, 63), (4, 64),
                                   (9, 65), (6, 131), (64, 160), (640, 64), (641, 60), (320, 256),
                                   (1280, 61), (1281, 64)])
@pytest.mark.parametrize("precision, flags, density", [(64, 0, 1.0), (64, 1, 1.0), (64, 2, 1.0),
                                                       (32, 0, 1.0), (32, 1, 20.0), (32, 2, 1.0)])
def test_alone_equals_batch(torch_cuda, shape, precision, flags, density):
    from paper_1904_10070_amd import TorusBatch
    p = params(shape, flags)
    alone, batched = make(p, precision, density), make(p, precision, density)
    batch = TorusBatch([batched])
    alone.step(3)
    batch.step(3)
    torch_cuda.cuda.synchronize()
    for a, b in zip(alone.get_state(), batched.get_state()):
        assert torch_cuda.equal(a, b), float((a - b).abs().max())
    batch.close()
    alone.close()
    batched.close()


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("shape", [(331, 258), (324, 256)])
def test_tile_heights_agree_above_the_small_sizes(torch_cuda, shape, precision):
    out = []
    for rows in (4, 8, 16):
        g = make(params(shape), precision)
        g.set_tile_rows(rows)
        g.step(3)
        out.append(g.get_state())
        g.close()
    for f, phi in out[1:]:
        assert torch_cuda.equal(f, out[0][0]) and torch_cuda.equal(phi, out[0][1])


@pytest.mark.parametrize("precision, tol", [(64, 1e-12), (32, 1e-5)])
@pytest.mark.parametrize("shape", [(2, 2), (64, 130), (331, 258), (324, 256)])
def test_fourth_order_matches_oracle(torch_cuda, shape, precision, tol):
    from oracle import ref
    p = params(shape, flags=32)
    g = make(p, precision)
    g.step(4)
    f, phi = (x.double().cpu().numpy() for x in g.get_state())
    o = ref.RefGrid(**p.as_dict())
    o.set_state(*inputs.random_state(p, seed=3))
    o.step(4)
    f_ref, phi_ref = o.get_state()
    ef = np.abs(f - f_ref).max() / np.abs(f_ref).max()
    ep = np.abs(phi - phi_ref).max() / np.abs(phi_ref).max()
    print(shape, precision, f"{ef:.1e} {ep:.1e}", flush=True)
    assert ef <= tol and ep <= tol
    g.close()
