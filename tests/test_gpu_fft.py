"""tlb_structure_length at the sizes where its FFTs can go wrong, against numpy's FFT
(oracle/structure.py): lengths 1 and 2, primes, odd numbers of rows (two rows share a transform),
mixed factors, the longest row held twice in LDS (5120) and the direct sum beyond it.  Bar: 1e-11
relative (FP64 throughout; an n-term sum errs by about sqrt(n) 1e-16, n <= 8192)."""
import numpy as np
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 2), (2, 1), (1, 7), (5, 4), (7, 11), (30, 77), (101, 103),
                                   (64, 257), (121, 169), (96, 135), (4093, 8), (4096, 9),
                                   (3, 5119), (16, 5120), (9, 5121), (8, 8192)])
@pytest.mark.parametrize("precision", [32, 64])
def test_structure_length_of_any_size(torch_cuda, shape, precision):
    from paper_1904_10070_amd import TorusGrid
    from oracle import structure
    p = inputs.TorusParams(1.0, 2.5, shape[0], shape[1], 0.5, 2e-3, 0.05, 0.3, 1e-6)
    phi = 0.3 + np.random.default_rng(shape[0] + shape[1]).uniform(-1, 1, shape)
    if precision == 32:
        phi = phi.astype(np.float32).astype(np.float64)
    g = TorusGrid(p, precision=precision)
    g.set_state(phi, *inputs.rest_moments(*shape))
    got = g.structure_length()
    ref = structure.structure_length(phi, 1.0, 2.5)
    print(shape, precision, got, ref, flush=True)
    assert all(abs(a - b) <= 1e-11 * abs(b) for a, b in zip(got, ref)), (got, ref)
    g.close()
