"""A batch of FP32 tori of different densities.  Each stores its populations relative to its own
reference density, and one that is not 1 puts the whole batch on the kernels that read it: every
member, those of unit density too, still ends bit for bit where it does alone."""
import pytest

from paper_1904_10070_amd import inputs

pytestmark = pytest.mark.gpu


def make(shape, density, seed):
    from paper_1904_10070_amd import TorusGrid
    p = inputs.params_three_cells(1.0, 2.5, shape[0], shape[1], A=0.5, M=2.5e-3, tau=0.6, dt=1.0)
    g = TorusGrid(p.with_(dt=0.25 * inputs.stable_dt(p)), precision=32)
    phi, n, ut, up = inputs.random_state(p, seed=seed)
    g.set_state(phi, density * n, ut, up)
    return g


# the second shape of each is above the sizes of the small-grid kernel, so that a member alone runs
# the tile kernel without a reference density; 130 columns have no 16-byte copies
@pytest.mark.parametrize("shapes", [((40, 96), (660, 128)), ((40, 130), (430, 194))])
def test_members_end_where_they_do_alone(torch_cuda, shapes):
    from paper_1904_10070_amd import TorusBatch
    members = [(shapes[0], 1.0), (shapes[1], 1.0), (shapes[0], 20.0), (shapes[1], 0.35)]
    alone = [make(*m, seed=i) for i, m in enumerate(members)]
    batched = [make(*m, seed=i) for i, m in enumerate(members)]
    batch = TorusBatch(batched)
    batch.step(20)
    for i, (g, h) in enumerate(zip(alone, batched)):
        g.step(20)
        for a, b in zip(g.get_state(), h.get_state()):
            assert torch_cuda.equal(a, b), (members[i], float((a - b).abs().max()))
    batch.close()
    for g in alone + batched:
        g.close()
