"""Dispatches of a V-cycle on levels that run a dispatch per colour: with C
colours a level takes 2 C - 1 each way and its two transfers, no more; counted
by the batch's statistics (dispatches of an iteration pair), against the same
grid with level 1 as the coarsest."""
import pytest

from paper_1204_5125_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def glnk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_5125_amd import glnk as g
    g.lib()
    return g


def dispatches(glnk, N, max_levels):
    m = glnk.Mesh(3, N, tuple(0.4 * (n - 1) for n in N), mu=0.6)
    psi = torch.from_numpy(inputs.random_phase_state(m.n, seed=4)).cuda()
    kw = dict(max_coarse=8, max_levels=max_levels)
    info = glnk.Precond(m, psi, **kw).info()
    batch = glnk.Batch([m])
    batch.set_tiles(bottom_rows=1)
    batch.newton_solve([psi], fixed_steps=1, krylov_max_iter=4, raise_on_fail=False, **kw)
    return batch.stats()["dispatches_per_graph"] / 2, info


@pytest.mark.parametrize("N", [(9, 8, 7), (17, 17, 17), (23, 21, 22), (61, 5, 5)])
def test_colour_pass_dispatches(glnk, N):
    deep, info = dispatches(glnk, N, 16)
    flat, two = dispatches(glnk, N, 2)
    assert two["nlev"] == 2 and info["sizes"][:2] == two["sizes"] and info["nlev"] > 2
    assert deep - flat == sum(4 * c for c in info["ncolors"][1:-1])
