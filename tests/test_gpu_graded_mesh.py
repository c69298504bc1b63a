"""A level whose rows crowd into one of the equal tiles of its plane (a finely
resolved square and a triangle far away) keeps its dispatch per colour, and finds
that out in time: sorting the rows of such a tile, and building patches from it,
takes steps that grow with their square (90 000 rows: 1.3e8 steps of one wave a
try, at eight tries; a million rows: 1.6e10).  The V-cycle against the oracle's
within the bounds of the other patch tests; the setup, a few hundredths of a
second, within one."""
import time

import numpy as np
import pytest

import oracle
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


def square_and_far_triangle(k, side, far):
    t = np.linspace(0.0, side, k)
    x = np.stack(np.meshgrid(t, t, indexing="ij"), -1).reshape(-1, 2)
    i = np.arange(k * k).reshape(k, k)
    a, b, c, d = i[:-1, :-1].ravel(), i[1:, :-1].ravel(), i[:-1, 1:].ravel(), i[1:, 1:].ravel()
    tri = np.concatenate([np.stack([a, b, d], 1), np.stack([a, d, c], 1), [[k * k, k * k + 1, k * k + 2]]])
    return np.concatenate([x, far + np.array([[0.0, 0.0], [1.0, 0.0], [0.3, 0.9]])]), tri


# all in one tile; a few tiles around a patch's limit; a level in the largest patches' range
@pytest.mark.parametrize("k,side,far", [(60, 10.0, 3000.0), (60, 10.0, 20.0), (300, 30.0, 9000.0)])
def test_crowded_tile(glnk, k, side, far):
    x, t = square_and_far_triangle(k, side, far)
    mg, mo = glnk.Mesh.simplicial(x, t, mu=0.2), oracle.Mesh.simplices(x, t, mu=0.2)
    psi = inputs.random_phase_state(mo.n, seed=4)
    r = inputs.random_complex(mo.n, seed=5)
    want = oracle.Amg.for_state(mo, psi, max_coarse=64).precond(mo, r, cycles=1)
    glnk.Precond(mg, torch.from_numpy(psi).cuda(), max_coarse=64).close()
    for prec, tol in ((glnk.GL_FP64, 1e-11), (glnk.GL_FP32, 1e-5)):
        t0 = time.perf_counter()
        pre = glnk.Precond(mg, torch.from_numpy(psi).cuda(), precision=prec, max_coarse=64)
        torch.cuda.synchronize()
        assert time.perf_counter() - t0 < 1.0
        z = torch.empty(mo.n, dtype=torch.complex128, device="cuda")
        pre.apply(torch.from_numpy(r).cuda(), z)
        assert np.abs(z.cpu().numpy() - want).max() <= tol * np.abs(want).max(), prec


def disc_handle_bytes(glnk, k, power):
    """Device memory of a handle on a disc of k rings with radii r^power."""
    from paper_1204_5125_amd import meshes
    x, t = meshes.disc(k)
    rel = np.linalg.norm(x, axis=1, keepdims=True) / meshes.RADIUS
    held, sizes = [0], {}

    def alloc(n):
        p = torch.cuda.caching_allocator_alloc(n)
        sizes[p] = n
        held[0] += n
        return p

    def release(p):
        held[0] -= sizes.pop(p)
        torch.cuda.caching_allocator_delete(p)

    glnk.gl_set_allocator(alloc, release)
    try:
        m = glnk.Mesh.simplicial(x * rel ** (power - 1), t, mu=0.3)
        before = held[0]
        pre = glnk.Precond(m, torch.from_numpy(inputs.random_phase_state(m.n, seed=1)).cuda(), max_coarse=64)
        used = held[0] - before
        pre.close()
        m.close()
        assert held[0] == 0
    finally:
        glnk.gl_set_allocator(None, None)
    return used


@pytest.mark.parametrize("k,power", [(64, 2.5), (128, 1.8), (128, 2.0)])
def test_tries_that_do_not_fit_hold_nothing(glnk, k, power):
    """Rings moved towards the centre leave the connectivity, and with it the
    hierarchy, as they were.  With radii r^5 no level's fullest tile fits a patch
    and nothing is built; with these, patches are built and found not to fit:
    the handle holds as much."""
    assert disc_handle_bytes(glnk, k, power) == disc_handle_bytes(glnk, k, 5)
