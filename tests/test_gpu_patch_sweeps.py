"""The V-cycle on hierarchies whose levels run in patches, and on those that
must not: against the oracle's V-cycle (FP64 1e-11, FP32 and mixed 1e-5 of the
largest entry, the bounds of the other V-cycle tests).  A long thin grid (tiles
one row high), sizes just below and above one patch, a disc (empty tiles at the
corners of its box), a disc whose rings crowd at the centre (a tile with
thousands of rows: the level falls back to a dispatch per colour), a fan (rows
of hundreds of neighbours), and splits that move levels between the patches,
the dense operator and the bottom kernel on one handle."""
import numpy as np
import pytest

import oracle
from paper_1204_5125_amd import inputs, meshes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def glnk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_5125_amd import glnk as g
    g.lib()
    return g


def crowded_disc(k):
    x, t = meshes.disc(k)
    r = np.linalg.norm(x, axis=1, keepdims=True) / meshes.RADIUS
    return x * r ** 2, t


def fan(m, rings):
    xy, tri = [(0.0, 0.0)], []
    t = 2 * np.pi / m
    for r in range(rings):
        xy += [((1.0 + r * t) * np.cos(t * k), (1.0 + r * t) * np.sin(t * k)) for k in range(m)]
    at = lambda r, k: 1 + r * m + k % m  # noqa: E731
    for k in range(m):
        tri.append((0, at(0, k), at(0, k + 1)))
        for r in range(rings - 1):
            tri += [(at(r, k), at(r + 1, k), at(r + 1, k + 1)), (at(r, k), at(r + 1, k + 1), at(r, k + 1))]
    return np.array(xy), np.array(tri, dtype=np.int64)


SHAPES = {
    "thin": (700, 5), "small": (23, 25), "one patch": (60, 58), "ragged": (257, 101),
    "disc": meshes.disc(45), "crowded": crowded_disc(40), "fan": fan(300, 4),
}


def pair(glnk, name):
    s = SHAPES[name]
    if isinstance(s[0], int):
        side = tuple(0.25 * (n - 1) for n in s)
        return glnk.Mesh(2, s, side, mu=0.6), oracle.Mesh(2, s, side, mu=0.6)
    return glnk.Mesh.simplicial(*s, mu=0.3), oracle.Mesh.simplices(*s, mu=0.3)


def vcycle(pre, r, n):
    z = torch.empty(n, dtype=torch.complex128, device="cuda")
    pre.apply(torch.from_numpy(r).cuda(), z)
    return z.cpu().numpy()


@pytest.mark.parametrize("name", list(SHAPES))
def test_vcycle_against_oracle(glnk, name):
    mg, mo = pair(glnk, name)
    psi = inputs.random_phase_state(mo.n, seed=4)
    r = inputs.random_complex(mo.n, seed=5)
    for cycles in (1, 2):
        want = oracle.Amg.for_state(mo, psi, max_coarse=8).precond(mo, r, cycles=cycles)
        for prec, tol in ((glnk.GL_FP64, 1e-11), (glnk.GL_FP32, 1e-5), (glnk.GL_MIXED, 1e-5)):
            pre = glnk.Precond(mg, torch.from_numpy(psi).cuda(), precision=prec, cycles=cycles, max_coarse=8)
            z = vcycle(pre, r, mo.n)
            assert np.abs(z - want).max() <= tol * np.abs(want).max(), (name, prec, cycles)
            assert np.array_equal(z, vcycle(pre, r, mo.n))  # every call the same bits


def test_splits_on_one_handle(glnk):
    """Levels that move between the patches, an explicit sub-cycle and back
    keep their values current."""
    mg, mo = pair(glnk, "ragged")
    psi = inputs.random_phase_state(mo.n, seed=4)
    r = inputs.random_complex(mo.n, seed=5)
    want = oracle.Amg.for_state(mo, psi, max_coarse=8).precond(mo, r)
    pre = glnk.Precond(mg, torch.from_numpy(inputs.random_phase_state(mo.n, seed=9)).cuda(), max_coarse=8)
    glnk.gl_precond_set_tiles(pre, 0, 64, 1000, 0)
    pre.update(torch.from_numpy(psi).cuda())
    for tiles in ((0, 64, 1000, 0), (0, 0, 0, 0), (1, 8192, 0, 2), (0, 64, 200, 1), (0, 0, 0, 0)):
        glnk.gl_precond_set_tiles(pre, *tiles)
        z = vcycle(pre, r, mo.n)
        assert np.abs(z - want).max() <= 1e-11 * np.abs(want).max(), tiles


@pytest.mark.parametrize("name", ["ragged", "disc"])
def test_solves_follow_the_values(glnk, name):
    """The explicit sub-cycle that solves use belongs to the values of the last
    setup: after an update, with applications in between and across precisions,
    a kept handle solves as a fresh one does."""
    mg, mo = pair(glnk, name)
    b = torch.from_numpy(inputs.random_complex(mo.n, seed=5)).cuda()
    x, y, z = (torch.empty_like(b) for _ in range(3))
    states = [torch.from_numpy(inputs.random_phase_state(mo.n, seed=s)).cuda() for s in (1, 2, 3)]
    kept = glnk.Precond(mg, states[0], max_coarse=8)
    glnk.gl_jacobian_solve(mg, states[0], kept, b, x, max_iter=5, raise_on_fail=False)
    for psi, prec in ((states[1], glnk.GL_FP64), (states[2], glnk.GL_FP32), (states[1], glnk.GL_MIXED)):
        kept.update(psi, precision=prec)
        kept.apply(b, z)
        fresh = glnk.Precond(mg, psi, precision=prec, max_coarse=8)
        for p, out in ((kept, x), (fresh, y)):
            rc, info = glnk.gl_jacobian_solve(mg, psi, p, b, out, max_iter=6, inner_rtol=1e-3, raise_on_fail=False)
            assert info["iterations"] == 6
        assert torch.equal(x, y)
        fresh.apply(b, x)
        assert torch.equal(x, z)


@pytest.mark.parametrize("shape", [(660, 650), (9000, 50)])
def test_large_levels(glnk, shape):
    """Levels of more than 65 536 rows take larger patches; bounds as above."""
    side = tuple(0.25 * (n - 1) for n in shape)
    mg, mo = glnk.Mesh(2, shape, side, mu=0.6), oracle.Mesh(2, shape, side, mu=0.6)
    psi = inputs.random_phase_state(mo.n, seed=4)
    r = inputs.random_complex(mo.n, seed=5)
    want = oracle.Amg.for_state(mo, psi, max_coarse=64).precond(mo, r, cycles=1)
    for prec, tol in ((glnk.GL_FP64, 1e-11), (glnk.GL_FP32, 1e-5)):
        pre = glnk.Precond(mg, torch.from_numpy(psi).cuda(), precision=prec, cycles=1, max_coarse=64)
        z = vcycle(pre, r, mo.n)
        assert np.abs(z - want).max() <= tol * np.abs(want).max(), prec


@pytest.mark.parametrize("shift", [-1, 0, 1])
@pytest.mark.parametrize("shape", [(9, 8, 7), (23, 5, 17), (30, 31, 29)])
def test_colour_passes(glnk, shape, shift):
    """3D levels, a dispatch per colour on the halves of the rows, with fewer and
    more lanes per row; bounds as above."""
    side = tuple(0.4 * (n - 1) for n in shape)
    mg, mo = glnk.Mesh(3, shape, side, mu=0.6), oracle.Mesh(3, shape, side, mu=0.6)
    psi = inputs.random_phase_state(mo.n, seed=4)
    r = inputs.random_complex(mo.n, seed=5)
    want = oracle.Amg.for_state(mo, psi, max_coarse=8).precond(mo, r, cycles=1)
    for prec, tol in ((glnk.GL_FP64, 1e-11), (glnk.GL_FP32, 1e-5), (glnk.GL_MIXED, 1e-5)):
        pre = glnk.Precond(mg, torch.from_numpy(psi).cuda(), precision=prec, cycles=1, max_coarse=8)
        glnk.gl_precond_set_tiles(pre, shift, 1, 0, 0)
        z = vcycle(pre, r, mo.n)
        assert np.abs(z - want).max() <= tol * np.abs(want).max(), prec
