"""gl_precond_set_tiles: the request alone decides what a handle does, whatever
was set before it; all fields 0 is the automatic choice of a new handle and
{0, 512, 0, 0} one dispatch per pass with no explicit sub-cycle.  A handle that
went through other choices gives the bits of a new one with the same tiles, in
applications and in solves; the level-0 forms are told apart by the profiler's
count of level-0 residual launches (the tiled forms have none) and agree with
the one-pass form within the bounds of the other level-0 tests."""
import numpy as np
import pytest

import oracle
from paper_1204_5125_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

AUTO, PLAIN = (0, 0, 0, 0), (0, 512, 0, 0)
L0_RESIDUAL = 3  # profile id


@pytest.fixture(scope="module")
def glnk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1204_5125_amd import glnk as g
    g.lib()
    return g


def mesh(glnk, N):
    return glnk.Mesh(2, N, tuple(0.25 * (n - 1) for n in N), mu=0.6)


def vec(n, seed):
    return torch.from_numpy(inputs.random_complex(n, seed=seed)).cuda()


def results(glnk, m, pre, psi, b):
    """An application, and a few iterations of a solve."""
    z, x = torch.empty_like(b), torch.empty_like(b)
    pre.apply(b, z)
    glnk.gl_jacobian_solve(m, psi, pre, b, x, rtol=0.0, max_iter=6, poll_every=6, raise_on_fail=False)
    return z, x


def residual_launches(glnk, pre, b):
    z = torch.empty_like(b)
    glnk.gl_profile_start(L0_RESIDUAL)
    pre.apply(b, z)
    torch.cuda.synchronize()
    return glnk.gl_profile_stop()[2]


@pytest.mark.parametrize("tiles", [AUTO, PLAIN, (0, 512, 0, 2), (0, 64, 1000, 0), (1, 0, 0, 0)])
def test_request_decides_not_history(glnk, tiles):
    m = mesh(glnk, (65, 71))
    psi = torch.from_numpy(inputs.random_phase_state(m.n, seed=1)).cuda()
    b = vec(m.n, 2)
    new = glnk.Precond(m, psi, max_coarse=16)
    glnk.gl_precond_set_tiles(new, *tiles)
    want = results(glnk, m, new, psi, b)
    used = glnk.Precond(m, psi, max_coarse=16)
    for other in ((0, 64, 1000, 1), PLAIN, AUTO, (2, 8192, 0, 3)):
        glnk.gl_precond_set_tiles(used, *other)
        results(glnk, m, used, psi, b)
        glnk.gl_precond_set_tiles(used, *tiles)
        for got, ref in zip(results(glnk, m, used, psi, b), want):
            assert torch.equal(got, ref), (tiles, other)
    assert residual_launches(glnk, used, b) == residual_launches(glnk, new, b) == (0 if tiles == AUTO or tiles[3] else 1)


def test_read_and_restored(glnk):
    m = mesh(glnk, (65, 71))
    psi = torch.from_numpy(inputs.random_phase_state(m.n, seed=1)).cuda()
    b = vec(m.n, 2)
    pre = glnk.Precond(m, psi, max_coarse=16)
    want = results(glnk, m, pre, psi, b)
    read = glnk.gl_precond_get_tiles(pre)
    assert read == {"lane_shift": 0, "bottom_rows": 0, "dense_rows": 0, "l0_tiled": 0}
    for other in (PLAIN, (0, 64, 4096, 3)):
        glnk.gl_precond_set_tiles(pre, *other)
        assert tuple(glnk.gl_precond_get_tiles(pre).values()) == other
        glnk.gl_precond_set_tiles(pre, **read)
        for got, ref in zip(results(glnk, m, pre, psi, b), want):
            assert torch.equal(got, ref), other


@pytest.mark.parametrize("N", [(33, 33), (37, 23), (24, 17), (129, 129), (70, 45), (5, 3), (3, 70)])
def test_level0_forms_against_one_pass(glnk, N):
    """Every tile shape and the automatic choice against one dispatch per pass,
    which is asked for on the handle as it is built; and that against the oracle."""
    m = mesh(glnk, N)
    mo = oracle.Mesh(2, N, tuple(0.25 * (n - 1) for n in N), mu=0.6)
    psi = inputs.random_phase_state(m.n, seed=17)
    r = inputs.random_complex(m.n, seed=18)
    dpsi, dr = torch.from_numpy(psi).cuda(), torch.from_numpy(r).cuda()
    z = torch.empty_like(dr)
    for prec, cycles in ((glnk.GL_FP64, 1), (glnk.GL_FP32, 1), (glnk.GL_MIXED, 1), (glnk.GL_FP64, 3)):
        pre = glnk.Precond(m, dpsi, precision=prec, cycles=cycles, max_coarse=8)
        glnk.gl_precond_set_tiles(pre, *PLAIN)
        assert residual_launches(glnk, pre, dr) == cycles
        pre.apply(dr, z)
        ref = z.cpu().numpy()
        want = oracle.Amg.for_state(mo, psi, max_coarse=8).precond(mo, r, cycles=cycles)
        assert np.abs(ref - want).max() <= (1e-11 if prec == glnk.GL_FP64 else 1e-5) * np.abs(want).max()
        for tiles in ((0, 512, 0, 1), (0, 512, 0, 2), (0, 512, 0, 3), AUTO):
            glnk.gl_precond_set_tiles(pre, *tiles)
            assert residual_launches(glnk, pre, dr) == 0
            pre.apply(dr, z)
            e = np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max()
            assert e < (1e-13 if prec == glnk.GL_FP64 else 1e-6), (prec, cycles, tiles, e)
