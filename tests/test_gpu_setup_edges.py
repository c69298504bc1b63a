"""The setup kernels at the sizes where they can go wrong, bit-exact against
the oracle (integer arrays equal, values within 1e-12): grids whose rows are a
single node past a work-group, the smallest grids that coarsen, and a fan (a
hub whose matrix row, restriction row and coarse row are hundreds of entries
long, several chunks of a wave), and a coarse row past the limit of 512 columns
refused."""
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


def fan(m, rings):
    """A hub and `rings` rings of m nodes, the quadrilaterals between rings split."""
    xy, tri = [(0.0, 0.0)], []
    t = 2 * np.pi / m
    for r in range(rings):
        rad = 1.0 + r * t
        xy += [(rad * np.cos(t * k), rad * np.sin(t * k)) for k in range(m)]
    at = lambda r, k: 1 + r * m + k % m  # noqa: E731
    for k in range(m):
        tri.append((0, at(0, k), at(0, k + 1)))
        for r in range(rings - 1):
            tri += [(at(r, k), at(r + 1, k), at(r + 1, k + 1)), (at(r, k), at(r + 1, k + 1), at(r, k + 1))]
    return np.array(xy), np.array(tri, dtype=np.int64)


def compare(glnk, mg, mo, max_coarse):
    psi = inputs.random_phase_state(mo.n, seed=3)
    pre = glnk.Precond(mg, torch.from_numpy(psi).cuda(), max_coarse=max_coarse)
    amg = oracle.Amg.for_state(mo, psi, max_coarse=max_coarse)
    assert pre.info()["nlev"] == amg.nlev >= 2
    for l, L in enumerate(amg.levels):
        assert np.array_equal(pre.export(l, "color"), L["color"])
        names = ["A"] if l == amg.nlev - 1 else ["A", "P", "R"]
        for M in names:
            assert np.array_equal(pre.export(l, M + "_rp"), L[M].indptr)
            assert np.array_equal(pre.export(l, M + "_ci"), L[M].indices)
            v, w = pre.export(l, M + "_v"), L[M].data
            scale = np.abs(w).max()
            if M == "A" and l > 0:  # a Galerkin product's rounding is that of its terms, which may cancel
                up = amg.levels[l - 1]
                scale = (abs(up["R"]) @ abs(up["A"]) @ abs(up["P"])).max()
            assert np.abs(v - w).max() <= 1e-12 * scale
        if l < amg.nlev - 1:
            assert np.array_equal(pre.export(l, "agg"), L["agg"])
            assert np.array_equal(pre.export(l, "root"), L["root"])
    return pre


@pytest.mark.parametrize("dim,N,max_coarse", [(2, (257, 2), 4), (2, (2, 300), 8), (2, (3, 3), 2), (2, (129, 131), 8),
                                              (3, (2, 2, 2), 1), (3, (4, 33, 3), 4), (3, (17, 15, 16), 8)])
def test_grid_hierarchies(glnk, dim, N, max_coarse):
    side = tuple(0.3 * (n - 1) for n in N)
    kw = dict(mu=0.7)
    compare(glnk, glnk.Mesh(dim, N, side, **kw), oracle.Mesh(dim, N, side, **kw), max_coarse)


@pytest.mark.parametrize("m,rings", [(130, 3), (700, 5)])
def test_fan_hierarchy(glnk, m, rings):
    x, t = fan(m, rings)
    pre = compare(glnk, glnk.Mesh.simplicial(x, t, mu=0.5), oracle.Mesh.simplices(x, t, mu=0.5), 16)
    longest = max(np.diff(pre.export(0, M + "_rp")).max() for M in ("A", "R"))
    assert longest > m


def test_too_long_coarse_row_refused(glnk):
    x, t = fan(4000, 5)
    mesh = glnk.Mesh.simplicial(x, t, mu=0.5)
    psi = torch.ones(mesh.n, dtype=torch.complex128, device="cuda")
    with pytest.raises(glnk.GlnkError, match="GL_ERR_UNSUPPORTED"):
        glnk.Precond(mesh, psi, max_coarse=16)


def test_memory_given_back_and_taken_again(glnk):
    """Hierarchies built in the memory that others of the mesh gave back, with some
    still alive beside them, and one that outlives its mesh: each applies as one
    on a mesh of its own does, to the bit."""
    shapes = [(33, 33), (70, 41), (129, 65)]
    r = [torch.from_numpy(inputs.random_complex(s[0] * s[1], seed=7)).cuda() for s in shapes]
    psi = [[torch.from_numpy(inputs.random_phase_state(s[0] * s[1], seed=q)).cuda() for q in (1, 2, 3)] for s in shapes]
    mesh_of = lambda s: glnk.Mesh(2, s, tuple(0.25 * (n - 1) for n in s), mu=0.6)  # noqa: E731

    def applied(pre, b):
        z = torch.empty_like(b)
        pre.apply(b, z)
        return z

    for k, s in enumerate(shapes):
        want = []
        for p in psi[k]:
            m = mesh_of(s)
            pre = glnk.Precond(m, p, max_coarse=16)
            want.append(applied(pre, r[k]))
            pre.close()
            m.close()
        m = mesh_of(s)
        kept = glnk.Precond(m, psi[k][0], max_coarse=16)
        for q in (1, 2, 1):
            pre = glnk.Precond(m, psi[k][q], max_coarse=16)
            assert torch.equal(applied(pre, r[k]), want[q])
            pre.close()
        assert torch.equal(applied(kept, r[k]), want[0])
        last = glnk.Precond(m, psi[k][2], max_coarse=16)
        kept.close()
        assert torch.equal(applied(last, r[k]), want[2])
        m.close()
        last.close()


@pytest.mark.parametrize("shape", [(64, 32), (683, 3), (32, 32), (25, 41), (8, 8, 8), (11, 31, 6)])
def test_power_iteration_of_small_levels(glnk, shape):
    """Levels at and past the sizes whose spectral-radius estimate one work-group
    runs (2048 and 1024 rows of up to 8 entries, 512 and 1024 of seven in 3D): the
    prolongator and the coarse operators against the oracle, as above."""
    side = tuple(0.3 * (n - 1) for n in shape)
    compare(glnk, glnk.Mesh(len(shape), shape, side, mu=0.7), oracle.Mesh(len(shape), shape, side, mu=0.7), 8)
