"""The explicit sub-cycle that solves on automatic tiles use: its memory comes
with the first solve (a handle that only serves applications holds none), a
batch has one bounded workspace for forming all of them, in as many turns as
that takes, with the bits of single solves; and where there is no memory for it
solves do without."""
import gc

import numpy as np
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


@pytest.fixture
def allocator(glnk):
    """torch's allocator, counting what is held, refusing requests above .most"""
    class A:
        held, most, sizes, asked = 0, None, {}, []

        def alloc(self, n):
            self.asked.append(n)
            if self.most is not None and n > self.most:
                return 0
            p = torch.cuda.caching_allocator_alloc(n)
            self.sizes[p] = n
            self.held += n
            return p

        def release(self, p):
            self.held -= self.sizes.pop(p)
            torch.cuda.caching_allocator_delete(p)

    a = A()
    a.sizes, a.asked = {}, []
    glnk.gl_set_allocator(a.alloc, a.release)
    try:
        yield a
    finally:
        gc.collect()
        glnk.gl_set_allocator(None, None)


def mesh(glnk, N):
    return glnk.Mesh(2, (N, N), (0.25 * (N - 1),) * 2, mu=0.6)


def state(n, seed):
    return torch.from_numpy(inputs.random_phase_state(n, seed=seed)).cuda()


def solve(glnk, m, psi, pre, b):
    x = torch.empty_like(b)
    rc, info = glnk.gl_jacobian_solve(m, psi, pre, b, x, rtol=1e-10, max_iter=200)
    assert info["converged"]
    return x, info["iterations"]


def test_allocated_by_the_first_solve(glnk, allocator):
    m = mesh(glnk, 65)
    psi, b = state(m.n, 1), torch.from_numpy(inputs.random_complex(m.n, seed=2)).cuda()
    pre = glnk.Precond(m, psi, max_coarse=16)
    smallest = pre.info()["sizes"][-2]  # of the levels whose sub-cycle may be explicit
    built = allocator.held
    z = torch.empty_like(b)
    pre.apply(b, z)
    pre.update(psi)
    assert allocator.held == built
    solve(glnk, m, psi, pre, b)
    first = allocator.held
    assert first - built >= 24 * smallest ** 2
    pre.update(psi)
    solve(glnk, m, psi, pre, b)
    assert allocator.held == first
    pre.close()
    m.close()
    assert allocator.held == 0


def test_no_memory_for_it(glnk, allocator):
    m = mesh(glnk, 65)
    psi, b = state(m.n, 1), torch.from_numpy(inputs.random_complex(m.n, seed=2)).cuda()
    ref = glnk.Precond(m, psi, max_coarse=16)
    want, its = solve(glnk, m, psi, ref, b)
    pre = glnk.Precond(m, psi, max_coarse=16)
    allocator.most = 0
    asked = len(allocator.asked)
    for _ in range(2):
        got, its2 = solve(glnk, m, psi, pre, b)
        assert abs(its2 - its) <= 1
        assert float((got - want).abs().max() / want.abs().max()) < 1e-8
        pre.update(psi)
    assert len(allocator.asked) == asked + 1  # asked for once
    allocator.most = None
    glnk.gl_precond_set_tiles(pre, 0, 512, 0, 0)
    glnk.gl_precond_set_tiles(pre, 0, 0, 0, 0)  # chosen again
    assert torch.equal(solve(glnk, m, psi, pre, b)[0], want)


def batch_run(glnk, N, count, **kw):
    ms = [mesh(glnk, N) for _ in range(count)]
    psis = [state(m.n, 10 + i) for i, m in enumerate(ms)]
    batch = glnk.Batch(ms)
    batch.newton_solve(psis, fixed_steps=1, krylov_rtol=1e-3, krylov_max_iter=200, max_coarse=16, **kw)
    torch.cuda.synchronize()
    return [p.cpu().numpy() for p in psis]


def test_no_memory_for_it_in_a_batch(glnk, allocator):
    want = batch_run(glnk, 33, 12)
    gc.collect()
    shared = max(allocator.asked)
    others = sorted(allocator.asked)[-2]
    assert shared > 2 * others
    allocator.most = others
    allocator.asked.clear()
    got = batch_run(glnk, 33, 12)
    assert max(allocator.asked) == shared
    for a, b in zip(got, want):
        assert np.abs(a - b).max() <= 1e-2 * np.abs(b).max()  # solves to 1e-3, counts may differ by one


@pytest.mark.parametrize("N,count", [(33, 3), (110, 9)])
def test_workspace_in_turns(glnk, allocator, N, count):
    """(110: sub-cycles of about 2000 rows, 0.2 GB of workspace each)"""
    got = batch_run(glnk, N, count)
    gc.collect()
    assert max(allocator.asked) <= 3 << 29
    if count == 9:
        assert max(allocator.asked) > 1 << 30  # all nine do not fit
    for i in range(count):
        m, psi = mesh(glnk, N), state(mesh(glnk, N).n, 10 + i)
        glnk.gl_newton_solve(m, psi, fixed_steps=1, krylov_rtol=1e-3, krylov_max_iter=200, max_coarse=16)
        assert np.array_equal(psi.cpu().numpy(), got[i])


def test_batch_leaves_nothing_with_its_meshes(glnk):
    """The memory that a batch's handles took is gone with the batch, also while
    its meshes live (hipMalloc; the first batch is for what the runtime keeps)."""
    def used():
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free

    ms = [mesh(glnk, 129) for _ in range(8)]
    psis = [state(m.n, 10 + i) for i, m in enumerate(ms)]
    for _ in range(2):
        before = used()
        batch = glnk.Batch(ms)
        batch.newton_solve(psis, fixed_steps=1, krylov_rtol=1e-2, krylov_max_iter=50, raise_on_fail=False)
        held = used() - before
        batch.close()
        left = used() - before
    assert held > 8 * 20e6
    assert left <= 8e6
