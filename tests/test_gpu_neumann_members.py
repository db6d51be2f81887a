"""Pure-Neumann solves of several members: each member's mean of the preconditioned residual is its
own, in workgroups that hold some of the members, all of them or several elements of each, and with
the members in turn; the host looks at the states at every third iteration only.

Tolerance: the members' solves and the single ones end at relative residuals of 1e-11; on these
meshes the smallest non-zero eigenvalue of the Jacobi-scaled operator is above 1e-4 of the largest,
so that they differ by less than 1e-6 (and by far less where the residuals are unrelated)."""
import numpy as np
import pytest

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu

# at p = 1..4 the last sizes are just above 400 workgroups of elements
CASES = [(8, 2, 2), (8, 2, 3), (8, 2, 5), (8, 2, 9), (5, 2, 9), (3, 3, 2), (1, 3, 30),
         (1, 23, 3), (2, 19, 3), (3, 16, 3), (4, 15, 2), (4, 15, 5), (2, 19, 9)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("p,n,nb", CASES)
def test_members_have_their_own_means(p, n, nb, mode):
    from paper_1910_03032_amd import DIFFUSION, Operator
    m = BoxMesh(n, p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p)
    rng = np.random.default_rng(p + nb)
    b = rng.uniform(-1, 1, (nb, m.ndof)) * 10.0 ** np.arange(nb)[:, None] + rng.uniform(-1, 1, (nb, 1))
    u, res = op.pcg(gpu(b), op=DIFFUSION, rtol=1e-11, mode=mode, check_every=3, nullspace=True)
    assert res.converged, res
    for k in sorted({0, 1, nb // 2, nb - 1}):
        w, one = op.pcg(gpu(b[k]), op=DIFFUSION, rtol=1e-11, mode=mode, check_every=3, nullspace=True)
        e = rel(host(u[k]), host(w))
        say(f"[neumann] p={p} n={n} nb={nb} mode={mode} k={k} iters={res.iters[k]} {one.iters[0]} rel={e:.1e}")
        assert one.converged and e <= 1e-6, (k, e)
        assert abs(res.iters[k] - one.iters[0]) <= 0.1 * one.iters[0] + 2, (k, res.iters[k], one.iters[0])
    op.close()
