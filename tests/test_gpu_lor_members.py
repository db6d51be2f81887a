"""LOR-preconditioned CG of several right-hand sides, which are solved one after another: each as its
single solve, also after a Jacobi solve of the same members has left its partial sums in the
workspace that both use.

Tolerance: two solves to relative residual 1e-12 of these operators (condition numbers below 1e4,
pure Neumann below 1e5) differ by less than 1e-7."""
import numpy as np
import pytest

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("neumann", [False, True])
@pytest.mark.parametrize("lor32", [False, True])
@pytest.mark.parametrize("p,n,nb", [(1, 6, 3), (2, 4, 2), (4, 3, 3), (8, 2, 3)])
def test_members_one_after_another(p, n, nb, lor32, neumann):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, Operator, PRECOND_LOR, PRECOND_LOR32
    m = BoxMesh(n, p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=None if neumann else m.ess)
    op.set_coeffs(10.0, 1.0)
    kind = DIFFUSION if neumann else HELMHOLTZ
    b = gpu(np.random.default_rng(p).uniform(-1, 1, (nb, m.ndof)))
    args = dict(op=kind, rtol=1e-12, nullspace=neumann)
    op.pcg(b, **args)
    pc = PRECOND_LOR32 if lor32 else PRECOND_LOR
    u, res = op.pcg(b, precond=pc, **args)
    assert res.converged, res
    for k in range(nb):
        w, one = op.pcg(b[k], precond=pc, **args)
        e = rel(host(u[k]), host(w))
        say(f"[lor] p={p} n={n} nb={nb} lor32={lor32} neumann={neumann} k={k} iters={res.iters[k]} {one.iters[0]} "
            f"rel={e:.1e}")
        assert one.converged and res.iters[k] == one.iters[0] and e <= 1e-7, (k, e, res.iters[k], one.iters[0])
    op.close()
