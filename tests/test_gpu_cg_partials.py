"""CG of several members where the partial sums of p.Ap are many: more than 32768 a member, which a
launch of its own folds, with fewer and with more members than a workgroup has pairs.

Tolerance: two solves to relative residual 1e-12 of an operator with a condition number below 1e3
differ by less than 1e-9."""
import numpy as np
import pytest

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu


def same_as_single_solves(p, n, nb, mode, members, check_every=4):
    from paper_1910_03032_amd import Operator
    m = BoxMesh(n, p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    op.set_coeffs(100.0 * n * n, 1.0)
    b = gpu(np.random.default_rng(p + nb).uniform(-1, 1, (nb, m.ndof)))
    u, res = op.pcg(b, rtol=1e-12, mode=mode, check_every=check_every)
    assert res.converged, res
    for k in members:
        w, one = op.pcg(b[k], rtol=1e-12, mode=0)
        e = rel(host(u[k]), host(w))
        say(f"[cg] p={p} n={n} nb={nb} mode={mode} k={k} iters={res.iters[k]} {one.iters[0]} rel={e:.1e}")
        assert one.converged and e <= 1e-9, (k, e)
        assert mode == 1 or abs(res.iters[k] - one.iters[0]) <= 1, (res.iters[k], one.iters)
    op.close()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("p,n,nb", [(1, 33, 32), (1, 49, 8)])
def test_folded_partials(p, n, nb, mode):
    same_as_single_solves(p, n, nb, mode, (0, 1, nb - 1))
