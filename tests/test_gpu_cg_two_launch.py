"""The two-launch CG iteration at the sizes where its bookkeeping can go wrong: more members than
a workgroup holds, a single element (no shared DoF), DoFs shared by more than 8 elements, and
essential DoFs with a nonzero right-hand side (each counted once in p.Ap).  Also the factors
formed from the trilinear map on stretched and sheared elements.

Tolerances: a solve to relative residual 1e-12 of operators with condition numbers below 1e3 is
within 1e-9 of the direct solution; an apply in float64 is within 1e-12 of the oracle, in
float32 within 1e-5."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
import torch

from gpu_common import gpu, host, rel, say
from oracle import Discretization
from workloads import BoxMesh, FanMesh

pytestmark = pytest.mark.gpu


def _solve_case(m, p, nb, ess_rhs, mode, seed=5):
    from paper_1910_03032_amd import Operator
    d = Discretization(m.elem_xyz, m.elem_dofs, m.ess, m.ndof, p, p + 2)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    op.set_coeffs(100.0, 1.0)
    b = np.random.default_rng(seed).uniform(-1, 1, (nb, m.ndof))
    if not ess_rhs:
        b[:, m.ess.astype(bool)] = 0.0
    x, res = op.pcg(gpu(b if nb > 1 else b[0]), rtol=1e-12, mode=mode, check_every=3)
    assert res.converged, res
    lu = spla.splu(d.assemble(100.0, 1.0).tocsc())
    xd = np.stack([lu.solve(v) for v in b])
    e = rel(host(x).reshape(nb, -1), xd)
    say(f"[cg] p={p} ndof={m.ndof} nb={nb} mode={mode} iters={res.iters} rel={e:.1e}")
    op.close()
    assert e <= 1e-9, e


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("ne,p,nb", [(1, 3, 1), (1, 8, 3), (2, 8, 5), (2, 7, 4), (3, 1, 30), (2, 4, 8)])
def test_members_beyond_a_workgroup_and_single_elements(ne, p, nb, mode):
    _solve_case(BoxMesh(ne, p), p, nb, True, mode)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("p,ess_rhs", [(1, True), (2, False), (3, True), (5, True)])
def test_dofs_of_more_than_eight_elements(p, ess_rhs, mode):
    _solve_case(FanMesh(p, nsect=6, nlayer=2), p, 2, ess_rhs, mode)


@pytest.mark.parametrize("p", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("stretch,shear,shift", [(1e-3, 0.0, 0.0), (30.0, 2.0, 1e3)])
def test_factors_of_stretched_and_sheared_elements(p, stretch, shear, shift):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, Operator
    m = BoxMesh(2, p)
    xyz = m.elem_xyz.copy()
    xyz[..., 2] *= stretch
    xyz[..., 0] += shear * xyz[..., 1] + shift
    d = Discretization(xyz, m.elem_dofs, m.ess, m.ndof, p, p + 2)
    op = Operator(xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    nu = np.random.default_rng(2).uniform(0.5, 2.0, (m.nelem, (p + 2) ** 3))
    x = np.random.default_rng(3).uniform(-1, 1, m.ndof)
    # the coordinates carry 2^-53 shift; the element size is 0.5 (and stretch)
    tol = 1e-12 + 1e-15 * abs(shift)
    for use_nu in (False, True):
        op.set_coeffs(10.0, 0.5, gpu(nu) if use_nu else None)
        for kind, a, b in ((DIFFUSION, 0.0, 1.0), (HELMHOLTZ, 10.0, 0.5)):
            ref = d.apply(x, a, b, nu if use_nu else None)
            e64 = rel(host(op.apply(gpu(x), op=kind)), ref)
            e32 = rel(host(op.apply(gpu(x, torch.float32), op=kind)), ref)
            say(f"[geom] p={p} stretch={stretch} nu={use_nu} op={kind}: {e64:.1e} {e32:.1e}")
            assert e64 <= tol and e32 <= 1e-5 + tol, (e64, e32)
    op.close()
