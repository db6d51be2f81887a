"""Several float32 members of one coefficient, which from 400 workgroups of elements on are taken
in turn (p <= 4), against the same members one at a time and, where each has its own coefficient
or there are more than 8 in a solve, the (element, member) pairs.

Tolerances: two float32 applies differ by their roundings (1e-5 of the oracle each, 2e-6 of each
other at these orders); two solves to relative residual 1e-12 of an operator with a condition
number below 1e3 by 1e-9."""
import numpy as np
import pytest
import torch

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu

# elements per direction with just more than 400 workgroups of the CG kernels, and just fewer
SIZES = {1: (23, 22), 2: (19, 18), 3: (16, 15), 4: (15, 14)}


@pytest.mark.parametrize("use_nu", [False, True])
@pytest.mark.parametrize("big", [0, 1])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_members_in_turn(p, big, use_nu):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, Operator
    m = BoxMesh(SIZES[p][big], p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    rng = np.random.default_rng(p)
    nu = gpu(rng.uniform(0.5, 2.0, (m.nelem, (p + 2) ** 3))) if use_nu else None
    op.set_coeffs(1000.0, 1.0, nu)
    x = gpu(rng.uniform(-1, 1, (3, m.ndof)), torch.float32)
    for kind in (DIFFUSION, HELMHOLTZ):
        y = op.apply(x, op=kind)
        for k in range(3):
            e = rel(host(y[k]), host(op.apply(x[k], op=kind)))
            assert e <= 2e-6, (kind, k, e)
    for nb in (2, 3, 9):
        b = gpu(rng.uniform(-1, 1, (nb, m.ndof)))  # (essential entries not zero)
        u, res = op.pcg(b, rtol=1e-12, mode=1, check_every=4)
        assert res.converged, res
        for k in (0, nb - 1):
            w, one = op.pcg(b[k], rtol=1e-12, mode=0)
            e = rel(host(u[k]), host(w))
            assert one.converged and e <= 1e-9, (nb, k, e)
    say(f"[members] p={p} ne={m.ne} nu={use_nu} iters={res.iters}")
    op.close()


@pytest.mark.parametrize("p", [1, 4])
def test_own_coefficients_go_by_pairs(p):
    from paper_1910_03032_amd import HELMHOLTZ, Operator
    m = BoxMesh(SIZES[p][0], p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    rng = np.random.default_rng(p)
    nu = rng.uniform(0.5, 2.0, (2, m.nelem * (p + 2) ** 3))
    x = gpu(rng.uniform(-1, 1, (2, m.ndof)), torch.float32)
    op.set_coeffs(10.0, 1.0, gpu(nu))
    y = host(op.apply(x, op=HELMHOLTZ))
    for k in range(2):
        op.set_coeffs(10.0, 1.0, gpu(nu[k]))
        e = rel(y[k], host(op.apply(x[k], op=HELMHOLTZ)))
        assert e <= 2e-6, (k, e)
    op.close()
