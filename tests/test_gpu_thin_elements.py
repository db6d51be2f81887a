"""Float32 operators on elements whose edges are nearly parallel (boxes sheared by up to 1e6 and
turned): their factors come from adj(J), whose entries keep their digits there, not from the metric.

Tolerance: float32 results are within 1e-5 of the float64 ones, as on ordinary elements; the shear
enters both through the same adj(J) and |J| in float64.  The refined solve to 1e-12 of an operator
that its mass term dominates (condition number below 1e3) is within 1e-9 of the float64 one."""
import numpy as np
import pytest
import torch

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu


def _sheared(n, p, kind, a):
    from paper_1910_03032_amd import Operator
    m = BoxMesh(n, p)
    xyz = m.elem_xyz.copy()
    if kind == "one":      # needles: xi_1 and xi_3 almost along z
        xyz[..., 2] += a * xyz[..., 0]
    else:                  # all three directions almost along x
        xyz[..., 0] += a * (xyz[..., 1] + xyz[..., 2])
    q, _ = np.linalg.qr(np.random.default_rng(11).standard_normal((3, 3)))
    q *= np.sign(np.linalg.det(q))
    return m, Operator(xyz @ q.T, m.elem_dofs, m.ndof, p, ess=m.ess)


# shears of 300 are below the limit for the metric, of 3000 just above it; 23^3 elements at p = 1 are
# above 400 workgroups (their vertices in float64 are too coarse for the last shear)
SMALL = [(1, 3), (2, 3), (3, 2), (4, 2), (5, 2), (6, 2), (7, 2), (8, 2)]
CASES = [(p, n, k, a) for p, n in SMALL + [(1, 23)]
         for k, a in (("one", 300.0), ("one", 3000.0), ("one", 1e6), ("all", 1e6)) if (n, k) != (23, "all")]


@pytest.mark.parametrize("p,n,kind,a", CASES)
def test_float32_applies(p, n, kind, a):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ
    m, op = _sheared(n, p, kind, a)
    rng = np.random.default_rng(p)
    nu = gpu(rng.uniform(0.5, 2.0, (m.nelem, (p + 2) ** 3)))
    x = rng.uniform(-1, 1, (3, m.ndof))
    for use_nu in (False, True):
        op.set_coeffs(10.0, 0.5, nu if use_nu else None)
        for op_kind in (DIFFUSION, HELMHOLTZ):
            y64 = host(op.apply(gpu(x), op=op_kind))
            y32 = host(op.apply(gpu(x, torch.float32), op=op_kind))
            e = max(rel(y32[k], y64[k]) for k in range(3))
            e1 = rel(host(op.apply(gpu(x[0], torch.float32), op=op_kind)), y64[0])
            say(f"[thin] p={p} n={n} {kind} {a:.0e} nu={use_nu} op={op_kind}: {e:.1e} {e1:.1e}")
            assert e <= 1e-5 and e1 <= 1e-5, (e, e1)
    op.close()


@pytest.mark.parametrize("p,n", [(1, 23), (2, 3), (4, 2), (5, 2), (8, 2)])
def test_refined_solve(p, n):
    a = 3000.0
    m, op = _sheared(n, p, "one", a)
    op.set_coeffs(100.0 * (a * n * p * p) ** 2, 1.0)
    b = gpu(np.random.default_rng(p).uniform(-1, 1, (2, m.ndof)))
    u, res = op.pcg(b, rtol=1e-12, mode=1, check_every=3)
    w, one = op.pcg(b, rtol=1e-12, mode=0)
    e = rel(host(u), host(w))
    say(f"[thin] solve p={p} n={n} iters={res.iters} {one.iters} rel={e:.1e}")
    assert res.converged and one.converged and e <= 1e-9, e
    op.close()
