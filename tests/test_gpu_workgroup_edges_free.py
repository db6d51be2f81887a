"""Applies and flow kernels without essential DoFs, every row compared: one element, workgroups partly
filled, filled and followed by another that is partly filled (at p = 1 a flow workgroup takes 28
elements and an apply's 7, so 27 and 64 elements).

Tolerances: float64 results are within 1e-12 of the oracle, float32 ones within 1e-5."""
import numpy as np
import pytest
import torch

from gpu_common import gpu, host, rel, say
from oracle import Discretization
from oracle.flow import weak_curl, weak_divergence, weak_gradient
from oracle.stokes import convection
from workloads import BoxMesh

pytestmark = pytest.mark.gpu

CASES = [(p, n) for p in range(1, 9) for n in (1, 2, 3)] + [(1, 4), (2, 4)]


def _setup(n, p):
    from paper_1910_03032_amd import Operator
    m = BoxMesh(n, p)
    free = np.zeros(m.ndof, dtype=np.uint8)
    return m, Discretization(m.elem_xyz, m.elem_dofs, free, m.ndof, p, p + 2), \
        Operator(m.elem_xyz, m.elem_dofs, m.ndof, p)


@pytest.mark.parametrize("nb", [1, 3])
@pytest.mark.parametrize("p,n", CASES)
def test_applies(p, n, nb):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, MASS
    m, d, op = _setup(n, p)
    op.set_coeffs(10.0, 0.5)
    x = np.random.default_rng(p).uniform(-1, 1, (nb, m.ndof))
    for kind, a, b in ((MASS, 1.0, 0.0), (DIFFUSION, 0.0, 1.0), (HELMHOLTZ, 10.0, 0.5)):
        ref = np.stack([d.apply(v, a, b, None) for v in x])
        e64 = rel(host(op.apply(gpu(x), op=kind)), ref)
        e32 = rel(host(op.apply(gpu(x, torch.float32), op=kind)), ref)
        say(f"[free] p={p} n={n} nb={nb} op={kind} {e64:.1e} {e32:.1e}")
        assert np.linalg.norm(ref) > 0 and e64 <= 1e-12 and e32 <= 1e-5, (kind, e64, e32)
    op.close()


@pytest.mark.parametrize("p,n", CASES)
def test_flow_kernels(p, n):
    from paper_1910_03032_amd import WEAK_CURL, WEAK_DIVERGENCE, WEAK_GRADIENT
    m, d, op = _setup(n, p)
    u = np.random.default_rng(p).uniform(-1, 1, (3, m.ndof))
    for name, got, ref in (("convection", op.convection(gpu(u)), convection(d, u)),
                           ("curl", op.weak_op(WEAK_CURL, gpu(u)), weak_curl(d, u)),
                           ("divergence", op.weak_op(WEAK_DIVERGENCE, gpu(u)), weak_divergence(d, u)),
                           ("gradient", op.weak_op(WEAK_GRADIENT, gpu(u[0])), weak_gradient(d, u[0]))):
        ref = np.asarray(ref)
        e = rel(host(got), ref)
        say(f"[free] p={p} n={n} {name} {e:.1e}")
        assert np.linalg.norm(ref) > 0 and e <= 1e-12, (name, e)
    op.close()
