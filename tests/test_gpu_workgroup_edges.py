"""Applies and flow kernels where a workgroup is not full or holds several waves' elements: meshes
of one element, and of numbers of elements around the 2 to 28 that a workgroup takes, for every
order (one wave per workgroup at p = 1, elements inside a wave at p = 2 and 6, two waves at p = 3).

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


def _setup(n, p):
    from paper_1910_03032_amd import Operator
    m = BoxMesh(n, p)
    return m, Discretization(m.elem_xyz, m.elem_dofs, m.ess, m.ndof, p, p + 2), \
        Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)


@pytest.mark.parametrize("nb", [1, 3])
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("p", range(1, 9))
def test_applies(p, n, nb):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, MASS
    m, d, op = _setup(n, p)
    op.set_coeffs(10.0, 0.5)
    x = np.random.default_rng(p).uniform(-1, 1, (nb, m.ndof))
    for kind, a, b in ((MASS, 1.0, 0.0), (DIFFUSION, 0.0, 1.0), (HELMHOLTZ, 10.0, 0.5)):
        ref = np.stack([d.apply(v, a, b, None) for v in x])
        e64 = rel(host(op.apply(gpu(x), op=kind)), ref)
        e32 = rel(host(op.apply(gpu(x, torch.float32), op=kind)), ref)
        say(f"[edges] p={p} n={n} nb={nb} op={kind} {e64:.1e} {e32:.1e}")
        assert e64 <= 1e-12 and e32 <= 1e-5, (kind, e64, e32)
    op.close()


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("p", range(1, 9))
def test_flow_kernels(p, n):
    from paper_1910_03032_amd import WEAK_CURL, WEAK_DIVERGENCE, WEAK_GRADIENT
    m, d, op = _setup(n, p)
    u = np.random.default_rng(p).uniform(-1, 1, (3, m.ndof))
    free = ~m.ess.astype(bool)
    for name, got, ref in (("convection", op.convection(gpu(u)), convection(d, u)),
                           ("curl", op.weak_op(WEAK_CURL, gpu(u)), weak_curl(d, u)),
                           ("divergence", op.weak_op(WEAK_DIVERGENCE, gpu(u)), weak_divergence(d, u)),
                           ("gradient", op.weak_op(WEAK_GRADIENT, gpu(u[0])), weak_gradient(d, u[0]))):
        got, ref = host(got)[..., free], np.asarray(ref)[..., free]
        e = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-300) if free.any() else 0.0
        say(f"[edges] p={p} n={n} {name} {e:.1e}")
        assert e <= 1e-12, (name, e)
    op.close()
