"""Float32 applies of several members of one coefficient at p = 5 and 6, in turn from 3200 waves on (16^3
elements at p = 5, 15^3 at p = 6), on both sides of the rule against the members one at a time.

Tolerance: two float32 applies differ by their roundings, by less than 2e-6 at these orders."""
import numpy as np
import pytest
import torch

from gpu_common import gpu, host, rel, say
from workloads import BoxMesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [2, 3, 9])
@pytest.mark.parametrize("use_nu", [False, True])
@pytest.mark.parametrize("p,n", [(5, 15), (5, 16), (6, 14), (6, 15)])
def test_members_in_turn(p, n, use_nu, nb):
    from paper_1910_03032_amd import DIFFUSION, HELMHOLTZ, Operator
    m = BoxMesh(n, p)
    op = Operator(m.elem_xyz, m.elem_dofs, m.ndof, p, ess=m.ess)
    rng = np.random.default_rng(p)
    op.set_coeffs(1000.0, 1.0, gpu(rng.uniform(0.5, 2.0, (m.nelem, (p + 2) ** 3))) if use_nu else None)
    x = gpu(rng.uniform(-1, 1, (nb, m.ndof)), torch.float32)
    for kind in (DIFFUSION, HELMHOLTZ):
        y = op.apply(x, op=kind)
        e = max(rel(host(y[k]), host(op.apply(x[k], op=kind))) for k in range(nb))
        say(f"[members] p={p} n={n} nb={nb} nu={use_nu} op={kind}: {e:.1e}")
        assert e <= 2e-6, (kind, e)
    op.close()
