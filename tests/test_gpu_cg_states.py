"""CG of several members on both sides of the rule that has a launch of its own form the members'
states: few workgroups of few members, many workgroups, many members, by pairs and in turn.

Tolerance: as in test_gpu_cg_partials."""
import pytest

from test_gpu_cg_partials import same_as_single_solves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("p,n,nb", [(2, 14, 3), (2, 17, 3), (1, 6, 7), (1, 6, 8), (2, 4, 8), (8, 3, 7), (8, 3, 8),
                                    (2, 20, 3), (4, 19, 3), (5, 3, 9), (4, 19, 1), (1, 43, 1)])
def test_states_apart(p, n, nb, mode):
    same_as_single_solves(p, n, nb, mode, sorted({0, nb // 2, nb - 1}), check_every=5)
