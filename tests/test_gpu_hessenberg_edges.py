"""Real Ritz analyses at the orders where the eigenvectors' place changes: one per lane up
to 64, two beyond, in LDS up to 86, in global memory from 87 on."""
import pytest

from test_gpu_hessenberg import _hess, _real_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [63, 65, 85, 86, 87])
def test_real_solver_matches_lapack_at_the_edges(tsk, p):
    print(f"real hessenberg p={p}", flush=True)
    _real_check(tsk, _hess(p, 20 + p, False), 0.61)
