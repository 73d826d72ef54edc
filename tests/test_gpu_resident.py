"""MINRES with its vectors on chip (registers and LDS), against the oracle.

In the problem array each chain length takes its own number of rows per
thread, and n falls just above or below whole rows of the workgroup
(n = 6, 20, 70, 252 of 512 threads; 924 of 2 x 512; 3432 of 7 x 512). Bars:
those of the problem-array tests against dense eigenpairs.
"""
import numpy as np
import pytest

from test_gpu_problems import _check_dense
from workloads import disorder_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,nev,precond", [(4, 2, "row"), (6, 3, "id"), (8, 5, "row"),
                                           (10, 4, "jacobi"), (12, 4, "id"), (14, 3, "row")])
def test_problem_array_on_chip(gpu, L, nev, precond):
    f = disorder_fields(L, 3.0, 600 + L)
    st, res = gpu.si_lanczos_problems([dict(L=L, h=f, nev=nev)], seed=4, precond=precond,
                                      minres_kmax=400_000)
    print(f"L={L} {precond}: steps {res[0].steps}, {res[0].minres_iters} iterations", flush=True)
    assert st == 0
    _check_dense(L, f, res[0], nev)


def test_problem_array_iteration_limit(gpu):
    """kmax iterations per solve and no more, and a warning."""
    f = disorder_fields(12, 3.0, 612)
    st, res = gpu.si_lanczos_problems([dict(L=12, h=f, nev=2, sigma=0.1)], mmax=3, minres_kmax=7)
    assert st == 1 and res[0].status == 1
    assert res[0].steps == 3 and res[0].minres_iters == 21
