"""qrk_set_tsqr_shape: odd leaf counts, whose trees pass a leaf or a node up a level, and the fan-in argument,
which is accepted and has no effect (the same bits).  Bounds of the other tests of the dense part: 1e-11
float64, 1e-5 float32."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import gpu_solve_blockangular, log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(np.float32, 1e-5), (np.float64, 1e-11)])
@pytest.mark.parametrize("nB", [30, 100])
def test_odd_leaves_and_ignored_fan_in(nB, dtype, tol):
    inst = gen.make_blockangular(15, K=400, m=12, n=3, nB=nB, lam=1e-2, dtype=dtype)
    p_ref, _ = refine.reference_solution(inst)
    for leaves in (5, 7, 33, 255, 1001):
        log(f"leaves={leaves} nB={nB} {np.dtype(dtype).name}")
        p, st = gpu_solve_blockangular(inst, leaves=leaves)
        assert st[0] == 0
        assert p_err(p, p_ref, inst.d) <= tol
        for fanin in (2, 64):
            assert np.array_equal(gpu_solve_blockangular(inst, leaves=leaves, fanin=fanin)[0], p)
