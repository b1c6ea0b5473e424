"""The dense triangular sweeps (csrc/solve.hip: back-substitution, refinement and adjoint), which go
by 16 x 16 blocks of the diagonal, at the edges of the blocks and of the triangle sizes 32, 64, 96
and 128.  Float32 after two refinement sweeps holds the 1e-10 of the other float32 tests; the float64
adjoint holds 1e-9 (the triangle's condition twice, times a few hundred roundings of 1e-16)."""
import numpy as np
import pytest

from oracle import adjoint, refine
from tests.gpu_util import gpu_solve_blockangular, log, p_err, rel_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 80, 95, 96, 97, 112, 113, 127]


@pytest.mark.parametrize("nB", WIDTHS)
def test_refined_step(nB):
    K = 90
    inst = gen.make_blockangular(700 + nB, K=K, m=(np.arange(K) % 9) + 4, n=3, nB=nB, lam=1e-2, dtype=np.float32)
    p_ref, _ = refine.reference_solution(inst)
    log(f"dense sweeps, refined step nB={nB}")
    p, st = gpu_solve_blockangular(inst, sweeps=2)
    assert st[0] == 0, st
    assert p_err(p, p_ref, inst.d) <= 1e-10


@pytest.mark.parametrize("nB", WIDTHS)
def test_adjoint(nB):
    import torch
    K = 90
    inst = gen.make_blockangular(800 + nB, K=K, m=(np.arange(K) % 9) + 4, n=3, nB=nB, lam=1e-2, dtype=np.float64)
    p_ref, f = refine.reference_solution(inst)
    log(f"dense sweeps, adjoint nB={nB}")
    p, st, solver, _ = gpu_solve_blockangular(inst, sweeps=1, return_solver=True)
    assert st[0] == 0, st
    g = np.cos(np.arange(inst.N))
    ref = adjoint.adjoint_blockangular(inst, f, p_ref, g)
    out = solver.solve_adjoint(torch.from_numpy(p).cuda(), torch.from_numpy(g).cuda())
    for k in ("dA", "dB", "db", "dd", "dlam"):
        assert rel_err(np.ravel(out[k].cpu().numpy()), np.ravel(ref[k])) <= 1e-9, k
