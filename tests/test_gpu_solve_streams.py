"""Row streams of the solve kernels (csrc/solve.hip): units of the block solves and packs of the
refinement at their edges -- one block, units and packs just full and one over, blocks without rows,
every block width class -- at the stream widths 16, 32, 64 and 128.  Float32 after two refinement
sweeps holds the 1e-10 of the other float32 tests, float64 the 1e-11 of the float64 tests."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import gpu_solve_blockangular, log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nB", [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 127])
@pytest.mark.parametrize("n", [1, 3, 8])
def test_units_and_packs(n, nB):
    for K in [1, 2, 5, 16, 21, 22, 64, 65, 300]:
        tall = n + 9 + nB // K  # enough rows in all for the coupled columns
        if tall > 56:
            continue
        m = np.where(np.arange(K) % 3 == 2, tall, tall - (np.arange(K) % 4))
        for dtype, sweeps, tol in ((np.float32, 2, 1e-10), (np.float64, 1, 1e-11)):
            inst = gen.make_blockangular(40 + nB + K, K=K, m=m, n=n, nB=nB, lam=1e-2, dtype=dtype)
            p_ref, _ = refine.reference_solution(inst)
            log(f"streams n={n} nB={nB} K={K} {np.dtype(dtype).name}")
            p, st = gpu_solve_blockangular(inst, sweeps=sweeps)
            assert st[0] == 0, st
            assert p_err(p, p_ref, inst.d) <= tol


@pytest.mark.parametrize("nB", [0, 6, 30, 60, 90])
@pytest.mark.parametrize("heights", [[0, 9], [0, 0, 0, 20], [1], [56, 0, 8], [2, 1, 0, 3, 40]])
def test_block_heights(heights, nB):
    """Blocks without rows (damped only), packs that end on one, one-row and 56-row blocks."""
    K = 200
    m = np.resize(heights, K)
    inst = gen.make_blockangular(70 + nB, K=K, m=m, n=3, nB=nB, lam=1.0, dtype=np.float32)
    inst.d = np.ones_like(inst.d)  # fewer rows than unknowns: the damping alone bounds the condition
    p_ref, _ = refine.reference_solution(inst)
    log(f"streams heights={heights} nB={nB}")
    p, st = gpu_solve_blockangular(inst, sweeps=2)
    assert st[0] == 0, st
    assert p_err(p, p_ref, inst.d) <= 1e-10


@pytest.mark.parametrize("n,nB", [(1, 16), (3, 30), (3, 90), (5, 64), (8, 127)])
@pytest.mark.parametrize("heights", [[0, 9], [0, 0, 0, 20], [12], [56, 0, 8]])
def test_adjoint_rows(heights, n, nB):
    """The adjoint's streams in float64 on the same heights; 1e-9 as in the other adjoint tests."""
    import torch
    from oracle import adjoint
    from tests.gpu_util import rel_err
    K = 150
    inst = gen.make_blockangular(30 + nB, K=K, m=np.resize(heights, K), n=n, nB=nB, lam=1.0, dtype=np.float64)
    inst.d = np.ones_like(inst.d)
    p_ref, f = refine.reference_solution(inst)
    log(f"adjoint streams heights={heights} n={n} nB={nB}")
    p, st, solver, _ = gpu_solve_blockangular(inst, sweeps=1, return_solver=True)
    assert st[0] == 0, st
    g = np.cos(np.arange(inst.N))
    ref = adjoint.adjoint_blockangular(inst, f, p_ref, g)
    out = solver.solve_adjoint(torch.from_numpy(p).cuda(), torch.from_numpy(g).cuda())
    for k in ("dA", "dB", "db", "dd", "dlam"):
        assert rel_err(np.ravel(out[k].cpu().numpy()), np.ravel(ref[k])) <= 1e-9, k
