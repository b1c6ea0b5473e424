"""Float64 batches whose problems have fewer rows than a leaf takes: one leaf each, no merge slots are
allocated for them, and their steps are those of the oracle (1e-11)."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


def test_one_leaf_each():
    import torch
    from paper_1802_03773_amd import BlockAngularBatch
    P, K, m, nB, dtype, tol = 300, 3, 8, 127, np.float64, 1e-11
    insts = [gen.make_blockangular(20 + i, K=K, m=m, n=3, nB=nB, lam=1e-1, dtype=dtype) for i in range(6)]
    s = gen.stack_batch([insts[i % 6] for i in range(P)])
    dev = [torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")]
    solver = BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype=np.dtype(dtype).name)
    es, L = np.dtype(dtype).itemsize, nB + 1
    # R_B | c_B, S | c and the reduced rows, and 8 KiB for all the rest of a problem
    per = es * L * (L + K * 3 + K * m) + 8192
    log(f"one leaf each {np.dtype(dtype).name}: {solver.workspace_bytes() / P:.0f} bytes a problem, bound {per}")
    assert solver.workspace_bytes() <= P * per
    solver.factor(*dev)
    p = solver.solve(sweeps=0).cpu().numpy().reshape(P, -1)
    assert not solver.status_problems().any()
    for i, inst in enumerate(insts):
        p_ref = refine.reference_solution(inst)[0]
        assert p_err(p[i], p_ref, inst.d) <= tol
        assert np.array_equal(p[i], p[i + P - 6])
