"""Float32 batches of 8 column blocks with more rows than a tile of 96 for each wave of a round: their leaves
are whole tiles (108,000 rows: two).  Batches of fewer rows are in test_gpu_batch_tree.py.  Bounds of the
other float32 tests: 1e-5 unrefined, 1e-10 after two sweeps."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nBs,Ks", [((120,), (6000, 11900, 100))])
def test_wide_leaves(nBs, Ks):
    import torch
    from paper_1802_03773_amd import BlockAngularBatch
    insts = [gen.make_blockangular(80 + i, K=K, m=6, n=3, nB=nBs[i % len(nBs)], lam=1e-2, dtype=np.float32)
             for i, K in enumerate(Ks)]
    refs = [refine.reference_solution(i)[0] for i in insts]
    s = gen.stack_batch(insts)
    dev = [torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")]
    for mode in ("plain", "bf16x3"):
        solver = BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype="float32", mode=mode)
        solver.factor(*dev)
        for sweeps, tol in ((0, 1e-5), (2, 1e-10)):
            p = solver.solve(sweeps=sweeps).cpu().numpy()
            assert not solver.status_problems().any()
            at = 0
            for i, inst in enumerate(insts):
                e = p_err(p[at:at + inst.N], refs[i], inst.d)
                log(f"wide leaves {mode} nBs={nBs} sweeps={sweeps} problem {i}: {e:.2e}")
                assert e <= tol
                at += inst.N
