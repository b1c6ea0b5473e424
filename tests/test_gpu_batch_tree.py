"""Float32 batches through the pipelined merge trees: every column-block count next to others, odd and
even leaf counts, problems of one leaf, and a second factor that finds the flags of the first.  Bounds
of the other float32 tests: 1e-5 unrefined, 1e-10 after two sweeps."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["plain", "bf16x3"])
@pytest.mark.parametrize("nBs", [(6,), (0, 30, 90), (14, 15, 16, 40, 63, 64, 75, 100, 127)])
def test_batch_trees(nBs, mode):
    import torch
    from paper_1802_03773_amd import BlockAngularBatch
    rng = np.random.default_rng(len(nBs))
    Ks = [40, 700, 90, 333, 170, 61, 512, 29, 250]
    insts = [gen.make_blockangular(60 + i, K=K, m=rng.integers(4, 20, size=K), n=3, nB=nBs[i % len(nBs)], lam=1e-2,
                                   dtype=np.float32) for i, K in enumerate(Ks)]
    refs = [refine.reference_solution(i)[0] for i in insts]
    s = gen.stack_batch(insts)
    dev = {k: torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")}
    solver = BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype="float32", mode=mode)
    for sweeps, tol in ((0, 1e-5), (2, 1e-10)):
        solver.factor(dev["A"], dev["B"], dev["b"], dev["d"], dev["lam"])
        p = solver.solve(sweeps=sweeps).cpu().numpy()
        assert not solver.status_problems().any()
        at = 0
        for i, inst in enumerate(insts):
            log(f"batch trees {mode} nBs={nBs} sweeps={sweeps} problem {i}")
            assert p_err(p[at:at + inst.N], refs[i], inst.d) <= tol
            at += inst.N
