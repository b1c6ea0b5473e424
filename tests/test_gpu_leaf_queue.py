"""The persistent leaf launch (k_tsqr_queue, k_tsqr_queue_keep) and the launches per width it stands in for,
each forced through the autotuner's cache: every column-block count the queue holds (1 .. 6) beside 7 and 8,
more leaves than the launch has waves, both modes, with and without the stored Q.  Bounds of the other float32
tests: 1e-5 unrefined, 1e-10 after two sweeps."""
import json

import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu

NBS = [6, 20, 40, 55, 70, 90, 100, 120, 14]
KEY = "/n2/"  # the block width of no other test's tuned batch


@pytest.fixture(scope="module")
def problems():
    rng = np.random.default_rng(12)
    insts = [gen.make_blockangular(700 + i, K=300 + 37 * (i % 11), m=rng.integers(4, 21, size=300 + 37 * (i % 11)), n=2,
                                   nB=NBS[i % 9], lam=1e-2, dtype=np.float32) for i in range(27)]
    return insts, [refine.reference_solution(i)[0] for i in insts], gen.stack_batch(insts)


def _solver(s, mode):
    from paper_1802_03773_amd import BlockAngularBatch
    return BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype="float32", mode=mode)


@pytest.mark.parametrize("mode", ["plain", "bf16x3"])
@pytest.mark.parametrize("queue", [1, 0])
def test_both_leaf_launches(problems, tmp_path, mode, queue):
    import torch
    from paper_1802_03773_amd import qrkit
    insts, refs, s = problems
    dev = [torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")]
    path = tmp_path / "tune.json"
    qrkit.set_tune_cache(path)
    try:
        first = _solver(s, mode)
        first.factor(*dev)
        first.autotune()  # writes the entry of this shape
        data = json.loads(path.read_text())
        mine = [k for k in data["entries"] if f"/{mode}/" in k and KEY in k]
        assert len(mine) == 1, list(data["entries"])
        data["entries"][mine[0]] = {"leaf_scale": 1, "leaf_queue": queue, "refine_scale": 1, "ms": 1}
        path.write_text(json.dumps(data))
        qrkit.set_tune_cache(path)
        for keep in (False, True):
            solver = _solver(s, mode)
            assert qrkit.tune_choice(solver) == {"leaf_scale": 1, "leaf_queue": queue, "refine_scale": 1}
            solver.set_keep_q(keep)
            for sweeps, tol in ((0, 1e-5), (2, 1e-10)):  # the second factor finds the first's queue head
                solver.factor(*dev)
                p = (solver.solve_qt(dev[2], sweeps=sweeps) if keep else solver.solve(sweeps=sweeps)).cpu().numpy()
                assert not solver.status_problems().any()
                at = 0
                for i, inst in enumerate(insts):
                    e = p_err(p[at:at + inst.N], refs[i], inst.d)
                    log(f"leaf queue {queue} {mode} keep={keep} sweeps={sweeps} problem {i} nB={inst.nB}: {e:.2e}")
                    assert e <= tol
                    at += inst.N
    finally:
        qrkit.set_tune_cache(None)


def test_reported_choice_is_the_one_used():
    """An untuned batch of several widths and few rows runs a launch per width, and says so; one width, or
    float64, has no queue to choose."""
    from paper_1802_03773_amd import BlockAngularBatch, qrkit
    off = np.arange(0, 8 * 60 + 1, 8)
    for nBs, dtype, queue in (((6, 30), "float32", 0), ((6, 6), "float32", 1), ((6, 30), "float64", 1)):
        bt = BlockAngularBatch([30, 30], nBs, off, 1, dtype=dtype)
        assert qrkit.tune_choice(bt) == {"leaf_scale": 1, "leaf_queue": queue, "refine_scale": 1}, (nBs, dtype)
