"""Merge trees of two handles on two streams at once: the nodes of each launch wait for nodes of the same
launch only once those have started, so neither can keep the other's out.  Every factor's step equals,
bit for bit, the one of the handle alone, and no status word is set."""
import numpy as np
import pytest

from tests.gpu_util import log
from workloads import generators as gen

pytestmark = pytest.mark.gpu


def _batch(seed, P, K, nB, dtype):
    import torch
    from paper_1802_03773_amd import BlockAngularBatch
    insts = [gen.make_blockangular(seed + i, K=K, m=10, n=3, nB=nB, lam=1e-2, dtype=dtype) for i in range(P)]
    s = gen.stack_batch(insts)
    dev = [torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")]
    return BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype=np.dtype(dtype).name), dev


# 30 trees of 55 leaves at 8 column blocks: more nodes than the GPU holds at once
@pytest.mark.parametrize("other", [(30, 700, 120, np.float32), (24, 250, 100, np.float64)])
def test_trees_on_two_streams(other):
    import torch
    sides = [_batch(500, 30, 700, 120, np.float32), _batch(900, *other)]
    alone = []
    for solver, dev in sides:
        solver.factor(*dev)
        alone.append(solver.solve(sweeps=0).clone())
        torch.cuda.synchronize()
        assert not solver.status_problems().any()
    streams = [torch.cuda.Stream() for _ in sides]
    for rep in range(6):
        log(f"two streams {other} pass {rep}")
        p = []
        for (solver, dev), st in zip(sides, streams):
            with torch.cuda.stream(st):
                for _ in range(3):
                    solver.factor(*dev)
                p.append(solver.solve(sweeps=0))
        torch.cuda.synchronize()
        for k, (solver, _) in enumerate(sides):
            assert torch.equal(p[k], alone[k])
            assert not solver.status_problems().any()
