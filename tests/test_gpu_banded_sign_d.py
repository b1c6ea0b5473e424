"""Banded Givens QR with damping values of either sign: only d^2 enters the step.  Columns that are small
next to their damping, so that a rotation's pivot is near -r before it.  Bounds of the other banded
tests (1e-11 float64, 1e-5 float32 unrefined, 1e-10 refined)."""
import dataclasses

import numpy as np
import pytest

from oracle import banded
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("w", [1, 12, 15, 16, 24])
def test_sign_of_d(w, dtype):
    import torch
    from paper_1802_03773_amd import BandedSolver
    rng = np.random.default_rng(w)
    inst = gen.make_banded(40 + w, N=77, w=w, lam=1.0, dtype=dtype)
    inst = dataclasses.replace(inst, d=inst.d * 10.0 ** rng.integers(0, 4 if dtype == np.float32 else 9, size=inst.N))
    p_ref = banded.reference_solution(inst)[0]
    d = inst.d * rng.choice([-1.0, 1.0], size=inst.N)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (inst.row_start, inst.vals, inst.b, d)]
    s = BandedSolver(inst.M, inst.N, w, dtype=np.dtype(dtype).name)
    s.factor(*dev, inst.lam)
    for sweeps, tol in ((0, 1e-11 if dtype == np.float64 else 1e-5), (2, 1e-10)):
        p = s.solve(sweeps=sweeps).cpu().numpy()
        log(f"sign of d w={w} {np.dtype(dtype).name} sweeps={sweeps}: {p_err(p, p_ref, inst.d):.2e}")
        assert s.status()[0] == 0
        assert p_err(p, p_ref, inst.d) <= tol
