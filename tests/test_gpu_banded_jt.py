"""J^T r of the banded refinement (k_banded_jt) over row ranges of one and of several chunks, with odd and
even chunk lengths and row counts, and many rows on few starts.  A float32 factor's refinement reaches 1e-10 in
two sweeps (a float64 one's stays at 1e-11) only if every row is counted once."""
import numpy as np
import pytest

from oracle import banded
from tests.gpu_util import log, p_err
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# a workgroup's range holds at most 576 rows and 24 KiB of values at a time (one value a column: fewer columns,
# more rows)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("N,w,rows", [(300, 1, 300), (400, 3, 511), (260, 4, 5000), (129, 12, 2600), (128, 15, 1811),
                                      (40, 12, 3000), (200, 16, 1601), (150, 31, 1203), (31, 31, 600)])
def test_rows_of_several_chunks(N, w, rows, dtype):
    import torch
    from paper_1802_03773_amd import BandedSolver
    rng = np.random.default_rng(N + w)
    insts = []
    for k in range(3):
        span = N - w + 1
        starts = np.sort(rng.integers(0, span, size=rows) if k != 1 else rng.choice([0, span // 2, span - 1], size=rows))
        vals, b = rng.standard_normal((rows, w)).astype(dtype), rng.standard_normal(rows).astype(dtype)
        rs = starts.astype(np.int32)
        insts.append(gen.Banded(N, w, rs, vals, b, gen.column_norms_banded(N, w, rs, vals), 1e-1, np.dtype(dtype)))
    dev = [torch.from_numpy(np.stack([getattr(i, k) for i in insts])).cuda() for k in ("row_start", "vals", "b", "d")]
    s = BandedSolver(rows, N, w, dtype=np.dtype(dtype).name, P=3)
    s.factor(*dev, 1e-1)
    p = s.solve(sweeps=2).cpu().numpy().reshape(3, N)
    for k, inst in enumerate(insts):
        e = p_err(p[k], banded.reference_solution(inst)[0], inst.d)
        log(f"J^T r N={N} w={w} rows={rows} {np.dtype(dtype).name} problem {k}: {e:.2e}")
        assert e <= (1e-10 if dtype == np.float32 else 1e-11)
