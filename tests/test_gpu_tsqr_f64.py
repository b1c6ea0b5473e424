"""Float64 dense parts on the matrix cores (csrc/tsqr_f64.hpp): every column-block count, the leaf
and tree edges, batches of several widths, and non-finite input.  Against the float64 oracle with
longdouble-refined references; the bounds are those of the other float64 tests (1e-11 on p and on
the factor up to row signs: the problems' condition times a few hundred roundings of 1e-16)."""
import numpy as np
import pytest

from oracle import refine
from tests.gpu_util import gpu_solve_blockangular, log, p_err, sign_fix_rows
from workloads import generators as gen

pytestmark = pytest.mark.gpu


def _check_rb(inst, solver, f):
    RB = solver.get_factor()[2].cpu().numpy()
    L = inst.nB + 1
    got, = sign_fix_rows(RB[:L - 1, :L - 1])
    want, = sign_fix_rows(np.asarray(f.R_B, np.float64))
    assert np.linalg.norm(got - want) <= 1e-11 * np.linalg.norm(want)
    assert not np.tril(RB, -1).any()


# L = nB + 1 at the edges of the 16-column blocks, one width per block count at least
@pytest.mark.parametrize("nB", [0, 1, 14, 15, 16, 31, 40, 47, 60, 63, 64, 79, 90, 95, 96, 111, 112, 126, 127])
def test_every_width(nB):
    K = 120
    inst = gen.make_blockangular(900 + nB, K=K, m=(np.arange(K) % 9) + 4, n=3, nB=nB, lam=1e-2, dtype=np.float64)
    p_ref, f = refine.reference_solution(inst)
    for leaves in [1, 2, 3, 7, 16, 33, 0]:
        log(f"float64 dense part nB={nB} leaves={leaves}")
        p, st, solver, _ = gpu_solve_blockangular(inst, leaves=leaves, return_solver=True)
        assert st[0] == 0, st
        assert p_err(p, p_ref, inst.d) <= 1e-11
        if nB:
            _check_rb(inst, solver, f)


# rows per leaf around the tile heights (32, 48, 64, 96 and 128 rows) and one row over
@pytest.mark.parametrize("nB,tile", [(30, 128), (60, 128), (75, 96), (90, 64), (105, 48), (120, 32)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_tile_edges(nB, tile, extra):
    rows = 3 * (2 * tile + extra)
    m = np.full(rows // 8 + 1, 8)
    m[-1] = rows - 8 * (rows // 8)
    inst = gen.make_blockangular(31 + nB + extra, K=m.size, m=m, n=3, nB=nB, lam=1e-2, dtype=np.float64)
    p_ref, _ = refine.reference_solution(inst)
    log(f"float64 tile edge nB={nB} rows={rows}")
    p, st = gpu_solve_blockangular(inst, leaves=3)
    assert st[0] == 0, st
    assert p_err(p, p_ref, inst.d) <= 1e-11


@pytest.mark.parametrize("lam", [1e-2, 0.0])
@pytest.mark.parametrize("nB", [47, 90, 127])
def test_few_rows_per_leaf(nB, lam):
    """Leaves of far fewer rows than columns: the columns beyond their rank are reflected on
    roundoff that shrinks towards the subnormal range."""
    K = 40
    m = np.where(np.arange(K) % 2 == 0, 10, 56)
    inst = gen.make_blockangular(90 + nB, K=K, m=m, n=8, nB=nB, lam=lam, dtype=np.float64)
    p_ref, _ = refine.reference_solution(inst)
    for leaves in [1, 3, 40, 110, 1024]:
        log(f"float64 few rows per leaf nB={nB} lam={lam} leaves={leaves}")
        p, st = gpu_solve_blockangular(inst, leaves=leaves)
        assert st[0] == 0, st
        assert p_err(p, p_ref, inst.d) <= 1e-11


def test_batch_of_widths():
    import torch
    from paper_1802_03773_amd import BlockAngularBatch
    rng = np.random.default_rng(3)
    shapes = [(30, 0), (500, 90), (1, 20), (60, 127), (220, 6), (90, 60), (64, 75), (33, 100), (700, 30), (40, 90)]
    insts = [gen.make_blockangular(50 + i, K=K, m=rng.integers(3, 20, size=K), n=3, nB=nB, lam=10.0 ** (-1 - i % 3),
                                   dtype=np.float64) for i, (K, nB) in enumerate(shapes)]
    s = gen.stack_batch(insts)
    dev = {k: torch.from_numpy(np.ascontiguousarray(s[k])).cuda() for k in ("A", "B", "b", "d", "lam")}
    solver = BlockAngularBatch(s["K"], s["nB"], s["row_off"], s["n"], dtype="float64")
    for k in range(2):  # the second factor finds the flags of the first
        solver.factor(dev["A"], dev["B"], dev["b"], dev["d"], dev["lam"])
        p = solver.solve(sweeps=0).cpu().numpy()
        assert not solver.status_problems().any()
        at = 0
        for i, inst in enumerate(insts):
            p_ref, _ = refine.reference_solution(inst)
            log(f"float64 batch pass {k} problem {i} {shapes[i]}")
            assert p_err(p[at:at + inst.N], p_ref, inst.d) <= 1e-11
            at += inst.N


@pytest.mark.parametrize("nB", [20, 60, 90, 120])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite_reaches_the_status(nB, bad):
    inst = gen.make_blockangular(8, K=60, m=9, n=3, nB=nB, lam=1e-2, dtype=np.float64)
    inst.B[100, nB // 2] = bad
    log(f"float64 non-finite nB={nB} {bad}")
    _, st = gpu_solve_blockangular(inst, leaves=4)
    assert st[0] == 5, st  # QRK_ENONFINITE
