"""A banded batch of 2^31 unknowns (2^21 problems of 1,024, two rows of one value each): the refinement's
launches cover every problem.  Against the step in closed form; 1e-10 after one sweep."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


def test_refined_step_of_2_31_unknowns():
    import torch
    from paper_1802_03773_amd import BandedSolver
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs about 120 GiB of free device memory")
    P, N, lam = 1 << 21, 1024, 0.5
    g = torch.Generator(device="cuda").manual_seed(1)
    rs = torch.tensor([3, N - 1], dtype=torch.int32, device="cuda").repeat(P, 1)
    vals = 1 + torch.rand(P, 2, 1, generator=g, device="cuda")
    b = torch.randn(P, 2, generator=g, device="cuda")
    d = torch.ones(P, N, dtype=torch.float64, device="cuda")
    s = BandedSolver(2, N, 1, dtype="float32", P=P)
    s.factor(rs, vals, b, d, lam)
    log("2^31 unknowns: factored")
    p = s.solve(sweeps=1).view(P, N)
    assert s.status()[0] == 0
    v, bb = vals.double().view(P, 2), b.double()
    want = v * bb / (v * v + lam)
    got = p[:, [3, N - 1]]
    e = ((got - want).abs().max() / want.abs().max()).item()
    log(f"2^31 unknowns: error {e:.2e}")
    assert e <= 1e-10
    assert p.count_nonzero() == want.count_nonzero()
