"""Local solves of the pressure preconditioner and their overlapping sum at
every order they take (boxes of 5^3 to 16^3 points: each has its own tiling
of the matrix cores), on elements with random local frames."""
import numpy as np
import pytest

import fixtures as F
from oracle import hybrid as HY
from tests.common import Pair, relerr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2207_07098_amd as sem  # noqa: E402


def mesh(N):
    # the oracle inverts every box as a dense matrix: fewer elements above
    K = (3, 2, 2) if N <= 7 else (2, 1, 1)
    return F.box(K, hi=(2.0, 1.0, 1.5), widths=[[1.0, 0.7, 1.2][:K[0]], [1.0, 0.8][:K[1]],
                                                [0.9, 1.0][:K[2]]],
                 dirichlet=(1, 1, 0, 1, 0, 0), reorient_seed=N)


@pytest.mark.parametrize("N", list(range(2, 14)))
def test_every_order_matches_oracle(N):
    """FP64: the Schwarz part and both parts to 1e-12.  FP32: a refined solve
    (FP32 local solves inside) meets 1e-10 without a hand-over, in about the
    FP64 solver's steps."""
    p = Pair(mesh(N), N, precisions=("fp64", "fp32"))
    hs = HY.HybridSchwarz(p.mesh, p.ora)
    ps = sem.PressureSolver(p.op, restart=30)
    r = p.ora.rhs_unique(F.random_unique(p.op.n_unique, N))
    rd = p.to_dev(r)
    z = p.from_dev(ps.precondition(rd, parts=ps.SCHWARZ))
    assert relerr(z, hs.schwarz(r)) < 1e-12
    z = p.from_dev(ps.precondition(rd))
    assert relerr(z, hs.apply(r)) < 1e-12
    x, info = ps.solve(rd, tol=1e-10)
    y, low = ps.solve(rd, tol=1e-10, precision="fp32")
    assert low["status"] == "SEM_OK" and low["fallback"] == "none", low
    assert p.ora.true_residual(p.from_dev(y), r) <= 1.01e-10
    assert low["iterations"] <= 2 * info["iterations"] + 8, (info, low)


def test_repeats_bitwise():
    """The sum runs in a fixed order: the Schwarz part repeats bitwise."""
    op = sem.Operator(F.box((5, 4, 3), reorient_seed=1), 6, precisions=("fp64",))
    ps = sem.PressureSolver(op, restart=2)
    g = torch.Generator(device="cuda").manual_seed(1)
    r = torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda")
    z = [ps.precondition(r, parts=ps.SCHWARZ) for _ in range(3)]
    assert torch.equal(z[0], z[1]) and torch.equal(z[0], z[2])
