"""One application of the FP32 preconditioner against the FP64 one."""
import pytest

import fixtures as F
from tests.test_gpu_local_solves import mesh

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("N", list(range(2, 14)))
def test_fp32_application(N):
    """A refined solve whose inner cycle is one step, stopped by its tolerance
    after one correction: x = |b| y z with z the FP32 preconditioner's image of
    b / |b| and y from one least-squares coefficient, here with the FP64
    preconditioner.  FP32 rounding of six contractions of at most 16 terms is
    6 x 16 x 6e-8 of the terms' size, 16 times that (1e-4) where they cancel; a
    16-bit product or sum anywhere would leave 4e-3."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(mesh(N), N, precisions=("fp64", "fp32"))
    ps = sem.PressureSolver(op, restart=1)
    g = torch.Generator(device="cuda").manual_seed(N)
    b = op.rhs(f_unique=torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    bn = float(b.norm())
    z = ps.precondition(b / bn)
    w = op.ax(z)
    y = float(torch.dot(b / bn, w) / torch.dot(w, w))
    want = bn * y * z
    left = float((b - op.ax(want)).norm()) / bn
    assert left < 0.999
    x, info = ps.solve(b, tol=0.5 * (1.0 + left), precision="fp32")
    assert info["status"] == "SEM_OK" and info["iterations"] == 1 and info["outer_iterations"] == 1, info
    err = float((x - want).abs().max() / want.abs().max())
    print("N = %d: %.1e" % (N, err), flush=True)
    assert err <= 1e-4
