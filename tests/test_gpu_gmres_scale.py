"""FP32 local solves on meshes whose eigenvalue sums are subnormal in FP32."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("h", [4e19, 5e19, 1e20])
def test_subnormal_eigenvalue_sums(h):
    """Element lengths of 4e19 and more: the refined solve goes on as the FP64
    one does (at such lengths the elements at the boundary get no local solve,
    so neither converges in 100 steps) instead of meeting a NaN in its first
    step."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box((4, 4, 4), hi=(4 * h,) * 3), 5, precisions=("fp64", "fp32"))
    ps = sem.PressureSolver(op)
    g = torch.Generator(device="cuda").manual_seed(1)
    b = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    for prec in ("fp64", "fp32"):
        x, info = ps.solve(b, tol=1e-10, precision=prec, max_iter=100, raise_on_error=False)
        assert info["status"] in ("SEM_OK", "SEM_ERR_NOT_CONVERGED"), (prec, info)
        assert info["iterations"] >= 1 and info["true_rel_residual"] < 1.0, (prec, info)
        assert bool(torch.isfinite(x).all())
