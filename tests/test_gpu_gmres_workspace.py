"""Device memory of the pressure solver."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


# elements, N, precisions, restart, and the bytes of the solver that summed the
# local solutions with atomics and needed no array for them
@pytest.mark.gpu
@pytest.mark.parametrize("K, N, precisions, restart, limit", [
    ((1, 1, 1), 4, ("fp64",), 1, 17356032), ((6, 5, 4), 3, ("fp64", "fp32"), 30, 19862784),
    ((9, 8, 7), 7, ("fp64", "fp16"), 2, 37314816), ((5, 5, 5), 9, ("fp64", "fp32"), 30, 70785280),
    ((24, 24, 24), 7, ("fp64",), 1, 455665152), ((24, 24, 24), 7, ("fp64", "fp32"), 30, 2713555456),
    ((12, 12, 12), 10, ("fp64", "fp32"), 1, 165068544), ((12, 12, 12), 13, ("fp64",), 1, 316572928)])
def test_workspace_is_no_larger_than_with_atomics(K, N, precisions, restart, limit):
    """The whole boxes are held where other arrays lie when they are not: from
    N = 7 on and on small meshes a mesh that fitted still fits.  The solve, over
    restarts and refinement steps, is that of the operator."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box(K), N, precisions=precisions)
    ps = sem.PressureSolver(op, restart=restart)
    print(K, N, precisions, restart, ps.workspace.numel(), limit, flush=True)
    assert ps.workspace.numel() <= limit
    if restart == 1:                              # steepest descent: far from the solution
        return
    g = torch.Generator(device="cuda").manual_seed(N)
    b = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    for prec in precisions:
        x, info = ps.solve(b, tol=1e-9, precision=prec)
        assert info["status"] == "SEM_OK", info
        assert float((b - op.ax(x)).norm() / b.norm()) <= 1.01e-9
