"""The first steps of the pressure solver against a flexible GMRES written
with tensor operations on the same operator and preconditioner."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


def _fgmres(op, ps, b, cycles):
    x = torch.zeros_like(b)
    for steps in cycles:
        r = b - op.ax(x)
        V, Z = [r / r.norm()], []
        H = torch.zeros(steps + 1, steps, dtype=torch.float64)
        for j in range(steps):
            Z.append(ps.precondition(V[j]))
            w = op.ax(Z[j])
            for _ in range(2):
                for i in range(j + 1):
                    h = torch.dot(V[i], w)
                    H[i, j] += h.cpu()
                    w = w - h * V[i]
            H[j + 1, j] = w.norm().cpu()
            V.append(w / w.norm())
        g = torch.zeros(steps + 1, 1, dtype=torch.float64)
        g[0] = r.norm().cpu()
        y = torch.linalg.lstsq(H, g).solution[:, 0]
        for j in range(steps):
            x = x + float(y[j]) * Z[j]
    return x


@pytest.mark.gpu
@pytest.mark.parametrize("K, N", [((3, 3, 2), 3), ((6, 5, 4), 6), ((11, 10, 9), 7)])
def test_capped_and_restarted_steps(K, N):
    """Caps of one to four steps in one cycle and, with cycles of two, over a
    restart: the iterate is that of the steps asked for, whatever the solver
    has queued beyond them, and a solve that runs to 1e-9 afterwards is not
    disturbed.  Odd and even lengths.  Four well-separated steps lose a few
    digits to the least squares at most: x agrees to 1e-9 of its largest
    entry."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box(K, deform=0.02), N, precisions=("fp64", "fp32"))
    g = torch.Generator(device="cuda").manual_seed(N)
    b = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    for m, cap, cycles in ((30, 1, [1]), (30, 2, [2]), (30, 4, [4]), (2, 2, [2]), (2, 3, [2, 1])):
        ps = sem.PressureSolver(op, restart=m)
        x, info = ps.solve(b, tol=1e-13, max_iter=cap, raise_on_error=False)
        assert info["iterations"] == cap, info
        want = _fgmres(op, ps, b, cycles)
        err = float((x - want).abs().max() / want.abs().max())
        print(K, N, m, cap, "rel diff %.2e" % err, flush=True)
        assert err <= 1e-9
        for prec in ("fp64", "fp32"):
            x, info = ps.solve(b, tol=1e-9, precision=prec)
            assert info["status"] == "SEM_OK", info
            assert float((b - op.ax(x)).norm() / b.norm()) <= 1.01e-9
