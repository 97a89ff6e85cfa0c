"""Launch shapes that a context starts with, where their rule changes: the
operator of the default tile against one element per workgroup."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K, N", [((13, 13, 13), 8), ((13, 13, 12), 8), ((32, 32, 32), 7),
                                  ((11, 7, 5), 2), ((11, 7, 5), 3), ((11, 7, 5), 5),
                                  ((5, 3, 3), 9), ((3, 3, 3), 11)])
def test_default_tile_against_single_elements(K, N):
    """Remainder groups and both sides of the element-count thresholds (2048
    at N = 8, 32768 at N = 7).  The sums of at most eight shared copies run
    in another order: a few units of rounding of the largest entry, FP64 and
    FP32 (the factors and the element arithmetic are the same)."""
    import paper_2207_07098_amd as sem
    m = F.box(K, hi=(F.meshgen.TWO_PI,) * 3, deform=0.02)
    op = sem.Operator(m, N, precisions=("fp64", "fp32", "fp16"), solver=False)
    g = torch.Generator(device="cuda").manual_seed(N)
    u = torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5
    for prec, tol in (("fp64", 1e-14), ("fp32", 4e-6), ("fp16", 4e-6)):
        v = u if prec == "fp64" else u.float()
        y = op.ax(v, precision=prec)
        op.set_tile(prec, elements_per_block=1, grid_cap=16, xcd_remap=0, pipeline=0)
        z = op.ax(v, precision=prec)
        assert float((y - z).abs().max()) <= tol * float(z.abs().max()), prec
    # the E-vector form takes its own planes in flight; Q does not mask, so
    # the Dirichlet entries of u are cleared first
    _, pos, dm, _ = op.numbering()
    u[torch.from_numpy(pos[dm == 1].astype("int64")).cuda()] = 0.0
    y, z = op.scatter(op.ax_local(op.gather(u))), op.ax(u)
    assert float((y - z).abs().max()) <= 1e-13 * float(z.abs().max())
