"""PCG on meshes whose vectors stay cached, where the number of the operator's
partial sums decides whether the reductions are fused."""
import pytest

import fixtures as F
from tests.test_gpu_cg_steps import _pcg

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K, N, prec, groups", [
    ((29, 29, 29), 3, "fp32", 24389), ((30, 29, 29), 3, "fp32", 25230),
    ((37, 37, 36), 4, "fp64", 24642), ((26, 26, 25), 6, "fp64", 16900),
    ((33, 32, 31), 5, "fp32", 32736), ((33, 32, 32), 5, "fp32", 33792)])
def test_both_sides_of_the_partials_limit(K, N, prec, groups):
    """24576 partial sums below N = 5 and 32768 from there, in the type named.
    Eight FP64 steps as in the step tests (1e-10), and the FP32 level to a true
    FP64 residual of 1e-9."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box(K, hi=(F.meshgen.TWO_PI,) * 3, deform=0.02), N,
                      precisions=("fp64", "fp32"))
    epb = op.get_tile(prec)["elements_per_block"]
    assert (K[0] * K[1] * K[2] + epb - 1) // epb == groups
    g = torch.Generator(device="cuda").manual_seed(N)
    b = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    want, _ = _pcg(op, b, torch.from_numpy(op.geometry()[2]).cuda(), 8)
    for kw in ({}, {"use_graph": False}, {"check_every": 3}):
        x, info = op.solve(b, tol=1e-14, max_iter=8, max_restart=0, raise_on_error=False, **kw)
        assert info["iterations"] == 8, (kw, info)
        err = float((x - want).abs().max() / want.abs().max())
        print(K, N, kw, "rel diff %.2e" % err, flush=True)
        assert err <= 1e-10, (kw, err)
    x, info = op.solve(b, tol=1e-9, precision="fp32")
    assert info["status"] == "SEM_OK" and info["fallback"] == "none", info
    assert float((b - op.ax(x)).norm() / b.norm()) <= 1.01e-9
