"""The kernels of a PCG iteration against a PCG written with tensor operations
on the same operator, on both sides of the rule that fuses the reductions
into the vector kernels."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


def _pcg(op, b, dinv, steps):
    x, r = torch.zeros_like(b), b.clone()
    p = dinv * r
    rz = torch.dot(r, p)
    for _ in range(steps):
        w = op.ax(p)
        alpha = rz / torch.dot(p, w)
        x += alpha * p
        r -= alpha * w
        z = dinv * r
        rz, old = torch.dot(r, z), rz
        p = z + (rz / old) * p
    return x, r


@pytest.mark.gpu
@pytest.mark.parametrize("K, N", [((3, 1, 1), 2), ((5, 4, 3), 4), ((9, 8, 7), 7), ((16, 16, 16), 7),
                                  ((30, 29, 29), 7)])
def test_pcg_steps(K, N):
    """One workgroup with a tail, several, more vectors than the fused grid
    has lanes (1.4 M nodes), and vectors of 350 MB, which take the separate
    reductions.  Eight steps, FP64: each scalar carries the rounding of sums
    in another order, below sqrt(n) units (1e-12 at 8.7 M nodes at worst),
    and eight steps from a random right-hand side stay far from the loss of
    conjugacy, so x agrees to 1e-10 of its largest entry."""
    import paper_2207_07098_amd as sem
    m = F.box(K, hi=(F.meshgen.TWO_PI,) * 3, deform=0.02)
    op = sem.Operator(m, N, precisions=("fp64", "fp32"))
    g = torch.Generator(device="cuda").manual_seed(N)
    b = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
    dinv = torch.from_numpy(op.geometry()[2]).cuda()
    steps = 4 if op.n_unique < 200 else 8
    want, _ = _pcg(op, b, dinv, steps)
    for kw in ({}, {"deterministic": True}, {"use_graph": False}, {"check_every": 3}):
        x, info = op.solve(b, tol=1e-14, max_iter=steps, max_restart=0, raise_on_error=False, **kw)
        assert info["iterations"] == steps, (kw, info)
        err = float((x - want).abs().max() / want.abs().max())
        print(K, N, kw, "rel diff %.2e" % err, flush=True)
        assert err <= 1e-10, (kw, err)
    # the FP32 level (its replacement points pause the iteration) to a true
    # FP64 residual of 1e-9
    x, info = op.solve(b, tol=1e-9, precision="fp32")
    r = b - op.ax(x)
    assert info["status"] == "SEM_OK" and info["fallback"] == "none", info
    assert float(r.norm() / b.norm()) <= 1.01e-9


@pytest.mark.gpu
@pytest.mark.parametrize("meshes", [[((2, 1, 1), 2)], [((3, 2, 1), 4), ((1, 1, 1), 3), ((7, 6, 5), 7)],
                                    [((12, 11, 10), 9), ((2, 2, 2), 5)],
                                    [((21, 21, 21), 7)] * 3])
def test_batch_steps(meshes):
    """Eight batched FP64 steps against the single solves of the same
    problems (sums in another order only, as above): one item, items of
    several problems with odd sizes, more nodes than items of the smallest
    size hold, and 390 MB of vectors, which take the separate reductions.
    Then the FP32 inner iteration to a true FP64 residual of 1e-9."""
    import paper_2207_07098_amd as sem
    ops = [sem.Operator(F.box(K, hi=(F.meshgen.TWO_PI,) * 3, deform=0.02), N,
                        precisions=("fp64", "fp32")) for K, N in meshes]
    g = torch.Generator(device="cuda").manual_seed(3)
    rhs = [op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5)
           for op in ops]
    steps = 3 if min(op.n_unique for op in ops) < 200 else 8
    batch = sem.Batch(ops)
    for kw in ({}, {"use_graph": False}):
        xs, infos = batch.solve(rhs, tol=1e-14, max_iter=steps, raise_on_error=False, **kw)
        for op, b, x, info in zip(ops, rhs, xs, infos):
            want, one = op.solve(b, tol=1e-14, max_iter=steps, max_restart=0, raise_on_error=False)
            assert info["iterations"] == one["iterations"], (info, one)
            err = float((x - want).abs().max() / want.abs().max())
            print(op.n_unique, kw, info["iterations"], "rel diff %.2e" % err, flush=True)
            assert err <= 1e-10
    xs, infos = batch.solve(rhs, tol=1e-9, precision="fp32")
    for op, b, x, info in zip(ops, rhs, xs, infos):
        assert info["status"] == "SEM_OK" and info["fallback"] == "none", info
        assert float((b - op.ax(x)).norm() / b.norm()) <= 1.01e-9
