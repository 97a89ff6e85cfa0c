"""Launch shapes of the operator's forms that store whole element blocks
(ax_local, the fixed-order sum): the result does not depend on the shape, and
the shape that a context starts with is not the one of the assembled operator
where that one is slow for them."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


def _op(K, N, precisions=("fp64", "fp32", "fp16"), **kw):
    import paper_2207_07098_amd as sem
    return sem.Operator(F.box(K, hi=(F.meshgen.TWO_PI,) * 3, deform=0.02), N,
                        precisions=precisions, solver=False, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15])
def test_results_do_not_depend_on_the_shape(N):
    """75 and 77 elements leave remainders of every group size.  An element's
    arithmetic is the same in any group, so the results are equal bitwise;
    against the atomic sum of the same factors they differ by the order of at
    most eight copies (a few units of rounding of the largest entry)."""
    for K in ((5, 5, 3), (11, 7, 1)):
        op = _op(K, N)
        g = torch.Generator(device="cuda").manual_seed(N)
        u = torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5
        uL = torch.rand(op.n_local, generator=g, dtype=torch.float64, device="cuda") - 0.5
        for prec, tol in (("fp64", 1e-14), ("fp32", 4e-6), ("fp16", 4e-6)):
            v, vL = (u, uL) if prec == "fp64" else (u.float(), uL.float())
            w, y = op.ax_local(vL, precision=prec), op.ax(v, precision=prec, deterministic=True)
            z = op.ax(v, precision=prec)
            assert float((y - z).abs().max()) <= tol * float(z.abs().max()), (K, prec)
            t = op.get_tile(prec)
            op.set_tile(prec, **t)               # changes nothing
            assert torch.equal(op.ax_local(vL, precision=prec), w)
            op.set_tile(prec, elements_per_block=1, grid_cap=0, xcd_remap=0, pipeline=0)
            assert torch.equal(op.ax_local(vL, precision=prec), w), (K, prec)
            assert torch.equal(op.ax(v, precision=prec, deterministic=True), y), (K, prec)


def _us(fn, reps=20, rounds=5):
    for _ in range(3):
        fn()
    out = []
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        b.synchronize()
        out.append(a.elapsed_time(b) / reps * 1e3)
    return min(out)


@pytest.mark.gpu
@pytest.mark.parametrize("K, N, prec, elements", [(45, 3, "fp32", 4), (45, 3, "fp16", 4),
                                                  (43, 4, "fp16", 5)])
def test_block_forms_fill_their_waves(K, N, prec, elements):
    """One element of low order per workgroup, good for the atomic form, leaves
    most of a wave idle: ax_local took 1.6 to 2 times as long with it."""
    op = _op((K, K, K), N, precisions=("fp64", prec))
    g = torch.Generator(device="cuda").manual_seed(N)
    uL = torch.rand(op.n_local, generator=g, dtype=torch.float32, device="cuda")
    wL = torch.empty_like(uL)
    first = _us(lambda: op.ax_local(uL, wL, precision=prec))
    op.set_tile(prec, elements_per_block=elements, grid_cap=0, xcd_remap=0, pipeline=0)
    shared = _us(lambda: op.ax_local(uL, wL, precision=prec))
    print("ax_local %s N = %d, %d^3: %.1f us, %d elements per workgroup %.1f us"
          % (prec, N, K, first, elements, shared), flush=True)
    assert first <= 1.25 * shared


@pytest.mark.gpu
@pytest.mark.parametrize("K, N, prec, better", [
    ((15, 15, 15), 5, "fp64", dict(elements_per_block=7, xcd_remap=1)),
    ((10, 10, 10), 10, "fp32", dict(elements_per_block=1, xcd_remap=1, pipeline=1)),
    ((9, 9, 9), 15, "fp16", dict(elements_per_block=1, xcd_remap=1, pipeline=1)),
    ((76, 76, 76), 3, "fp64", dict(elements_per_block=2, xcd_remap=1))])
def test_first_shape_is_not_a_slow_one(K, N, prec, better):
    """Sizes where the shape that fits larger or smaller meshes loses 10% and
    more: a second round of workgroups that is nearly empty, all factor planes
    in flight with few workgroups or at the largest order, no remap at a low
    order.  Both sides measured alike; equal shapes differ by 2%."""
    op = _op(K, N, precisions=("fp64", prec))
    g = torch.Generator(device="cuda").manual_seed(N)
    u = torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda")
    u = u if prec == "fp64" else u.float()
    y = torch.zeros_like(u)
    first = _us(lambda: op.ax(u, y, precision=prec), reps=50)
    z = op.ax(u, precision=prec)
    op.set_tile(prec, **{"grid_cap": 0, "pipeline": 0, **better})
    other = _us(lambda: op.ax(u, y, precision=prec), reps=50)
    tol = 1e-14 if prec == "fp64" else 4e-6       # copies summed in another order
    assert float((z - op.ax(u, precision=prec)).abs().max()) <= tol * float(z.abs().max())
    print("%s N = %d, %s: %.1f us, %s %.1f us" % (prec, N, K, first, better, other), flush=True)
    assert first <= 1.08 * other
