"""A preconditioner application that ends with an error leaves nothing behind
for the next one."""
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("parts", [2, 3])
def test_failed_application_leaves_no_restriction_behind(parts):
    """The error is one that an unrelated call of the HIP runtime left on the
    thread (a device number that does not exist, which the host refuses): the
    launch check after the first kernel, which has summed the restriction by
    then, returns it.  The next application agrees with the one before (the
    restriction is summed by atomics: rounding)."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box((4, 3, 3), hi=(2.0, 1.0, 1.5), deform=0.02), 5, precisions=("fp64",))
    ps = sem.PressureSolver(op, restart=4)
    g = torch.Generator(device="cuda").manual_seed(7)
    r, other = (torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda") - 0.5
                for _ in range(2))
    want, z = op.vector(), op.vector()
    ps.precondition(r, want, parts=parts)
    torch.cuda.synchronize()
    assert sem.lib().hipSetDevice(1 << 20) != 0
    with pytest.raises(sem.SemError) as e:
        ps.precondition(other, z, parts=parts)
    assert e.value.status == 3                               # SEM_ERR_DEVICE
    torch.cuda.synchronize()
    ps.precondition(r, z, parts=parts)
    assert float((z - want).abs().max()) <= 1e-12 * float(want.abs().max())
