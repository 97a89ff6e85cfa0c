"""Coarse part of the pressure preconditioner (ten Jacobi-PCG iterations on
the assembled N = 1 operator) against the oracle, on both sides of the size
where one workgroup stops solving it (1024 vertices), with zero and with
non-finite right-hand sides."""
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

MESHES = {
    "1024_vertices": F.box((15, 7, 7), hi=(3.0, 2.0, 2.0), reorient_seed=5),
    "1088_vertices": F.box((16, 7, 7), hi=(3.0, 2.0, 2.0), reorient_seed=6),
    "natural_faces": F.box((16, 8, 7), hi=(3.0, 2.0, 1.0), dirichlet=(1, 0, 0, 0, 0, 0)),
    "ogrid": F.ogrid(16, 9, 8),
}


@pytest.mark.parametrize("name", list(MESHES))
def test_coarse_part_matches_oracle(name):
    p = Pair(MESHES[name], 2, precisions=("fp64",))
    hs = HY.HybridSchwarz(MESHES[name], p.ora)
    ps = sem.PressureSolver(p.op, restart=4)
    for seed in (3, 4):
        # the second application starts from the right-hand side that the
        # first one cleared
        r = p.ora.rhs_unique(F.random_unique(p.op.n_unique, seed))
        z = p.from_dev(ps.precondition(p.to_dev(r), parts=ps.COARSE))
        assert relerr(z, hs.coarse(r)) < 1e-12
    z = ps.precondition(p.op.vector(), parts=ps.COARSE)
    assert float(z.abs().max()) == 0.0


@pytest.mark.parametrize("name", ["1024_vertices", "1088_vertices"])
def test_non_finite_residual_is_reported(name):
    op = sem.Operator(MESHES[name], 2, precisions=("fp64",))
    ps = sem.PressureSolver(op, restart=4)
    r = torch.ones(op.n_unique, dtype=torch.float64, device="cuda")
    r[op.n_unique // 2] = float("nan")
    with pytest.raises(sem.SemError) as e:
        ps.precondition(r, parts=ps.COARSE)
    assert e.value.status == 7                               # SEM_ERR_NAN
    # and leaves nothing behind for the next application
    z = ps.precondition(torch.zeros_like(r), parts=ps.COARSE)
    assert float(z.abs().max()) == 0.0


@pytest.mark.parametrize("K", [(32, 31, 30), (32, 31, 31)])
def test_coarse_part_around_the_one_kernel_form(K):
    """32,736 and 33,792 vertices, on both sides of the 32768 up to which an
    iteration is one kernel: ten PCG iterations on the same operator, written
    with tensor operations on an N = 1 context, to 1e-11 (the forms of the
    recurrence differ by rounding only)."""
    m = F.box(K, hi=(3.0, 2.0, 2.0))
    op = sem.Operator(m, 2, precisions=("fp64",))
    ps = sem.PressureSolver(op, restart=4)
    r = op.ax(torch.rand(op.n_unique, generator=torch.Generator(device="cuda").manual_seed(1),
                         dtype=torch.float64, device="cuda"))
    z = ps.precondition(r, parts=ps.COARSE)
    c = sem.Operator(m, 1, precisions=("fp64",))
    gid, pos, _, _ = op.numbering()
    cgid, cpos, cdm, _ = c.numbering()
    x1 = np.array([-1.0, 0.0, 1.0])
    h = np.stack([(1 - x1) / 2, (1 + x1) / 2])                     # [2][3]
    P = np.einsum("ai,bj,ck->cbakji", h, h, h).reshape(8, 27)      # corner, point
    rc = r.cpu().numpy()[pos]
    first = np.zeros(gid.size, dtype=bool)
    first[np.unique(gid.ravel(), return_index=True)[1]] = True     # one copy of each node
    b = np.zeros(c.n_unique)
    np.add.at(b, cgid.ravel(), ((rc[gid] * first.reshape(gid.shape)) @ P.T).ravel())
    b[cdm == 1] = 0.0
    bs = np.empty_like(b)
    bs[cpos] = b
    rv = torch.from_numpy(bs).cuda()
    d = torch.from_numpy(c.geometry()[2]).cuda()
    x, p = torch.zeros_like(rv), d * rv
    rz = torch.dot(rv, p)
    for _ in range(10):
        w = c.ax(p)
        a = rz / torch.dot(p, w)
        x += a * p
        rv = rv - a * w
        rz, o = torch.dot(rv, d * rv), rz
        p = d * rv + (rz / o) * p
    xc = x.cpu().numpy()[cpos]
    want = np.zeros(op.n_unique)
    want[gid.ravel()] = (xc[cgid] @ P).ravel()
    got = z.cpu().numpy()[pos]
    assert relerr(got, want) < 1e-11
