"""The in-place E-vector gather-scatter against a sum over the exported
numbering, on both sides of the rule that gives a lane one or two nodes."""
import numpy as np
import pytest

import fixtures as F

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K, N", [((1, 1, 1), 1), ((5, 4, 3), 2), ((2, 1, 1), 15), ((13, 12, 11), 7),
                                  ((17, 16, 16), 7)])
def test_gs_against_numbering(K, N):
    """One element, the longest position table (N = 15), and 219 and 559
    thousand boundary nodes around the 524288 of one resident set of lanes.
    At most eight copies (more on a folded periodic box) are summed: within
    16 units of rounding of the sum of their magnitudes."""
    import paper_2207_07098_amd as sem
    op = sem.Operator(F.box(K, deform=0.02), N, solver=False)
    gid, _, dmask, _ = op.numbering()
    rng = np.random.default_rng(N)
    v = rng.uniform(-1.0, 1.0, gid.size)
    for prec, dt, eps in (("fp64", np.float64, 2.3e-16), ("fp32", np.float32, 1.2e-7)):
        x = v.astype(dt)
        tot, mag = np.zeros(op.n_unique), np.zeros(op.n_unique)
        np.add.at(tot, gid.ravel(), x.astype(np.float64))
        np.add.at(mag, gid.ravel(), np.abs(x).astype(np.float64))
        tot[dmask == 1] = 0.0
        got = op.gs(torch.from_numpy(x.copy()).cuda(), precision=prec).cpu().numpy()
        assert np.all(np.abs(got - tot[gid.ravel()]) <= 16 * eps * mag[gid.ravel()]), prec
