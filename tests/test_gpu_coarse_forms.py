"""The coarse solve with two kernels per iteration (above 32768 vertices, and
rows of more than 28 entries): repeated applications, first-step stops and
non-finite residuals, against ten PCG iterations on the N = 1 operator."""
import types

import numpy as np
import pytest

import fixtures as F
from tests.common import relerr

torch = pytest.importorskip("torch")


def star(layers, sectors=5):
    """`sectors` quadrilaterals around one vertex, extruded: the inner vertices
    of the axis have 3 (2 sectors + 1) neighbours."""
    a = 2.0 * np.pi * np.arange(sectors) / sectors
    half = a + np.pi / sectors
    ring = np.concatenate([[[0.0, 0.0]], np.stack([np.cos(a), np.sin(a)], 1),
                           1.4 * np.stack([np.cos(half), np.sin(half)], 1)])
    nv = ring.shape[0]
    ids, bc = [], []
    for z in range(layers):
        for s in range(sectors):
            q = np.array([0, 1 + s, 1 + (s + 1) % sectors, 1 + sectors + s])
            ids.append(np.concatenate([q + z * nv, q + (z + 1) * nv]))
            bc.append([0, 0, 0, 0, int(z == 0), 0])
    xyz = np.concatenate([np.c_[ring, np.full(nv, 0.5 * z)] for z in range(layers + 1)])
    return types.SimpleNamespace(num_elements=len(ids), corner_ids=np.array(ids, dtype=np.int64),
                                 face_bc=np.array(bc, dtype=np.uint8), num_vertices=xyz.shape[0],
                                 vertex_xyz=xyz)


MESHES = {"33792_vertices": lambda: F.box((32, 31, 31), hi=(3.0, 2.0, 2.0)),
          "33_neighbours": lambda: star(40)}


class Reference:
    """Restriction, ten PCG iterations from zero and interpolation, written
    with tensor operations on an N = 1 context."""

    def __init__(self, sem, m, op):
        self.c = sem.Operator(m, 1, precisions=("fp64",))
        self.gid, self.pos, _, _ = op.numbering()
        self.cgid, self.cpos, self.cdm, _ = self.c.numbering()
        x1 = np.array([-1.0, 0.0, 1.0])
        h = np.stack([(1 - x1) / 2, (1 + x1) / 2])
        self.P = np.einsum("ai,bj,ck->cbakji", h, h, h).reshape(8, 27)
        first = np.zeros(self.gid.size, dtype=bool)
        first[np.unique(self.gid.ravel(), return_index=True)[1]] = True
        self.first = first.reshape(self.gid.shape)
        self.d = torch.from_numpy(self.c.geometry()[2]).cuda()

    def __call__(self, r):
        rc = r.cpu().numpy()[self.pos]
        b = np.zeros(self.c.n_unique)
        np.add.at(b, self.cgid.ravel(), ((rc[self.gid] * self.first) @ self.P.T).ravel())
        b[self.cdm == 1] = 0.0
        bs = np.empty_like(b)
        bs[self.cpos] = b
        rv = torch.from_numpy(bs).cuda()
        x, p = torch.zeros_like(rv), self.d * rv
        rz = torch.dot(rv, p)
        for _ in range(10):
            w = self.c.ax(p)
            a = rz / torch.dot(p, w)
            x += a * p
            rv = rv - a * w
            rz, o = torch.dot(rv, self.d * rv), rz
            p = self.d * rv + (rz / o) * p
        want = np.zeros(rc.size)
        want[self.gid.ravel()] = (x.cpu().numpy()[self.cpos][self.cgid] @ self.P).ravel()
        return want


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(MESHES))
def test_two_kernel_form(name):
    """1e-11, as in the comparison around 32768 vertices: the recurrences are
    the same and differ by rounding."""
    import paper_2207_07098_amd as sem
    m = MESHES[name]()
    op = sem.Operator(m, 2, precisions=("fp64",))
    ps = sem.PressureSolver(op, restart=2)
    ref = Reference(sem, m, op)
    dm = torch.from_numpy(op.numbering()[2].astype(bool))
    g = torch.Generator(device="cuda").manual_seed(1)
    for _ in range(2):                 # the second starts from what the first cleared
        r = op.ax(torch.rand(op.n_unique, generator=g, dtype=torch.float64, device="cuda"))
        z = ps.precondition(r, parts=ps.COARSE)
        assert relerr(z.cpu().numpy()[ref.pos][~dm.numpy()], ref(r)[~dm.numpy()]) < 1e-11
    assert float(ps.precondition(torch.zeros_like(r), parts=ps.COARSE).abs().max()) == 0.0
    bad = r.clone()
    bad[op.n_unique // 2] = float("nan")
    with pytest.raises(sem.SemError) as e:
        ps.precondition(bad, parts=ps.COARSE)
    assert e.value.status == 7                               # SEM_ERR_NAN
    assert float(ps.precondition(torch.zeros_like(r), parts=ps.COARSE).abs().max()) == 0.0
    z2 = ps.precondition(r, parts=ps.COARSE)
    assert relerr(z2.cpu().numpy(), z.cpu().numpy()) < 1e-12
