"""The sliced matrix kernels of the implicit-step system at the edges of
their 64-row slices: K in row order, A x and the CG solve against the dense
FP64 oracle, with and without a contact matrix, for vertex counts below, at
and above a slice and rows of very different lengths; the solve stops at an
iteration limit that is no multiple of the check interval, and a zero
right-hand side takes no iteration.

Tolerances: sums of at most 64 x 3 products, so 1e-13 of the largest term
for A x; a solve to rtol has a true residual within rtol plus the rounding
of its recurrence (1e-12 |b| at these sizes).
"""
import numpy as np
import pytest

from gen import meshes
from gpu_helpers import need_gpu, to_dev
from oracle import fem as ofem

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

E_Y, NU, RHO, DT, H = 3e5, 0.45, 1000.0, 1e-3, 3.125e-4


def _contact_matrix(V, rng):
    """A symmetric positive semidefinite BSR on some rows: B^T B of a few rank-one blocks."""
    from paper_2605_24339_amd.gmcp import BSR
    D = np.zeros((3 * V, 3 * V))
    for _ in range(5):
        v = np.zeros(3 * V)
        for i in rng.choice(V, size=min(V, 12), replace=False):
            v[3 * i:3 * i + 3] = rng.normal(size=3)
        D += np.outer(v, v) * 10.0
    rp, col, val = [0], [], []
    for i in range(V):
        for j in range(V):
            b = D[3 * i:3 * i + 3, 3 * j:3 * j + 3]
            if np.any(b):
                col.append(j)
                val.append(b)
        rp.append(len(col))
    dev = lambda a, t: torch.tensor(np.array(a), dtype=t, device="cuda")
    return BSR(dev(rp, torch.int32), dev(col, torch.int32), dev(val, torch.float64)), D


@pytest.mark.parametrize("shape,contact", [((1, 1, 1), False), ((2, 2, 6), True), ((3, 3, 3), False), ((4, 2, 4), True),
                                           ((7, 3, 3), True), ((12, 1, 4), False)])
def test_rows_and_solve_match_dense(shape, contact):
    need_gpu()
    from paper_2605_24339_amd.fem import Fem
    X, tets, top, bottom = meshes.tet_block(*shape, H)
    V = X.shape[0]
    rng = np.random.default_rng(V)
    fem = Fem(X, tets, E_Y, NU, RHO, DT, bottom)
    fem.constrain(top.ravel()[:1], 2)                       # one vertex held along y
    held = fem.fixed.cpu().numpy().ravel()
    K = ofem.stiffness(X, tets, E_Y, NU).toarray()
    B = fem.stiffness()
    Kg = np.zeros_like(K)
    rp, col, val = B.row_ptr.cpu().numpy(), B.col.cpu().numpy(), B.val.cpu().numpy()
    for i in range(V):
        for j in range(rp[i], rp[i + 1]):
            Kg[3 * i:3 * i + 3, 3 * col[j]:3 * col[j] + 3] = val[j]
    assert np.abs(Kg - K).max() <= 1e-12 * np.abs(K).max()
    H_bsr, Hd = _contact_matrix(V, rng) if contact else (None, 0.0)
    A = K + Hd + np.diag(np.repeat(ofem.lumped_mass(X, tets, RHO), 3)) / DT ** 2
    A[held], A[:, held] = 0.0, 0.0
    x = rng.normal(size=(V, 3))
    y = fem.apply(H_bsr, to_dev(x, torch.float64)).cpu().numpy().ravel()
    assert np.abs(y - A @ x.ravel()).max() <= 1e-12 * np.abs(A).max() * np.abs(x).max()
    b = rng.normal(size=(V, 3))
    bm = np.where(held, 0.0, b.ravel())
    rtol = 1e-8
    d, it, rr = fem.solve(H_bsr, to_dev(b, torch.float64), rtol=rtol)
    d = d.cpu().numpy().ravel()
    assert it % 8 == 0 and rr <= rtol
    assert np.all(d[held] == 0.0)
    assert np.linalg.norm(bm - A @ d) <= (rtol + 1e-12) * np.linalg.norm(bm)
    free = ~held
    ref = np.linalg.solve(A[np.ix_(free, free)], bm[free])
    cond = np.linalg.cond(A[np.ix_(free, free)])
    assert np.linalg.norm(d[free] - ref) <= 2 * rtol * cond * np.linalg.norm(ref)
    _, it, _ = fem.solve(H_bsr, to_dev(b, torch.float64), rtol=1e-300, max_iter=11)
    assert it == 11
    z, it, rr = fem.solve(H_bsr, torch.zeros(V, 3, dtype=torch.float64, device="cuda"))
    assert it == 0 and rr == 0.0 and not z.any()
