"""The tree search of the dual-mesh embedding gives exactly what the scan of
all triangles gives (gmcp_dualmesh_embed, which the oracle tests cover): the
same triangle, coordinates, offset and distance, bit for bit - on surfaces
of the smallest size the tree takes, at the edges of its leaves and levels
(a level more from 4097 and from 32769 triangles), vertices in their own and in the curve's order (from 131072), on flat and shuffled meshes, with
duplicate, degenerate and non-finite triangles, and for vertices that
coincide with the surface's own, lie far away or are not finite.
"""
import ctypes as C

import numpy as np
import pytest

from gen import meshes
from gpu_helpers import need_gpu, to_dev

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _p(t):
    return C.c_void_p(t.data_ptr())


def _embed(P, V, F, tree):
    from paper_2605_24339_amd.dualmesh import _lib
    L = _lib()
    N, nT = P.shape[0], F.shape[0]
    out = [torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(N, 3, dtype=torch.float64, device="cuda"),
           torch.empty(N, dtype=torch.float64, device="cuda"), torch.empty(N, dtype=torch.float64, device="cuda")]
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    args = [_p(P), N, _p(V), _p(F), nT, *[_p(o) for o in out]]
    if tree:
        nbytes = L.gmcp_dualmesh_embed_work_bytes(N, nT)
        assert nbytes > 0
        work = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")   # nothing is expected of its contents
        assert L.gmcp_dualmesh_embed_ws(*args, _p(work), nbytes - 1, st) == 1
        assert L.gmcp_dualmesh_embed_ws(*args, _p(work), nbytes, st) == 0
    else:
        assert L.gmcp_dualmesh_embed(*args, st) == 0
    return [o.cpu().numpy() for o in out]


def _surface(kind, n_tri, rng):
    if kind == "flat":
        n = int(np.ceil(np.sqrt(n_tri / 2)))
        V, F = meshes.pad(n, 1.0)
    else:
        V, F = meshes.geodesic_sphere(int(np.ceil(np.sqrt(n_tri / 20))), 1.0)
        V = V * (1 + 0.02 * rng.uniform(-1, 1, size=(V.shape[0], 1)))
    F = F[rng.permutation(F.shape[0])[:n_tri]] if kind != "sphere" else F[:n_tri]
    if kind == "mixed":
        F = F.copy()
        F[5:25] = F[30:50]                    # duplicates: ties go to the smaller index
        F[60:70, 2] = F[60:70, 1]             # zero area
        V = np.concatenate([V, [[np.nan, 0, 0], [np.inf, 0, 0]]])
        F[80, 0], F[81, 1] = V.shape[0] - 2, V.shape[0] - 1
    return V, np.ascontiguousarray(F, dtype=np.int32)


@pytest.mark.parametrize("kind,n_tri,n_vis", [("sphere", 256, 1), ("sphere", 513, 65), ("flat", 800, 1000),
                                              ("shuffled", 4100, 3000), ("mixed", 2000, 4097), ("sphere", 4097, 5000), ("sphere", 33000, 2000), ("shuffled", 300, 131100)])
def test_tree_equals_scan(kind, n_tri, n_vis):
    need_gpu()
    rng = np.random.default_rng(n_tri + n_vis)
    V, F = _surface(kind, n_tri, rng)
    T = rng.integers(0, F.shape[0], size=n_vis)
    b = rng.dirichlet((1.0, 1.0, 1.0), size=n_vis)
    P = (b[:, :, None] * V[F[T]]).sum(1) + 0.02 * rng.normal(size=(n_vis, 3))
    k = n_vis // 8
    P[:k] = V[F[T[:k], 0]]                     # the surface's own vertices
    P[k:2 * k] = 0.5 * (V[F[T[k:2 * k], 0]] + V[F[T[k:2 * k], 1]])   # on shared edges
    P[2 * k:2 * k + k // 4] *= 50.0            # far away
    if kind == "mixed":
        P[-3:] = [[np.nan, 0, 0], [np.inf, 0, 0], [0, -np.inf, np.nan]]
    P, V, F = to_dev(P, torch.float64), to_dev(V, torch.float64), torch.tensor(F, device="cuda")
    a, t = _embed(P, V, F, False), _embed(P, V, F, True)
    for name, x, y in zip(("tri", "bary", "delta", "dist2"), a, t):
        np.testing.assert_array_equal(x, y, err_msg=name)


def test_no_valid_triangle():
    need_gpu()
    P = torch.zeros(70, 3, dtype=torch.float64, device="cuda")
    V = torch.zeros(3, 3, dtype=torch.float64, device="cuda")
    F = torch.tensor([[0, 1, 2]], dtype=torch.int32, device="cuda").repeat(600, 1)
    for x, y in zip(_embed(P, V, F, False), _embed(P, V, F, True)):
        np.testing.assert_array_equal(x, y)
        assert (x == -1).all() or np.isnan(x).all() or np.isinf(x).all()
