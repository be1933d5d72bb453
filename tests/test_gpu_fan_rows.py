"""BSR rows of a master vertex under a fan of triangles (Sec. 4.2 Hessian
scatter).

The master blocks of a row are gathered from up to 32 incident triangles
through a mask of 96 bits in two words and two blocks at a time; beyond 32
triangles the row walks its adjacency instead.  A fan over a pad has one
vertex with as many triangles as wanted: around the words' edge (21 and 22
triangles, 63 and 66 entries), the table's edge (32 and 33) and odd and even
counts.  Tolerances are those of the other comparisons with the oracle."""
import numpy as np
import pytest

from gen import meshes, workloads
from gpu_helpers import bsr_rel_error, need_gpu, rel_fro, run_gpu, run_oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def fan(n, fp32):
    xs, ts = meshes.pad(10, 1e-2)
    a = 2 * np.pi * (np.arange(n) + 0.31) / n
    r = 9e-3 / np.cos(np.pi / n)
    xm = np.vstack([[2.3e-4, -1.7e-4, 3e-4], np.c_[r * np.cos(a), r * np.sin(a), np.full(n, 3e-4)]])
    i = np.arange(n)
    tm = np.c_[np.zeros(n, int), 1 + (i + 1) % n, 1 + i].astype(np.int32)  # normal -z, towards the pad
    w = workloads.Workload("fan", xs, ts, xm, tm, 2, 1e5, 1e-3, 0.0, np.zeros_like(xs), np.zeros_like(xm))
    return workloads._finish(w, fp32)


@pytest.mark.parametrize("n", [3, 4, 21, 22, 32, 33, 40])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_master_row_of_a_fan(n, dtype):
    need_gpu()
    w = fan(n, dtype == "f32")
    g = run_gpu(w, torch.float32 if dtype == "f32" else torch.float64, ccd=False)
    o = run_oracle(w, g["M"], ccd=False)
    O, tol = o["A"], 1e-4 if dtype == "f32" else 1e-10
    clear = ~o["flagged"]
    assert np.array_equal(g["M"][clear], o["nr"].M[clear]) and (g["M"] >= 0).sum() > 0.9 * len(g["M"])
    assert np.diff(O.row_ptr)[len(w.xs)] > len(w.xs) // 2  # the centre's row couples to most of the pad
    assert rel_fro(g["grad"], O.grad) <= tol
    assert bsr_rel_error(g["row_ptr"], g["col"], g["val"], O.row_ptr, O.col, O.val) <= tol
