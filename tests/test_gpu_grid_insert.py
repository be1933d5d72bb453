"""Placing master triangles in their grid cells (Sec. 4.2 broad phase): 16
lanes per triangle up to 16384 triangles, one from there on.  Flat punches of
few triangles over many cells (fewer cells than lanes, remainders, hundreds)
and just below and above the line; a sample's triangle would be missed if a
cell were, so the selection is compared with the oracle, and the candidate
total with the exported list."""
import numpy as np
import pytest

import oracle
from gen import workloads
from gpu_helpers import make_ctx, need_gpu, to_dev

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_punch", [1, 2, 7, 90, 91])  # 2, 8, 98, 16200, 16562 triangles
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_no_cell_is_missed(n_punch, dtype):
    need_gpu()
    fp32 = dtype == "f32"
    tdt = torch.float32 if fp32 else torch.float64
    w = workloads.flat_punch(n_pad=24, n_punch=n_punch, rule_n=2, fp32=fp32)
    ctx = make_ctx(w, tdt)
    assert (ctx.Tm <= 16384) == (n_punch <= 90)
    xs, xm = to_dev(w.xs, tdt), to_dev(w.xm, tdt)
    ctx.build_samples(to_dev(w.xs_rest, tdt))
    ctx.broadphase(xs, xm)
    ctx.assemble(xs, xm)
    M = ctx.sample_results()["M"].cpu().numpy()
    nr = oracle.narrow(workloads.to_problem(w))
    assert np.array_equal(M[nr.flags == 0], nr.M[nr.flags == 0]) and (M >= 0).mean() > 0.9
    off, cand = ctx.candidates()
    n = int(off[-1])
    assert n == int(ctx.status().n_candidates) and n >= int((M >= 0).any())
    T = np.repeat(np.arange(ctx.Ts), np.diff(off.cpu().numpy()))
    held = set(zip(T.tolist(), cand[:n].cpu().numpy().tolist()))
    k = np.nonzero(M >= 0)[0]
    assert all((int(i) // 4, int(M[i])) in held for i in k)  # 2 x 2 samples per triangle
