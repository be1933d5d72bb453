"""The two launch shapes of the BSR row kernels (Sec. 4.2 Hessian scatter):
one launch over light and heavy rows below 16384 rows, separate launches from
there on.  The scan of the row counts crosses from one tile of 16384 entries
to two at the same place.  A pad under a punch of coarse triangles (light slave rows, heavy
master rows) just below and just above the line, full and kinematic, against
the oracle; the gradient-only assembly takes the same lists and must repeat
the gradient.  Tolerances are those of the other comparisons with the oracle."""
import numpy as np
import pytest

import oracle
from gen import workloads
from gpu_helpers import bsr_rel_error, make_ctx, need_gpu, rel_fro, to_dev

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pad,kinematic", [(125, False), (126, False), (126, True), (127, True)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_both_sides_of_the_line(n_pad, kinematic, dtype):
    need_gpu()
    fp32 = dtype == "f32"
    tdt, tol = (torch.float32, 1e-4) if fp32 else (torch.float64, 1e-10)
    w = workloads.flat_punch(n_pad=n_pad, n_punch=15, rule_n=1, fp32=fp32)
    ctx = make_ctx(w, tdt, kinematic=kinematic)
    # 16132 | 16385 rows, kinematic (slave rows only) 16129 | 16384
    assert (ctx.V >= 16384) == (n_pad == (127 if kinematic else 126))
    xs, xm = to_dev(w.xs, tdt), to_dev(w.xm, tdt)
    ctx.build_samples(to_dev(w.xs_rest, tdt))
    ctx.broadphase(xs, xm)
    A = ctx.assemble(xs, xm)
    H, g = A.hessian, A.grad.clone()
    M = ctx.sample_results()["M"].cpu().numpy()
    P = workloads.to_problem(w)
    nr = oracle.narrow(P)
    assert np.array_equal(M[nr.flags == 0], nr.M[nr.flags == 0])
    O = oracle.assemble(P, np.where(nr.flags == 0, nr.M, M), kinematic=kinematic, project=False)
    nv = ctx.V
    assert rel_fro(g.double().cpu().numpy(), O.grad[:nv]) <= tol
    rp = H.row_ptr.cpu().numpy()
    assert rp[-1] == int(ctx.status().nnzb) and (kinematic or np.diff(rp).max() > 128)
    assert bsr_rel_error(rp, H.col.cpu().numpy(), H.val.double().cpu().numpy(), O.row_ptr[:nv + 1], O.col,
                         O.val) <= tol
    ctx.broadphase(xs, xm)
    assert torch.equal(ctx.assemble(xs, xm, hessian=False).grad, g)
