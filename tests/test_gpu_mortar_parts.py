"""Clipped mortar samples (Sec. 4.1, face samples) over the four waves of a
work tile: tiles of 64, 16, 7 and 4 triangles (rules 1 to 4), a pad whose
triangle count leaves a partial last tile in each, and more than 64 candidate
pairs per triangle (two chunks), against the oracle.  Tolerances are those of
the other comparisons with the oracle."""
import numpy as np
import pytest


from gen import workloads
from gpu_helpers import bsr_rel_error, need_gpu, rel_fro
from oracle import mortar as om
from test_gpu_mortar import _oracle_bsr, _run

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule_n,n_pad,n_punch", [(1, 7, 5), (2, 7, 5), (3, 5, 4), (4, 5, 4), (2, 2, 17)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_every_part_of_a_tile(rule_n, n_pad, n_punch, dtype):
    need_gpu()
    fp32 = dtype == "f32"
    w = workloads.flat_punch(n_pad=n_pad, n_punch=n_punch, rule_n=rule_n, fp32=fp32)
    ctx, xs, xm, A = _run(w, torch.float32 if fp32 else torch.float64)
    P = workloads.to_problem(w)
    O = om.assemble(P, om.samples(P))
    off, _ = ctx.candidates()
    assert n_punch < 17 or int(np.diff(off.cpu().numpy()).max()) > 64
    te, tg = (1e-5, 1e-4) if fp32 else (1e-10, 1e-10)
    assert abs(float(A.energy.double().sum()) / O.energy - 1) <= te
    assert rel_fro(A.grad.double().cpu().numpy(), O.grad) <= tg
    rp, col, val = _oracle_bsr(O.blocks, P.Vs + P.Vm)
    H = A.hessian
    assert bsr_rel_error(H.row_ptr.cpu().numpy(), H.col.cpu().numpy(), H.val.double().cpu().numpy().reshape(-1, 9),
                         rp, col, val) <= tg
    e, g = A.energy.clone(), A.grad.clone()
    ctx.broadphase(xs, xm)
    A2 = ctx.assemble(xs, xm)
    assert torch.equal(A2.energy, e) and torch.equal(A2.grad, g)
