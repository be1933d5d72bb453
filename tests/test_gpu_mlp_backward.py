"""The fused backward pass of the warm-start MLP against the same products in
float64 with the same bf16 operands (dY, W, H, x and each layer's dZ are
rounded to bf16 as matrix operands, bias gradients sum the unrounded dZ), at
the edges of its 16-row waves and 256-row blocks and beyond one block per
partial, and for parameters that start at any float.

Tolerance: float32 dZ differs from the float64 one by a few 1e-7, which moves
about 1e-4 of its values to the other side of a bf16 rounding (2^-9): 2e-5
of a gradient's norm for sums over many rows, at most 2^-9 sqrt(1e-4) of it
otherwise; 1e-4 covers both and the accumulation in float32.
"""
import numpy as np
import pytest

from gpu_helpers import need_gpu
from oracle import mlp as omlp

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _bf(a):
    return a.float().bfloat16().double()


def _reference(p, x, act, dy):
    w, o = {}, 0
    for name, shp in omlp.SHAPES:
        n = int(np.prod(shp))
        w[name] = p[o:o + n].reshape(shp).double()
        o += n
    Z1, H1, Z2, H2, Z3, H3 = (a.double() for a in act.split(128, dim=1))
    def dsilu(z):
        s = torch.sigmoid(z)
        return s * (1.0 + z * (1.0 - s))

    g = {"W4": _bf(H3).T @ _bf(dy), "b4": dy.double().sum(0)}
    d = dy.double()
    for k, (Z, H, W) in ((3, (Z3, H2, "W4")), (2, (Z2, H1, "W3")), (1, (Z1, x, "W2"))):
        d = (_bf(d) @ _bf(w[W]).T) * dsilu(Z)
        g[f"W{k}"], g[f"b{k}"] = _bf(H).T @ _bf(d), d.sum(0)
    return g


@pytest.mark.parametrize("B,shift", [(1, 0), (15, 1), (16, 0), (255, 3), (256, 0), (257, 2), (1000, 0), (66000, 0)])
def test_fused_backward_matches_products(B, shift):
    need_gpu()
    from paper_2605_24339_amd.gmcp import _ptr
    from paper_2605_24339_amd.mlp import MLP, _lib, _stream
    gen = torch.Generator(device="cuda").manual_seed(B)
    net = MLP(torch.tensor(omlp.init(seed=3), dtype=torch.float32, device="cuda"))
    x = torch.zeros(B, 16, device="cuda")
    x[:, :9] = torch.randn(B, 9, generator=gen, device="cuda")
    dy = torch.zeros(B, 16, device="cuda")
    dy[:, :3] = torch.randn(B, 3, generator=gen, device="cuda")
    y, act = net.forward(x)
    buf = torch.zeros(net.n + 4, device="cuda")
    buf[shift:shift + net.n] = net.p                      # parameters at any float
    p = buf[shift:shift + net.n]
    y2 = torch.empty_like(y)
    assert _lib().gmcp_mlp_forward(_ptr(p), _ptr(x), B, _ptr(y2), None, _stream(x.device)) == 0
    assert torch.equal(y, y2)
    g = torch.full((net.n,), float("nan"), device="cuda")
    nb = int(_lib().gmcp_mlp_work_bytes(B))
    work = torch.full((nb // 4,), float("nan"), device="cuda")
    args = (_ptr(p), _ptr(x), _ptr(act), _ptr(dy), B, _ptr(g), _ptr(work))
    assert _lib().gmcp_mlp_backward(*args, nb - 1, _stream(x.device)) == 1
    assert _lib().gmcp_mlp_backward(*args, nb, _stream(x.device)) == 0
    ref, o = _reference(net.p, x, act, dy), 0
    for name, shp in omlp.SHAPES:
        n = int(np.prod(shp))
        got = g[o:o + n].reshape(shp).double()
        o += n
        assert (got - ref[name]).norm() <= 1e-4 * ref[name].norm() + 1e-30, name
    assert torch.equal(net.backward(x, act, dy), g)       # and the same bits again
