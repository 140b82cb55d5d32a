"""BF16 adjoint of the H = 128 layer, weight gradients formed beside it.

The meshes end inside a 16-edge block, leave waves of a workgroup without a
tile, and have more tiles than workgroups.  The reference is FP64 autograd on
the same inputs.  Every factor is rounded to BF16 (2^-9) once before a product
and at most five products follow one another: 5 x 2^-9 = 1e-2 in norm, doubled
for the LayerNorms' gain in the tolerance.
"""

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from mpinputs import box_mesh, slab_partition

from _util import layer_params

pytestmark = pytest.mark.gpu

DEV, H = "cuda", 128
MESHES = {"tail": ((1, 1, 1), 1, 1), "odd": ((3, 5, 2), 3, 2), "many_tiles": ((7, 6, 8), 5, 4)}


def _graph(name):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    nel, P, R = MESHES[name]
    m = box_mesh(nel, P)
    part = slab_partition(nel, R) if R > 1 else np.zeros(m.n_elem, np.int32)
    return DeviceGraph(build_graph(m.elem_gid, P, part, R), DEV)


def _mlp(p, pre, z, ln):
    z = F.elu(z @ p[f"W{pre}1"].T + p[f"b{pre}1"]) @ p[f"W{pre}2"].T + p[f"b{pre}2"]
    return F.layer_norm(z, (H,), p[f"g{pre}"], p[f"bg{pre}"], 1e-5) if ln else z


def _layer(dg, p, x, e, ln, agg):
    recv, col = dg.recv.long(), dg.col.long()
    m = _mlp(p, "e", torch.cat([x[recv], x[col], e], 1), ln)
    e2 = e + m
    a = torch.zeros_like(x).index_add(0, recv, (m if agg == "message" else e2) / dg.edge_mult.double()[:, None])
    gid = torch.from_numpy(dg.host.row_gid).to(DEV)
    a = torch.zeros(int(gid.max()) + 1, H, dtype=x.dtype, device=DEV).index_add(0, gid, a)[gid]
    return x + _mlp(p, "n", torch.cat([a, x], 1), ln), e2


@pytest.mark.parametrize("mesh,ln,agg,estate,with_ge", [
    ("tail", True, "state", "f32", True), ("tail", False, "message", "bf16", False),
    ("odd", False, "state", "f32", True), ("odd", True, "message", "f32", False), ("odd", True, "state", "bf16", True),
    ("many_tiles", True, "state", "f32", True), ("many_tiles", False, "message", "bf16", True)])
def test_adjoint_against_fp64(mesh, ln, agg, estate, with_ge):
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg, layer_forward
    dg = _graph(mesh)
    _, o, names = layer_params(H, ln)
    p = {k: torch.from_numpy(o[v].astype(np.float32)).to(DEV) for k, v in names.items()}
    gen = torch.Generator().manual_seed(9)
    et = torch.bfloat16 if estate == "bf16" else torch.float32
    r = lambda n: torch.randn(n, H, generator=gen).to(DEV)
    x, e, gx, ge = r(dg.n_rows), r(dg.n_edges).to(et), r(dg.n_rows), r(dg.n_edges).to(et)
    cfg = layer_cfg(H, ln, gemm="bf16", aggregate=agg, estate=estate)
    _, _, a = layer_forward(cfg, p, dg, x, e)
    g_x, g_e, grads = layer_backward(cfg, p, dg, x, e, a, gx, ge if with_ge else None)
    ref = {k: v.double().requires_grad_(True) for k, v in p.items()}
    rx, re = x.double().requires_grad_(True), e.double().requires_grad_(True)
    out = _layer(dg, ref, rx, re, ln, agg)
    want = torch.autograd.grad(list(out), [rx, re] + [ref[k] for k in names],
                               [gx.double(), ge.double() if with_ge else torch.zeros_like(re)])
    for k, got, w in zip(["g_x", "g_e"] + list(names), [g_x, g_e] + [grads[k] for k in names], want):
        assert ((got.double() - w).norm() / w.norm()).item() < 2e-2, k
    again = layer_backward(cfg, p, dg, x, e, a, gx, ge if with_ge else None)
    assert torch.equal(again[0], g_x) and torch.equal(again[1], g_e)
    assert all(torch.equal(again[2][k], grads[k]) for k in names)


@pytest.mark.parametrize("mesh,ln", [("tail", True), ("odd", False), ("many_tiles", True)])
def test_fp32_weight_gradients_against_fp64(mesh, ln):
    """The separate weight-gradient passes of the FP32 layer, over row counts
    that end inside 16- and 32-row blocks.  A sum of n products rounds to some
    sqrt(n) 2^-24 of a term's size: 1e-5 of the sum leaves a factor of ten."""
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg, layer_forward
    dg = _graph(mesh)
    _, o, names = layer_params(H, ln)
    p = {k: torch.from_numpy(o[v].astype(np.float32)).to(DEV) for k, v in names.items()}
    gen = torch.Generator().manual_seed(5)
    r = lambda n: torch.randn(n, H, generator=gen).to(DEV)
    x, e, gx, ge = r(dg.n_rows), r(dg.n_edges), r(dg.n_rows), r(dg.n_edges)
    cfg = layer_cfg(H, ln)
    _, _, a = layer_forward(cfg, p, dg, x, e)
    _, _, grads = layer_backward(cfg, p, dg, x, e, a, gx, ge)
    ref = {k: v.double().requires_grad_(True) for k, v in p.items()}
    out = _layer(dg, ref, x.double(), e.double(), ln, "state")
    want = torch.autograd.grad(list(out), [ref[k] for k in names], [gx.double(), ge.double()])
    for k, w in zip(names, want):
        assert ((grads[k].double() - w).norm() / w.norm()).item() < 1e-5, k
