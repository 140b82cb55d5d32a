"""FP32 gradients per edge, and what their errors add up to over many edges.

The gradient of an edge depends on that edge alone: it is bitwise the same under
every schedule, and the same for edges with the same inputs, whichever sub-graph,
tile or workgroup holds them.

The weight gradients add E terms of either sign.  With W waves the roundings of
the partial sums (of size sqrt(E / W), three or more a block of 16 edges) come to
about 2^-24 / sqrt(12) sqrt(3 E / 16) sqrt(E / W) in all; the bound, 2^-24 E /
sqrt(W), is eight times that.  An error of 2^-28 of the partial sum in one
direction in every step would come to 3 E / 16 2^-28 sqrt(E / W), 3 times the
bound for the smallest E here.
"""

import numpy as np
import pytest
import torch

from mpinputs import box_mesh, slab_partition

from _util import layer_params

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _graph(nel=(7, 6, 8), P=5, R=4):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    m = box_mesh(nel, P)
    part = slab_partition(nel, R) if R > 1 else np.zeros(m.n_elem, np.int32)
    return DeviceGraph(build_graph(m.elem_gid, P, part, R), DEV)


def _layer_inputs(H, dg, seed=5):
    _, o, names = layer_params(H, True)
    p = {k: torch.from_numpy(o[v].copy()).to(DEV) for k, v in names.items()}
    gen = torch.Generator().manual_seed(seed)
    r = lambda n: torch.randn(n, H, generator=gen).to(DEV)
    return p, r(dg.n_rows), r(dg.n_edges), r(dg.n_rows), r(dg.n_edges)


@pytest.mark.parametrize("agg", ["state", "message"])
@pytest.mark.parametrize("H", [32, 64, 128])
def test_edge_gradients_do_not_depend_on_the_schedule(H, agg):
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg, layer_forward
    dg = _graph((5, 4, 6), 4, 3)
    p, x, e, gx, ge = _layer_inputs(H, dg)
    cfg = layer_cfg(H, True, aggregate=agg)
    _, _, a = layer_forward(cfg, p, dg, x, e)
    ref = layer_backward(cfg, p, dg, x, e, a, gx, ge)[1]
    for te in (0, 16, 128, 512):
        for grid in (0, 1, 8, 24, 512):
            cfg.tile_edges, cfg.edge_bwd_grid = te, grid
            assert torch.equal(layer_backward(cfg, p, dg, x, e, a, gx, ge)[1], ref), (te, grid)


@pytest.mark.parametrize("H,nh", [(32, None), (64, None), (128, None), (8, 2), (32, 0), (32, 2), (32, 5)])
def test_equal_edges_have_equal_gradients(H, nh):
    from paper_2410_01657_amd.ops import DeepLayerFn, MPLayerFn, LAYER_FIELDS, deep_layer_cfg, deep_theta_size, layer_cfg
    dg = _graph()
    gen = torch.Generator().manual_seed(H)
    row = lambda n: torch.randn(1, H, generator=gen).to(DEV).repeat(n, 1)
    x, e, ge = row(dg.n_rows).requires_grad_(True), row(dg.n_edges).requires_grad_(True), row(dg.n_edges)
    if nh is None:
        p = _layer_inputs(H, dg)[0]
        out = MPLayerFn.apply(layer_cfg(H, True), dg, True, x, e, *[p[f] for f in LAYER_FIELDS])
    else:
        th = [(torch.rand(deep_theta_size(k * H, H, nh, H, True), generator=gen) - 0.5).to(DEV) for k in (3, 2)]
        out = DeepLayerFn.apply(deep_layer_cfg(H, nh, True), dg, x, e, *th)
    g_e, = torch.autograd.grad([out[0], out[1]], [e], [torch.zeros_like(x), ge])
    assert torch.equal(g_e, g_e[:1].expand_as(g_e))


@pytest.mark.parametrize("H,grid,waves", [(32, 0, 2048), (64, 0, 1024), (64, 8, 32), (32, 1, 4), (128, 0, 256)])
def test_weight_gradient_sums_have_no_bias(H, grid, waves):
    """u = 1 for zero We1 and be1 = 1, and without LayerNorm gm = g_e': every
    column of dW2 is the sum of g_e'."""
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg, layer_forward
    dg = _graph()
    E = dg.n_edges
    _, o, names = layer_params(H, False)
    p = {k: torch.zeros(o[v].shape, device=DEV) for k, v in names.items()}
    p["be1"] += 1.0
    x, e = torch.zeros(dg.n_rows, H, device=DEV), torch.zeros(E, H, device=DEV)
    ge = torch.randn(E, H, generator=torch.Generator().manual_seed(H)).to(DEV)
    cfg = layer_cfg(H, False)
    cfg.edge_bwd_grid = grid
    _, _, a = layer_forward(cfg, p, dg, x, e)
    _, _, grads = layer_backward(cfg, p, dg, x, e, a, torch.zeros_like(x), ge)
    ref = ge.double().sum(0)
    err = (grads["We2"].double() - ref[:, None]).square().mean().sqrt().item()
    assert err <= 2.0 ** -24 * E / waves ** 0.5


def test_deep_weight_gradient_sums_have_no_bias():
    """Width 32, one extra layer, W0 = W1 = 0 and biases of one: the hidden values
    are one, so the last matrix's gradient is in every column the sum of g_e' (or
    g_x'), the hidden one's the sum of Wo^T g."""
    from paper_2410_01657_amd.ops import DeepLayerFn, deep_layer_cfg
    H, dg = 32, _graph()
    gen = torch.Generator().manual_seed(1)
    Wo = torch.randn(H, H, generator=gen).to(DEV) * H ** -0.5

    def theta(k):
        z, one = torch.zeros, torch.ones(H, device=DEV)
        return torch.cat([z(k * H * H, device=DEV), one, z(H * H, device=DEV), one, Wo.reshape(-1),
                          z(H, device=DEV)]).requires_grad_(True)
    te, tn = theta(3), theta(2)
    x, e = torch.zeros(dg.n_rows, H, device=DEV), torch.zeros(dg.n_edges, H, device=DEV)
    gx, ge = (torch.randn(n, H, generator=gen).to(DEV) for n in (dg.n_rows, dg.n_edges))
    # one set of gradients at a time: through the node update g_x' reaches the edges too
    for t, k, gs, g in ((te, 3, [torch.zeros_like(gx), ge], ge), (tn, 2, [gx, torch.zeros_like(ge)], gx)):
        out = DeepLayerFn.apply(deep_layer_cfg(H, 1, False), dg, x, e, te, tn)
        d, = torch.autograd.grad(list(out), [t], gs)
        hid, last = d[k * H * H + H:].double().split([H * H + H, H * H + H])
        s = g.double().sum(0)
        h = s @ Wo.double()
        tol = 2.0 ** -24 * g.shape[0] / 1024 ** 0.5
        for got, ref in ((hid, h), (last, s)):
            for v in (got[:H * H].view(H, H) - ref[:, None], got[H * H:] - ref):
                assert v.square().mean().sqrt().item() <= tol
