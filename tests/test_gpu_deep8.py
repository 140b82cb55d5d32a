"""Width-8 deep layers: forward and adjoint against FP64.

The meshes end inside a 64-row chunk or have more chunks than waves; six and
more extra layers stay on the record-writing kernels.  Bounds are
those of the one-layer parity tests (FP32 forward 1e-5, gradients 1e-4).
"""

import numpy as np
import pytest
import torch

from mpinputs import box_mesh, slab_partition

from _util import normwise

pytestmark = pytest.mark.gpu

DEV, H = "cuda", 8
MESHES = {"tail": ((1, 1, 1), 1, 1), "odd": ((3, 5, 2), 3, 2), "many_tiles": ((12, 12, 12), 5, 4)}


def _graph(name):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    nel, P, R = MESHES[name]
    m = box_mesh(nel, P)
    part = slab_partition(nel, R) if R > 1 else np.zeros(m.n_elem, np.int32)
    return DeviceGraph(build_graph(m.elem_gid, P, part, R), DEV)


def _theta(gen, n_in, nh, ln):
    """Flat parameters (torch.nn.Linear order) and the same as FP64 pieces."""
    flat, dims = [], [n_in] + [H] * (nh + 2)
    for k in range(nh + 2):
        a = (6.0 / (dims[k] + dims[k + 1])) ** 0.5
        flat += [(torch.rand(dims[k + 1] * dims[k], generator=gen) * 2 - 1) * a,
                 (torch.rand(dims[k + 1], generator=gen) * 2 - 1) * 0.2]
    if ln:
        flat += [torch.rand(H, generator=gen) + 0.5, (torch.rand(H, generator=gen) * 2 - 1) * 0.2]
    return torch.cat(flat).to(DEV)


def _mlp64(theta, z, n_in, nh, ln):
    o, k = 0, n_in
    for layer in range(nh + 2):
        W = theta[o:o + H * k].view(H, k)
        b = theta[o + H * k:o + H * k + H]
        o, k = o + H * k + H, H
        z = z @ W.T + b
        if layer < nh + 1:
            z = torch.nn.functional.elu(z)
    return torch.nn.functional.layer_norm(z, (H,), theta[o:o + H], theta[o + H:], 1e-5) if ln else z


def _layer64(dg, te, tn, x, e, nh, ln, agg):
    recv, col = dg.recv.long(), dg.col.long()
    m = _mlp64(te, torch.cat([x[recv], x[col], e], 1), 3 * H, nh, ln)
    e2 = e + m
    a = torch.zeros_like(x).index_add(0, recv, (m if agg == "message" else e2) / dg.edge_mult.double()[:, None])
    gid = torch.from_numpy(dg.host.row_gid).to(DEV)
    a = torch.zeros(int(gid.max()) + 1, H, dtype=x.dtype, device=DEV).index_add(0, gid, a)[gid]
    return x + _mlp64(tn, torch.cat([a, x], 1), 2 * H, nh, ln), e2


@pytest.mark.parametrize("mesh,nh,ln,agg", [("tail", 5, True, "state"), ("odd", 0, False, "state"),
                                            ("odd", 1, True, "message"), ("odd", 4, False, "message"),
                                            ("odd", 6, True, "state"), ("many_tiles", 2, True, "state"),
                                            ("many_tiles", 5, True, "state"), ("many_tiles", 3, False, "state")])
def test_forward_and_adjoint(mesh, nh, ln, agg):
    from paper_2410_01657_amd.ops import DeepLayerFn, deep_layer_cfg
    dg = _graph(mesh)
    gen = torch.Generator().manual_seed(nh + 10 * ln)
    te, tn = _theta(gen, 3 * H, nh, ln), _theta(gen, 2 * H, nh, ln)
    r = lambda n: torch.randn(n, H, generator=gen).to(DEV)
    x, e, gx, ge = r(dg.n_rows), r(dg.n_edges), r(dg.n_rows), r(dg.n_edges)
    cfg = deep_layer_cfg(H, nh, ln, aggregate=agg)
    ins = [t.clone().requires_grad_(True) for t in (x, e, te, tn)]
    out = DeepLayerFn.apply(cfg, dg, *ins)
    grads = torch.autograd.grad(list(out), ins, [gx, ge])
    ref_in = [t.double().requires_grad_(True) for t in (x, e, te, tn)]
    ref = _layer64(dg, ref_in[2], ref_in[3], ref_in[0], ref_in[1], nh, ln, agg)
    ref_g = torch.autograd.grad(list(ref), ref_in, [gx.double(), ge.double()])
    for got, want in zip(out, ref):
        assert normwise(got.detach().cpu(), want.detach().cpu()) < 1e-5
    for got, want in zip(grads, ref_g):
        assert normwise(got.cpu(), want.cpu()) < 1e-4
    # the same again, bitwise, and with parameters that are not 16-byte aligned
    for shift in (0, 1):
        ps = []
        for t in (te, tn):
            buf = torch.empty(t.numel() + 4, device=DEV)
            ps.append(buf[shift:shift + t.numel()].copy_(t).requires_grad_(True))
        ins2 = [x.clone().requires_grad_(True), e.clone().requires_grad_(True)] + ps
        out2 = DeepLayerFn.apply(cfg, dg, *ins2)
        grads2 = torch.autograd.grad(list(out2), ins2, [gx, ge])
        assert all(torch.equal(p, q) for p, q in zip(out + grads, out2 + grads2))
