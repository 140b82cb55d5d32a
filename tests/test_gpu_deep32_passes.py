"""Width-32 deep adjoint on a graph long enough that its weight gradients are summed
in two passes (16384 tiles of 128 edges and more), against FP64.

Tiles that end unevenly over the eighths of the graph and over the passes; the
bound is that of the one-layer gradient tests (1e-4).  A pass left out, or added
twice, is an error of the gradient's own size.
"""

import pytest
import torch

from mpinputs import box_mesh, slab_partition

from _util import normwise

pytestmark = pytest.mark.gpu

DEV, H, ROWS = "cuda", 32, 1 << 20


@pytest.mark.parametrize("nh,ln", [(1, True), (5, False)])
def test_two_passes(nh, ln):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    from paper_2410_01657_amd.ops import DeepLayerFn, deep_layer_cfg, deep_theta_size
    nel = (15, 16, 14)
    m = box_mesh(nel, 5)
    dg = DeviceGraph(build_graph(m.elem_gid, 5, slab_partition(nel, 2), 2), DEV)
    assert dg.n_edges // 128 >= 16384 and (dg.n_edges + 127) // 128 % 16
    gen = torch.Generator(device=DEV).manual_seed(nh)
    r = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    te, tn = (r(deep_theta_size(k * H, H, nh, H, ln)) * 0.2 for k in (3, 2))
    x, e, ge = r(dg.n_rows, H), r(dg.n_edges, H), r(dg.n_edges, H)
    te.requires_grad_(True)
    out = DeepLayerFn.apply(deep_layer_cfg(H, nh, ln), dg, x, e, te, tn)
    got, = torch.autograd.grad([out[1]], [te], [ge])

    # no gradient at x': d(theta) = sum over the edges of J^T g_e', in chunks
    t64 = te.detach().double().requires_grad_(True)
    recv, col = dg.recv.long(), dg.col.long()
    want = torch.zeros_like(t64)
    for k in range(0, dg.n_edges, ROWS):
        s = slice(k, k + ROWS)
        z, o, n_in = torch.cat([x[recv[s]], x[col[s]], e[s]], 1).double(), 0, 3 * H
        for layer in range(nh + 2):
            W, b = t64[o:o + H * n_in].view(H, n_in), t64[o + H * n_in:o + H * n_in + H]
            o, n_in = o + H * n_in + H, H
            z = torch.nn.functional.linear(z, W, b)
            if layer <= nh:
                z = torch.nn.functional.elu(z)
        if ln:
            z = torch.nn.functional.layer_norm(z, (H,), t64[o:o + H], t64[o + H:], 1e-5)
        want += torch.autograd.grad(z, t64, ge[s].double())[0]
    assert normwise(got.cpu(), want.cpu()) < 1e-4
