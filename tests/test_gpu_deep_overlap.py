"""Deep layers whose x_out or g_x_in takes the place of a buffer that is dead by
then.

The node update is the last to run, so x_out may lie where e_in or e_out was:
a caller that needs x' alone saves an array.  In the adjoint g_x_in is written
last and may lie where e_in or g_e_out was.  The results are those of separate
buffers, in the forward within the FP32 forward bound (1e-5).
"""

import ctypes as C

import pytest
import torch

from mpinputs import box_mesh, slab_partition

from _util import normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,nh", [(8, 2), (16, 2), (32, 0), (32, 2), (32, 5), (32, 6)])
@pytest.mark.parametrize("over", ["e_in", "e_out", "inside e_out"])
def test_x_out_over_an_edge_array(H, nh, over):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    from paper_2410_01657_amd._lib import call
    from paper_2410_01657_amd.ops import deep_layer_cfg, deep_theta_size
    m = box_mesh((3, 5, 2), 3)
    dg = DeviceGraph(build_graph(m.elem_gid, 3, slab_partition((3, 5, 2), 2), 2), "cuda")
    gen = torch.Generator().manual_seed(H + nh)
    te, tn = ((torch.rand(deep_theta_size(k * H, H, nh, H, True), generator=gen) - 0.5).cuda() for k in (3, 2))
    x = torch.randn(dg.n_rows, H, generator=gen).cuda()
    e = torch.randn(dg.n_edges, H, generator=gen).cuda()
    cfg = deep_layer_cfg(H, nh, True)

    def forward(e_in, x_out, e_out):
        a = torch.empty_like(x)
        call("mp_deep_layer_forward", C.byref(cfg), te.data_ptr(), tn.data_ptr(), C.byref(dg.desc), x.data_ptr(),
             e_in.data_ptr(), x_out.data_ptr(), e_out.data_ptr(), a.data_ptr(),
             torch.cuda.current_stream().cuda_stream)
        return a

    want, e_want = torch.empty_like(x), torch.empty_like(e)
    a_want = forward(e, want, e_want)
    e_in, e_out = e.clone(), torch.empty_like(e)
    row0 = 4 if over == "inside e_out" else 0
    buf = e_in if over == "e_in" else e_out
    x_out = buf[row0:row0 + dg.n_rows]
    a = forward(e_in, x_out, e_out)
    assert normwise(x_out.cpu(), want.cpu()) < 1e-5
    assert normwise(a.cpu(), a_want.cpu()) < 1e-5
    rest = e_out if over == "e_in" else e_out[row0 + dg.n_rows:]
    ref = e_want if over == "e_in" else e_want[row0 + dg.n_rows:]
    assert normwise(rest.cpu(), ref.cpu()) < 1e-5


@pytest.mark.parametrize("H,nh", [(8, 2), (16, 2), (32, 0), (32, 5), (32, 6)])
@pytest.mark.parametrize("over", ["e_in", "g_e_out"])
def test_g_x_in_over_an_edge_array(H, nh, over):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    from paper_2410_01657_amd._lib import call
    from paper_2410_01657_amd.ops import deep_layer_cfg, deep_theta_size
    m = box_mesh((3, 5, 2), 3)
    dg = DeviceGraph(build_graph(m.elem_gid, 3, slab_partition((3, 5, 2), 2), 2), "cuda")
    gen = torch.Generator().manual_seed(H + nh)
    te, tn = ((torch.rand(deep_theta_size(k * H, H, nh, H, True), generator=gen) - 0.5).cuda() for k in (3, 2))
    r = lambda n: torch.randn(n, H, generator=gen).cuda()
    x, a, gx, e, ge = r(dg.n_rows), r(dg.n_rows), r(dg.n_rows), r(dg.n_edges), r(dg.n_edges)
    cfg = deep_layer_cfg(H, nh, True)
    nb = C.c_size_t()
    call("mp_deep_layer_workspace_size", C.byref(cfg), C.byref(dg.desc), 1, C.byref(nb))

    def adjoint(e_in, g_e_out, g_x):
        g_e, gt = torch.empty_like(e), [torch.empty_like(t) for t in (te, tn)]
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        call("mp_deep_layer_backward", C.byref(cfg), te.data_ptr(), tn.data_ptr(), C.byref(dg.desc), x.data_ptr(),
             e_in.data_ptr(), a.data_ptr(), gx.data_ptr(), g_e_out.data_ptr(), g_x.data_ptr(), g_e.data_ptr(),
             gt[0].data_ptr(), gt[1].data_ptr(), ws.data_ptr(), nb.value, torch.cuda.current_stream().cuda_stream)
        return [g_x, g_e] + gt

    want = adjoint(e, ge, torch.empty_like(x))
    e_in, g_e_out = e.clone(), ge.clone()
    got = adjoint(e_in, g_e_out, (e_in if over == "e_in" else g_e_out)[:dg.n_rows])
    assert all(torch.equal(p, q) for p, q in zip(got, want))
