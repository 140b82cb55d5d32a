"""The accuracy of one FP32 product alone, on the paths that form it from three
BF16 parts per operand (H = 32 and 64).

Left out are m_w l_x + l_w m_x: with weights split by rounding (parts of 2^-8 and
2^-17 of the value) and inputs by cutting (2^-7 and 2^-16), 2^-23 at most; the sum
of the rest rounds within 2^-23.
"""

import numpy as np
import pytest
import torch

from mpinputs import box_mesh

from _util import layer_params

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("H", [32, 64])
def test_one_nonzero_input(H):
    from paper_2410_01657_amd import DeviceGraph, build_graph
    from paper_2410_01657_amd.ops import layer_cfg, layer_forward
    m = box_mesh((6, 5, 4), 4)
    dg = DeviceGraph(build_graph(m.elem_gid, 4, np.zeros(m.n_elem, np.int32), 1), DEV)
    E = dg.n_edges
    _, o, names = layer_params(H, False)
    p = {k: torch.zeros(o[v].shape, device=DEV) for k, v in names.items()}
    gen = torch.Generator().manual_seed(H)
    p["We1"][:, 2 * H:] = torch.rand(H, H, generator=gen).to(DEV) + 0.01
    p["We2"] += torch.eye(H, device=DEV)       # h > 0, so e' = e + h
    col = torch.arange(E, device=DEV) % H
    v = (torch.rand(E, generator=gen) + 0.01).to(DEV)
    e = torch.zeros(E, H, device=DEV)
    e[torch.arange(E, device=DEV), col] = v
    e2 = layer_forward(layer_cfg(H, False), p, dg, torch.zeros(dg.n_rows, H, device=DEV), e)[1]
    want = p["We1"][:, 2 * H:].double().T[col] * v.double()[:, None]
    rel = ((e2.double() - want) / want).abs()
    rel[torch.arange(E, device=DEV), col] = 0   # those hold the residual as well
    assert rel.max().item() <= 2.0 ** -22
