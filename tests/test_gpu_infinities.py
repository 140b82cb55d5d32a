"""FP32 arithmetic at the ends of its range, on the paths whose products are formed
from BF16 parts (H = 32 and 64, and the width-32 deep layers).

An infinite operand has no parts; the results must be those of FP32 arithmetic all
the same: infinite where the reference (FP64) is, NaN where it is, and elsewhere
within the bounds of the parity tests (forward 1e-5, gradients 1e-4).  Only edge
arrays are compared where the aggregate of a row is infinite (the segmented sum of
a block multiplies by zero).
"""

import numpy as np
import pytest
import torch

from mpinputs import box_mesh, slab_partition

from _util import layer_params, normwise

pytestmark = pytest.mark.gpu

DEV, INF = "cuda", float("inf")


def _graph():
    from paper_2410_01657_amd import DeviceGraph, build_graph
    m = box_mesh((3, 5, 2), 3)
    return DeviceGraph(build_graph(m.elem_gid, 3, slab_partition((3, 5, 2), 2), 2), DEV)


def _same(got, want, tol):
    """Equal infinities and NaNs, the rest within tol of the largest finite value."""
    got, want = got.detach().double().cpu(), want.detach().double().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    inf = torch.isinf(want)
    assert torch.equal(torch.isinf(got), inf) and torch.equal(got[inf], want[inf])
    fin = torch.isfinite(want)
    assert normwise(got[fin], want[fin]) < tol


def _mlp(z, pairs, ln):
    for k, (W, b) in enumerate(pairs):
        z = torch.nn.functional.linear(z, W, b)
        if k + 1 < len(pairs):
            z = torch.nn.functional.elu(z)
    return torch.nn.functional.layer_norm(z, z.shape[-1:], *ln, 1e-5) if ln is not None else z


def _ref(dg, edge, node, lne, lnn, x, e):
    """x', e', a* in FP64 for MLPs given as lists of (W, b)."""
    recv, col = dg.recv.long(), dg.col.long()
    e2 = e + _mlp(torch.cat([x[recv], x[col], e], 1), edge, lne)
    a = torch.zeros_like(x).index_add(0, recv, e2 / dg.edge_mult.double()[:, None])
    gid = torch.from_numpy(dg.host.row_gid).to(DEV)
    a = torch.zeros(int(gid.max()) + 1, x.shape[1], dtype=x.dtype, device=DEV).index_add(0, gid, a)[gid]
    return x + _mlp(torch.cat([a, x], 1), node, lnn), e2, a


def _layer(H, ln, seed=11):
    _, o, names = layer_params(H, ln, seed)
    return {k: torch.from_numpy(o[v].astype(np.float32)).to(DEV) for k, v in names.items()}


def _layer_ref(dg, p, x, e):
    d = {k: (v if v.dtype == torch.float64 else v.double()) for k, v in p.items()}
    return _ref(dg, [(d["We1"], d["be1"]), (d["We2"], d["be2"])], [(d["Wn1"], d["bn1"]), (d["Wn2"], d["bn2"])],
                (d["ge"], d["bge"]) if "ge" in d else None, (d["gn"], d["bgn"]) if "gn" in d else None, x, e)


def _rows(H, *ns, seed=2):
    gen = torch.Generator().manual_seed(seed)
    return [torch.randn(n, H, generator=gen).to(DEV) for n in ns]


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("ln", [False, True])
def test_minus_infinity_in_a_node_state(H, ln):
    """Positive node columns: every pre-activation the row reaches is -inf, ELU -1,
    and the layer's other results are finite."""
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg, layer_forward
    dg, p = _graph(), _layer(H, ln)
    p["We1"][:, :2 * H].abs_().add_(0.01)
    p["Wn1"][:, H:].abs_().add_(0.01)
    x, e, gx, ge = _rows(H, dg.n_rows, dg.n_edges, dg.n_rows, dg.n_edges)
    x[dg.n_rows // 2, 3] = -INF
    cfg = layer_cfg(H, ln)
    x2, e2, a, pq = layer_forward(cfg, p, dg, x, e, want_pq=True)
    ins = [x.double().requires_grad_(True), e.double().requires_grad_(True)]
    pd = {k: v.double().requires_grad_(True) for k, v in p.items()}
    want = _layer_ref(dg, pd, *ins)
    assert torch.isfinite(want[1]).all() and torch.isfinite(want[2]).all()
    for got, ref in zip((x2, e2, a), want):
        _same(got, ref, 1e-5)
    g_x, g_e, grads = layer_backward(cfg, p, dg, x, e, a, gx, ge, pq)
    names = ["We2", "be2", "Wn2", "bn2", "be1", "bn1"]
    ref = torch.autograd.grad(list(want[:2]), ins + [pd[k] for k in names], [gx.double(), ge.double()])
    for got, r in zip([g_x, g_e] + [grads[k] for k in names], ref):
        assert torch.isfinite(r).all()
        _same(got, r, 1e-4)


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("case", ["x", "e", "both signs", "We1 node", "We1 edge", "We2", "overflow"])
def test_infinite_operands_of_the_edge_update(H, case):
    from paper_2410_01657_amd.ops import layer_cfg, layer_forward
    dg, p = _graph(), _layer(H, False)
    x, e = _rows(H, dg.n_rows, dg.n_edges)
    k = dg.n_edges // 3
    if case == "x":
        x[5, 1] = INF
    elif case == "e":
        e[k, H - 1] = -INF
    elif case == "both signs":
        e[k, 0], e[k, 1], e[k + 40, 7] = INF, -INF, INF
    elif case == "We1 node":
        p["We1"][4, H + 2] = INF
    elif case == "We1 edge":
        p["We1"][H - 2, 2 * H + 9] = -INF
    elif case == "We2":
        p["We2"][H // 2 + 1, 6] = INF
    else:
        # finite, but one first pre-activation is beyond FP32's range
        p["We1"][3, 2 * H] = 1e20
        e[k, 0] = 1e20
    _, e2, _ = layer_forward(layer_cfg(H, False), p, dg, x, e)
    if case == "overflow":
        pd = {n: v.double() for n, v in p.items()}
        want = _layer_ref(dg, pd, x.double(), e.double())[1]
        h = torch.nn.functional.linear(torch.cat([x[dg.recv.long()], x[dg.col.long()], e], 1).double(), pd["We1"], pd["be1"])
        u = torch.nn.functional.elu(torch.where(h.abs() > 3.4e38, torch.sign(h) * INF, h))
        want = e.double() + torch.nn.functional.linear(u, pd["We2"], pd["be2"])
    else:
        want = _layer_ref(dg, p, x.double(), e.double())[1]
    assert not torch.isfinite(want).all()
    _same(e2, want, 1e-5)


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("agg", ["state", "message"])
def test_infinite_gradient_of_an_edge(H, agg):
    from paper_2410_01657_amd.ops import layer_backward, layer_cfg
    dg, p = _graph(), _layer(H, False)
    x, e, a, gx, ge = _rows(H, dg.n_rows, dg.n_edges, dg.n_rows, dg.n_rows, dg.n_edges)
    ge[dg.n_edges // 2, 9] = INF
    g_e = layer_backward(layer_cfg(H, False, aggregate=agg), p, dg, x, e, a, torch.zeros_like(gx), ge)[1]
    # with no gradient at x', g_e = g_e' + J^T g_e' edge by edge; zero times infinity is left to IEEE
    d = {k: v.double() for k, v in p.items()}
    recv, col = dg.recv.long(), dg.col.long()
    h = torch.nn.functional.linear(torch.cat([x[recv], x[col], e], 1).double(), d["We1"], d["be1"])
    gh = (ge.double() @ d["We2"]) * torch.where(h > 0, torch.ones_like(h), torch.exp(h))
    _same(g_e, ge.double() + gh @ d["We1"][:, 2 * H:], 1e-4)


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("form", ["eenc", "nenc", "wide", "dec"])
def test_minus_infinity_into_an_mlp(H, form):
    from paper_2410_01657_amd.ops import MLP_FIELDS, mlp_cfg, mlp_forward
    k, o = {"eenc": (4, H), "nenc": (3, H), "wide": (H, H), "dec": (H, 3)}[form]
    gen = torch.Generator().manual_seed(H)
    w = [torch.rand(H, k, generator=gen) + 0.01, torch.randn(H, generator=gen),
         torch.randn(o, H, generator=gen), torch.randn(o, generator=gen)]
    w = [t.to(DEV) for t in w]
    x = torch.randn(1000, k, generator=gen).to(DEV)
    x[77, 1] = -INF
    for dead in (False, True):
        if dead:    # and an infinite pre-activation of the other sign
            x[500, 0] = INF
        out = mlp_forward(mlp_cfg(k, H, o, False), dict(zip(MLP_FIELDS, w)), x)
        _same(out, _mlp(x.double(), [(w[0].double(), w[1].double()), (w[2].double(), w[3].double())], None), 1e-5)


def _theta(gen, n_in, H, nh, ln):
    flat, pairs, k = [], [], n_in
    for _ in range(nh + 2):
        W = (torch.rand(H, k, generator=gen) * 2 - 1) * (6.0 / (k + H)) ** 0.5
        pairs.append((W.to(DEV), ((torch.rand(H, generator=gen) * 2 - 1) * 0.2).to(DEV)))
        k = H
    g = [(torch.rand(H, generator=gen) + 0.5).to(DEV), ((torch.rand(H, generator=gen) * 2 - 1) * 0.2).to(DEV)] if ln else None
    return pairs, g


def _flat(pairs, g):
    return torch.cat([t.reshape(-1) for pr in pairs for t in pr] + ([] if g is None else g))


@pytest.mark.parametrize("nh,ln", [(0, False), (1, True), (2, False), (5, True), (5, False), (6, True)])
def test_minus_infinity_in_a_deep_layer(nh, ln):
    from paper_2410_01657_amd.ops import DeepLayerFn, deep_layer_cfg
    H, dg = 32, _graph()
    gen = torch.Generator().manual_seed(nh)
    edge, lne = _theta(gen, 3 * H, H, nh, ln)
    node, lnn = _theta(gen, 2 * H, H, nh, ln)
    edge[0][0][:, :2 * H].abs_().add_(0.01)
    node[0][0][:, H:].abs_().add_(0.01)
    x, e, gx, ge = _rows(H, dg.n_rows, dg.n_edges, dg.n_rows, dg.n_edges)
    x[dg.n_rows // 2, 3] = -INF
    ins = [x.requires_grad_(True), e.requires_grad_(True)]
    out = DeepLayerFn.apply(deep_layer_cfg(H, nh, ln), dg, *ins, _flat(edge, lne), _flat(node, lnn))
    got = torch.autograd.grad(list(out), ins, [gx, ge])
    d = [t.detach().double().requires_grad_(True) for t in ins]
    dbl = lambda ps: [(W.double(), b.double()) for W, b in ps]
    ln64 = lambda g: None if g is None else [t.double() for t in g]
    want = _ref(dg, dbl(edge), dbl(node), ln64(lne), ln64(lnn), *d)
    assert torch.isfinite(want[1]).all()
    for u, v in zip(out, want):
        _same(u, v, 1e-5)
    for u, v in zip(got, torch.autograd.grad(list(want[:2]), d, [gx.double(), ge.double()])):
        assert torch.isfinite(v).all()
        _same(u, v, 1e-4)


@pytest.mark.parametrize("where", ["e", "W0", "Wo"])
@pytest.mark.parametrize("nh", [0, 2, 5])
def test_infinite_operands_of_a_deep_edge_update(nh, where):
    from paper_2410_01657_amd.ops import DeepLayerFn, deep_layer_cfg
    H, dg = 32, _graph()
    gen = torch.Generator().manual_seed(nh + 20)
    edge, _ = _theta(gen, 3 * H, H, nh, False)
    node, _ = _theta(gen, 2 * H, H, nh, False)
    x, e = _rows(H, dg.n_rows, dg.n_edges)
    if where == "e":
        e[dg.n_edges // 2, 5] = INF
    elif where == "W0":
        edge[0][0][7, H + 3] = -INF
    else:
        edge[-1][0][20, 4] = INF
    _, e2 = DeepLayerFn.apply(deep_layer_cfg(H, nh, False), dg, x, e, _flat(edge, None), _flat(node, None))
    want = _ref(dg, [(W.double(), b.double()) for W, b in edge], [(W.double(), b.double()) for W, b in node], None, None,
                x.double(), e.double())[1]
    assert not torch.isfinite(want).all()
    _same(e2, want, 1e-5)


@pytest.mark.parametrize("H", [32, 64])
def test_identity_weights_at_the_ends_of_the_range(H):
    """e' = 2 e exactly up to the largest e whose double is finite; below 2^-100
    parts under 2^-133 (the smallest BF16 value) are lost: two products of three
    parts each, 6 x 2^-133 at most."""
    from paper_2410_01657_amd.ops import layer_cfg, layer_forward
    dg = _graph()
    _, o, names = layer_params(H, False)
    p = {k: torch.zeros(o[v].shape, device=DEV) for k, v in names.items()}
    eye = torch.eye(H, device=DEV)
    p["We1"][:, 2 * H:] = eye
    p["We2"] += eye
    x = torch.zeros(dg.n_rows, H, device=DEV)
    gen = torch.Generator().manual_seed(H)
    bits = lambda lo, hi: ((torch.randint(lo, hi, (dg.n_edges, H), generator=gen, dtype=torch.int32) << 23)
                           | torch.randint(0, 1 << 23, (dg.n_edges, H), generator=gen, dtype=torch.int32)).view(torch.float32).to(DEV)
    big, tiny = bits(220, 254), bits(1, 27)
    big[3, 5] = torch.finfo(torch.float32).max / 2
    run = lambda e: layer_forward(layer_cfg(H, False), p, dg, x, e)[1]
    assert torch.equal(run(big), 2 * big)
    assert (run(tiny).double() - 2 * tiny.double()).abs().max().item() <= 6 * 2.0 ** -133
