"""The work that users of this framework have it do, as timed cases.

Every case is one call (or one training step) on a partitioned spectral-element
or tetrahedral mesh graph, through the package's public entry points, in the
library's default schedule.  Kinds:

  infer       the whole encode-process-decode model, no gradients
  train       the whole model: forward, consistent MSE, all parameter gradients
  layer_fwd   one message-passing layer, no gradients
  layer_step  one message-passing layer, forward and adjoint
  deep_step   the same for the narrow deep MLPs (Table I's models)
  mlp_step    an encoder or decoder MLP, forward and adjoint

Graphs come from the library's own builder (a mesh is partitioned once and
kept for a whole run); states are LayerNorm-sized, weights Xavier-uniform with
trained-looking biases and gains, upstream gradients those of a mean over all
outputs.
"""

import functools
from dataclasses import dataclass

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2410_01657_amd import ops
from paper_2410_01657_amd.graph import DeviceGraph, build_graph
from paper_2410_01657_amd.model import ConsistentGNN

DEV = "cuda"


@dataclass(frozen=True)
class Spec:
    H: int
    n_layers: int
    n_hidden: int = 0
    layernorm: bool = True
    node_in: int = 3
    edge_in: int = 4
    out: int = 3
    ln_eps: float = 1e-5
    aggregate: str = "state"


# ------------------------------------------------------------------- cases

def _mesh(nx, ny, nz, P, R, part="slabs", elem="hex", drop=0.0):
    return {"nx": nx, "ny": ny, "nz": nz, "P": P, "R": R, "part": part, "elem": elem, "drop": drop}


def listed():
    return [
        # the smallest whole call: a 2,197-node mesh in eight blocks, as in a
        # consistency check or a coupled solver's small test; launches and
        # host work count
        dict(name="infer_tiny_f32_h32", kind="infer", H=32, layers=2, ln=False, gemm="f32", estate="f32",
             **_mesh(4, 4, 4, 3, 8, "blocks")),
        # one layer called by itself on a small odd mesh in BF16 (a roll-out
        # on a coarse grid)
        dict(name="layer_small_bf16_h64", kind="layer_fwd", H=64, ln=True, gemm="bf16", estate="f32",
             **_mesh(5, 7, 3, 5, 3, "uneven")),
        # a training step of the medium workload (16^3 elements of order 5,
        # 16 z-slabs, 4 layers) with BF16 products: encoders, layers, decoder,
        # loss and every gradient
        dict(name="train_medium_bf16_h64", kind="train", H=64, layers=4, ln=True, gemm="bf16", estate="f32",
             **_mesh(16, 16, 16, 5, 16)),
        # the same mesh through one layer in FP32, the library's default type
        dict(name="layer_medium_f32_h64", kind="layer_step", H=64, ln=True, gemm="f32", estate="f32",
             **_mesh(16, 16, 16, 5, 16)),
        # inference on a larger mesh in FP32: one layer forward
        dict(name="layer_fwd_f32_h64", kind="layer_fwd", H=64, ln=True, gemm="f32", estate="f32",
             **_mesh(18, 20, 22, 6, 8, "uneven")),
        # the large batched workload (order 7, uneven sub-graphs), one layer
        # forward and adjoint, at a size that is still quick to prepare
        dict(name="layer_large_bf16_h64", kind="layer_step", H=64, ln=True, gemm="bf16", estate="f32",
             **_mesh(17, 16, 18, 7, 16, "uneven")),
        # the same layer with BF16 edge states (the storage option)
        dict(name="layer_large_es_bf16_h64", kind="layer_step", H=64, ln=True, gemm="bf16", estate="bf16",
             **_mesh(16, 16, 33, 5, 8, "uneven")),
        # the wide model (H = 128), BF16 products, one unpartitioned graph
        dict(name="layer_wide_bf16_h128", kind="layer_step", H=128, ln=True, gemm="bf16", estate="f32",
             **_mesh(20, 20, 20, 5, 1)),
        # the wide model in FP32 on eight blocks (its gradient checks)
        dict(name="layer_wide_f32_h128", kind="layer_step", H=128, ln=True, gemm="f32", estate="f32",
             **_mesh(12, 12, 12, 5, 8, "blocks")),
        # an unstructured tetrahedral mesh with holes: in-degrees of 3 to 14,
        # H = 32, no LayerNorm
        dict(name="layer_tet_f32_h32", kind="layer_step", H=32, ln=False, gemm="f32", estate="f32",
             **_mesh(37, 41, 29, 1, 5, "uneven", "tet", 0.05)),
        # Table I's small model (H = 8, two hidden layers) on two slabs of
        # Table II's size
        dict(name="deep_small_h8", kind="deep_step", H=8, hidden=2, ln=True,
             **_mesh(16, 16, 32, 5, 2)),
        # Table I's large model (H = 32, five hidden layers)
        dict(name="deep_large_h32", kind="deep_step", H=32, hidden=5, ln=True,
             **_mesh(16, 16, 16, 5, 16)),
    ]


def _edges(case):
    if case["elem"] == "tet":
        return 14 * (case["nx"] + 1) * (case["ny"] + 1) * (case["nz"] + 1)
    n = [case[k] * case["P"] + 1 for k in ("nx", "ny", "nz")]
    return 6 * n[0] * n[1] * n[2]


def draw(rng):
    """A case of the same ranges: 300 to 2 million rows, any kind, width,
    type and partition."""
    kind = rng.choice(["infer", "train", "layer_fwd", "layer_step", "layer_step", "deep_step", "mlp_step"])
    gemm = rng.choice(["f32", "bf16"])
    H = rng.choice([32, 64, 64, 128])
    # the largest cost drawn stays below the largest listed case's
    top = {"infer": 4e6, "train": 2e6, "layer_fwd": 9e6, "layer_step": 6e6, "deep_step": 3e6, "mlp_step": 9e6}[kind]
    if H == 128 and kind != "deep_step":
        top /= 4
    target = 10.0 ** rng.uniform(3.5, np.log10(top))   # directed edges
    elem = rng.choice(["hex", "hex", "hex", "tet"])
    P = 1 if elem == "tet" else rng.choice([1, 2, 3, 4, 5, 6, 7])
    side = (target / (14.0 if elem == "tet" else 6.0)) ** (1.0 / 3.0) / P
    nel = [max(2, int(round(side * rng.uniform(0.75, 1.3)))) for _ in range(3)]
    R = rng.choice([1, 1, 2, 3, 4, 7, 8, 16])
    R = min(R, nel[2])
    case = dict(kind=kind, H=H, ln=rng.random() < 0.8, **_mesh(*nel, P, R, "uneven" if R > 1 else "slabs", elem,
                                                              0.03 if elem == "tet" else 0.0))
    if kind == "deep_step":
        case["H"], case["hidden"] = rng.choice([(8, 2), (8, 1), (16, 2), (32, 5), (32, 3), (32, 0)])
        return case
    case["gemm"] = gemm
    case["estate"] = rng.choice(["f32", "bf16"]) if gemm == "bf16" else "f32"
    if kind in ("infer", "train"):
        case["layers"] = rng.choice([2, 4])
    if kind == "mlp_step":
        case["form"] = rng.choice(["eenc", "nenc", "dec"])
        case["estate"] = "f32"
    return case


# -------------------------------------------------------------- mesh graphs

def _axis(n, P):
    """Gauss-Legendre-Lobatto positions of n elements of order P on [0, 1]."""
    x = np.array([-1.0, 1.0])
    if P > 1:
        d = np.polynomial.legendre.Legendre.basis(P).deriv().roots()
        x = np.concatenate([[-1.0], np.sort(d.real), [1.0]])
    t = (x + 1.0) / 2.0
    return np.concatenate([(e + t[:-1]) / n for e in range(n)] + [[1.0]])


def _key(case):
    return tuple(case[k] for k in ("nx", "ny", "nz", "P", "R", "part", "elem", "drop"))


@functools.lru_cache(maxsize=None)
def _host_graph(key):
    """(partitioned host graph, node positions) of a mesh: hexahedra of order
    P, or each cell of the box cut into six tetrahedra with a fraction of the
    cells missing."""
    nx, ny, nz, P, R, part, elem, drop = key
    rng = np.random.default_rng(7)
    npts = (nx * P + 1, ny * P + 1, nz * P + 1)
    e = np.arange(nx * ny * nz)
    ex, ey, ez = e % nx, (e // nx) % ny, e // (nx * ny)
    q = np.arange(P + 1)
    la, lb, lc = np.tile(q, (P + 1) ** 2), np.tile(np.repeat(q, P + 1), P + 1), np.repeat(q, (P + 1) ** 2)
    gid = ((ex[:, None] * P + la) + npts[0] * ((ey[:, None] * P + lb)
           + npts[1] * (ez[:, None] * P + lc).astype(np.int64)))
    if part == "blocks":
        p = (ex * 2 // nx) + 2 * (ey * 2 // ny) + 4 * (ez * 2 // nz)
    elif part == "slabs":
        p = ez * R // nz
    else:  # uneven slabs along z, the thickest about three times the thinnest
        w = np.cumsum(rng.uniform(1.0, 3.0, R))
        cut = np.maximum.accumulate(np.round(w[:-1] / w[-1] * nz).astype(int)) if R > 1 else np.zeros(0, int)
        cut = np.array([min(max(c, i + 1), nz - (R - 1 - i)) for i, c in enumerate(cut)], int)
        p = np.searchsorted(cut, ez, side="right")
    links = None
    if elem == "tet":
        # the six tetrahedra around a cell's long diagonal
        order = [(0, 1, 3, 7), (0, 1, 5, 7), (0, 2, 3, 7), (0, 2, 6, 7), (0, 4, 5, 7), (0, 4, 6, 7)]
        keep = rng.random(e.shape[0]) >= drop
        first = np.unique(p, return_index=True)[1]   # every part keeps a cell
        keep[first] = True
        gid = np.concatenate([gid[keep][:, o] for o in order])
        p = np.tile(p[keep], 6)
        used, gid = np.unique(gid, return_inverse=True)
        gid = gid.reshape(-1, 4)
        links = np.array([(i, j) for i in range(4) for j in range(i + 1, 4)], np.int32)
    else:
        used = np.arange(npts[0] * npts[1] * npts[2], dtype=np.int64)
    ax = [_axis(n, P) for n in (nx, ny, nz)]
    pos = np.stack([ax[0][used % npts[0]], ax[1][(used // npts[0]) % npts[1]], ax[2][used // (npts[0] * npts[1])]], 1)
    return build_graph(gid, P, p.astype(np.int32), R, links), pos


# ------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, *shape, scale=1.0):
    return torch.randn(*shape, generator=g, device=DEV).mul_(scale)


def _mlp_shapes(prefix, k, H, out, hidden, ln):
    dims = [k] + [H] * (hidden + 1) + [out]
    s = []
    for i in range(len(dims) - 1):
        s += [(f"{prefix}.lin{i}.W", (dims[i + 1], dims[i])), (f"{prefix}.lin{i}.b", (dims[i + 1],))]
    if ln:
        s += [(f"{prefix}.ln.g", (out,)), (f"{prefix}.ln.b", (out,))]
    return s


def _weights(shapes, seed):
    """Xavier-uniform weights; biases, gains and shifts as after training."""
    r = np.random.default_rng(seed)
    out = {}
    for name, shape in shapes:
        if name.endswith(".W"):
            a = np.sqrt(6.0 / (shape[0] + shape[1]))
            v = r.uniform(-a, a, shape)
        elif name.endswith(".ln.g"):
            v = r.uniform(0.5, 1.5, shape)
        else:
            v = r.uniform(-0.2, 0.2, shape)
        out[name] = v.astype(np.float32)
    return out


def _spec(case):
    return Spec(H=case["H"], n_layers=case["layers"], layernorm=case["ln"])


def _model_shapes(case):
    H, ln = case["H"], case["ln"]
    s = _mlp_shapes("nenc", 3, H, H, 0, ln) + _mlp_shapes("eenc", 4, H, H, 0, ln)
    for m in range(case["layers"]):
        s += _mlp_shapes(f"mp{m}.edge", 3 * H, H, H, 0, ln) + _mlp_shapes(f"mp{m}.node", 2 * H, H, H, 0, ln)
    return s + _mlp_shapes("dec", H, H, 3, 0, False)


def _field(case, seed):
    """Taylor-Green-like velocity at the rows, with noise, and its target."""
    hg, pos = _host_graph(_key(case))
    r = np.random.default_rng(seed)
    ph = r.uniform(0.0, 2.0 * np.pi, 3)

    def u(shift):
        t = 2.0 * np.pi * pos + ph + shift
        f = np.stack([np.sin(t[:, 0]) * np.cos(t[:, 1]) * np.cos(t[:, 2]),
                      -np.cos(t[:, 0]) * np.sin(t[:, 1]) * np.cos(t[:, 2]), np.zeros(len(pos))], 1)
        return f
    X = (u(0.0) + r.normal(0.0, 0.01, pos.shape)).astype(np.float32)
    T = u(0.1).astype(np.float32)
    return (torch.from_numpy(X[hg.row_gid]).to(DEV), torch.from_numpy(T[hg.row_gid]).to(DEV),
            torch.from_numpy(pos[hg.row_gid]).to(DEV))


def _states(case, seed):
    """(x, e, g_x, g_e): node and edge states and the gradients arriving at
    a layer's outputs."""
    hg, _ = _host_graph(_key(case))
    g, H = _gen(seed), case["H"]
    edt = torch.bfloat16 if case.get("estate") == "bf16" else torch.float32
    x, e = _randn(g, hg.n_rows, H), _randn(g, hg.n_edges, H).to(edt)
    if case["kind"] == "layer_fwd":
        return x, e, None, None
    s = 1.0 / hg.n_rows
    return x, e, _randn(g, hg.n_rows, H, scale=s), _randn(g, hg.n_edges, H, scale=s).to(edt)


def _layer_weights(case, seed):
    H, ln, nh = case["H"], case["ln"], case.get("hidden", 0)
    return _weights(_mlp_shapes("edge", 3 * H, H, H, nh, ln) + _mlp_shapes("node", 2 * H, H, H, nh, ln), seed)


_LAYER = ["edge.lin0.W", "edge.lin0.b", "edge.lin1.W", "edge.lin1.b", "edge.ln.g", "edge.ln.b",
          "node.lin0.W", "node.lin0.b", "node.lin1.W", "node.lin1.b", "node.ln.g", "node.ln.b"]
_FORMS = {"eenc": (4, None), "nenc": (3, None), "dec": (None, 3)}


def _mlp_dims(case):
    k, o = _FORMS[case["form"]]
    return k or case["H"], o or case["H"], case["ln"] and o is None


def _mlp_inputs(case, seed):
    hg, _ = _host_graph(_key(case))
    k, o, _ = _mlp_dims(case)
    n = hg.n_edges if case["form"] == "eenc" else hg.n_rows
    g = _gen(seed)
    x = _randn(g, n, k, scale=0.1 if case["form"] == "eenc" else 1.0)
    return x, _randn(g, n, o, scale=1.0 / n)


def _tensors(w):
    return {k: torch.from_numpy(v).to(DEV) for k, v in w.items()}


def _flat(w, prefix):
    return torch.cat([v.reshape(-1) for k, v in w.items() if k.startswith(prefix)])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp_step":
        k, o, ln = _mlp_dims(case)
        x, go = _mlp_inputs(case, seed)
        w = _tensors(_weights(_mlp_shapes("m", k, case["H"], o, 0, ln), seed))
        params = [v.requires_grad_(True) for v in w.values()]
        return {"kind": kind, "cfg": ops.mlp_cfg(k, case["H"], o, ln, case["gemm"]),
                "x": x.requires_grad_(case["form"] == "dec"), "go": go, "params": params}
    hg, _ = _host_graph(_key(case))
    dg = DeviceGraph(hg, DEV)
    st = {"kind": kind, "dg": dg}
    if kind in ("infer", "train"):
        X, T, pos = _field(case, seed)
        model = ConsistentGNN(_spec(case), _weights(_model_shapes(case), seed), DEV, gemm=case["gemm"],
                              estate=case["estate"])
        st.update(model=model.requires_grad_(kind == "train"), X=X, T=T, E0=ops.edge_inputs(dg, pos))
        return st
    x, e, gx, ge = _states(case, seed)
    w = _tensors(_layer_weights(case, seed))
    if kind == "layer_fwd":
        names = ops.LAYER_FIELDS
        p = {f: w.get(n) for f, n in zip(names, _LAYER)}
        st.update(cfg=ops.layer_cfg(case["H"], case["ln"], True, case["gemm"], estate=case["estate"]), p=p, x=x, e=e)
        return st
    st.update(x=x.requires_grad_(True), e=e.requires_grad_(True), gx=gx, ge=ge)
    if kind == "deep_step":
        st["cfg"] = ops.deep_layer_cfg(case["H"], case["hidden"], case["ln"])
        st["params"] = [_flat(w, "edge").requires_grad_(True), _flat(w, "node").requires_grad_(True)]
    else:
        st["cfg"] = ops.layer_cfg(case["H"], case["ln"], True, case["gemm"], estate=case["estate"])
        st["params"] = [w[n].requires_grad_(True) if n in w else None for n in _LAYER]
    return st


def run(st):
    kind = st["kind"]
    if kind == "infer":
        with torch.no_grad():
            return st["model"].forward(st["dg"], st["X"], st["E0"])
    if kind == "train":
        model = st["model"]
        for t in model.params.values():
            t.grad = None
        Y = model.forward(st["dg"], st["X"], st["E0"])
        loss = model.loss(st["dg"], Y, st["T"])
        loss.backward()
        return Y.detach(), loss.detach(), torch.cat([t.grad.reshape(-1) for t in model.params.values()])
    if kind == "layer_fwd":
        return ops.layer_forward(st["cfg"], st["p"], st["dg"], st["x"], st["e"])
    if kind == "mlp_step":
        out = ops.MLPFn.apply(st["cfg"], st["x"], *(st["params"] + [None] * (6 - len(st["params"]))))
        wrt = ([st["x"]] if st["x"].requires_grad else []) + st["params"]
        return (out.detach(),) + torch.autograd.grad(out, wrt, st["go"])
    if kind == "deep_step":
        out = ops.DeepLayerFn.apply(st["cfg"], st["dg"], st["x"], st["e"], *st["params"])
    else:
        out = ops.MPLayerFn.apply(st["cfg"], st["dg"], True, st["x"], st["e"], *st["params"])
    wrt = [st["x"], st["e"]] + [p for p in st["params"] if p is not None]
    return (out[0].detach(), out[1].detach()) + torch.autograd.grad(list(out), wrt, [st["gx"], st["ge"]])


# --------------------------------------------------------------------- work

def work(case):
    """Each input read once and each output written once; the products of the
    forward, and for a step those of the two adjoint products as well."""
    kind, H = case["kind"], case["H"]
    hg, _ = _host_graph(_key(case))
    N, E = hg.n_rows, hg.n_edges
    if kind == "mlp_step":
        k, o, _ = _mlp_dims(case)
        n = E if case["form"] == "eenc" else N
        gin = k if case["form"] == "dec" else 0
        return {"bytes": 4 * n * (k + 2 * o + gin), "flops": 3 * 2 * n * (k * H + H * o)}
    es = 2 if case.get("estate") == "bf16" else 4
    nh = case.get("hidden", 0)
    if nh or kind == "deep_step":
        fl = 2 * E * (3 * H * H + (nh + 1) * H * H) + 2 * N * (2 * H * H + (nh + 1) * H * H)
    else:
        fl = 2 * E * 2 * H * H + 2 * N * 5 * H * H
    graph = 9 * E + 4 * N
    fwd = E * H * 2 * es + N * H * 2 * 4
    if kind == "layer_fwd":
        return {"bytes": fwd + N * H * 4 + graph, "flops": fl}
    if kind in ("layer_step", "deep_step"):
        return {"bytes": fwd + E * H * 2 * es + N * H * 2 * 4 + graph + 4 * E, "flops": 3 * fl}
    enc = 2 * E * (4 * H + H * H) + 2 * N * (2 * 3 * H + 2 * H * H)
    fl = case["layers"] * fl + enc
    # the mesh inputs and the outputs alone; what passes between the layers
    # (the edge states) does not fit on the chip and counts once each way
    mid = case["layers"] * E * H * 2 * es
    if kind == "infer":
        return {"bytes": 16 * E + 24 * N + graph + mid, "flops": fl}
    return {"bytes": 16 * E + 36 * N + graph + 3 * mid, "flops": 3 * fl}


# ------------------------------------------------------- 64-bit references

_CHUNK = 1 << 21   # rows of one library product (some fail on very many rows)


def _mlp64(p, prefix, z, ln, hidden=0):
    if z.shape[0] > _CHUNK:
        return torch.cat([_mlp64(p, prefix, c, ln, hidden) for c in z.split(_CHUNK)])
    n = hidden + 2
    for k in range(n):
        z = torch.nn.functional.linear(z, p[f"{prefix}.lin{k}.W"], p[f"{prefix}.lin{k}.b"])
        if k < n - 1:
            z = torch.nn.functional.elu(z)
    if ln:
        z = torch.nn.functional.layer_norm(z, z.shape[-1:], p[f"{prefix}.ln.g"], p[f"{prefix}.ln.b"], 1e-5)
    return z


class _Graph64:
    def __init__(self, case):
        hg, self.pos = _host_graph(_key(case))
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        self.recv, self.col = t(hg.recv).long(), t(hg.col).long()
        self.inv_d = 1.0 / t(hg.edge_mult).double()
        self.gid, self.n, self.row_gid = t(hg.row_gid), hg.n_rows, hg.row_gid
        self.n_gid = int(hg.row_gid.max()) + 1
        self.node_mult = t(hg.node_mult).double()


def _layer64(G, p, pre, x, e, H, ln, hidden=0):
    """(x', e', a*) of one consistent layer, the first edge Linear applied to
    its three inputs one by one, chunks of edges at a time."""
    W = p[pre + "edge.lin0.W"]
    lin = torch.nn.functional.linear
    P, Q = lin(x, W[:, :H]), lin(x, W[:, H:2 * H])
    n = hidden + 2
    out = []
    for ec, rc, cc in zip(e.split(_CHUNK), G.recv.split(_CHUNK), G.col.split(_CHUNK)):
        z = torch.nn.functional.elu(lin(ec, W[:, 2 * H:], p[pre + "edge.lin0.b"]) + P[rc] + Q[cc])
        for k in range(1, n):
            z = lin(z, p[f"{pre}edge.lin{k}.W"], p[f"{pre}edge.lin{k}.b"])
            if k < n - 1:
                z = torch.nn.functional.elu(z)
        if ln:
            z = torch.nn.functional.layer_norm(z, z.shape[-1:], p[pre + "edge.ln.g"], p[pre + "edge.ln.b"], 1e-5)
        out.append(ec + z)
    e2 = torch.cat(out)
    a = torch.zeros_like(x).index_add(0, G.recv, e2 * G.inv_d[:, None])
    s = torch.zeros(G.n_gid, H, dtype=x.dtype, device=x.device).index_add(0, G.gid, a)
    a = s[G.gid]
    return x + _mlp64(p, pre + "node", torch.cat([a, x], 1), ln, hidden), e2, a


def _p64(w, grad):
    return {k: torch.from_numpy(v).to(DEV).double().requires_grad_(grad) for k, v in w.items()}


def exact(case, seed):
    kind, H, ln = case["kind"], case["H"], case["ln"]
    if kind == "mlp_step":
        k, o, mln = _mlp_dims(case)
        x, go = _mlp_inputs(case, seed)
        p = _p64(_weights(_mlp_shapes("m", k, H, o, 0, mln), seed), True)
        x = x.double().requires_grad_(case["form"] == "dec")
        out = _mlp64(p, "m", x, mln)
        wrt = ([x] if x.requires_grad else []) + list(p.values())
        return (out.detach(),) + torch.autograd.grad(out, wrt, go.double())
    G = _Graph64(case)
    if kind in ("infer", "train"):
        X, T, pos = _field(case, seed)
        d = pos[G.col] - pos[G.recv]
        E0 = torch.cat([d, d.norm(dim=1, keepdim=True)], 1).float().double()
        p = _p64(_weights(_model_shapes(case), seed), kind == "train")
        with torch.set_grad_enabled(kind == "train"):
            x = _mlp64(p, "nenc", X.double(), ln)
            ck = functools.partial(checkpoint, use_reentrant=False)
            e = ck(lambda z: _mlp64(p, "eenc", z, ln), E0)
            for m in range(case["layers"]):
                x, e = ck(lambda x_, e_, m_=m: _layer64(G, p, f"mp{m_}.", x_, e_, H, ln)[:2], x, e)
            Y = _mlp64(p, "dec", x, False)
        if kind == "infer":
            return Y
        w = 1.0 / G.node_mult
        loss = (w[:, None] * (Y - T.double()) ** 2).sum() / (w.sum() * 3)
        grads = torch.autograd.grad(loss, list(p.values()))
        return Y.detach(), loss.detach(), torch.cat([t.reshape(-1) for t in grads])
    x, e, gx, ge = _states(case, seed)
    nh = case.get("hidden", 0)
    w = _layer_weights(case, seed)
    if kind == "layer_fwd":
        with torch.no_grad():
            return _layer64(G, _p64(w, False), "", x.double(), e.double(), H, ln)
    p = _p64(w, True)
    x, e = x.double().requires_grad_(True), e.double().requires_grad_(True)
    x2, e2, _ = _layer64(G, p, "", x, e, H, ln, nh)
    if kind == "deep_step":
        wrt = [x, e] + list(p.values())
        g = torch.autograd.grad([x2, e2], wrt, [gx.double(), ge.double()])
        ne = sum(k.startswith("edge") for k in p)
        flat = lambda ts: torch.cat([t.reshape(-1) for t in ts])
        return (x2.detach(), e2.detach(), g[0], g[1], flat(g[2:2 + ne]), flat(g[2 + ne:]))
    wrt = [x, e] + [p[n] for n in _LAYER if n in p]
    return (x2.detach(), e2.detach()) + torch.autograd.grad([x2, e2], wrt, [gx.double(), ge.double()])
