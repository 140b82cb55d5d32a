"""Algorithmic work of each kernel of one layer: the bytes it must move
through HBM and the flops it must execute, independent of how it is built.

Units: N rows (node copies over all sub-graphs), E directed sub-graph edges,
G halo groups with M members, hidden width H, FP32 node states, FP32 or BF16
edge states.
Index arrays: int32 receiver and sender per edge plus a uint8 degree;
int32 reverse-edge and row-offset arrays where a kernel follows them.
Each row or edge is counted once per kernel even when it is gathered several
times (repeat gathers are cache traffic, not algorithmic traffic).

Flops count the MLP products (2 per multiply-add); elementwise work (ELU,
LayerNorm, the 1/d sums) is below 1% and left out.
"""

from dataclasses import dataclass

# MI355X published peaks
PEAK_HBM = 8.0e12          # bytes/s
PEAK = {"f32": 157.3e12, "bf16": 2.5e15}   # dense MFMA flop/s by operand type
# FP32 products formed from three BF16 parts per operand take six BF16 products
PEAK_F32_PARTS = PEAK["bf16"] / 6
# FP32 vector ALU: 256 CUs x 4 SIMDs x 16 lanes x 2 flops (FMA) x 2 (packed
# FP32) x 2.4 GHz.  The library is built without packed FP32 operations, so
# its own ceiling is half of this (78.6 TFLOP/s).
PEAK_VALU = 157.3e12


@dataclass(frozen=True)
class Work:
    bytes: float
    flops: float


def edge_bwd_split(H, gemm="f32"):
    """Whether the edge adjoint runs in two passes (per-edge factors, then the
    weight-gradient sums): FP32 at widths above 64."""
    return H > 64 and gemm == "f32"


def node_bwd_split(H):
    return H > 64


def gq_split(H, gemm):
    return H > 64 and gemm == "f32"


def matrix_peak(kernel, H, gemm):
    """Matrix flop/s that a layer kernel's products can reach: FP32 products
    run from BF16 parts at H <= 64 (but for the node update's adjoint and the
    sender-side pass) and in the weight-gradient passes above."""
    parts = kernel.endswith("_dw") if H > 64 else kernel in ("proj", "edge_fwd", "node_fwd", "edge_bwd")
    return PEAK_F32_PARTS if gemm == "f32" and parts else PEAK[gemm]


def layer_kernels(N, E, G, M, H, gemm="bf16", n_layers=1, estate="f32"):
    """Per launch, for one layer; keys match the library's profile names.

    gemm: "bf16" stores the edge-state adjoint g_h in BF16 (2 bytes per
    value), "f32" in FP32.  n_layers: the adjoint kernels are averaged over
    the layers of a model, whose last layer gets no gradient at its edge
    output (g_e' is absent there).  estate: storage type of the edge states
    e, e' and their gradients ("bf16": 2 bytes per value).

    At H > 64 the edge and node adjoints (and, in FP32, the sender-side
    pass) are counted split: the first pass recomputes the MLP and forms the input
    gradients, a second pass (edge_dw / node_dw / gq_dw) sums the weight
    gradients from per-row factors the first pass stored.  The products are
    then counted where they run; the stored factors are implementation
    traffic, and each second pass is charged only the bytes of the factors
    it must read (one launch of edge_dw / node_dw / gq_dw stands for all of
    that pass's launches in a layer).  The BF16 edge adjoint forms its weight
    gradients itself: launched_kernels has it as it runs."""
    f = 4.0                              # bytes per FP32 value
    fe = 2.0 if estate == "bf16" else 4.0  # bytes per edge-state value
    fh = 2.0 if gemm == "bf16" else 4.0  # bytes per g_h value (and per stored factor)
    ge = (n_layers - 1) / n_layers if n_layers > 1 else 1.0  # launches that read g_e'
    w = {
        # x -> P = W1a x + b1, Q = W1b x
        "proj": Work(N * 3 * H * f, N * 2 * 2 * H * H),
        # e, P_i, Q_j -> e', a ; per edge 2 H x H products
        "edge_fwd": Work(E * (2 * H * fe + 9) + N * 3 * H * f, E * 2 * 2 * H * H),
        # every member row read and written once, plus the plan
        "halo": Work(M * 2 * H * f + 4 * (M + G + 1), 0.0),
        "halo_adj": Work(M * 2 * H * f + 4 * (M + G + 1), 0.0),
        # [a*, x] -> x' ; products 2H x H and H x H
        "node_fwd": Work(N * 3 * H * f, N * 2 * 3 * H * H),
        # a*, x, g_x' -> g_a*, g_x ; recompute (3H^2) + input grads (3H^2) + weight grads (3H^2)
        "node_bwd": Work(N * 5 * H * f, N * 2 * 9 * H * H),
        # e, [g_e'], P_i, Q_j, g_a_i -> g_e, g_h, g_P ; 6 H x H products per edge
        "edge_bwd": Work(E * ((2 + ge) * H * fe + H * fh + 9) + N * 4 * H * f, E * 2 * 6 * H * H),
        # g_P, g_h (through reverse edges), x, g_x -> g_x ; 2 (2H x H) products per node
        "gq": Work(E * (H * fh + 4) + N * (4 * H * f + 4), N * 2 * 4 * H * H),
    }
    if H > 64:
        # pass 1: recompute (W1c, W2) and the input-gradient products (W2^T, W1c^T)
        w["edge_bwd"] = Work(w["edge_bwd"].bytes, E * 2 * 4 * H * H)
        # pass 2: dW1c = sum g_h e^T, dW2 = sum gm u^T (+ LayerNorm sums)
        w["edge_dw"] = Work(E * (H * fh + H * fe + 2 * H * fh + 2 * H * fh), E * 2 * 2 * H * H)
    if node_bwd_split(H):
        w["node_bwd"] = Work(w["node_bwd"].bytes, N * 2 * 6 * H * H)
        # dW1 = sum g_y u^T, dW0 = sum g_z [a*, x]^T (+ LayerNorm sums)
        w["node_dw"] = Work(N * (2 * H * fh + H * fh + 2 * H * f + H * fh + H * f), N * 2 * 3 * H * H)
    if gq_split(H, gemm):
        w["gq"] = Work(w["gq"].bytes, N * 2 * 2 * H * H)
        # dW1a = sum g_P x^T, dW1b = sum g_Q x^T
        w["gq_dw"] = Work(N * 3 * H * f, N * 2 * 2 * H * H)
    return w


def launched_kernels(N, E, G, M, H, gemm="bf16", n_layers=1, estate="f32"):
    """layer_kernels by the launches that run: in BF16 at H > 64 one kernel
    forms the edge adjoint and its weight gradients, so its products are
    edge_bwd's and no factor is stored or read."""
    w = layer_kernels(N, E, G, M, H, gemm, n_layers, estate)
    if "edge_dw" in w and not edge_bwd_split(H, gemm):
        w["edge_bwd"] = Work(w["edge_bwd"].bytes, w["edge_bwd"].flops + w.pop("edge_dw").flops)
    return w


# kernels that belong to the message-passing layers (the rest of a model
# step: encoders, decoder, loss, edge inputs)
LAYER_KERNEL_NAMES = ("pack", "tiles", "proj", "edge_fwd", "halo", "halo_adj", "node_fwd", "node_bwd",
                      "edge_bwd", "edge_dw", "node_dw", "gq", "gq_dw", "wreduce")


def layer_roof_seconds(N, E, G, M, H, gemm, n_layers, hbm=None, peak=None, estate="f32"):
    """Lower bound on the time of the message-passing layers' forward and
    adjoint: every kernel of every layer at the higher of its HBM floor
    (algorithmic bytes / bandwidth) and its product floor (flops / matrix
    peak of the operand type, FP32 from parts where the kernel runs so).
    hbm / peak default to the published MI355X figures."""
    hbm = PEAK_HBM if hbm is None else hbm
    w = launched_kernels(N, E, G, M, H, gemm, n_layers, estate)
    return n_layers * sum(max(k.bytes / hbm, k.flops / (peak or matrix_peak(n, H, gemm))) for n, k in w.items())


def bound_of(work, gemm, peak=None):
    """'hbm' or 'mfma': whichever roof takes longer for this work."""
    return "hbm" if work.bytes / PEAK_HBM >= work.flops / (peak or PEAK[gemm]) else "mfma"


def mlp_flops(K, H, NH, O):
    """Flops of one row through Linear(K->H), NH x Linear(H->H), Linear(H->O)."""
    return 2.0 * (K * H + NH * H * H + O * H)


def deep_split(H, NH):
    """Whether a deep layer runs on the kernels of its own width (8: FP32 FMAs,
    32: the matrix unit, from BF16 parts), whose adjoint has the first edge
    Linear's node parts split off and forms its weight gradients itself."""
    return H in (8, 32) and NH <= 5


def deep_peak(H, NH):
    """(bound, flop/s) of the deep kernels' products."""
    return ("mfma", PEAK_F32_PARTS) if H == 32 and deep_split(H, NH) else ("alu", PEAK_VALU)


def deep_kernels(N, E, G, M, H, NH, n_layers=1):
    """Per launch, one layer of the narrow deep-MLP kernels (keys match the
    library's profile names).  Bytes: the layer's inputs and outputs and what
    passes between its launches (each row once); the per-row adjoint records
    of H = 16 and deeper MLPs are an implementation choice and not counted.
    Flops: the MLP products (recomputed forward, transposed products, and one
    product per weight per row for the weight gradients, where they run)."""
    f = 4.0
    ge = (n_layers - 1) / n_layers if n_layers > 1 else 1.0
    fe, fn = mlp_flops(3 * H, H, NH, H), mlp_flops(2 * H, H, NH, H)
    halo = Work(M * 2 * H * f + 4 * (M + G + 1), 0.0)
    w = {
        "deep_edge_fwd": Work(E * (2 * H * f + 5) + N * (3 * H * f + 4), E * fe),
        "halo": halo,
        "halo_adj": halo,
        "deep_node_fwd": Work(N * 3 * H * f, N * fn),
    }
    if deep_split(H, NH):
        w.update({
            # x -> P = W0a x + b0, Q = W0b x
            "proj": Work(N * 3 * H * f, N * 2 * 2 * H * H),
            "deep_node_bwd": Work(N * 5 * H * f, N * 3 * fn),
            # e, [g_e'], P_i, Q_j, g_a_i -> g_e, g_h (and at H = 32 g_P)
            "deep_edge_bwd": Work(E * ((3 + ge) * H * f + 9) + N * (4 if H == 32 else 3) * H * f,
                                  E * 3 * mlp_flops(H, H, NH, H)),
            # g_h through the reverse edges (g_P given, or summed here as well), x, g_x -> g_x
            "gq": Work(E * ((1 if H == 32 else 2) * H * f + 4) + N * ((4 if H == 32 else 3) * H * f + 4),
                       N * 2 * 4 * H * H),
        })
    else:
        w.update({
            "deep_node_bwd": Work(N * 5 * H * f, N * 2 * fn),
            "deep_edge_bwd": Work(E * ((2 + ge) * H * f + 5) + N * (3 * H * f + 4), E * 2 * fe),
            "deep_gather": Work(E * (H * f + 4) + N * (3 * H * f + 4), 0.0),
            "deep_edge_dw": Work(0.0, E * fe),
            "deep_node_dw": Work(0.0, N * fn),
        })
    return w
