"""The work bench.py prices: the launches that run, at the rate their products can
reach."""

import pytest

from paper_2410_01657_amd import roofline as rl

N, E, G, M = 1771561, 10541520, 1000, 4000


@pytest.mark.parametrize("estate", ["f32", "bf16"])
def test_wide_bf16_edge_adjoint_is_one_launch(estate):
    """Six H x H products per edge, and the bytes of the edge arrays alone."""
    H = 128
    two = rl.layer_kernels(N, E, G, M, H, "bf16", 4, estate)
    one = rl.launched_kernels(N, E, G, M, H, "bf16", 4, estate)
    assert "edge_dw" not in one and set(two) - set(one) == {"edge_dw"}
    assert one["edge_bwd"].flops == E * 12 * H * H
    assert one["edge_bwd"].bytes == two["edge_bwd"].bytes
    assert rl.launched_kernels(N, E, G, M, H, "f32", 4) == rl.layer_kernels(N, E, G, M, H, "f32", 4)
    t = rl.layer_roof_seconds(N, E, G, M, H, "bf16", 4, estate=estate)
    assert t == pytest.approx(4 * sum(max(w.bytes / 8e12, w.flops / 2.5e15) for w in one.values()))


def test_fp32_products_from_parts_are_priced_at_a_sixth_of_bf16():
    assert rl.matrix_peak("edge_bwd", 64, "f32") == rl.matrix_peak("edge_dw", 128, "f32") == rl.PEAK["bf16"] / 6
    assert rl.matrix_peak("node_bwd", 64, "f32") == rl.matrix_peak("edge_bwd", 128, "f32") == rl.PEAK["f32"]
    assert {rl.matrix_peak(k, H, "bf16") for k in ("edge_bwd", "gq") for H in (64, 128)} == {rl.PEAK["bf16"]}
    # at H = 64 the FP32 edge kernels are then bound by memory
    w = rl.launched_kernels(N, E, G, M, 64, "f32", 4)
    assert all(rl.bound_of(w[k], "f32", rl.matrix_peak(k, 64, "f32")) == "hbm" for k in ("edge_fwd", "edge_bwd"))


@pytest.mark.parametrize("H,NH,own", [(8, 2, True), (32, 5, True), (32, 6, False), (16, 2, False)])
def test_deep_layers_have_the_launches_that_run(H, NH, own):
    w = rl.deep_kernels(N, E, G, M, H, NH, 4)
    records = {"deep_gather", "deep_edge_dw", "deep_node_dw"}
    assert set(w) == {"deep_edge_fwd", "halo", "halo_adj", "deep_node_fwd", "deep_node_bwd", "deep_edge_bwd"} | (
        {"proj", "gq"} if own else records)
    fe, fn = rl.mlp_flops(3 * H, H, NH, H), rl.mlp_flops(2 * H, H, NH, H)
    adj = sum(w[k].flops for k in w if k not in ("deep_edge_fwd", "deep_node_fwd"))
    if own:   # W0's node parts once per node instead of per edge: recomputed, back, and their gradients
        assert adj == 3 * (E * (fe - 4 * H * H) + N * fn) + N * 12 * H * H
    else:
        assert adj == 3 * (E * fe + N * fn)
    assert rl.deep_peak(H, NH) == (("mfma", rl.PEAK["bf16"] / 6) if (H, own) == (32, True) else ("alu", rl.PEAK_VALU))
