"""What the layer workspaces hold (no GPU)."""

import ctypes as C

import pytest

from test_abi_host import L, _fake_desc  # noqa: F401


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("backward", [0, 1])
def test_no_room_for_fragments_that_nothing_packs(L, H, backward):
    """The edge kernels stage their matrices themselves at H <= 64 and in BF16;
    packed are the node update's alone (6 H x H matrices with the transposes), so
    the forward workspaces of the two types differ by those and nothing else, and
    an H = 128 adjoint in FP32 adds W1a, W1b, W1c and W2 once."""
    from paper_2410_01657_amd._lib import call
    from paper_2410_01657_amd.ops import layer_cfg
    d = _fake_desc(L)

    def size(H, gemm, backward):
        cfg, nb = layer_cfg(H, gemm=gemm), C.c_size_t()
        cfg.tile_edges, cfg.edge_bwd_grid = 128, 1
        call("mp_layer_workspace_size", C.byref(cfg), C.byref(d), backward, C.byref(nb))
        return nb.value

    if not backward:
        assert size(H, "f32", 0) - size(H, "bf16", 0) == 6 * H * H * 2
        assert size(128, "f32", 0) - size(128, "bf16", 0) == 6 * 128 * 128 * 2 + 4 * 128 * 128 * 4
    else:   # the edge array g_h is FP32 in FP32
        up = lambda n: (n + 255) // 256 * 256
        g_h = up(d.n_edges * H * 4) - up(d.n_edges * H * 2)
        assert size(H, "f32", 1) - size(H, "bf16", 1) == 6 * H * H * 2 + g_h
