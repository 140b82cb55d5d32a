"""The schedule search space and its cache key (no GPU)."""

import types

import pytest

import paper_2410_01657_amd.autotune as at


@pytest.mark.parametrize("H", [32, 64, 128])
@pytest.mark.parametrize("gemm", ["f32", "bf16"])
def test_the_default_schedule_is_a_candidate(H, gemm):
    """0 (the library's own choice) for every field but the waves, whose default
    is one of the values searched: 8 where there are two forms, else 4."""
    cs = at.candidates(H, gemm)
    zero = [c for c in cs if not any(c[f] for f in ("tile_edges", "edge_grid", "edge_bwd_grid", "edge_fwd_queue"))]
    assert (8 if (gemm == "bf16") == (H <= 64) else 4) in {c["edge_bwd_waves"] for c in zero}
    # no two candidates launch the same kernels
    assert (gemm == "bf16") == (H <= 64) or {c["edge_bwd_waves"] for c in cs} == {4}


def test_a_schedule_is_kept_for_the_library_it_was_timed_on(tmp_path, monkeypatch):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one")
    monkeypatch.setattr(at, "LIB_PATH", str(lib))
    monkeypatch.setattr(at.torch.cuda, "get_device_properties", lambda d: types.SimpleNamespace(gcnArchName="gfx950:x"))
    monkeypatch.setenv("MPLAYER_TUNE_CACHE", str(tmp_path / "tune.json"))
    calls = []
    monkeypatch.setattr(at, "tune_layer", lambda *a, **k: calls.append(a) or {"ms": float(len(calls))})
    dg = types.SimpleNamespace(device="cuda", n_rows=10, n_edges=20, host=types.SimpleNamespace(R=2))
    assert at.tuned_schedule(dg, 64, True, "f32") == at.tuned_schedule(dg, 64, True, "f32") == {"ms": 1.0}
    lib.write_bytes(b"other")
    assert at.tuned_schedule(dg, 64, True, "f32") == {"ms": 2.0}
    lib.write_bytes(b"one")
    assert at.tuned_schedule(dg, 64, True, "f32") == {"ms": 1.0} and len(calls) == 2
