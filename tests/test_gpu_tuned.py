"""Decoders built from the committed tuning cache run the kernels that the
library's own choice runs, at every call size."""
import pytest

from tests.helpers import HO_ROWS, ensure_built

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["bch63_45", "bch63_36", "bch127_64", "bch127_99"])
def test_tuned_decoder_runs_the_default_kernels(name, precision):
    B = ensure_built()
    from paper_2412_20828_amd import autotune
    assert autotune.key(name, HO_ROWS[name], precision, 9, autotune._gpu_name()) in autotune.load()
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1)
    dec = B.Decoder(c, p, n_branches=9, max_iter=8, precision=precision)
    tuned = autotune.tuned_decoder(c, p, name, HO_ROWS[name], precision=precision)
    for F in (1, 1000, 16_384, 100_000, 1_000_000, 4_000_000, 11_000_000):
        assert tuned.running_kernel(F) == dec.running_kernel(F)
    assert autotune.apply_cached(dec, name, HO_ROWS[name])


@pytest.mark.parametrize("name,frames", [("bch127_99", 50_000), ("bch63_45", 8_000_000), ("bch63_36", 10_000)])
def test_grid_is_tuned_where_it_applies(name, frames, tmp_path, monkeypatch):
    """In fixed point another kernel runs these sizes (matrix cores, packed,
    row-parallel): the cached grid, which smaller calls would take, stays the default."""
    B = ensure_built()
    from paper_2412_20828_amd import autotune
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "tuning.json"))
    monkeypatch.setattr(autotune, "_batch", lambda n, N, F, *a, **k: (
        torch.zeros((F, 64 if N <= 64 else 128), device="cuda"), torch.zeros(F, dtype=torch.uint8, device="cuda")))
    d = B.CODE_DEFS[name]
    c = B.Code(d.m, d.prim, d.t)
    p = B.Pcm.build(c, target_rows=HO_ROWS[name], seed=1)
    dec = B.Decoder(c, p, n_branches=9, max_iter=8, precision=B.FIX8)
    best, results = autotune.tune(dec, name, HO_ROWS[name], frames=frames, reps=1)
    assert best["waves_per_cu"] == 0 and len(results) == 1 and not best["packed16"]
