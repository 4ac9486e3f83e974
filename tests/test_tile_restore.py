"""CPU: what a tile getter reports can be set again, on lattices of fewer planes than the shortest
slab that is otherwise accepted too, and a saved autotuner choice can be read back; other short
slabs stay refused."""
import ctypes
import json

import pytest

from paper_2604_25876_amd import skyr

# (lattices that no other test sets a tile of)
SHAPES = [(5, 7, 6), (9, 41, 40), (19, 30, 31), (20, 30, 31), (21, 18, 71)]


@pytest.mark.parametrize("prec", [skyr.F64, skyr.F32_BULK])
@pytest.mark.parametrize("n", SHAPES)
def test_default_tile_can_be_set_again(prec, n):
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    for get, put in ((skyr.get_tile, skyr.set_tile), (skyr.get_batch_tile, skyr.set_batch_tile)):
        default = get(lat, prec)
        other = (default[0] + 1) % len(skyr.tile_variants(prec))
        put(lat, prec, other, 16)
        assert get(lat, prec) == (other, 16)
        put(lat, prec, *default)
        assert get(lat, prec) == default
        refused = [(other, 15), (default[0], 0)] + [(default[0], x) for x in (1, 15) if x != default[1]]
        for v, xc in refused:
            with pytest.raises(skyr.SkyrError):
                put(lat, prec, v, xc)
        assert get(lat, prec) == default


def test_saved_choice_of_a_small_lattice(tmp_path, monkeypatch):
    lat = skyr.Lattice((ctypes.c_int32 * 3)(9, 42, 40), 0, 0.2)
    v, xc = skyr.get_tile(lat, skyr.F64)
    assert xc < 16
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"9x42x40:f64": {"variant": v, "xchunk": xc, "us": 20.0}}))
    monkeypatch.setenv("SKYR_TUNE_CACHE", str(path))
    got = skyr.autotune_cached(lat, skyr.F64, skyr.Model(1.0), skyr.Flow(0.01, 0.0, 1, 0, 0), None, None, None, None)
    assert got == (v, xc, 20.0)
