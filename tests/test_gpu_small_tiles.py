"""GPU: on a lattice of fewer planes than the shortest slab that can be set, the default choice with
that length in its place is the default: the same launch, so the same bytes of every sum."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
# (lattices that no other test sets a tile of)
@pytest.mark.parametrize("n", [(5, 6, 7), (7, 41, 9), (9, 70, 71), (19, 41, 100)])
def test_restored_default_is_the_default(prec, n):
    import torch

    import skyr_inputs
    from paper_2604_25876_amd import skyr
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    phi0 = torch.tensor(skyr_inputs.random_unit_field(n, seed=n[1], spread=0.3), dtype=skyr.field_dtype(prec), device="cuda")
    work, model, flow = skyr.new_workspace(lat, prec), skyr.Model(1.0), skyr.Flow(0.004, 0.0, 5, 0, 0)

    def results():
        phi, st = phi0.clone(), skyr.anf_state()
        skyr.anf_step(lat, prec, model, flow, phi, torch.zeros_like(phi), torch.zeros_like(phi), st, 5, work)
        phi_b, work_b = phi0.clone(), skyr.new_workspace(lat, prec)
        with skyr.Batch(1) as b:
            slot = b.add(lat, prec, model, flow, phi_b, torch.zeros_like(phi), torch.zeros_like(phi), work_b)
            for _ in range(3):
                b.run(4)
            batch = bytes(b.poll(slot))
        return bytes(st), batch, skyr.observables(lat, prec, model, phi0, work)

    default, batch_default = skyr.get_tile(lat, prec), skyr.get_batch_tile(lat, prec)
    assert default[1] < 16 and batch_default[1] < 16
    want = results()
    try:
        for length in (16, None):
            skyr.set_tile(lat, prec, default[0], length or default[1])
            skyr.set_batch_tile(lat, prec, batch_default[0], length or batch_default[1])
            assert results() == want
    finally:
        skyr.set_tile(lat, prec, *default)
        skyr.set_batch_tile(lat, prec, *batch_default)
