"""GPU: a batch tile that was set is used as it was set, and a field on it gives the bytes of the
single-field flow on the same tile: the same blocks, partial sums and decisions.  Slab lengths that
do not divide the planes (100 + 24 of 124, 16 and a last slab of 4, one slab), every shape, flows
that arrest by energy and by power, alone and beside fields on default tiles."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skyr():
    from paper_2604_25876_amd import skyr as s
    return s


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("n,xchunk", [((128, 20, 40), 100), ((40, 37, 36), 16), ((57, 24, 70), 1000)])
@pytest.mark.parametrize("mode", [0, 1])
def test_set_batch_tile_equals_single_flow(skyr, prec, variant, n, xchunk, mode):
    import torch

    import skyr_inputs
    model, flow = skyr.Model(1.0), skyr.Flow(0.03, 0.0, 12, 5, mode)

    def setup(n, seed):
        lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
        phi = torch.tensor(skyr_inputs.random_unit_field(n, seed=seed, spread=0.05),
                           dtype=skyr.field_dtype(prec), device="cuda")
        return lat, phi, torch.zeros_like(phi), torch.zeros_like(phi), skyr.new_workspace(lat, prec)

    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    solo, saved = skyr.get_tile(lat, prec), skyr.get_batch_tile(lat, prec)
    if (variant, xchunk) in (solo, saved):
        pytest.skip("the default choice: its launch is the library's")
    try:
        skyr.set_tile(lat, prec, variant, xchunk)
        skyr.set_batch_tile(lat, prec, variant, xchunk)
        _, phi, alt, vel, work = setup(n, 7)
        st = skyr.anf_state()
        skyr.anf_step(lat, prec, model, flow, phi, alt, vel, st, 12, work)
        assert st.steps == 12 and st.arrests > 0
        for others in (0, 3):
            with skyr.Batch(4) as b:
                keep = [setup((30, 31, 32), k) for k in range(others)]
                for k in keep:
                    b.add(k[0], prec, model, flow, *k[1:])
                f = setup(n, 7)
                slot = b.add(f[0], prec, model, flow, *f[1:])
                for _ in range(7):
                    b.run(4)
                got = b.poll(slot)
            assert torch.equal(f[1], phi) and torch.equal(f[3], vel)
            assert bytes(got) == bytes(st), (got.E_prev - st.E_prev, got.arrests, st.arrests)
    finally:
        skyr.set_tile(lat, prec, *solo)
        skyr.set_batch_tile(lat, prec, *saved)
