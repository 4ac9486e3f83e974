"""GPU: a slab may be set longer than the lattice, up to the largest 32-bit length: one slab, the
fields of any other tile, from the single-field flow, the gradient, a batch and a block."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
def test_slab_longer_than_the_lattice(prec):
    import torch

    import skyr_inputs
    from paper_2604_25876_amd import skyr
    n = (43, 22, 39)  # (no other test sets a tile of it or of its region)
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    phi0 = torch.tensor(skyr_inputs.random_unit_field(n, seed=1, spread=0.1), dtype=skyr.field_dtype(prec), device="cuda")
    model, flow, work = skyr.Model(1.0), skyr.Flow(0.01, 0.0, 3, 2, skyr.NEWTON_FLOW), skyr.new_workspace(lat, prec)

    def results():
        phi, vel, grad = phi0.clone(), torch.zeros_like(phi0), torch.zeros_like(phi0)
        st = skyr.anf_state()
        skyr.anf_step(lat, prec, model, flow, phi, torch.zeros_like(phi0), vel, st, 3, work)
        skyr.energy_gradient(lat, prec, model, phi0, work, grad)
        other = phi0.clone()
        with skyr.Batch(1) as b:
            slot = b.add(lat, prec, model, flow, other, torch.zeros_like(phi0), torch.zeros_like(phi0),
                         skyr.new_workspace(lat, prec))
            b.run(4)
            assert b.poll(slot).steps == 3
        blk = skyr.Block.of(lat, (0, 0, 0), n)
        box = torch.nn.functional.pad(phi0, (4,) * 6)
        own = torch.zeros(box.shape[1:], dtype=torch.bool, device="cuda")
        own[4:-4, 4:-4, 4:-4] = True
        out, bv = torch.zeros_like(box), torch.zeros_like(box)
        skyr.block_sweep(blk, prec, model, skyr.BLOCK_STEP, box, box[:, ~own].contiguous(), out, vel=bv,
                         work=skyr.new_block_workspace(blk, prec), dt=0.01)
        return phi, vel, grad, other, out, bv

    want = results()
    solo, batch = skyr.get_tile(lat, prec), skyr.get_batch_tile(lat, prec)
    try:
        for length in (1000, 2 ** 31 - 1):
            skyr.set_tile(lat, prec, 1, length)
            skyr.set_batch_tile(lat, prec, 1, length)
            assert skyr.get_tile(lat, prec) == skyr.get_batch_tile(lat, prec) == (1, length)
            for a, b in zip(results(), want):
                assert torch.equal(a, b)
    finally:
        skyr.set_tile(lat, prec, *solo)
        skyr.set_batch_tile(lat, prec, *batch)
