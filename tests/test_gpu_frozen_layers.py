"""GPU: the two outermost layers of a gradient are zero and those of a flow's second buffer are the
field's, whatever the arrays held, on lattices with one interior site along an axis, odd rows and
unequal edges; exactly."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 5, 5), (5, 9, 6), (16, 5, 33), (17, 18, 70), (70, 23, 5)])
@pytest.mark.parametrize("prec", [0, 1])
def test_frozen_layers(prec, shape):
    import torch

    import skyr_inputs
    from paper_2604_25876_amd import skyr
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*shape), 0, 0.2)
    phi = torch.tensor(skyr_inputs.random_unit_field(shape, seed=shape[2], spread=0.05),
                       dtype=skyr.field_dtype(prec), device="cuda")
    work, model = skyr.new_workspace(lat, prec), skyr.Model(1.0)
    frozen = torch.ones(shape, dtype=torch.bool, device="cuda")
    frozen[2:-2, 2:-2, 2:-2] = False
    for projected in (False, True):
        grad = torch.full_like(phi, float("nan"))
        skyr.energy_gradient(lat, prec, model, phi, work, grad, projected)
        torch.cuda.synchronize()
        assert bool((grad[:, frozen] == 0).all()) and bool(torch.isfinite(grad[:, ~frozen]).all())
    before, alt, st = phi.clone(), torch.full_like(phi, float("nan")), skyr.anf_state()
    skyr.anf_step(lat, prec, model, skyr.Flow(0.01, 0.0, 1, 0, 0), phi, alt, torch.zeros_like(phi), st, 1, work)
    assert torch.equal(alt[:, frozen], before[:, frozen]) and torch.equal(phi[:, frozen], before[:, frozen])
