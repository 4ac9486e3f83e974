"""GPU: the printed-form step takes another kernel instance where the steps of every slab, four more
than its planes, are whole groups of five.  One step from rest must be that of the gradient call
(whose instance never is): v = -dt g, phi' = (phi + dt v) / |phi + dt v|, to a few roundings of the
field's type (v: the two products and the unscaling of g, 4 eps; phi': 4 eps and those of v).  Slabs
of one plane (one or two tiles), a last slab shorter than the others, whole and ragged lattices."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(5, 5, 5), (6, 20, 36), (60, 20, 36), (125, 40, 70), (130, 132, 133), (70, 200, 100), (64, 64, 64)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("model", [(1.0,), (1.0, 0.6, 0.5, 0.4)])
@pytest.mark.parametrize("n", SHAPES)
def test_one_step_is_the_gradient(prec, model, n):
    import torch

    import skyr_inputs
    from paper_2604_25876_amd import skyr
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    phi = torch.tensor(skyr_inputs.random_unit_field(n, seed=n[0], spread=0.05), dtype=skyr.field_dtype(prec), device="cuda")
    work, m, dt = skyr.new_workspace(lat, prec), skyr.Model(*model), 0.01
    m.form = skyr.FORM_PRINTED
    grad = torch.full_like(phi, float("nan"))
    skyr.energy_gradient(lat, prec, m, phi, work, grad, True)
    want_v = -dt * grad.double()
    q = phi.double() + dt * want_v
    want = q / q.square().sum(0, keepdim=True).sqrt()
    out, vel, st = phi.clone(), torch.zeros_like(phi), skyr.anf_state()
    skyr.anf_step(lat, prec, m, skyr.Flow(dt, 0.0, 1, 0, skyr.NEWTON_FLOW), out, torch.zeros_like(phi), vel, st, 1, work)
    eps = torch.finfo(phi.dtype).eps
    inner = (slice(None),) + (slice(2, -2),) * 3
    assert st.steps == 1 and torch.isfinite(vel).all()
    assert ((vel.double() - want_v).abs() <= 4 * eps * want_v.abs())[inner].all()
    assert ((out.double() - want).abs() <= 4 * eps + 4 * eps * dt * want_v.abs())[inner].all()
