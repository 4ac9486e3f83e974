"""GPU: a lattice never set or tuned runs on the launch of least estimated time, which may take
another tile shape and shorter slabs than the tile it reports.  Field values must not depend on
that: flow, gradient and printed-form flow equal the same calls on explicitly set tiles bit for bit,
and the sums to the rounding of their order (N terms of one sign: at most N eps, below 1e-10 here)."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skyr():
    from paper_2604_25876_amd import skyr as s
    return s


# one interior site; one row; fewer planes than a slab; cubes; ragged tiles; more rows than a round
SHAPES = [(5, 5, 5), (7, 40, 9), (9, 40, 40), (40, 40, 40), (23, 70, 37), (66, 18, 130), (30, 260, 100)]


@pytest.mark.parametrize("n", SHAPES)
@pytest.mark.parametrize("prec_name", ["f32", "f64"])
def test_default_launch_equals_set_tiles(skyr, prec_name, n):
    import torch
    prec = skyr.F32_BULK if prec_name == "f32" else skyr.F64
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
    g = torch.Generator(device="cuda").manual_seed(sum(n))
    phi0 = torch.randn((4,) + n, generator=g, device="cuda", dtype=torch.float64) * 0.3
    phi0[0] += 1.0
    phi0 = (phi0 / phi0.square().sum(0, keepdim=True).sqrt()).to(skyr.field_dtype(prec))
    model = skyr.Model(1.0, 0.5, 0.4, 0.3, 0.2)
    flow = skyr.Flow(0.002, 0.0, 4, 2, skyr.NEWTON_FLOW)
    work = skyr.new_workspace(lat, prec)

    def calls():
        phi, alt, vel, st = phi0.clone(), torch.zeros_like(phi0), torch.zeros_like(phi0), skyr.anf_state()
        skyr.anf_step(lat, prec, model, flow, phi, alt, vel, st, 4, work)
        grad = torch.zeros_like(phi0)
        parts = skyr.energy_gradient(lat, prec, model, phi0, work, grad=grad)
        obs = skyr.observables(lat, prec, model, phi0, work)
        return phi, vel, grad, [st.E, st.max_force, parts["E"], parts["E2"], parts["E4"], obs["E"], obs["E6"]]

    default = skyr.get_tile(lat, prec)
    want = calls()
    assert all(torch.isfinite(t).all() for t in want[:3])
    try:
        for v in range(len(skyr.tile_variants(prec))):
            for xc in (16, 19):
                if (v, xc) == default:
                    continue
                skyr.set_tile(lat, prec, v, xc)
                assert skyr.get_tile(lat, prec) == (v, xc)
                got = calls()
                for a, b in zip(got[:3], want[:3]):
                    assert torch.equal(a, b), (v, xc)
                assert got[3] == pytest.approx(want[3], rel=1e-10)
    finally:
        skyr.set_tile(lat, prec, default[0], max(16, default[1]))
    if default[1] >= 16:  # the default choice, set, is the default
        again = calls()
        assert again[3] == want[3] and torch.equal(again[0], want[0])
