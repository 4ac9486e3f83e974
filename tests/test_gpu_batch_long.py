"""GPU: batched fields of more planes than a 32-bit product of unit and plane numbers can hold
(200,000 of them, on thin lattices) equal the single-field flow bit for bit, alone and beside a small
field, dense and in padded rows."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [(0, (200004, 5, 6)), (1, (200004, 6, 9)), (1, (185356, 5, 5))])
def test_long_thin_batch(prec, n):
    import torch

    from paper_2604_25876_amd import skyr
    model, flow = skyr.Model(1.0), skyr.Flow(0.01, 0.0, 3, 2, skyr.NEWTON_FLOW)

    def field(n):
        lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
        g = torch.Generator(device="cuda").manual_seed(n[2])
        phi = torch.randn((4,) + n, generator=g, device="cuda", dtype=torch.float64) * 0.1
        phi[0] += 1.0
        return lat, (phi / phi.square().sum(0, keepdim=True).sqrt()).to(skyr.field_dtype(prec))

    lat, phi0 = field(n)
    want, vel, st = phi0.clone(), torch.zeros_like(phi0), skyr.anf_state()
    skyr.anf_step(lat, prec, model, flow, want, torch.zeros_like(phi0), vel, st, 3, skyr.new_workspace(lat, prec))
    layout = skyr.batch_layout(lat, prec)
    for others, padded in ((0, False), (1, False), (0, True)):
        with skyr.Batch(2) as b:
            keep = []
            for _ in range(others):
                l2, p2 = field((20, 21, 22))
                keep.append((p2, torch.zeros_like(p2), torch.zeros_like(p2), skyr.new_workspace(l2, prec)))
                b.add(l2, prec, model, flow, *keep[-1])
            phi = skyr.to_padded(phi0, layout) if padded else phi0.clone()
            alt, v, work = torch.zeros_like(phi), torch.zeros_like(phi), skyr.new_workspace(lat, prec)
            slot = (b.add_padded(lat, prec, model, flow, phi, alt, v, work, layout) if padded
                    else b.add(lat, prec, model, flow, phi, alt, v, work))
            b.run(4)
            got = b.poll(slot)
        if padded:
            phi, v = skyr.from_padded(phi, layout, n[2]), skyr.from_padded(v, layout, n[2])
        assert got.steps == st.steps == 3
        assert torch.equal(phi, want) and torch.equal(v, vel), (others, padded)
        assert got.E_prev == pytest.approx(st.E_prev, rel=1e-12)
