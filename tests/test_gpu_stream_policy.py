"""GPU: the step kernels of every cache policy give the same field, bit for bit.

Which kernel runs depends on the bytes of phi, phi_alt and vel (plain accesses up to
256 MB, streamed ones above) and on whether rows are whole 128-byte lines, so one lattice
just above that line reaches the streaming kernels (dense and padded rows, a batch) and a
block of it, whose arrays are smaller, the plain ones."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skyr():
    from paper_2604_25876_amd import skyr as s
    return s


# (precision, extents): just above 256 MB in all, rows of whole lines and not
CASES = [("f32", (24, 530, 448)), ("f32", (24, 530, 451)), ("f64", (24, 360, 336)), ("f64", (24, 360, 333))]


@pytest.mark.parametrize("prec_name,n", CASES)
def test_policies_agree_bitwise(skyr, prec_name, n):
    import ctypes

    import torch
    prec = skyr.F32_BULK if prec_name == "f32" else skyr.F64
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.15)
    elem = 4 if prec_name == "f32" else 8
    assert 3 * 4 * n[0] * n[1] * n[2] * elem > 256 << 20
    model, flow = skyr.Model(1.0), skyr.Flow(0.015, 0.0, 3, 16, skyr.ARREST_POWER)
    g = torch.Generator(device="cuda").manual_seed(n[2])
    phi0 = torch.randn((4,) + n, generator=g, device="cuda", dtype=torch.float64) * 0.3
    phi0[0] += 1.0
    phi0 /= phi0.square().sum(0, keepdim=True).sqrt()
    phi0 = phi0.to(skyr.field_dtype(prec))
    work = skyr.new_workspace(lat, prec)

    def flow_of(dense: bool):
        layout = skyr.batch_layout(lat, prec)
        phi = phi0.clone() if dense else skyr.to_padded(phi0, layout)
        alt, vel, st = torch.zeros_like(phi), torch.zeros_like(phi), skyr.anf_state()
        if dense:
            skyr.anf_step(lat, prec, model, flow, phi, alt, vel, st, 3, work)
            return phi, vel
        skyr.anf_step_padded(lat, prec, model, flow, phi, alt, vel, st, 3, work, layout)
        return skyr.from_padded(phi, layout, n[2]), skyr.from_padded(vel, layout, n[2])

    phi, vel = flow_of(True)
    other = flow_of(False)
    assert torch.equal(phi, other[0]) and torch.equal(vel, other[1])
    layout = skyr.batch_layout(lat, prec)
    p = skyr.to_padded(phi0, layout)
    alt, v = torch.zeros_like(p), torch.zeros_like(p)
    with skyr.Batch(1) as b:
        slot = b.add_padded(lat, prec, model, flow, p, alt, v, work, layout)
        while b.poll(slot).steps < 3:
            b.run(3)
    assert torch.equal(skyr.from_padded(p, layout, n[2]), phi)
    # the first step of a block of the lattice, whose arrays stay below the line
    one, alt, vel, st = phi0.clone(), torch.zeros_like(phi0), torch.zeros_like(phi0), skyr.anf_state()
    skyr.anf_step(lat, prec, model, flow, one, alt, vel, st, 1, work)
    blk = skyr.Block.of(lat, (0, 0, 0), (n[0], 64, n[2]))
    at = [torch.arange(-4, e + 4, device="cuda").clamp(0, m - 1) for e, m in zip(blk.extent, n)]
    box = phi0[:, at[0][:, None, None], at[1][None, :, None], at[2][None, None, :]].contiguous()
    own = torch.zeros(box.shape[1:], dtype=torch.bool, device="cuda")
    own[4:-4, 4:-4, 4:-4] = True
    out, bv = torch.zeros_like(box), torch.zeros_like(box)
    skyr.block_sweep(blk, prec, model, skyr.BLOCK_STEP, box, box[:, ~own].contiguous(), out, vel=bv,
                     work=skyr.new_block_workspace(blk, prec), dt=0.015)
    inner = (slice(None), slice(2, -2), slice(2, 64), slice(2, -2))
    assert torch.equal(out[:, 4:-4, 4:-4, 4:-4][inner], one[inner])
    assert torch.equal(bv[:, 4:-4, 4:-4, 4:-4][inner], vel[inner])
