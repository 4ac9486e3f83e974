"""GPU: a field's result in a batch is the same bytes whatever the other fields need: the kernel of a
chain is that of the most general model in it (extra potentials, the sextic term), and its cache
policy goes by the bytes of all fields (streamed outputs above 256 MB).  State and field of plain,
potential and sextic fields, alone and beside the others, in both precisions; the arithmetic is the
same, so nothing may differ."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

MODELS = {"plain": (1.0,), "massless": (0.0,), "potentials": (1.0, 0.7, 0.6, 0.5), "sextic": (1.0, 0.0, 0.0, 0.0, 0.3),
          "all": (0.8, 0.5, 0.4, 0.3, 0.2)}


@pytest.fixture(scope="module")
def skyr():
    from paper_2604_25876_amd import skyr as s
    return s


@pytest.mark.parametrize("prec", [0, 1])
def test_result_is_independent_of_the_other_models(skyr, prec):
    import torch

    import skyr_inputs
    flow = skyr.Flow(0.004, 0.0, 6, 4, 0)

    def setup(shape, seed):
        lat = skyr.Lattice((ctypes.c_int32 * 3)(*shape), 0, 0.2)
        phi = torch.tensor(skyr_inputs.random_unit_field(shape, seed=seed, spread=0.3),
                           dtype=skyr.field_dtype(prec), device="cuda")
        return lat, phi, torch.zeros_like(phi), torch.zeros_like(phi), skyr.new_workspace(lat, prec)

    def run(names, big=False):
        keep, slots = [], []
        with skyr.Batch(len(names) + 1) as b:
            for name in names:
                keep.append(setup((24, 26, 40), len(name)))
                slots.append(b.add(keep[-1][0], prec, skyr.Model(*MODELS[name]), flow, *keep[-1][1:]))
            if big:  # more than 256 MB with it
                lat = skyr.Lattice((ctypes.c_int32 * 3)(24, 530, 452), 0, 0.2)
                phi = torch.zeros((4, 24, 530, 452), dtype=skyr.field_dtype(prec), device="cuda")
                phi[0] = 1.0
                b.add(lat, prec, skyr.Model(1.0), flow, phi, torch.zeros_like(phi), torch.zeros_like(phi),
                      skyr.new_workspace(lat, prec))
            for _ in range(4):
                b.run(4)
            states = [bytes(b.poll(s)) for s in slots]
        return [(st, k[1], k[3]) for st, k in zip(states, keep)]

    alone = {name: run([name])[0] for name in MODELS}
    mixes = [list(MODELS), ["plain", "potentials"], ["plain", "massless", "sextic"], ["potentials", "sextic"]]
    for names, big in [(m, False) for m in mixes] + [([m], True) for m in MODELS]:
        for name, (st, phi, vel) in zip(names, run(names, big)):
            assert torch.equal(phi, alone[name][1]) and torch.equal(vel, alone[name][2]), (name, names, big)
            a, s = (skyr.AnfState.from_buffer_copy(x) for x in (alone[name][0], st))
            assert st == alone[name][0], (name, names, big, a.E_prev - s.E_prev, a.max_force - s.max_force)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(6, 24, 40), (37, 20, 21), (132, 20, 70)])
def test_padded_fields_are_independent_of_the_slabs(skyr, prec, shape):
    """Padded rows, alone (short slabs) and beside 24 large fields (long ones), and dense: one result."""
    import torch

    import skyr_inputs
    model, flow = skyr.Model(1.0), skyr.Flow(0.02, 0.0, 6, 4, 0)

    def setup(n, seed, padded):
        lat = skyr.Lattice((ctypes.c_int32 * 3)(*n), 0, 0.2)
        phi = torch.tensor(skyr_inputs.random_unit_field(n, seed=seed, spread=0.05),
                           dtype=skyr.field_dtype(prec), device="cuda")
        layout = skyr.batch_layout(lat, prec) if padded else None
        phi = skyr.to_padded(phi, layout) if padded else phi
        return lat, phi, torch.zeros_like(phi), torch.zeros_like(phi), skyr.new_workspace(lat, prec), layout

    def run(padded, others):
        f = setup(shape, 3, padded)
        with skyr.Batch(1 + len(others)) as b:
            for o in others:
                b.add(o[0], prec, model, flow, *o[1:5])
            slot = b.add_padded(f[0], prec, model, flow, *f[1:]) if padded else b.add(f[0], prec, model, flow, *f[1:5])
            for _ in range(4):
                b.run(4)
            st = bytes(b.poll(slot))
        return st, skyr.from_padded(f[1], f[5], shape[2]) if padded else f[1]

    dense, alone = run(False, []), run(True, [])
    mixed = run(True, [setup((132, 132, 68), k, False) for k in range(24)])
    assert dense[0] == alone[0] == mixed[0]
    assert torch.equal(dense[1], alone[1]) and torch.equal(alone[1], mixed[1])
