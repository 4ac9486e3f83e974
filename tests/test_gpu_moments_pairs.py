"""GPU: the moment passes take sites of a row in pairs and an eighth of the lattice per XCD: rows
of one, an odd and an even number of sites, fewer pairs than blocks, and every potential in the
energy.  Tolerances: FP64 sums of at most 60,000 terms of either sign against the oracle's, whose
rounding stays below N eps of the sum of magnitudes (1e-10 here); the energy against the
observables sweep (the density in the field's precision: 2e-6 in single).  A noise field may have
no charge or a negative second moment, where centre or radius are undefined: the call has to say
so exactly there, and every quantity that the oracle defines is compared."""
import ctypes
import math
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skyr():
    from paper_2604_25876_amd import skyr as s
    return s


@pytest.mark.parametrize("shape", [(5, 5, 5), (6, 7, 6), (8, 9, 40), (9, 8, 41), (31, 20, 67)])
@pytest.mark.parametrize("prec", [0, 1])
def test_moments_of_ragged_rows(skyr, prec, shape, monkeypatch):
    import torch

    import skyr_inputs
    from oracle.moments import moments as oracle_moments
    # the oracle's radius of a negative second moment: undefined instead of an exception
    monkeypatch.setattr("oracle.moments.math", types.SimpleNamespace(
        pi=math.pi, sqrt=lambda v: math.sqrt(v) if v >= 0 else math.nan))
    h = 0.3
    phi = skyr_inputs.random_unit_field(shape, seed=shape[2], spread=0.5)
    if prec == 1:
        phi = phi.astype(np.float32).astype(np.float64)
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*shape), 0, h)
    t = torch.tensor(phi, dtype=skyr.field_dtype(prec), device="cuda")
    work = skyr.new_workspace(lat, prec)
    torch.cuda.synchronize()

    def moments(model):
        out = skyr.MomentObs()
        rc = skyr.lib().skyr_moments(ctypes.byref(lat), prec, ctypes.byref(model), ctypes.c_void_p(t.data_ptr()),
                                     ctypes.byref(out), ctypes.c_void_p(work.data_ptr()), None)
        return rc, out.as_dict()

    rc, got = moments(skyr.Model(1.0))
    with np.errstate(all="ignore"):
        ref = oracle_moments(phi, h, 1.0)
    defined = all(np.isfinite(v).all() for v in ref.values())
    assert rc == (skyr.OK if defined else skyr.E_NONFINITE)
    tensors = [k for k in ("U", "V", "W") if np.isfinite(ref[k]).all()]
    size = max([np.abs(ref[k]).max() for k in tensors if k in "UV"] + [1.0])
    assert got["E"] == pytest.approx(ref["E"], rel=1e-10)
    assert got["B"] == pytest.approx(ref["B"], rel=1e-9, abs=1e-12)
    for k in tensors:
        assert np.abs(got[k] - ref[k]).max() <= 1e-9 * size, k
    model = skyr.Model(1.0, 0.7, 0.6, 0.5, 0.4)
    e = skyr.observables(lat, prec, model, t, work)["E"]
    assert moments(model)[1]["E"] == pytest.approx(2.0 * e, rel=1e-12 if prec == 0 else 2e-6)
