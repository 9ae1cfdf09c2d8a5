"""Models that are not numbers, or become so, stay so: TCM from a theta0 with a
NaN, with a negative entry (a NaN logarithm) and with columns that lose all
their mass (beta = 0), by every DNA form and the protein one.  The oracle says
where NaN and -inf belong; models beside them are not touched."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _models(rng, A, l, kind):
    th0 = rng.dirichlet(np.full(A, 0.8), size=(4, l)).transpose(0, 2, 1).copy()
    for b in (0, 2):  # the others stay ordinary
        if kind == "nan":
            th0[b, 1, 1] = np.nan
        if kind == "negative":
            th0[b, 1, 0] = -0.1
        if kind == "no mass":
            th0[b, :, 0] = 0.0
    return th0


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("mix0", [0.1, 1.0])
@pytest.mark.parametrize("kind,beta", [("nan", 1.0), ("negative", 1.0), ("no mass", 0.0)])
@pytest.mark.parametrize("A,l,copies", [(4, 9, 1), (4, 9, 150), (4, 9, 700), (20, 6, 1)],
                         ids=["eight waves", "four waves", "tiles", "protein"])
def test_tcm(A, l, copies, kind, beta, mix0, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] not a number", A, copies, kind, mix0, prec, flush=True)
    rng = np.random.default_rng([A, l])
    seqs = random_sequences(rng, 4, [60, 120, l, 300], "dna" if A == 4 else "protein")
    bg = np.full(A, 1.0 / A)
    th0 = _models(rng, A, l, kind)
    iters, B = 2, 4 * copies
    with np.errstate(all="ignore"):
        r_th, r_mix, r_J, r_LL, _ = oracle.em_model(oracle.Seqs(A, seqs), l, pm.PM_TCM, mix0, th0, bg, iters, beta)
    assert np.isnan(r_th[::2]).any() and np.isfinite(r_th[1::2]).all()
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    th = torch.zeros((B, A, l), dtype=torch.float64, device="cuda")
    mix = torch.zeros(B, dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL, sites = torch.zeros_like(J), torch.zeros((B, len(seqs)), dtype=torch.int32, device="cuda")
    pm.em_refine_model(pm.Seqs(A, seqs), l, pm.PM_TCM, mix0, d(np.tile(th0, (copies, 1, 1))), d(bg), B, None, iters,
                       beta, prec, th, mix, J, LL, sites)
    torch.cuda.synchronize()
    rtol = 1e-12 if prec == pm.PM_FP64 else 1e-5  # the vector forms' tolerances
    for got, ref in ((th, r_th), (J, r_J), (LL, r_LL)):
        got = got.cpu().numpy()[-4:]
        scale = np.abs(ref[np.isfinite(ref)]).max()
        np.testing.assert_allclose(got[1::2], ref[1::2], rtol=2 * rtol, atol=2 * rtol * scale)
        assert (np.isnan(got[::2]) == np.isnan(ref[::2])).all()
        assert (np.isfinite(got[::2]) == np.isfinite(ref[::2])).all()
