"""The vector EM of protein models (FP64 and FP32): motif lengths around the four
positions read ahead, sequences around a lane's 16 held scores, inputs staged
by bytes, packed and not at all.  Against the oracle; tolerances are those of the
forms: 1e-12 relative in FP64, 1e-5 in FP32."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WINDOWS = {"short": [1, 2, 63, 64, 65, 5], "held": [1023, 1024, 1025, 1], "packed": [1000] * 45,
           "global": [2000] * 45}


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("model,mix0", [(pm.PM_OOPS, 0.0), (pm.PM_ZOOPS, 0.5), (pm.PM_TCM, 0.05)],
                         ids=["oops", "zoops", "tcm"])
@pytest.mark.parametrize("l,windows", [(1, "short"), (3, "short"), (4, "short"), (5, "short"), (32, "short"),
                                       (10, "held"), (15, "packed"), (12, "global")])
def test_lengths_and_staging(l, windows, model, mix0, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case]", l, windows, model, prec, flush=True)
    rng = np.random.default_rng([l, len(windows), model])
    seqs = random_sequences(rng, len(WINDOWS[windows]), [n + l - 1 for n in WINDOWS[windows]], "protein")
    B, iters, beta, bg = 3, 2, 0.7, np.full(20, 0.05)
    th0 = np.maximum(rng.dirichlet(np.full(20, 0.6), size=(B, l)).transpose(0, 2, 1), 1e-6)
    th0 /= th0.sum(axis=1, keepdims=True)
    r_th, r_mix, r_J, r_LL, r_sites = oracle.em_model(oracle.Seqs(20, seqs), l, model, mix0, th0, bg, iters, beta)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 20, l), dtype=torch.float64, device="cuda")
    mix = torch.zeros(B, dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    sites = torch.zeros((B, len(seqs)), dtype=torch.int32, device="cuda")
    S = pm.Seqs(20, seqs)
    if model == pm.PM_OOPS:
        pm.em_refine(S, l, d(th0), d(bg), B, None, iters, beta, prec, th, J, LL, sites)
    else:
        pm.em_refine_model(S, l, model, mix0, d(th0), d(bg), B, None, iters, beta, prec, th, mix, J, LL, sites)
    torch.cuda.synchronize()
    rtol = 1e-12 if prec == pm.PM_FP64 else 1e-5
    scale = max(np.abs(r_J).max(), 1.0)
    np.testing.assert_allclose(J.cpu().numpy(), r_J, rtol=rtol, atol=rtol * scale)
    np.testing.assert_allclose(LL.cpu().numpy(), r_LL, rtol=rtol, atol=rtol * scale)
    np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=2 * rtol, atol=2 * rtol)
    if model != pm.PM_OOPS:
        np.testing.assert_allclose(mix.cpu().numpy(), r_mix, rtol=2 * rtol, atol=1e-15)
    if prec == pm.PM_FP64:
        assert np.array_equal(sites.cpu().numpy(), r_sites)
