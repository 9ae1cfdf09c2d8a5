"""The vector EM of DNA models (FP64 and FP32) where its three-letter tables
and register-held scores have edges: motif lengths around multiples of three
and at 31 and 32 (the last table's letters past the 32nd symbol), sequences of
one window, of 64 and 1024 windows give or take one (a lane's 16 windows, and
beyond them the twice-scored form), and models with zero entries.  Against the
oracle; tolerances are those derived for the forms: 1e-12 relative in FP64,
1e-5 in FP32."""
import sys

import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# sequence lengths as numbers of windows
WINDOWS = {"short": [1, 2, 63, 64, 65, 128, 5], "long": [1024, 1023, 1025, 1, 2100]}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield
    torch.cuda.synchronize()


def _theta0(rng, B, l, zeros):
    th = rng.dirichlet(np.full(4, 0.6), size=(B, l)).transpose(0, 2, 1).copy()
    th = np.maximum(th, 1e-6)
    if zeros:  # one letter of one column never occurs
        for b in range(B):
            th[b, rng.integers(4), rng.integers(l)] = 0.0
    return th / th.sum(axis=1, keepdims=True)


def _check(seqs, l, th0, bg, iters, beta, model, mix0, prec):
    B = len(th0)
    ref = oracle.Seqs(4, seqs)
    r_th, r_mix, r_J, r_LL, r_sites = oracle.em_model(ref, l, model, mix0, th0, bg, iters, beta)
    S = pm.Seqs(4, seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 4, l), dtype=torch.float64, device="cuda")
    mix = torch.zeros(B, dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    sites = torch.zeros((B, len(seqs)), dtype=torch.int32, device="cuda")
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


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("model,mix0", [(pm.PM_OOPS, 0.0), (pm.PM_ZOOPS, 0.5), (pm.PM_TCM, 0.05)],
                         ids=["oops", "zoops", "tcm"])
@pytest.mark.parametrize("l,windows", [(1, "short"), (2, "short"), (3, "short"), (16, "short"), (17, "short"),
                                       (24, "short"), (31, "short"), (32, "short"), (15, "long"), (32, "long")])
def test_table_and_register_edges(l, windows, model, mix0, prec):
    print("[case] vector em", l, windows, model, prec, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng([l, len(windows), model])
    seqs = random_sequences(rng, len(WINDOWS[windows]), [n + l - 1 for n in WINDOWS[windows]], "dna")
    _check(seqs, l, _theta0(rng, 5, l, False), np.full(4, 0.25), 3, 0.7, model, mix0, prec)


@pytest.mark.parametrize("model,mix0", [(pm.PM_OOPS, 0.0), (pm.PM_ZOOPS, 0.5), (pm.PM_TCM, 0.05)],
                         ids=["oops", "zoops", "tcm"])
@pytest.mark.parametrize("windows", [[300, 80, 64], [1100, 70]], ids=["short", "long"])
def test_models_with_zero_entries(windows, model, mix0):
    l = 7
    rng = np.random.default_rng(len(windows))
    seqs = random_sequences(rng, len(windows), [n + l - 1 for n in windows], "dna")
    _check(seqs, l, _theta0(rng, 6, l, True), np.array([0.3, 0.2, 0.2, 0.3]), 3, 0.0, model, mix0, pm.PM_FP64)
