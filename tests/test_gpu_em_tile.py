"""EM of many DNA models in FP64 (sixteen models per workgroup, the M-step on
the FP64 matrix instructions) where it has edges: motif lengths around multiples
of three and four, sequences of one window and of several steps of a wave, more
sequences than sums are kept for, sequences whose terms all underflow against
the highest score, models with zero entries, and numbers of models on the
device on either side of the rule.  Each call refines a few models many times
over: against the oracle (1e-12 relative in FP64, 1e-5 for FP32 calls, as for the
other form), and equal models must have equal results bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WINDOWS = {"short": [1, 2, 63, 64, 65, 128, 5], "long": [1024, 97, 1500], "many": [3, 9, 1, 17, 30] * 27}
ROUND = 4096  # models of a full round (sixteen per CU)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield
    torch.cuda.synchronize()


def _theta0(rng, B, l, kind):
    th = rng.dirichlet(np.full(4, 0.6), size=(B, l)).transpose(0, 2, 1).copy()
    th = np.maximum(th, 1e-6)
    if kind == "zeros":  # one letter of one column never occurs
        for b in range(B):
            th[b, rng.integers(4), rng.integers(l)] = 0.0
    if kind == "sharp":  # most windows are hundreds of orders below the highest score
        th = np.full((B, 4, l), 1e-30)
        for b in range(B):
            th[b, rng.integers(0, 4, l), np.arange(l)] = 1.0
    return th / th.sum(axis=1, keepdims=True)


def _refine(S, seqs, l, th0, copies, bg, iters, beta, model, mix0, prec, n_dev=None):
    B = len(th0) * copies
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 4, l), dtype=torch.float64, device="cuda")
    mix = torch.zeros(B, dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    sites = torch.full((B, len(seqs)), -7, dtype=torch.int32, device="cuda")
    t0 = d(np.tile(th0, (copies, 1, 1)))
    nd = None if n_dev is None else torch.tensor([n_dev], dtype=torch.int64, device="cuda")
    if model == pm.PM_OOPS:
        pm.em_refine(S, l, t0, d(bg), B, nd, iters, beta, prec, th, J, LL, sites)
    else:
        pm.em_refine_model(S, l, model, mix0, t0, d(bg), B, nd, iters, beta, prec, th, mix, J, LL, sites)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (th, mix, J, LL, sites)]


def _check(windows, l, kind, model, mix0, prec, iters=3, beta=0.7, n=2900, n_dev=None):
    rng = np.random.default_rng([l, len(windows), model])
    seqs = random_sequences(rng, len(WINDOWS[windows]), [w + l - 1 for w in WINDOWS[windows]], "dna")
    bg = np.array([0.3, 0.2, 0.2, 0.3])
    th0 = _theta0(rng, 5, l, kind)
    r_th, r_mix, r_J, r_LL, r_sites = oracle.em_model(oracle.Seqs(4, seqs), l, model, mix0, th0, bg, iters, beta)
    got = _refine(pm.Seqs(4, seqs), seqs, l, th0, n // 5, bg, iters, beta, model, mix0, prec, n_dev)
    used = n if n_dev is None else n_dev
    for x in got:  # equal models, equal results; nothing written past the last
        for k in range(5):
            assert (x[k:used:5] == x[k]).all()
    th, mix, J, LL, sites = (x[:5] for x in got)
    rtol = 1e-12 if prec == pm.PM_FP64 else 1e-5
    scale = max(np.abs(r_J).max(), 1.0)
    np.testing.assert_allclose(J, r_J, rtol=rtol, atol=rtol * scale)
    np.testing.assert_allclose(LL, r_LL, rtol=rtol, atol=rtol * scale)
    np.testing.assert_allclose(th, r_th, rtol=2 * rtol, atol=2 * rtol)
    if model != pm.PM_OOPS:
        np.testing.assert_allclose(mix, r_mix, rtol=2 * rtol, atol=1e-15)
    if prec == pm.PM_FP64:
        assert np.array_equal(sites, r_sites)
    if n_dev is not None:
        assert (got[4][n_dev:] == -7).all() and (got[2][n_dev:] == 0).all()


MODELS = pytest.mark.parametrize("model,mix0", [(pm.PM_OOPS, 0.0), (pm.PM_ZOOPS, 0.5), (pm.PM_TCM, 0.05)],
                                 ids=["oops", "zoops", "tcm"])


@MODELS
@pytest.mark.parametrize("l", [1, 4, 9, 12, 13, 15, 16, 17, 18, 19, 20, 21, 22, 24])
def test_motif_lengths(l, model, mix0):
    _check("short", l, "plain", model, mix0, pm.PM_FP64)


@MODELS
@pytest.mark.parametrize("windows,prec", [("long", pm.PM_FP64), ("many", pm.PM_FP64), ("long", pm.PM_FP32)],
                         ids=["long", "many", "fp32"])
def test_sequences(windows, prec, model, mix0):
    _check(windows, 15, "plain", model, mix0, prec)


@MODELS
def test_zero_entries(model, mix0):
    _check("long", 8, "zeros", model, mix0, pm.PM_FP64)


@pytest.mark.parametrize("model,mix0", [(pm.PM_OOPS, 0.0), (pm.PM_ZOOPS, 0.5)], ids=["oops", "zoops"])
def test_terms_below_the_highest_score(model, mix0):
    _check("short", 24, "sharp", model, mix0, pm.PM_FP64, iters=1)


@pytest.mark.parametrize("n,n_dev", [(2900, 10), (2900, 2250), (2900, 2255), (4600, 4500), (4600, 4510), (4600, 4096),
                                     (4600, 4100)])
def test_models_on_the_device(n, n_dev):
    _check("short", 11, "plain", pm.PM_OOPS, 0.0, pm.PM_FP64, n=n, n_dev=n_dev)
