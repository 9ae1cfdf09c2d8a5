"""The matrix-core EM where its posteriors' references have edges: models whose
largest scores fall by far more than the margin from one iteration to the next
(the iteration is repeated from the lowest scores) beside ones whose scores
rise, more sequences than the kernel keeps maxima of, every ceil(l/4) class of
the sparse E-step's operands, and lists of few and of many models (workgroups
of several parts and of one).  Split FP16 against the FP64 oracle, with the
form's tolerances (1e-5 of the largest |J|, 2e-5 on theta); the single-FP16
form's first objective within t * l * 2^-11 * max |log2-odds|."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _theta0(rng, seqs, l, B):
    """Models peaked on one window of one sequence (their fit to that sequence
    falls in the first iteration), and flat ones (which rise)."""
    th = np.empty((B, 4, l))
    for b in range(B):
        if b % 3 == 2:
            th[b] = rng.dirichlet(np.full(4, 20.0), size=l).T
            continue
        s = seqs[int(rng.integers(len(seqs)))]
        a = int(rng.integers(len(s) - l + 1))
        th[b] = 0.01
        for p, ch in enumerate(s[a:a + l]):
            th[b, pm.DNA_CODE_ORDER.index(ch), p] = 0.97
    return th


@pytest.mark.parametrize("t,room", [(9, 70), (60, 70), (61, 70), (1, 70), (9, 60000)])
@pytest.mark.parametrize("l", [3, 7, 11, 14, 18, 22, 26, 30])
def test_references_and_sparse_operands(l, t, room):
    print("[case] em reference", l, t, room, flush=True)
    rng = np.random.default_rng([l, t])
    seqs = random_sequences(rng, t, [l + int(n) for n in rng.integers(0, 150, size=t)], "dna")
    B, iters, beta = 70, 4, 1.0
    th0, bg = _theta0(rng, seqs, l, B), np.full(4, 0.25)
    r_th, r_J, r_LL, _ = oracle.em(oracle.Seqs(4, seqs), l, th0, bg, iters, beta)
    S = pm.Seqs(4, seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    n_dev = torch.tensor([B], device="cuda")
    in0 = torch.zeros((room, 4, l), dtype=torch.float64, device="cuda")
    in0[:B] = d(th0)
    for prec in (pm.PM_F16X2, pm.PM_F16):
        th = torch.zeros((room, 4, l), dtype=torch.float64, device="cuda")
        J = torch.zeros((room, iters + 1), dtype=torch.float64, device="cuda")
        LL = torch.zeros_like(J)
        pm.em_refine(S, l, in0, d(bg), room, n_dev, iters, beta, prec, th, J, LL)
        torch.cuda.synchronize()
        assert not th[B:].any() and not J[B:].any()
        th, J, LL = th[:B], J[:B], LL[:B]
        if prec == pm.PM_F16X2:
            scale = np.abs(r_J).max()
            np.testing.assert_allclose(J.cpu().numpy(), r_J, rtol=1e-5, atol=1e-5 * scale)
            np.testing.assert_allclose(LL.cpu().numpy(), r_LL, rtol=1e-5, atol=1e-5 * scale)
            np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=2e-5, atol=2e-5)
        else:
            bound = t * l * 2.0 ** -11 * np.abs(np.log2(th0 / 0.25)).max()
            assert np.abs(J[:, 0].cpu().numpy() - r_J[:, 0]).max() <= bound
            assert np.isfinite(J.cpu().numpy()).all()


@pytest.mark.parametrize("l", [7, 18, 30])
def test_two_sequences(l):
    """Fewer sequences than parts of a workgroup; one iteration (with two
    sequences, later ones multiply any rounding of the first)."""
    print("[case] em two sequences", l, flush=True)
    rng = np.random.default_rng([l, 2])
    seqs = random_sequences(rng, 2, [l + 40, l + 131], "dna")
    B = 70
    th0, bg = _theta0(rng, seqs, l, B), np.full(4, 0.25)
    r_th, r_J, _, r_sites = oracle.em(oracle.Seqs(4, seqs), l, th0, bg, 1, 1.0)
    S = pm.Seqs(4, seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 4, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((B, 2), dtype=torch.float64, device="cuda")
    sites = torch.full((B, 2), -5, dtype=torch.int32, device="cuda")
    pm.em_refine(S, l, d(th0), d(bg), B, None, 1, 1.0, pm.PM_F16X2, th, J, None, sites)
    torch.cuda.synchronize()
    np.testing.assert_allclose(J.cpu().numpy(), r_J, rtol=1e-5, atol=1e-5 * np.abs(r_J).max())
    np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=2e-5, atol=2e-5)
    assert (sites.cpu().numpy() == r_sites).mean() > 0.9
