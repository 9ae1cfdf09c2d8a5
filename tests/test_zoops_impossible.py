"""ZOOPS where a sequence holds no window of positive probability (theta with
zeros and beta = 0): the sequence holds no site, LLR_i = ln(1 - gamma), its
posteriors are 0 and its site is -1.  The oracle against products written out,
and the GPU forms (workgroup per model with four and eight waves, tiles of
sixteen models, protein) against the oracle, with such sequences short, within
a lane's registers and past them."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences


def _problem(A, l, B, seed):
    """Sequences of which some hold windows of the models and some cannot, and
    theta0 with two letters per column."""
    rng = np.random.default_rng([A, l, seed])
    order = pm.DNA_CODE_ORDER if A == 4 else pm.PROTEIN_CODE_ORDER
    last = order[A - 1]  # the letter that no model takes
    seqs = random_sequences(rng, 4, [l, B * l, B * l + 37, 300], "dna" if A == 4 else "protein")
    seqs += [last * n for n in (l, l + 70, l + 1100)]
    th = np.zeros((B, A, l))
    for b in range(B):
        for p in range(l):
            c = rng.choice(A - 1, 2, replace=False)
            th[b, c[0], p], th[b, c[1], p] = (w := rng.uniform(0.2, 0.8)), 1 - w
        for i in range(3):  # a window of the model in three sequences
            s = seqs[i + 1]
            w = "".join(order[rng.choice(A, p=th[b, :, p])] for p in range(l))
            a = len(s) - (b + 1) * l
            seqs[i + 1] = s[:a] + w + s[a + l:]
    return seqs, th


def test_oracle_equals_products():
    l, gamma = 5, 0.3
    seqs, th = _problem(4, l, 1, 0)
    bg = np.array([0.3, 0.2, 0.2, 0.3])
    S = oracle.Seqs(4, seqs)
    LL, s, Z, q = oracle.estep_model(S, l, pm.PM_ZOOPS, gamma, th[0], bg)
    codes = [np.array([pm.DNA_CODE_ORDER.index(c) for c in x]) for x in seqs]
    w0, want = 0, 0.0
    dead = 0
    for i, c in enumerate(codes):
        L = len(c) - l + 1
        r = np.array([np.prod([th[0, c[a + p], p] / bg[c[a + p]] for p in range(l)]) for a in range(L)])
        total = (1 - gamma) + gamma / L * r.sum()
        want += np.log(total)
        np.testing.assert_allclose(Z[w0:w0 + L], gamma / L * r / total, rtol=1e-12, atol=1e-300)
        np.testing.assert_allclose(q[i], gamma / L * r.sum() / total, rtol=1e-12, atol=1e-300)
        dead += not r.any()
        w0 += L
    assert dead >= 3
    np.testing.assert_allclose(LL, want, rtol=1e-12)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("A,l,copies", [(4, 8, 1), (4, 25, 1), (4, 9, 150), (4, 14, 700), (4, 23, 700), (20, 6, 1)],
                         ids=["eight waves", "long motif", "four waves", "tiles", "tiles l=23", "protein"])
def test_gpu_matches_oracle(A, l, copies, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nm, iters, mix0 = 4, 3, 0.5
    seqs, th0 = _problem(A, l, nm, 1)
    bg = np.full(A, 1.0 / A)
    r_th, r_mix, r_J, r_LL, r_sites = oracle.em_model(oracle.Seqs(A, seqs), l, pm.PM_ZOOPS, mix0, th0, bg, iters, 0.0)
    assert np.isfinite(r_th).all() and np.isfinite(r_J).all() and (r_sites[:, -3:] == -1).all()
    B = nm * copies
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    th = torch.zeros((B, A, l), dtype=torch.float64, device="cuda")
    mix = torch.zeros(B, dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL, sites = torch.zeros_like(J), torch.full((B, len(seqs)), -7, dtype=torch.int32, device="cuda")
    print("[case] zoops without a finite score", A, l, B, prec, flush=True)
    pm.em_refine_model(pm.Seqs(A, seqs), l, pm.PM_ZOOPS, mix0, d(np.tile(th0, (copies, 1, 1))), d(bg), B, None, iters,
                       0.0, prec, th, mix, J, LL, sites)
    torch.cuda.synchronize()
    # the vector forms' tolerances: 1e-12 relative in FP64, 1e-5 in FP32
    rtol = 1e-12 if prec == pm.PM_FP64 else 1e-5
    scale = max(np.abs(r_J).max(), 1.0)
    for got, ref in ((J, r_J), (LL, r_LL)):
        np.testing.assert_allclose(got.cpu().numpy()[-nm:], ref, rtol=rtol, atol=rtol * scale)
    np.testing.assert_allclose(th.cpu().numpy()[-nm:], r_th, rtol=2 * rtol, atol=2 * rtol)
    np.testing.assert_allclose(mix.cpu().numpy()[-nm:], r_mix, rtol=2 * rtol)
    if prec == pm.PM_FP64:
        assert np.array_equal(sites.cpu().numpy()[-nm:], r_sites)
