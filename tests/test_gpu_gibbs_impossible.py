"""Gibbs sampling from a theta0 with zeros under which a sequence holds no start
of positive probability: it begins at the first start, as the oracle does (a
start of -1 read outside the input).  DNA and protein, the first sequence and
later ones, fewer starts than lanes and more: equal sites, F and theta to 1e-12."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from test_zoops_impossible import _problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("A,l", [(4, 7), (4, 15), (4, 32), (20, 5), (20, 12)])
def test_starts_without_a_finite_score(A, l):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] gibbs without a finite score", A, l, flush=True)
    B, sweeps, seed = 4, 3, 17
    seqs, th0 = _problem(A, l, B, 5)
    seqs = seqs[-3:-1] + seqs  # impossible ones first too
    bg = np.full(A, 1.0 / A)
    r_th, r_F, r_sites = oracle.gibbs(oracle.Seqs(A, seqs), l, th0, bg, sweeps, 1.0, seed)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, A, l), dtype=torch.float64, device="cuda")
    F = torch.zeros((B, sweeps + 1), dtype=torch.float64, device="cuda")
    sites = torch.zeros((B, len(seqs)), dtype=torch.int32, device="cuda")
    pm.gibbs_refine(pm.Seqs(A, seqs), l, d(th0), d(bg), B, None, sweeps, 1.0, seed, th, F, sites)
    torch.cuda.synchronize()
    assert np.array_equal(sites.cpu().numpy(), r_sites)
    np.testing.assert_allclose(F.cpu().numpy(), r_F, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=1e-12, atol=1e-15)
