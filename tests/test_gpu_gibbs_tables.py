"""Gibbs sampling of DNA models where its three-letter tables and register-held
weights have edges: motif lengths around multiples of three and at 31 and 32,
sequences of 1024 starts give or take one (a lane's 16 starts), one sequence,
more sequences than lanes, the largest staged input with the most sequences, and
pseudocounts so small that l ratios leave the
FP64 range (tables of logarithms).  Against the oracle's chain: equal sites,
F and theta to 1e-12."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # l, starts per sequence, beta, sweeps
    (1, [1, 2, 64, 65, 200], 1.0, 4),
    (2, [63, 64, 65, 3], 0.5, 4),
    (17, [1024, 1023, 1025, 1, 90], 1.0, 4),
    (31, [40, 1500, 16, 17], 1.0, 4),
    (32, [1024, 1100, 1, 15], 1.0, 4),
    (12, [300], 1.0, 3),
    (9, [30 + (7 * i) % 50 for i in range(70)], 1.0, 3),
    (32, [200, 1030, 64, 33], 1e-12, 4),
    (12, [360] * 512, 1.0, 2),
]


@pytest.mark.parametrize("l,starts,beta,sweeps", CASES)
def test_table_and_register_edges(l, starts, beta, sweeps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] gibbs tables", l, starts[:6], beta, flush=True)
    rng = np.random.default_rng([l, len(starts)])
    seqs = random_sequences(rng, len(starts), [n + l - 1 for n in starts], "dna")
    B, seed = 6, 11
    th0 = rng.dirichlet(np.full(4, 0.7), size=(B, l)).transpose(0, 2, 1)
    th0 = np.ascontiguousarray(np.maximum(th0, 1e-6))
    bg = np.array([0.3, 0.2, 0.2, 0.3])
    r_th, r_F, r_sites = oracle.gibbs(oracle.Seqs(4, seqs), l, th0, bg, sweeps, beta, seed)
    S = pm.Seqs(4, seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 4, l), dtype=torch.float64, device="cuda")
    F = torch.zeros((B, sweeps + 1), dtype=torch.float64, device="cuda")
    sites = torch.zeros((B, len(seqs)), dtype=torch.int32, device="cuda")
    pm.gibbs_refine(S, l, d(th0), d(bg), B, None, sweeps, beta, seed, th, F, sites)
    torch.cuda.synchronize()
    assert np.array_equal(sites.cpu().numpy(), r_sites)
    np.testing.assert_allclose(F.cpu().numpy(), r_F, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=1e-12, atol=1e-15)
