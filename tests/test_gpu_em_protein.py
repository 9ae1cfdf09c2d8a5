"""The protein matrix-core EM at the edges of its tiles: every number of column
blocks, sequences of one window, of whole and partial blocks of 32 and steps of
128 windows, the longest sequence and the most sequences it takes, a last
workgroup of few models.  Against the FP64 oracle, one iteration, models near
the background: with W the log2-odds, a score is off by at most
delta = l * 2^-11 * max |W| (one FP16 value each) and what FP32 sums of l terms
add, so J by t * delta * ln 2, a posterior by a factor 2^(2 delta) and its own
FP16 rounding, and theta by as much."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # l, windows per sequence, models
    (1, [1, 2, 31, 32, 33, 64, 127, 128, 129, 300], 5),
    (3, [1, 128, 129, 40], 70),
    (6, [33, 257, 5], 65),
    (10, [96, 97, 500, 1], 9),
    (13, [64, 160, 161], 64),
    (16, [200, 31, 1], 33),
    (19, [130, 128, 2], 17),
    (20, [981, 400, 33], 66),
    (24, [1, 64, 2048 - 23, 90], 7),
    (9, [20 + i for i in range(64)], 20),
]


@pytest.mark.parametrize("l,windows,B", CASES)
def test_protein_tiles(l, windows, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] protein em", l, windows[:5], B, flush=True)
    rng = np.random.default_rng([l, B])
    t = len(windows)
    seqs = random_sequences(rng, t, [n + l - 1 for n in windows], "protein")
    bg = rng.dirichlet(np.full(20, 20.0))
    th0 = rng.dirichlet(bg * 400, size=(B, l)).transpose(0, 2, 1)
    th0 = np.maximum(th0, bg[:, None] / 8)
    th0 = np.ascontiguousarray(th0 / th0.sum(axis=1, keepdims=True))
    r_th, r_J, r_LL, r_sites = oracle.em(oracle.Seqs(20, seqs), l, th0, bg, 1, 1.0)
    S = pm.Seqs(20, seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 20, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((B, 2), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    sites = torch.full((B, t), -5, dtype=torch.int32, device="cuda")
    pm.em_refine(S, l, d(th0), d(bg), B, None, 1, 1.0, pm.PM_F16, th, J, LL, sites)
    torch.cuda.synchronize()
    delta = l * np.abs(np.log2(th0 / bg[:, None])).max() * (2.0 ** -11 + l * 2.0 ** -24)
    assert np.abs(LL[:, 0].cpu().numpy() - r_LL[:, 0]).max() <= t * delta * np.log(2) + 1e-12
    factor = 2.0 ** (2 * delta) * (1 + 2.0 ** -10) - 1
    np.testing.assert_allclose(th.cpu().numpy(), r_th, rtol=factor, atol=1e-12)
    got = sites.cpu().numpy()
    assert ((got >= 0) & (got < np.array(windows))).all()
