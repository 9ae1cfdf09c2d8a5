"""The protein matrix-core EM against the FP64 oracle where its operands are
exact, and over two iterations.

With theta = bg times powers of two, every log2-odds is a whole number, every
score too, and every term 2^(score - reference) a power of two: all that is left
to round in the first E-step is the sum of the terms, which is FP64, so LLR and
J agree to 1e-12.  With ordinary models the bounds are those of one FP16 value
per operand."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _refine(seqs, l, th0, bg, iters):
    B, t = len(th0), len(seqs)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    th = torch.zeros((B, 20, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    sites = torch.full((B, t), -5, dtype=torch.int32, device="cuda")
    pm.em_refine(pm.Seqs(20, seqs), l, d(th0), d(bg), B, None, iters, 1.0, pm.PM_F16, th, J, LL, sites)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (th, J, LL, sites)]


@pytest.mark.parametrize("l,windows,B", [(24, [300, 31, 1000, 64, 1], 70), (20, [981, 400, 33], 5), (10, [129, 500], 65)])
def test_sums_of_terms_are_fp64(l, windows, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] protein sums", l, windows, B, flush=True)
    rng = np.random.default_rng([l, B])
    seqs = random_sequences(rng, len(windows), [n + l - 1 for n in windows], "protein")
    bg = np.full(20, 0.05)
    odds = np.array([16.0] + [0.5] * 4 + [0.25] + [0.125] * 14)  # they sum to 20
    th0 = np.stack([np.stack([rng.permutation(odds) for _ in range(l)], axis=1) for _ in range(B)]) * 0.05
    r_th, r_J, r_LL, r_sites = oracle.em(oracle.Seqs(20, seqs), l, th0, bg, 0, 1.0)
    th, J, LL, sites = _refine(seqs, l, th0, bg, 0)
    scale = np.abs(r_LL).max()
    np.testing.assert_allclose(LL, r_LL, rtol=0, atol=1e-12 * scale)
    np.testing.assert_allclose(J, r_J, rtol=0, atol=1e-12 * np.abs(r_J).max())


@pytest.mark.parametrize("l,windows,B", [(3, [1, 128, 129, 40], 70), (6, [33, 257, 5], 65), (13, [64, 160, 161], 64),
                                         (16, [200, 31, 1], 33), (20, [981, 400, 33], 66), (24, [1, 64, 2025, 90], 7)])
def test_two_iterations_at_block_edges(l, windows, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] protein two iterations", l, windows, B, flush=True)
    rng = np.random.default_rng([l, B, 2])
    t = len(windows)
    seqs = random_sequences(rng, t, [n + l - 1 for n in windows], "protein")
    bg = rng.dirichlet(np.full(20, 20.0))
    th0 = rng.dirichlet(bg * 400, size=(B, l)).transpose(0, 2, 1)
    th0 = np.maximum(th0, bg[:, None] / 8)
    th0 = np.ascontiguousarray(th0 / th0.sum(axis=1, keepdims=True))
    R = oracle.Seqs(20, seqs)
    th1 = oracle.em(R, l, th0, bg, 1, 1.0)[0]
    r_th, r_J, r_LL, r_sites = oracle.em(R, l, th0, bg, 2, 1.0)
    th, J, LL, sites = _refine(seqs, l, th0, bg, 2)

    # a score's error (log2 units): one FP16 rounding of each log-odds, FP32 sums,
    # and what theta itself is off by
    def score_error(theta, off):
        return l * (np.abs(np.log2(theta / bg[:, None])).max() * (2.0 ** -11 + l * 2.0 ** -24) + np.log2(1 + off))

    # posteriors off by 2^(2 delta) and their FP16 rounding (2^-25 where subnormal)
    def theta_error(delta):
        return 2.0 ** (2 * delta) * (1 + 2.0 ** -10) - 1

    # the smallest theta is at least beta bg / (t + beta): absolute errors as relative ones
    tiny = sum(windows) * 2.0 ** -25 / bg.min()
    off0, ln2 = 0.0, np.log(2)
    for it, theta in ((0, th0), (1, th1), (2, r_th)):
        delta = score_error(theta, off0)
        assert np.abs(LL[:, it] - r_LL[:, it]).max() <= t * delta * ln2 + 1e-12
        prior = np.abs(np.log1p(off0)) if off0 else 0.0  # sum of bg over l columns
        assert np.abs(J[:, it] - r_J[:, it]).max() <= t * delta * ln2 + l * prior + 1e-12
        off0 = theta_error(delta) + tiny
        if it == 1:
            assert (np.abs(th / r_th - 1)).max() <= off0
    # every reported start is the best but for the error of two scores
    lo = np.log2(r_th / bg[:, None])
    codes = [np.array([pm.PROTEIN_CODE_ORDER.index(c) for c in q]) for q in seqs]
    for i, c in enumerate(codes):
        win = np.lib.stride_tricks.sliding_window_view(c, l)
        s = lo[:, win, np.arange(l)].sum(axis=2)
        assert (s[np.arange(B), sites[:, i]] >= s.max(axis=1) - 2 * delta).all()


def test_zero_in_theta0():
    """Its log-odds is -inf, which the one-hot multiplies by 0: the sequence's
    log-likelihood is -inf, and other models' are not touched."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] protein f16, a zero in theta0", flush=True)
    rng = np.random.default_rng(8)
    l, B = 6, 3
    seqs = random_sequences(rng, 3, [80, 200, 41], "protein")
    th0 = rng.dirichlet(np.full(20, 2.0), size=(B, l)).transpose(0, 2, 1).copy()
    th0[1, :, 2] = 0.0
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    th = torch.zeros((B, 20, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((B, 1), dtype=torch.float64, device="cuda")
    LL = torch.zeros_like(J)
    pm.em_refine(pm.Seqs(20, seqs), l, d(th0), d(np.full(20, 0.05)), B, None, 0, 1.0, pm.PM_F16, th, J, LL)
    LL = LL.cpu().numpy()[:, 0]
    assert LL[1] == -np.inf and np.isfinite(LL[[0, 2]]).all()
