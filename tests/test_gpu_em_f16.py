"""The single-FP16 matrix-core EM of DNA models against the FP64 oracle: LLR, J,
theta and starts over two iterations, with sequences at the edges of its 32-window
pairs, few models (parts of a workgroup) and room for many (one part), l on both
sides of its fragments.  With W the log2-odds, a score is off by one FP16 rounding
of each W, FP32 sums and the hardware logarithm (2^-20 a position is ample), a
posterior by a factor 2^(2 delta) and its own FP16 rounding, theta by as much, and
the next scores by that in turn."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("room", [0, 60000], ids=["parts", "one part"])
@pytest.mark.parametrize("l,windows,B", [(3, [1, 32, 33, 200], 70), (8, [129, 500], 5), (13, [31, 64, 65, 300], 64),
                                         (18, [983, 400, 33, 128, 90], 17), (22, [160, 161, 1], 66), (30, [300, 97], 9)])
def test_two_iterations(l, windows, B, room):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] dna f16", l, windows, B, room, flush=True)
    rng = np.random.default_rng([l, B])
    t, beta, iters = len(windows), 1.0, 2
    seqs = random_sequences(rng, t, [n + l - 1 for n in windows], "dna")
    bg = np.array([0.3, 0.2, 0.2, 0.3])
    th0 = rng.dirichlet(bg * 40, size=(B, l)).transpose(0, 2, 1)
    th0 = np.maximum(th0, bg[:, None] / 8)
    th0 = np.ascontiguousarray(th0 / th0.sum(axis=1, keepdims=True))
    R = oracle.Seqs(4, seqs)
    th1 = oracle.em(R, l, th0, bg, 1, beta)[0]
    r_th, r_J, r_LL, _ = oracle.em(R, l, th0, bg, iters, beta)
    n = max(B, room)
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    full = np.zeros((n, 4, l))
    full[:B] = th0
    th = torch.zeros((n, 4, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((n, iters + 1), dtype=torch.float64, device="cuda")
    LL, sites = torch.zeros_like(J), torch.full((n, t), -5, dtype=torch.int32, device="cuda")
    nd = torch.tensor([B], dtype=torch.int64, device="cuda")
    pm.em_refine(pm.Seqs(4, seqs), l, d(full), d(bg), n, nd, iters, beta, pm.PM_F16, th, J, LL, sites)
    torch.cuda.synchronize()
    th, J, LL, sites = (x[:B].cpu().numpy() for x in (th, J, LL, sites))

    def score_error(theta, off):
        return l * (np.abs(np.log2(theta / bg[:, None])).max() * (2.0 ** -11 + l * 2.0 ** -24) + 2.0 ** -20
                    + np.log2(1 + off))

    off, ln2 = 0.0, np.log(2)
    for it, theta in ((0, th0), (1, th1), (2, r_th)):
        delta = score_error(theta, off)
        assert np.abs(LL[:, it] - r_LL[:, it]).max() <= t * delta * ln2
        assert np.abs(J[:, it] - r_J[:, it]).max() <= t * delta * ln2 + beta * l * (2.0 ** -20 + np.log1p(off))
        # posteriors: 2^(2 delta), their FP16 rounding, 2^-25 where subnormal
        # (theta is at least beta bg / (t + beta))
        off = 2.0 ** (2 * delta) * (1 + 2.0 ** -10) - 1 + sum(windows) * 2.0 ** -25 / bg.min()
        if it == 1:
            assert np.abs(th / r_th - 1).max() <= off
    lo = np.log2(r_th / bg[:, None])
    for i, q in enumerate(seqs):
        c = np.array([pm.DNA_CODE_ORDER.index(x) for x in q])
        win = np.lib.stride_tricks.sliding_window_view(c, l)
        s = lo[:, win, np.arange(l)].sum(axis=2)
        assert (s[np.arange(B), sites[:, i]] >= s.max(axis=1) - 2 * delta).all()
