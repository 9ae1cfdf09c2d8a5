"""Which matrix-core EM kernel a call launches: a shape set by em_set_tuning is
taken by calls of few models too, em_autotune runs every candidate's own kernel
on them, and without a set shape they run in parts.  By the kernel names that
the profiler reports (k_em_mfma<ceil(l/4), source, split, pairs, groups,
parts>); results are the same bit for bit and within the split form's bound of
the oracle (1e-5 of J's scale)."""
import re

import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = (11, 12, 14, 21, 22, 24)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield
    torch.cuda.synchronize()


def _launched(call):
    """(pairs, groups, parts) of every k_em_mfma launch of call()."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "k_em_mfma" in e.name]
    found = [re.search(r"k_em_mfma<\d+, \d+, \w+, (\d+), (\d+), (\w+)>", n)
             or re.search(r"k_em_mfmaILi\d+ELi\d+ELb\dELi(\d+)ELi(\d+)ELb(\d)E", n) for n in names]
    assert found and all(found), names
    return [(int(m[1]), int(m[2]), m[3] in ("true", "1")) for m in found]


@pytest.mark.parametrize("l", [22, 20])
def test_kernels_of_few_models(l):
    rng = np.random.default_rng(l)
    iters, B, prec = 3, 130, pm.PM_F16X2
    seqs = random_sequences(rng, 7, [l, l + 31, l + 32, 300, 90, 64, 501], "dna")
    bg = np.full(4, 0.25)
    th0 = np.maximum(rng.dirichlet(np.full(4, 0.5), size=(B, l)).transpose(0, 2, 1), 1e-3)
    th0 /= th0.sum(axis=1, keepdims=True)
    _, r_J, r_LL, _ = oracle.em(oracle.Seqs(4, seqs), l, th0, bg, iters, 1.0)
    S = pm.Seqs(4, seqs)
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    d_th0, d_bg = d(th0), d(bg)
    th = torch.zeros((B, 4, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((B, iters + 1), dtype=torch.float64, device="cuda")

    def refine():
        pm.em_refine(S, l, d_th0, d_bg, B, None, iters, 1.0, prec, th, J)

    tuned = pm.em_autotune(S, l, d_th0, d_bg, B, iters, 1.0, prec, th, J)  # (no shape is set after it)
    print("[case] shapes", l, tuned, flush=True)
    assert _launched(refine) == [(4, 1, True)]
    base = J.cpu().numpy(), th.cpu().numpy()
    np.testing.assert_allclose(base[0], r_J, rtol=1e-5, atol=1e-5 * np.abs(r_J).max())
    try:
        for shape in SHAPES:
            pm.em_set_tuning(l, prec, shape)
            th.zero_()
            assert _launched(refine) == [(shape % 10, shape // 10, False)]
            assert np.array_equal(J.cpu().numpy(), base[0]) and np.array_equal(th.cpu().numpy(), base[1]), shape
    finally:
        ran = _launched(lambda: pm.em_autotune(S, l, d_th0, d_bg, B, iters, 1.0, prec, th, J))
    assert set(ran) == {(s % 10, s // 10, False) for s in SHAPES}
