"""bucket_select on trials of many buckets whose members are listed in LDS and
ranked: buckets too large for the list (skewed letters), one bitmap word of
more members than the list, bitmaps that leave LDS for one workgroup per CU,
more trials than workgroups.  Whole numbers: equal to the oracle's."""
import zlib

import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import projection_masks, random_sequences
from test_gpu_select_forms import _select

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name, alphabet, uniform lengths, lengths of mostly one letter, its share, l, k, s, m
CASES = [
    ("large buckets among small ones", 4, [1200] * 10, [800] * 10, 0.7, 12, 6, 1, 3),
    ("a word beyond the list", 4, [1200] * 10, [2500] * 10, 0.93, 12, 6, 1, 2),
    ("a word beyond the list, k = 7", 4, [1500] * 12, [2500] * 12, 0.95, 14, 7, 2, 2),
    ("one letter only", 4, [2000] * 8, [2100] * 9, 1.0, 12, 6, 1, 2),
    ("bitmap of half the LDS, k = 9", 4, [2000] * 12, [300] * 2, 0.9, 15, 9, 1, 2),
    ("protein, skewed", 20, [1000] * 8, [1500] * 10, 0.8, 10, 4, 1, 2),
    ("more trials than workgroups", 4, [700] * 6, [200], 0.8, 12, 6, 1, 600),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("cut", [False, True], ids=["whole", "cut"])
def test_heavy_trials_match_oracle(case, cut):
    name, A, lens, skewed, share, l, k, s, m = case
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case]", name, cut, flush=True)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    alpha = "dna" if A == 4 else "protein"
    seqs = random_sequences(rng, len(lens), lens, alpha)
    for n in skewed:
        q = np.array(list(random_sequences(rng, 1, [n], alpha)[0]))
        q[rng.random(n) < share] = "A"
        seqs.append("".join(q))
    masks = projection_masks(rng, l, k, m)
    RK, RN = oracle.hash_trials(oracle.Seqs(A, seqs), l, k, masks)
    rbk, rmem, (rnb, rnm), _ = oracle.select(oracle.Seqs(A, seqs), l, k, RK, RN, s)
    assert np.bincount(rbk[:, 0], minlength=m).min() > 1024
    S = pm.Seqs(A, seqs)
    if not cut:
        bk, mem, tot, st = _select(S, A, l, k, s, RK, RN)
        assert st == 0 and tot == [rnb, rnm]
        assert np.array_equal(bk[:rnb], rbk) and np.array_equal(mem[:rnm], rmem)
        return
    cap_b, cap_m = rnb - rnb // 5, rnm - rnm // 3
    bk, mem, tot, st = _select(S, A, l, k, s, RK, RN, cap_b=cap_b, cap_m=cap_m)
    assert st & pm.PM_STATUS_CAPACITY and tot == [rnb, rnm]
    assert np.array_equal(bk[:cap_b], rbk[:cap_b])
    end = min(cap_m, int(rbk[cap_b - 1][3] + rbk[cap_b - 1][2]))
    assert np.array_equal(mem[:end], rmem[:end])
    assert (mem[end:cap_m] == 0xffffffff).all()  # members of buckets that were not kept
