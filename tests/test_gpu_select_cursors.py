"""Selection of trials with many members per bucket or with single large
buckets, in instances of more than 32 768 windows: both are placed by cursors.
Trials shared by several workgroups and trials in more than one range of
buckets, ranges whose keys fit the kernel's table and ranges that do not, more
trials than workgroups, buckets past the capacity.  Whole numbers: equal to the
oracle's.  And the time of such a selection, which must not go with members per
bucket."""
import zlib

import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import projection_masks, random_sequences
from test_gpu_select_forms import _select

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name, alphabet, letters in use, uniform lengths, lengths of mostly one letter,
# its share, l, k, s, m, members per bucket at least (0: not dense)
CASES = [
    ("dense, ranges shared", 4, 4, [2600] * 56, [], 0, 12, 6, 3, 2, 32),
    ("dense, more trials than workgroups", 20, 11, [1100] * 42, [], 0, 10, 3, 2, 260, 32),
    ("dense, one large bucket", 20, 12, [1500] * 40, [2000] * 3, 1.0, 10, 3, 2, 3, 32),
    ("large buckets among small ones, k = 7", 4, 4, [1500] * 22, [1500] * 10, 0.8, 13, 7, 2, 9, 0),
    ("large buckets, sparse keys, k = 9", 4, 4, [2000] * 20, [900] * 9, 0.85, 15, 9, 1, 2, 0),
    ("large buckets, protein", 20, 20, [1300] * 24, [1200] * 9, 0.7, 10, 4, 1, 5, 0),
]


def _case(case):
    name, A, used, lens, skewed, share, l, k, s, m, per = case
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    letters = (pm.DNA_CODE_ORDER if A == 4 else pm.PROTEIN_CODE_ORDER)[:used]
    seqs = ["".join(rng.choice(list(letters), n)) for n in lens]
    for n in skewed:
        q = rng.choice(list(letters), n)
        q[rng.random(n) < share] = "A"
        seqs.append("".join(q))
    return seqs, projection_masks(rng, l, k, m)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("cut", [False, True], ids=["whole", "cut"])
def test_matches_oracle(case, cut):
    name, A, used, lens, skewed, share, l, k, s, m, per = case
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    seqs, masks = _case(case)
    print("[case]", name, cut, flush=True)
    assert sum(len(q) - l + 1 for q in seqs) > 32768
    RK, RN = oracle.hash_trials(oracle.Seqs(A, seqs), l, k, masks)
    rbk, rmem, (rnb, rnm), _ = oracle.select(oracle.Seqs(A, seqs), l, k, RK, RN, s)
    buckets = np.bincount(rbk[:, 0], minlength=m)
    members = np.bincount(rbk[:, 0], weights=rbk[:, 2], minlength=m)
    assert buckets.min() > 1024
    assert (members > 32 * buckets).all() if per else (members < 32 * buckets).all() and rbk[:, 2].max() > 128
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


def test_time_does_not_go_with_members_per_bucket():
    """64 trials of 520 000 windows, 127 members in each of 4096 buckets: the
    selection's time as a multiple of the hash's (6 by cursors, 80 when each
    bucket was searched for by itself)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    l, k, s, m = 12, 6, 3, 64
    rng = np.random.default_rng(6)
    S = pm.Seqs(4, random_sequences(rng, 104, [5011] * 104, "dna"))
    x = S.nwin(l)
    masks = torch.from_numpy(projection_masks(rng, l, k, m).view(np.int32)).cuda()
    keys = torch.empty(m, x, dtype=torch.int32, device="cuda")
    counts = torch.empty(m, 4 ** k, dtype=torch.int32, device="cuda")
    nb, nm = m * 4 ** k, m * x
    buckets = torch.zeros(nb, 4, dtype=torch.int32, device="cuda")
    members = torch.zeros(nm, dtype=torch.int32, device="cuda")
    n_out = torch.zeros(2, dtype=torch.int64, device="cuda")
    ws = torch.empty(pm.pm_select_workspace(4, k, m, nb), dtype=torch.uint8, device="cuda")

    def ms(f):
        f()
        best = 1e9
        for _ in range(3):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            f()
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    print("[case] time at 127 members per bucket", flush=True)
    t_hash = ms(lambda: pm.projection_hash(S, l, k, masks, m, keys, counts))
    t_select = ms(lambda: pm.bucket_select(S, l, k, keys, counts, m, s, buckets, nb, members, nm, n_out, ws,
                                           ws.numel()))
    assert t_select < 20 * t_hash, (t_hash, t_select)
