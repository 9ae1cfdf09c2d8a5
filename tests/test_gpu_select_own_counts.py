"""bucket_select with counts of the caller's own that exceed the keys': every
bucket has the room that its count says, its members in window order in the
first slots of it, and the rest untouched -- whichever way the trial is placed
(few members, a list with ranks, one large bucket, cursors)."""
import numpy as np
import pytest

import oracle
import paper_1605_06904_amd as pm
from synth import projection_masks, random_sequences
from test_gpu_select_forms import _select

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("lens,l,k,s,m", [([300] * 6, 12, 7, 2, 3), ([1300] * 20, 12, 6, 3, 3),
                                          ([1300] * 15 + [-900], 12, 6, 2, 2), ([2600] * 56, 12, 6, 3, 2)],
                         ids=["few members", "list", "large bucket", "cursors"])
def test_counts_above_the_keys(lens, l, k, s, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] own counts", lens[-1], len(lens), flush=True)
    rng = np.random.default_rng([len(lens), k])
    seqs = [random_sequences(rng, 1, [n], "dna")[0] if n > 0 else "A" * -n for n in lens]
    masks = projection_masks(rng, l, k, m)
    K, N = oracle.hash_trials(oracle.Seqs(4, seqs), l, k, masks)
    N = N + np.where(N >= s, rng.integers(0, 3, N.shape), 0).astype(N.dtype)
    trial, key = np.nonzero(N >= s)
    size = N[trial, key].astype(np.int64)
    first = np.cumsum(size) - size
    want = np.full(int(size.sum()), 0xffffffff, dtype=np.uint32)
    for j in range(m):
        w = np.argsort(K[j], kind="stable")
        at = np.searchsorted(K[j][w], np.arange(4 ** k + 1))
        for b in np.nonzero(trial == j)[0]:
            ws = w[at[key[b]]:at[key[b] + 1]]
            want[first[b]:first[b] + len(ws)] = ws
    bk, mem, tot, st = _select(pm.Seqs(4, seqs), 4, l, k, s, K, N)
    assert len(size) > 0 and st == 0 and tot == [len(size), len(want)]
    assert np.array_equal(bk, np.stack([trial, key, size, first], axis=1).astype(np.uint32))
    assert np.array_equal(mem, want)
