"""Sorted selection behind its filter (s >= 2): windows around what a workgroup
keeps in registers (24576) and a slice of them takes, keys that all occur often
(more candidates than the sort buffer's 4096 pairs), few of them, and none.
Buckets and members are whole numbers: equal to the oracle's."""
import zlib

import numpy as np
import pytest
import torch

import paper_1605_06904_amd as pm
from synth import projection_masks, random_sequences
from test_gpu_sortsel import _oracle_sorted, _sorted

pytestmark = pytest.mark.gpu

# name, alphabet, lengths, l, k, m, s, period of the sequences (0: random)
CASES = [
    ("one window", 4, [16], 16, 13, 2, 2, 0),
    ("one wave of windows", 4, [40, 63], 20, 14, 3, 2, 0),
    ("last held window", 4, [3086] * 8, 15, 13, 2, 2, 0),
    ("first window not held", 4, [3086] * 8 + [15], 15, 13, 2, 2, 0),
    ("two slices", 4, [3100] * 8 + [77], 15, 13, 2, 3, 0),
    ("three slices", 4, [2000] * 27, 18, 14, 2, 2, 0),
    ("every key often", 4, [900] * 10, 18, 14, 3, 2, 301),
    ("candidates at the buffer's size", 4, [2065] * 4, 18, 14, 2, 2, 1024),
    ("every key often, two slices", 4, [2600] * 12, 16, 16, 2, 2, 1700),
    ("all one letter", 4, [3000] * 10, 18, 14, 2, 2, 1),
    ("protein", 20, [1300] * 20, 12, 6, 2, 2, 0),
    ("protein, every key often", 20, [800] * 8, 12, 7, 2, 3, 97),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_filtered_selection_matches_oracle(case):
    name, A, lens, l, k, m, s, period = case
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case]", name, flush=True)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    alpha = "dna" if A == 4 else "protein"
    if period:
        unit = random_sequences(rng, 1, [period], alpha)[0]
        seqs = [(unit * (n // period + 1))[:n] for n in lens]
    else:
        seqs = random_sequences(rng, len(lens), lens, alpha)
    masks = projection_masks(rng, l, k, m)
    rbk, rmem, rtot = _oracle_sorted(seqs, A, l, k, masks, s)
    bk, mem, tot, st = _sorted(pm.Seqs(A, seqs), l, k, masks, s)
    assert st == 0 and tot == rtot
    assert np.array_equal(bk, rbk) and np.array_equal(mem, rmem)
