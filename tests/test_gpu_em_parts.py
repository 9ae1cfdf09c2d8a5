"""Matrix-core EM: a model's result does not depend on how many models, or how
much room for them, a launch has.  The same models through launches of every
kind -- workgroups whose slots of sequences run side by side (few models) and
one after the other (more than 256 groups of 64 models, here by capacity), in a
list and in a batch -- must agree bit for bit."""
import numpy as np
import pytest

import paper_1605_06904_amd as pm
from synth import planted_instance, projection_masks, random_sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOM = 60000  # capacity of a launch in one part


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    yield
    torch.cuda.synchronize()


def _refine(S, l, th0, prec, iters, room):
    """th0's models at the front of a launch of `room`."""
    n, t = len(th0), S.t
    full = np.zeros((room,) + th0.shape[1:])
    full[:n] = th0
    bg = torch.full((4,), 0.25, dtype=torch.float64, device="cuda")
    nd = torch.tensor([n], dtype=torch.int64, device="cuda")
    th = torch.zeros((room, 4, l), dtype=torch.float64, device="cuda")
    J = torch.zeros((room, iters + 1), dtype=torch.float64, device="cuda")
    LL, sites = torch.zeros_like(J), torch.full((room, t), -7, dtype=torch.int32, device="cuda")
    pm.em_refine(S, l, torch.from_numpy(full).cuda(), bg, room, nd, iters, 0.7, prec, th, J, LL, sites)
    torch.cuda.synchronize()
    assert (sites[n:] == -7).all() and (th[n:] == 0).all()
    return [x[:n].cpu().numpy() for x in (th, J, LL, sites)]


# sequences: fewer than slots, as many, one more, many of other lengths; more
# than the launch keeps maxima of (60)
LENS = {"1": [150], "2": [90, 400], "3": [64, 65, 300], "4": [40, 200, 33, 500],
        "20": [37 + 53 * (i % 7) for i in range(20)], "61": [60 + 7 * (i % 5) for i in range(61)]}


@pytest.mark.parametrize("prec", [pm.PM_F16X2, pm.PM_F16], ids=["f16x2", "f16"])
@pytest.mark.parametrize("l,lens", [(14, "1"), (14, "2"), (18, "3"), (18, "4"), (18, "20"), (22, "20"), (27, "20"),
                                    (31, "4"), (15, "61"), (3, "20")])
def test_same_bits_with_any_room(l, lens, prec):
    rng = np.random.default_rng([l, len(lens)])
    seqs = random_sequences(rng, len(LENS[lens]), LENS[lens], "dna")
    # models far from the sequences and near one of their windows, so that
    # scores rise by many bits from one iteration to the next (repeated sweeps)
    th0 = rng.dirichlet(np.full(4, 0.4), size=(150, l)).transpose(0, 2, 1).copy()
    th0 = np.maximum(th0, 1e-4)
    th0 /= th0.sum(axis=1, keepdims=True)
    S = pm.Seqs(4, seqs)
    print("[case] parts", l, lens, prec, flush=True)
    few = _refine(S, l, th0, prec, 4, len(th0))
    many = _refine(S, l, th0, prec, 4, ROOM)
    assert np.isfinite(few[1]).all()
    for a, b in zip(few, many):
        assert np.array_equal(a, b)


def test_projection_run_alone_and_beside_many():
    """A problem of more models than a launch in parts takes beside two small ones:
    each alone and all in one batch."""
    rng = np.random.default_rng(77)
    problems = []
    for t, n, m in ((20, 600, 300), (17, 500, 12), (23, 700, 9)):
        inst = planted_instance(rng, t, n, 15, 4)
        problems.append(pm.Problem(inst.seqs, 4, 15, d=4, k=7, s=4, masks=projection_masks(rng, 15, 7, m),
                                   bg=np.full(4, 0.25)))
    kw = dict(em_iters=2, precision=pm.PM_F16X2)
    alone = [pm.projection_run([p], **kw)[0] for p in problems]
    assert alone[0]["n_enriched"] > 24576 and all(r["n_enriched"] < 4000 for r in alone[1:])
    batch = pm.projection_run(problems, batched=True, **kw)
    for a, b in zip(alone, batch):
        assert a["consensus"] == b["consensus"] and a["J"] == b["J"] and a["llr"] == b["llr"]
        assert np.array_equal(a["theta"], b["theta"]) and np.array_equal(a["sites"], b["sites"])
        assert (a["best_trial"], a["best_key"]) == (b["best_trial"], b["best_key"])
