"""Workloads of the library's public entry points, for timing them.

``listed()`` names the workloads, ``draw()`` gives more of the same ranges,
``prepare()`` makes the inputs, buffers and handles that a program has before
the call, ``run()`` is one pass, ``work()`` counts what a pass cannot do
without and ``exact()`` gives the results of the computed numbers in 64 bits,
by plain torch.

Every kind of case is one entry point or pipeline call:

  run     projection_run, host in and host out (packing, selection, EM, pick)
  pass    Pipeline.run: one instance, buffers kept between passes
  select  projection_hash_select: projection, counts and enriched buckets
  batch   projection_hash_select_batch: uneven instances of one shape class
  sort    bucket_sort_select: key spaces too large for a count table
  em      em_refine / em_refine_model: refinement of many buckets
  emb     em_refine_batch: refinement over a batch of instances
  gibbs   gibbs_refine: site sampling in place of EM

Sizes are those of the synthetic workloads ((15,4), (18,6), (21,7) DNA,
(20,6) protein, the uneven instances) or generic ones of the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1605_06904_amd as pm

BETA = 1.0
PRECISION = {"fp64": pm.PM_FP64, "fp32": pm.PM_FP32, "f16x2": pm.PM_F16X2, "f16": pm.PM_F16}
# The element type a program keeps a form's results in: the C ABI writes
# float64 whatever the form computes with.
RESULT = {"fp64": torch.float64, "fp32": torch.float32, "f16x2": torch.float32, "f16": torch.float16}
MODEL = {"oops": pm.PM_OOPS, "zoops": pm.PM_ZOOPS, "tcm": pm.PM_TCM}


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # a small problem through the one-call entry point with its default
        # options: latency, allocations and launches
        dict(name="run_13_3", kind="run", A=4, t=20, lo=300, hi=300, l=13, d=3, k=7, s=4, m=50, iters=5),
        # the plain (15,4) challenge instance, 200 trials, every bucket
        # refined in 64 bits
        dict(name="pass_15_4", kind="pass", A=4, t=20, lo=600, hi=600, l=15, d=4, k=7, s=4, m=200, iters=5),
        # projection, counting and selection of the large DNA workload: the
        # whole table of keys and counts is written
        dict(name="select_18_6", kind="select", A=4, t=20, lo=1000, hi=1000, l=18, d=6, k=8, s=4, m=5000),
        # the same step on proteins
        dict(name="select_protein", kind="select", A=20, t=30, lo=1000, hi=1000, l=20, d=6, k=4, s=3, m=2000),
        # the same step over uneven instances (other t and n in each), whose
        # buckets are crowded
        dict(name="batch_uneven", kind="batch", A=4, P=24, l=16, d=5, k=7, s=3, m=250),
        # a key space of 4^14: buckets from sorted keys
        dict(name="sort_k14", kind="sort", A=4, t=20, lo=1000, hi=1000, l=18, d=6, k=14, s=2, m=1000),
        # every enriched bucket of the large DNA workload refined on the
        # matrix cores (this is most of a pass there)
        dict(name="em_18_6", kind="em", form="f16x2", model="oops", A=4, t=20, lo=1000, hi=1000, l=18, d=6, k=8, s=4,
             B=89000, iters=10),
        # a batch of (15,4) instances refined together
        dict(name="em_batch_15_4", kind="emb", form="f16x2", A=4, P=24, t=20, lo=600, hi=600, l=15, d=4, k=7, s=4,
             m=200, iters=5),
        # the single-FP16 form on the long (21,7) sequences
        dict(name="em_f16_21_7", kind="em", form="f16", model="oops", A=4, t=50, lo=2000, hi=2000, l=21, d=7, k=9, s=3,
             B=16384, iters=5),
        # protein refinement in the precision form
        dict(name="em_protein", kind="em", form="f16", model="oops", A=20, t=30, lo=1000, hi=1000, l=20, d=6, k=4, s=3,
             B=16384, iters=5),
        # the ZOOPS model, single precision
        dict(name="em_zoops", kind="em", form="fp32", model="zoops", A=4, t=20, lo=1000, hi=1000, l=18, d=6, k=8, s=4,
             B=4096, iters=10),
        # Gibbs sampling of as many buckets
        dict(name="gibbs_18_6", kind="gibbs", A=4, t=20, lo=1000, hi=1000, l=18, d=6, k=8, s=4, B=4096, iters=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the most column updates of a refinement, by form: the listed cases' or fewer
_MOST = {("fp64", 4): 4e10, ("fp32", 4): 3e10, ("f16x2", 4): 4e11, ("f16", 4): 3e11, ("f16", 20): 1e11,
         ("fp64", 20): 2e10}


def _cut(case, form, key):
    """The case with fewer models (trials) where it would be one of the largest."""
    w = work(case)["flops"]
    most = _MOST[form, case["A"]] * (0.4 if case["kind"] == "gibbs" else 1.0)
    if w > most:
        case[key] = max(1, int(case[key] * most / w))
    return case


def draw(rng):
    kind = rng.choice(["run", "pass", "select", "select", "batch", "sort", "em", "em", "em", "em", "emb", "gibbs"])
    # t and n as in the uneven instances, every sequence its own length
    t = rng.randint(10, 40)
    lo = _log(rng, 300, 1400)
    hi = lo + rng.randint(0, 600)
    size = dict(t=t, lo=lo, hi=hi)
    x = t * (lo + hi) // 2
    if kind in ("run", "pass"):
        l = rng.randint(13, 18)
        return _cut(dict(kind=kind, A=4, **size, l=l, d=l // 2 - 3, k=7, s=4, m=_log(rng, 10, 100),
                         iters=rng.randint(3, 8)), "fp64", "m")
    if kind == "select" and rng.random() < 0.3:
        l = rng.randint(9, 24)
        return dict(kind=kind, A=20, **size, l=l, d=l // 3, k=rng.randint(2, 4), s=3, m=_log(rng, 20, 1200))
    if kind == "select":
        l, k = rng.randint(11, 24), rng.randint(6, 9)
        most = min(4000, int(1.2e9 / (4.0 * (4 ** k + x))))
        return dict(kind=kind, A=4, **size, l=l, d=l // 4 + 1, k=k, s=rng.randint(3, 5), m=_log(rng, 20, most))
    if kind == "batch":
        l = rng.randint(11, 21)
        d = l // 4 + 1
        return dict(kind=kind, A=4, P=rng.randint(4, 24), l=l, d=d, k=min(max(l - d - 4, 6), 8), s=3,
                    m=_log(rng, 10, 120))
    if kind == "sort" and rng.random() < 0.3:
        return dict(kind=kind, A=20, **size, l=rng.randint(12, 24), d=4, k=rng.randint(6, 7), s=2,
                    m=_log(rng, 20, 400))
    if kind == "sort":
        l = rng.randint(17, 26)
        return dict(kind=kind, A=4, **size, l=l, d=l // 4, k=rng.randint(13, 16), s=2, m=_log(rng, 20, 600))
    l = rng.randint(11, 22)
    if kind == "emb":
        form = rng.choice(["f16x2", "f16"])
        return _cut(dict(kind=kind, form=form, A=4, P=rng.randint(4, 16), t=rng.randint(10, 24), lo=300,
                         hi=rng.randint(400, 700), l=l, d=l // 4 + 1, k=7, s=4, m=_log(rng, 20, 100),
                         iters=rng.randint(3, 8)), form, "m")
    if kind == "gibbs":
        return _cut(dict(kind=kind, A=4, **size, l=l, d=l // 4 + 1, k=8, s=4, B=_log(rng, 60, 4000),
                         iters=rng.randint(3, 10)), "fp64", "B")
    form, A, model = rng.choice([("fp64", 4, "oops"), ("fp64", 4, "oops"), ("fp32", 4, "oops"), ("fp32", 4, "zoops"),
                                 ("fp64", 4, "tcm"), ("fp32", 4, "tcm"), ("f16x2", 4, "oops"), ("f16x2", 4, "oops"),
                                 ("f16", 4, "oops"), ("f16", 20, "oops"), ("fp64", 20, "oops")])
    if A == 20:
        return _cut(dict(kind="em", form=form, model=model, A=20, **size, l=l, d=l // 3, k=3, s=4,
                         B=_log(rng, 40, 8000), iters=rng.randint(2, 6)), form, "B")
    return _cut(dict(kind="em", form=form, model=model, A=4, **size, l=l, d=l // 4 + 1, k=8, s=4,
                     B=_log(rng, 40, 30000), iters=rng.randint(2, 10)), form, "B")


# ------------------------------------------------------------------ the inputs
class _Instance:
    """One planted (l, d) instance: symbol codes, strings, lengths, background."""

    def __init__(self, rng, A, lens, l, d):
        letters = pm.DNA_CODE_ORDER if A == 4 else pm.PROTEIN_CODE_ORDER
        p = np.full(4, 0.25) if A == 4 else rng.dirichlet(np.full(20, 2.0))
        self.lens = lens
        t = len(lens)
        motif = rng.integers(0, A, size=l)
        rows = []
        for n in self.lens:
            row = rng.choice(A, size=int(n), p=p).astype(np.uint8)
            copy = motif.copy()
            at = rng.choice(l, size=min(d, l), replace=False)
            copy[at] = (copy[at] + rng.integers(1, A, size=len(at))) % A
            a = int(rng.integers(0, n - l + 1))
            row[a:a + l] = copy
            rows.append(row)
        self.codes = np.concatenate(rows)
        table = np.frombuffer(letters.encode(), dtype=np.uint8)
        self.seqs = [bytes(table[r]).decode() for r in rows]
        self.A, self.t, self.l = A, t, l
        self.x = int(self.lens.sum()) - t * (l - 1)
        cnt = np.bincount(self.codes, minlength=A).astype(np.float64)
        self.bg = np.full(4, 0.25) if A == 4 else (cnt + 1) / (cnt.sum() + A)


def _masks(rng, l, k, m):
    """m random k-subsets of l positions, as bit masks."""
    keep = np.argsort(rng.random((m, l)), axis=1)[:, :k]
    return np.bitwise_or.reduce(np.uint32(1) << keep.astype(np.uint32), axis=1).astype(np.uint32)


def _rng(case, seed):
    return np.random.default_rng([int(seed) % (1 << 63), int(case["l"]), int(case["k"])])


def _sizes(case):
    """Sequence lengths of every instance: part of the case, not of the seed."""
    r = np.random.default_rng([case["l"], case["k"], case.get("t", 0), case.get("lo", 0), case.get("P", 1)])
    if case["kind"] == "batch":  # the uneven instances: t in 10..40, n in 300..2000
        return [np.full(int(r.integers(10, 41)), int(r.integers(300, 2001))) for _ in range(case["P"])]
    return [r.integers(case["lo"], case["hi"] + 1, size=case["t"]) for _ in range(case.get("P", 1))]


def _instance(case, rng, p=0):
    return _Instance(rng, case["A"], _sizes(case)[p], case["l"], case["d"])


def _room(case):
    """Capacities of the bucket and member lists: what random letters give and
    a margin (what can be at most, for a protein's uneven letters)."""
    A, l, k, s, m = case["A"], case["l"], case["k"], case["s"], case["m"]
    nb = nm = 0
    for lens in _sizes(case):
        x = int(lens.sum()) - len(lens) * (l - 1)
        most = m * min(A ** k, x // s), m * x
        if A == 4:
            b, q = _lists_expected(A, x, k, s, m)
            extra = m * len(lens) // 2 + 64
            most = min(most[0], int(1.1 * b) + extra), min(most[1], int(1.1 * q) + 4 * extra)
        nb, nm = nb + most[0], nm + most[1]
    return nb, nm


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _windows(inst):
    """Symbol codes of every window, [x, l]."""
    l = inst.l
    starts = np.cumsum(inst.lens) - inst.lens
    first = np.concatenate([s + np.arange(n - l + 1) for s, n in zip(starts, inst.lens)])
    dev = _device()
    codes = torch.from_numpy(inst.codes.astype(np.int64)).to(dev)
    return codes[torch.from_numpy(first).to(dev)[:, None] + torch.arange(l, device=dev)]


def _profiles(inst, masks, k, s, most=None):
    """Letter counts of the enriched buckets in (trial, key) order, at most
    `most` of them: (trial [B], size [B], profile [B, A, l])."""
    A, l = inst.A, inst.l
    win = _windows(inst)
    dev, nb = win.device, A ** k
    bits = (masks[:, None] >> np.arange(l)) & 1
    rank = np.cumsum(bits, axis=1) - 1
    weight = torch.from_numpy(np.where(bits == 1, float(A) ** (k - 1 - rank), 0.0)).to(dev)
    trials, sizes, profs, have = [], [], [], 0
    step = max(1, min((1 << 24) // nb, (1 << 23) // inst.x))
    for j0 in range(0, len(masks), step):
        w = weight[j0:j0 + step]
        key = (w @ win.double().T).round().long()                       # exact: below 2^53
        key += nb * torch.arange(len(w), device=dev)[:, None]
        key = key.reshape(-1)
        count = torch.bincount(key, minlength=nb * len(w))
        ids = torch.nonzero(count >= s).reshape(-1)
        if most is not None:
            ids = ids[:most - have]
        where = torch.full((nb * len(w),), -1, dtype=torch.long, device=dev)
        where[ids] = torch.arange(len(ids), device=dev)
        to = where[key]
        at = torch.nonzero(to >= 0).reshape(-1)
        cell = to[at][:, None] * (A * l) + win[at % inst.x] * l + torch.arange(l, device=dev)
        profs.append(torch.bincount(cell.reshape(-1), minlength=len(ids) * A * l).reshape(-1, A, l))
        trials.append(ids // nb + j0)
        sizes.append(count[ids])
        have += len(ids)
        if most is not None and have >= most:
            break
    return torch.cat(trials), torch.cat(sizes), torch.cat(profs)


def _theta0(inst, sizes, profs):
    bg = torch.from_numpy(inst.bg).to(profs.device)
    return ((profs.double() + BETA * bg[:, None]) / (sizes.double() + BETA)[:, None, None]).contiguous()


def _em_inputs(case, seed):
    """An instance and theta0 of its first B enriched buckets."""
    rng = _rng(case, seed)
    inst = _instance(case, rng)
    B, th, left = case["B"], [], case["B"]
    while left > 0:
        _, sizes, profs = _profiles(inst, _masks(rng, case["l"], case["k"], 1000), case["k"], case["s"], left)
        th.append(_theta0(inst, sizes, profs))
        left -= len(sizes)
    return inst, torch.cat(th)[:B].contiguous()


def _batch_inputs(case, seed):
    rng = _rng(case, seed)
    inst, masks = [], []
    for p in range(case["P"]):
        inst.append(_instance(case, rng, p))
        masks.append(_masks(rng, case["l"], case["k"], case["m"]))
    return inst, masks


def _batch_models(case, inst, masks):
    """Buckets {trial, key, size, first} of a batch (EM reads the trial) and
    theta0, in lists with room for more, and how many there are."""
    tr, th = [], []
    for p, (i, mk) in enumerate(zip(inst, masks)):
        t, sizes, profs = _profiles(i, mk, case["k"], case["s"])
        tr.append(t + p * case["m"])
        th.append(_theta0(i, sizes, profs))
    trial, n, room = torch.cat(tr), sum(map(len, tr)), _room(case)[0]
    buckets = torch.zeros(room, 4, dtype=torch.int32, device=trial.device)
    buckets[:n, 0] = trial.int()
    th0 = torch.zeros(room, 4, case["l"], dtype=torch.float64, device=trial.device)
    torch.cat(th, out=th0[:n])
    return buckets, th0, torch.tensor([n], device=trial.device)


# ----------------------------------------------------------- before the passes
def _empty(*shape, dtype=torch.float64):
    return torch.empty(*shape, dtype=dtype, device="cuda")


def _lists(case, size):
    """Bucket and member lists, their lengths and the selection's workspace."""
    nb, nm = _room(case)
    return (torch.zeros(nb, 4, dtype=torch.int32, device="cuda"), nb,
            torch.zeros(nm, dtype=torch.int32, device="cuda"), nm,
            torch.zeros(2, dtype=torch.int64, device="cuda"),
            torch.empty(max(size(nb), 256), dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    kind, A, l, k = case["kind"], case["A"], case["l"], case["k"]
    st = dict(case=case)
    if kind in ("run", "pass", "select", "sort"):
        rng = _rng(case, seed)
        inst = _instance(case, rng)
        masks = _masks(rng, l, k, case["m"])
        if kind == "run":
            st["problem"] = pm.Problem(inst.seqs, A, l, d=case["d"], k=k, s=case["s"], masks=masks, bg=inst.bg)
            return st
        S = st["S"] = pm.Seqs(A, inst.seqs)
        m, x = case["m"], S.nwin(l)
        st["masks"] = torch.from_numpy(masks.view(np.int32)).cuda()
        if kind == "pass":
            st["P"] = pm.Pipeline(S, l, k, case["s"], masks, case["iters"], BETA, pm.PM_FP64, inst.bg, *_room(case))
        elif kind == "select":
            st["keys"] = _empty(m, x, dtype=torch.int32)
            st["counts"] = _empty(m, A ** k, dtype=torch.int32)
            st["lists"] = _lists(case, lambda c: pm.pm_select_workspace(A, k, m, c))
        else:
            st["lists"] = _lists(case, lambda c: pm.pm_sort_select_workspace(S, l, k, m))
    elif kind == "batch":
        inst, masks = _batch_inputs(case, seed)
        Bt = st["Bt"] = pm.Batch(A, l, k, [i.seqs for i in inst], masks)
        st["keys"] = _empty(Bt.keys_total, dtype=torch.int32)
        st["counts"] = _empty(Bt.items, A ** k, dtype=torch.int32)
        st["lists"] = _lists(case, lambda c: pm.pm_select_workspace(A, k, Bt.items, c))
    elif kind == "emb":
        inst, masks = _batch_inputs(case, seed)
        Bt = st["Bt"] = pm.Batch(A, l, k, [i.seqs for i in inst], masks)
        st["buckets"], st["th0"], st["n"] = _batch_models(case, inst, masks)
        B = len(st["th0"])
        st["bg"] = torch.from_numpy(inst[0].bg).cuda()
        st["th"], st["J"], st["llr"] = (torch.zeros_like(st["th0"]), _empty(B, case["iters"] + 1).zero_(),
                                        _empty(B, case["iters"] + 1).zero_())
        st["ws"] = torch.empty(pm.pm_em_batch_workspace(Bt, PRECISION[case["form"]]), dtype=torch.uint8, device="cuda")
    else:
        inst, st["th0"] = _em_inputs(case, seed)
        S = st["S"] = pm.Seqs(A, inst.seqs)
        B = len(st["th0"])
        st["bg"] = torch.from_numpy(inst.bg).cuda()
        st["th"], st["J"], st["llr"] = (torch.empty_like(st["th0"]), _empty(B, case["iters"] + 1),
                                        _empty(B, case["iters"] + 1))
        if kind == "gibbs":
            st["sites"], st["seed"] = _empty(B, case["t"], dtype=torch.int32), int(seed) % 1000003
        else:
            st["mix"] = _empty(B)
            n = pm.pm_em_workspace(S, l, PRECISION[case["form"]])
            st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else False
    return st


# ------------------------------------------------------------------ the passes
def run(st):
    c = st["case"]
    kind, l = c["kind"], c["l"]
    if kind == "run":
        r = pm.projection_run(st["problem"], em_iters=c["iters"])[0]
        cons = np.frombuffer(r["consensus"].encode(), dtype=np.uint8)
        return dict(consensus=cons, sites=r["sites"], theta=r["theta"], J=np.array([r["J"]]), llr=np.array([r["llr"]]),
                    bucket=np.array([r["best_trial"], r["best_key"]]), n=r["n_enriched"])
    if kind == "pass":
        P = st["P"]
        P.run()
        b = P.b
        return dict(n_out=b.n_out, buckets=b.buckets, members=b.members, theta=b.theta, J=b.J, llr=b.llr,
                    sites=b.sites, consensus=b.consensus)
    if kind in ("select", "batch", "sort"):
        buckets, nb, members, nm, n_out, ws = st["lists"]
        if kind == "select":
            pm.projection_hash_select(st["S"], l, c["k"], st["masks"], c["m"], st["keys"], st["counts"], c["s"],
                                      buckets, nb, members, nm, n_out, ws, ws.numel())
        elif kind == "sort":
            pm.bucket_sort_select(st["S"], l, c["k"], st["masks"], c["m"], c["s"], buckets, nb, members, nm, n_out,
                                  ws, ws.numel())
        else:
            Bt = st["Bt"]
            pm.projection_hash_select_batch(Bt, Bt.masks, st["keys"], st["counts"], c["s"], buckets, nb, members, nm,
                                            n_out, ws, ws.numel())
        out = dict(n_out=n_out, buckets=buckets, members=members)
        if kind != "sort":
            out.update(keys=st["keys"], counts=st["counts"])
        return out
    B = len(st["th0"])
    if kind == "gibbs":
        pm.gibbs_refine(st["S"], l, st["th0"], st["bg"], B, None, c["iters"], BETA, st["seed"], st["th"], st["J"],
                        st["sites"])
        return dict(theta=st["th"], F=st["J"], sites=st["sites"])
    prec, dt = PRECISION[c["form"]], RESULT[c["form"]]
    if kind == "emb":
        pm.em_refine_batch(st["Bt"], st["buckets"], st["th0"], st["bg"], B, st["n"], c["iters"], BETA, prec, st["th"],
                           st["J"], st["llr"], None, st["ws"], st["ws"].numel())
    elif c["model"] == "oops":
        pm.em_refine(st["S"], l, st["th0"], st["bg"], B, None, c["iters"], BETA, prec, st["th"], st["J"], st["llr"],
                     ws=st["ws"])
    else:
        pm.em_refine_model(st["S"], l, MODEL[c["model"]], 0.5, st["th0"], st["bg"], B, None, c["iters"], BETA, prec,
                           st["th"], st["mix"], st["J"], st["llr"])
    out = dict(theta=st["th"].to(dt), J=st["J"].to(dt), llr=st["llr"].to(dt))
    if kind == "em" and c["model"] != "oops":
        out["mix"] = st["mix"].to(dt)
    return out


# ------------------------------------------------- what a pass cannot do without
def _lists_expected(A, x, k, s, m):
    """Expected enriched buckets and members of m trials of a random instance."""
    nb = float(A) ** k
    lam = x / nb
    below = [math.exp(-lam) * lam ** j / math.factorial(j) for j in range(s)]
    if lam < 1e-3:  # the tail by its first term
        tail = lam ** s / math.factorial(s)
        return m * nb * tail, m * nb * tail * s
    return m * nb * max(0.0, 1 - sum(below)), m * x * max(0.0, 1 - sum(below[:s - 1]))


def work(case):
    A, l, k, kind, m = case["A"], case["l"], case["k"], case["kind"], case.get("m", 0)
    got = {"bytes": 0.0, "flops": 0.0}
    for lens in _sizes(case):
        t, n = len(lens), float(lens.sum())
        x = n - t * (l - 1)
        moved = n * (0.25 if A == 4 else 5 / 8.0) + 4.0 * m  # packed letters and masks
        table = 4.0 * m * (x + float(A) ** k)
        nb, nm = _lists_expected(A, x, k, case["s"], m)
        if kind in ("select", "batch", "sort"):
            moved += (0.0 if kind == "sort" else table) + 16 * nb + 4 * nm
            flops = m * x * k
        else:
            it, B = case["iters"], case.get("B", nb)
            if kind == "gibbs":  # the letters of every start once per sweep, and before the first
                moved, flops = moved + B * (16.0 * A * l + 8 * (it + 1) + 4 * t), B * x * l * (it + 1)
            else:  # one update per column of every window in each E-step and each M-step
                flops = B * x * l * (2.0 * it + 1)
                if kind == "run":
                    moved = n + 8.0 * A * l + 4 * t
                else:
                    moved += B * (16.0 * A * l + 16 * (it + 1))
                if kind == "pass":
                    moved += table + B * (16 + 4 * t) + 4 * nm
        got["bytes"] += moved
        got["flops"] += flops
    return got


# -------------------------------------------------------------- in plain 64 bits
def _em(inst, theta0, iters, model="oops", mix0=0.5):
    """EM of every model in 64 bits: theta, J, llr, mixing parameter."""
    A, l, t = inst.A, inst.l, inst.t
    win = _windows(inst)
    dev, x = win.device, len(win)
    hot = torch.zeros(x, A * l, dtype=torch.float64, device=dev)
    hot.scatter_(1, win * l + torch.arange(l, device=dev), 1.0)
    bg = torch.from_numpy(inst.bg).to(dev)
    ends = np.cumsum(inst.lens - l + 1)
    parts = [(int(e - n), int(e)) for e, n in zip(ends, inst.lens - l + 1)]
    step = max(64, (1 << 27) // x)
    out = []
    for b in range(0, len(theta0), step):
        th = theta0[b:b + step].to(dev).double()
        mix = torch.full((len(th),), mix0, dtype=torch.float64, device=dev)
        J, llr = [], []
        for it in range(iters + 1):
            lth = th.log()
            S = hot @ (lth - bg.log()[:, None]).reshape(len(th), -1).T.contiguous()
            total = torch.zeros(len(th), dtype=torch.float64, device=dev)
            for lo, hi in parts:
                z = S[lo:hi]
                if model == "tcm":
                    li = torch.logaddexp(torch.log1p(-mix).expand_as(z), mix.log() + z)
                    total += li.sum(0)
                    S[lo:hi] = (mix.log() + z - li).exp()
                    continue
                lse = torch.logsumexp(z, 0)
                li = lse - math.log(hi - lo)
                if model == "zoops":
                    site = mix.log() + li
                    li = torch.logaddexp(torch.log1p(-mix), site)
                    S[lo:hi] = (z + mix.log() - math.log(hi - lo) - li).exp()
                else:
                    S[lo:hi] = (z - lse).exp()
                total += li
            llr.append(total)
            J.append(total + BETA * (bg[:, None] * lth).sum((1, 2)))
            if it == iters:
                break
            n = (hot.T.contiguous() @ S).T.reshape(-1, A, l)
            mass = n[:, :, 0].sum(1)
            th = (n + BETA * bg[:, None]) / (mass + BETA)[:, None, None]
            mix = (mass / (t if model == "zoops" else x)).clamp(max=1.0)
        out.append((th, torch.stack(J, 1), torch.stack(llr, 1), mix))
        del S
    return tuple(torch.cat(v) for v in zip(*out))


def _padded(v, rows):
    out = torch.zeros(rows, *v.shape[1:], dtype=v.dtype, device=v.device)
    out[:len(v)] = v
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "pass"):
        rng = _rng(case, seed)
        inst = _instance(case, rng)
        _, sizes, profs = _profiles(inst, _masks(rng, case["l"], case["k"], case["m"]), case["k"], case["s"])
        th, J, llr, _ = _em(inst, _theta0(inst, sizes, profs), case["iters"])
        if kind == "pass":
            th, J, llr = (_padded(v, _room(case)[0]) for v in (th, J, llr))
            return dict(n_out=None, buckets=None, members=None, theta=th, J=J, llr=llr, sites=None, consensus=None)
        b = int(J[:, -1].argmax())
        return dict(consensus=None, sites=None, theta=th[b], J=J[b, -1:], llr=llr[b, -1:], bucket=None, n=None)
    if kind == "em":
        inst, th0 = _em_inputs(case, seed)
        th, J, llr, mix = _em(inst, th0, case["iters"], case["model"])
        return dict(theta=th, J=J, llr=llr, **({} if case["model"] == "oops" else {"mix": mix}))
    if kind == "emb":
        inst, masks = _batch_inputs(case, seed)
        got = []
        for i, mk in zip(inst, masks):
            _, sizes, profs = _profiles(i, mk, case["k"], case["s"])
            got.append(_em(i, _theta0(i, sizes, profs), case["iters"])[:3])
        th, J, llr = (_padded(torch.cat(v), _room(case)[0]) for v in zip(*got))
        return dict(theta=th, J=J, llr=llr)
    return None  # lists are whole numbers; a Gibbs chain is a random draw
