"""The work that users of this package have it do, as cases to be timed and compared.

Every case starts from seeded random closed walks (``paper_1807_02119_amd.gen``): the case fixes the
walks, so that every seed meets networks of one shape, and the seed draws which strand passes over at
the crossings, and the couplings where the case takes its own.  Kinds of case:

``one``       Z of one knot per call (``kn.contract``, or ``kn.contract_noalloc``)
``batch``     Z of many knots in one launch (``kn.Batch.contract``)
``values``    a batch of several q, down to the Jones values V (``kn.jones_many``)
``sweep``     a captured launch of a batch replayed on couplings held on the GPU (``kn.Batch.graph``)
``gradient``  Z and d log Z / d J of a batch (``kn.Batch.contract_backward``)
``fit``       log Z of one knot as a term of a loss: forward and backward through autograd (``kn.log_z``)
``pipeline``  PD codes to Jones values: plans, device program, upload, contraction, V = A Z
"""

from __future__ import annotations

import cmath
import functools
import math
import random
from fractions import Fraction

import numpy as np
import torch

from paper_1807_02119_amd import gen, kn, tune

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # the smallest call: one knot of a table of small knots, launch latency and little else
        dict(name="one_tiny", kind="one", walk="lattice", walk_seed=0, knots=1, lo=12, hi=20, q=3,
             precision=0, couplings="jones"),
        # one ordinary knot per call at a real t, where a spin has five values
        dict(name="one_q5", kind="one", walk="lattice", walk_seed=1, knots=1, lo=150, hi=200, q=5,
             precision=0, couplings="jones"),
        # one of the most crossed lattice knots per call: a long chain of dependent steps
        dict(name="one_600", kind="one", walk="lattice", walk_seed=2, knots=1, lo=560, hi=600, q=3,
             precision=0, couplings="jones"),
        # the throughput workload: 256 knots of 200-600 crossings in one launch, both precisions
        dict(name="batch_c128", kind="batch", walk="lattice", walk_seed=0, knots=256, lo=200, hi=600,
             q=3, precision=0, couplings="jones", tuned="q3_200_600"),
        dict(name="batch_c64", kind="batch", walk="lattice", walk_seed=0, knots=256, lo=200, hi=600,
             q=3, precision=1, couplings="jones", tuned="q3_200_600"),
        # a table of knots at several q, small and ordinary ones together, down to the values of V
        dict(name="values_mixed_q", kind="values", walk="lattice", walk_seed=3, knots=512, lo=20,
             hi=250, q=0, precision=0, couplings="jones", tuned="batched"),
        # couplings swept on the GPU: a captured launch replayed on whatever J holds
        dict(name="sweep_graph", kind="sweep", walk="lattice", walk_seed=4, knots=64, lo=50, hi=200,
             q=3, precision=0, couplings="any"),
        # derivatives by every coupling, many knots in one launch
        dict(name="gradient_batch", kind="gradient", walk="lattice", walk_seed=5, knots=32, lo=150,
             hi=300, q=3, precision=0, couplings="any"),
        # a step of a fit: log Z of one knot through autograd, forward and backward
        dict(name="fit_one", kind="fit", walk="lattice", walk_seed=6, knots=1, lo=100, hi=150, q=3,
             precision=0, couplings="any"),
        # the paper's own random grid walks, wide enough for products on the matrix cores
        dict(name="wide_grid", kind="batch", walk="grid", walk_seed=60, knots=4, size=60, switches=8,
             q=3, precision=0, couplings="jones"),
        # such a knot too wide for one tensor: fixed spins, a loop over the slices on the device
        dict(name="sliced_543", kind="one", walk="grid", walk_seed=71, knots=1, size=72, switches=0,
             q=3, precision=0, couplings="any", slice_log2_budget=26),
        # the whole path from diagrams to values of V, planning on the host included
        dict(name="pipeline", kind="pipeline", walk="lattice", walk_seed=0, knots=256, lo=200, hi=600,
             q=3, precision=0, couplings="jones", tuned="q3_200_600"),
    ]


_MOST_FLOPS = 1.6e12  # the largest listed case's


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """A case of the listed kinds with sizes spread over their ranges."""
    while True:
        case = _draw(rng)
        try:
            if work(case)["flops"] <= _MOST_FLOPS:
                return case
        except kn.KnError:  # a walk too wide for one tensor
            pass


def _draw(rng):
    kind = rng.choice(["one", "one", "batch", "batch", "values", "sweep", "gradient", "fit", "wide",
                       "wide", "sliced", "pipeline"])
    seed = rng.randrange(1000, 1 << 20)
    lattice = dict(walk="lattice", walk_seed=seed, precision=0)
    if kind in ("wide", "sliced"):
        case = dict(walk="grid", walk_seed=seed, q=3, precision=0)
        if kind == "wide" and rng.random() < 0.5:
            return dict(case, kind="batch", knots=rng.randint(3, 6), size=rng.randint(36, 56),
                        switches=8, couplings="jones")
        case = dict(case, kind="one", knots=1, switches=0, couplings="any")
        if kind == "wide":
            return dict(case, size=rng.randint(36, 56))
        return dict(case, size=rng.randint(52, 64), slice_log2_budget=rng.randint(18, 22))
    if kind == "one":
        q = rng.choice([3, 3, 3, 5, 6, 7])
        mid = _log_uniform(rng, 14, {3: 560, 5: 180, 6: 140, 7: 120}[q])
        return dict(lattice, kind=kind, knots=1, lo=int(0.9 * mid), hi=int(1.1 * mid) + 2, q=q,
                    couplings=rng.choice(["jones", "any"]), library_workspace=rng.random() < 0.3)
    if kind == "fit":
        mid = _log_uniform(rng, 16, 270)
        return dict(lattice, kind=kind, knots=1, lo=int(0.9 * mid), hi=int(1.1 * mid) + 2, q=3,
                    couplings="any")
    if kind == "batch":
        single = rng.random() < 0.4
        lo = _log_uniform(rng, 20, 400)
        case = dict(lattice, kind=kind, knots=_log_uniform(rng, 64 if single else 3, 400), lo=lo,
                    hi=int(1.5 * lo), q=3, couplings="jones", precision=int(single))
        return dict(case, tuned="q3_200_600") if lo >= 150 else case
    if kind == "values":
        lo = _log_uniform(rng, 15, 100)
        return dict(lattice, kind=kind, knots=_log_uniform(rng, 20, 512), lo=lo, hi=2 * lo, q=0,
                    couplings="jones", tuned="batched")
    if kind == "pipeline":
        lo = _log_uniform(rng, 30, 400)
        return dict(lattice, kind=kind, knots=_log_uniform(rng, 16, 256), lo=lo, hi=int(1.5 * lo), q=3,
                    couplings="jones", tuned="q3_200_600")
    lo = _log_uniform(rng, 30, 200)
    return dict(lattice, kind=kind, knots=_log_uniform(rng, 4, 32 if kind == "gradient" else 100),
                lo=lo, hi=int(1.5 * lo), q=3, couplings="any")


# ------------------------------------------------------------------ inputs


@functools.lru_cache(maxsize=16)
def _shadows(walk, walk_seed, knots, lo, hi, size):
    """PD codes of the case's walks, with one choice of the strand on top."""
    if walk == "grid":
        return [gen.random_grid_diagram(np.random.default_rng(walk_seed + k), size).pd
                for k in range(knots)]
    out = []
    for k in range(knots):
        rng = np.random.default_rng(np.random.SeedSequence([11, walk_seed, k]))
        target = int(rng.integers(lo, hi + 1))
        tol = max(2, target // 8)
        out.append(gen.lattice_knot((10, walk_seed, k), max(lo, target - tol), min(hi, target + tol)).pd)
    return out


def _switch(pd, which):
    """The diagram with the crossings `which` switched: the over-strand, which comes in on arc d of a
    positive crossing and on b of a negative one, becomes the under-strand."""
    out = pd.copy()
    positive = (pd[:, 1] - pd[:, 3]) % (2 * len(pd)) == 1
    out[which & positive] = np.roll(pd, 1, axis=1)[which & positive]
    out[which & ~positive] = np.roll(pd, -1, axis=1)[which & ~positive]
    return out


def _diagrams(case, seed):
    """The case's PD codes (int32, (n, 4)) and q values for this seed."""
    rng = np.random.default_rng(np.random.SeedSequence([12, seed]))
    pds = []
    for pd in _shadows(case["walk"], case["walk_seed"], case["knots"], case.get("lo"), case.get("hi"),
                       case.get("size")):
        n = len(pd)
        which = rng.integers(0, 2, n).astype(bool)
        if "switches" in case:  # the walk's own strands on top, but for these many
            which = np.isin(np.arange(n), rng.permutation(n)[:case["switches"]])
        pds.append(np.ascontiguousarray(_switch(pd, which), dtype=np.int32))
    mix = np.random.default_rng(np.random.SeedSequence([13, case["walk_seed"]]))
    qs = [case["q"] or int(mix.choice((2, 3, 5, 6))) for _ in pds]
    return pds, qs


def _couplings(case, seed, taits, qs):
    """Couplings J (complex128, one per crossing, knot after knot): the Jones couplings moved by a
    tenth, as a fit or a sweep around them has."""
    rng = np.random.default_rng(np.random.SeedSequence([14, seed]))
    out = []
    for t, q in zip(taits, qs):
        _, eps = t.edges()
        n = len(eps)
        off = 0.1 * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
        out.append(np.log(_jones_weights(q, eps)) + off)
    return np.concatenate(out)


def _options(case):
    opts = dict(precision=case["precision"])
    if case["couplings"] != "jones":
        opts["jones_only"] = False
    if case["kind"] in ("gradient", "fit"):
        opts["gradient"] = True
    if "slice_log2_budget" in case:
        opts["slice_log2_budget"] = case["slice_log2_budget"]
    if case.get("tuned"):
        opts.update(tune.plan_options(tune.load(case["tuned"], case["precision"])))
        if case["tuned"] == "q3_200_600":
            opts["strategy"] = 2  # min-fill orders alone, as a program that plans many knots has it
    return opts


def prepare(case, seed):
    pds, qs = _diagrams(case, seed)
    kind, opts = case["kind"], _options(case)
    s = dict(kind=kind, precision=case["precision"], qs=qs)
    if kind == "pipeline":
        s.update(opts=opts, counts=np.array([len(p) for p in pds], np.int32),
                 flat=np.concatenate([p.reshape(-1) for p in pds]),
                 workspace=kn.alloc_workspace(1 << 20), z=kn.alloc_scalars(len(pds)))
        return s
    if kind in ("one", "fit"):
        tait = kn.Tait(pds[0])
        plan = kn.Plan(tait, qs[0], **opts)
        s.update(plan=plan, library=bool(case.get("library_workspace"))
                 and plan.workspace_bytes <= 64 << 20)
        taits = [tait]
        if kind == "one":
            s["z"] = kn.alloc_scalars(1)
            if not s["library"]:
                s["workspace"] = kn.alloc_workspace(plan.workspace_bytes)
    else:
        taits, plans = kn.plan_many(pds, qs, **opts)
        batch = kn.Batch(plans)
        if case.get("tuned"):
            grid = tune.load(case["tuned"], case["precision"]).get("grid")
            if grid:
                batch.set_grid(int(grid))
        batch.upload()
        s.update(batch=batch, taits=taits, z=kn.alloc_scalars(len(plans)))
    J = None
    if case["couplings"] != "jones":
        J = torch.from_numpy(_couplings(case, seed, taits, qs)).to("cuda")
    if kind == "gradient":
        s["grad"] = torch.empty((J.numel(), 2), dtype=torch.float64, device="cuda")
    if kind == "sweep":
        s["batch"].contract(J, z=s["z"])  # a batch is launched once before it is captured
        torch.cuda.synchronize()
        s["graph"] = s["batch"].graph(s["z"], J)
    s["J"] = J.requires_grad_(True) if kind == "fit" else J
    return s


# ------------------------------------------------------------------ one pass


def _scalars(z, precision):
    """Z as the library returns it: mantissas, and exponents of two.  A complex64 contraction's
    mantissas are kept in the precision they have."""
    m = z[:, :2]
    return {"mantissa": m.to(torch.float32) if precision else m, "exp2": z.view(torch.int64)[:, 2]}


def run(s):
    kind = s["kind"]
    if kind == "one":
        if s["library"]:
            kn.contract_noalloc(s["plan"], s["J"], z=s["z"])
        else:
            kn.contract(s["plan"], s["J"], workspace=s["workspace"], z=s["z"])
        return _scalars(s["z"], s["precision"])
    if kind == "batch":
        return _scalars(s["batch"].contract(s["J"], z=s["z"]), s["precision"])
    if kind == "sweep":
        s["graph"].replay()
        return _scalars(s["z"], s["precision"])
    if kind == "values":
        z = s["batch"].contract(z=s["z"])
        v, log2, _ = kn.jones_many(s["qs"], s["taits"], z.cpu().numpy())
        return {"v": v, "log2": log2}
    if kind == "gradient":
        z, grad = s["batch"].contract_backward(s["J"], z=s["z"], grad=s["grad"])
        return dict(_scalars(z, s["precision"]), grad=grad)
    if kind == "fit":
        s["J"].grad = None
        log_z = kn.log_z(s["J"], s["plan"])
        log_z.real.backward()
        return {"log_z": log_z.detach(), "grad": s["J"].grad}
    plans = kn.plan_set(s["counts"], s["flat"], s["qs"], **s["opts"])
    batch = kn.Batch(plans)
    if s["workspace"].numel() < batch.workspace_bytes + 256:
        s["workspace"] = kn.alloc_workspace(batch.workspace_bytes)
    batch.upload(s["workspace"])
    z = batch.contract(z=s["z"])
    v, log2, _ = kn.jones_many(s["qs"], plans, z.cpu().numpy())
    return {"v": v, "log2": log2}


@functools.lru_cache(maxsize=256)
def _work(items):
    case = dict(items)
    pds, qs = _diagrams(case, 0)
    opts = _options(case)
    _, plans = kn.plan_many(pds, qs, **opts)
    edges = sum(len(p) for p in pds)
    grads = 16 * edges if opts.get("gradient") else 0
    return {"bytes": float((16 if case["couplings"] != "jones" else 1) * edges + 24 * len(pds) + grads),
            "flops": sum(p.stats["flops"] for p in plans)}


def work(case):
    """The complex multiply-adds of a pairwise contraction order (8 operations each) and, of memory,
    the couplings or signs read and the results written: the tensors between them need not leave the
    chip where they are small, and are the order's own where they are large."""
    return dict(_work(tuple(sorted((k, v) for k, v in case.items() if k != "name"))))


# ------------------------------------------------------------------ the values in 64 bits


def _t(q):
    """t(q), a root of t + 1/t = q - 2: principal roots, sqrt(q (q - 4)) first."""
    return (q - 2 + cmath.sqrt(q) * cmath.sqrt(q - 4)) / 2


def _jones_weights(q, eps):
    t = _t(q)
    return np.array([-(t ** -int(e)) for e in eps], np.complex128)


def _tait(pd):
    """Signed Tait graph of a PD code: (spins, (n, 2) ends of every crossing's edge, signs, writhe)."""
    n = len(pd)
    m = 2 * n
    positive = (pd[:, 1] - pd[:, 3]) % m == 1
    flat = pd.reshape(-1)
    order = np.argsort(flat, kind="stable")
    far = np.empty(4 * n, np.int64)  # the other end of the arc at slot 4 i + k
    far[order[0::2]], far[order[1::2]] = order[1::2], order[0::2]
    face = np.full(4 * n, -1)  # corner (i, k) lies between slots k and k + 1
    count = 0
    for c in range(4 * n):
        if face[c] >= 0:
            continue
        while face[c] < 0:
            face[c] = count
            j = far[c]
            c = (j & ~3) | ((j - 1) & 3)
        count += 1
    corner = face.reshape(n, 4)
    colour = np.full(count, -1)
    touching = [[] for _ in range(count)]
    for a, b in zip(corner.reshape(-1), np.roll(corner, 1, axis=1).reshape(-1)):
        touching[a].append(b)
        touching[b].append(a)
    # the region on the left of arc 0, where it leaves its crossing, is white
    out_over = np.where(positive, 1, 3)
    rows = np.arange(n)
    left0 = np.concatenate([corner[pd[:, 2] == 0, 2], corner[rows, out_over][pd[rows, out_over] == 0]])
    colour[left0[0]] = 0
    stack = [left0[0]]
    while stack:
        f = stack.pop()
        for g in touching[f]:
            if colour[g] < 0:
                colour[g] = 1 - colour[f]
                stack.append(g)
    spin = np.cumsum(colour) - 1
    black = colour[corner[rows, out_over]] == 1
    first = np.where(black, out_over, (out_over + 1) % 4)
    ends = np.stack([spin[corner[rows, first]], spin[corner[rows, (first + 2) % 4]]], axis=1)
    eps = np.where(black, 1, -1)
    return int(colour.sum()), ends, eps, int(np.where(positive, 1, -1).sum())


def _split(x, e=0):
    """(mantissa, exponent of two) with the mantissa's larger part in [0.5, 1)."""
    big = max(abs(x.real), abs(x.imag))
    k = math.frexp(big)[1]
    return complex(math.ldexp(x.real, -k), math.ldexp(x.imag, -k)), e + k


def _gauss_sum(spins, ends, eps):
    """Z at q = 3 with the Jones couplings: there x = w^eps with w = exp(2 pi i / 3), and two spins are
    equal unless the square of their difference is 1 modulo 3, so that Z = w^tau sum_s w^-sum eps (s_u -
    s_v)^2, a Gauss sum: diagonalised over the integers modulo 3, each square a gives sum_s w^(a s^2)."""
    M = np.zeros((spins, spins), np.int64)
    u, v = ends[:, 0], ends[:, 1]
    np.add.at(M, (u, u), -eps)
    np.add.at(M, (v, v), -eps)
    np.add.at(M, (u, v), eps)
    np.add.at(M, (v, u), eps)
    M %= 3
    counts = [0, 0, 0]
    live = np.arange(spins)
    while len(live):
        d = M[live, live]
        at = np.flatnonzero(d)
        if not len(at):
            off = np.argwhere(M[np.ix_(live, live)])
            if not len(off):
                counts[0] += len(live)
                break
            i, j = live[off[0]]
            M[i] = (M[i] + M[j]) % 3
            M[:, i] = (M[:, i] + M[:, j]) % 3
            continue
        i = live[at[0]]
        a = int(M[i, i])
        counts[a] += 1
        near = np.flatnonzero(M[i])
        row = M[i, near]
        block = np.ix_(near, near)
        M[block] = (M[block] - a * np.outer(row, row)) % 3  # 1 / a = a modulo 3
        live = np.delete(live, at[0])
    powers = 2 * counts[0] + counts[1] + counts[2]  # of sqrt 3
    whole = 3 ** (powers // 2)
    shift = max(0, whole.bit_length() - 1)
    mantissa = float(Fraction(whole, 1 << shift)) * (math.sqrt(3) if powers % 2 else 1.0)
    # i^(counts1 - counts2) w^tau in twelfths of a turn, its cosine and sine without rounding 0 and 1/2
    turn = (3 * (counts[1] - counts[2]) + 4 * int(eps.sum())) % 12
    half, tall = 0.5, math.sqrt(3) / 2
    cosine = (1, tall, half, 0, -half, -tall, -1, -tall, -half, 0, half, tall)
    return _split(mantissa * complex(cosine[turn], cosine[(turn - 3) % 12]), shift)


def _order(spins, ends):
    """Spins in min-fill order, and the largest number of spins joined by one of them."""
    near = [set() for _ in range(spins)]
    for u, v in ends:
        if u != v:
            near[u].add(v)
            near[v].add(u)
    missing = lambda v: sum(len(near[v] - near[a]) - 1 for a in near[v])  # noqa: E731
    cost = {v: (missing(v), len(near[v])) for v in range(spins)}
    order, width = [], 0
    while cost:
        v = min(cost, key=lambda x: (cost[x], x))
        del cost[v]
        order.append(v)
        nb = near[v]
        width = max(width, len(nb) + 1)
        stale = set(nb)
        for a in nb:
            near[a].discard(v)
            near[a] |= nb - {a}
            stale |= near[a]
        for a in stale:
            if a in cost:
                cost[a] = (missing(a), len(near[a]))
    return order, width


def _log_z(spins, ends, x, q, order):
    """log Z (a complex128 tensor, differentiable in the weights x = e^J) by summing out one spin after
    another; every factor is divided by its largest entry."""
    merged, log_z = {}, torch.zeros((), dtype=torch.complex128)
    for (u, v), w in zip(ends.tolist(), x.unbind()):
        if u == v:
            log_z = log_z + torch.log(w)
        else:
            key = (min(u, v), max(u, v))
            merged[key] = merged[key] * w if key in merged else w
    eye = torch.eye(q, dtype=torch.complex128)
    factors, holders = [], {}  # (spins, tensor); the factors that each spin is in

    def add(spins_, f):
        for s in spins_:
            holders.setdefault(s, set()).add(len(factors))
        factors.append((spins_, f))

    for key, w in merged.items():
        add(key, 1 + (w - 1) * eye)
    for v in order:
        held = sorted(holders.pop(v, ()), key=lambda i: len(factors[i][0]))
        if not held:
            log_z = log_z + math.log(q)
            continue
        union = [v]
        product = None
        for i in held:
            spins_, f = factors[i]
            factors[i] = None
            for s in spins_:
                if s != v:
                    holders[s].discard(i)
            extra = [s for s in spins_ if s not in union]
            if product is not None:
                product = product.reshape(product.shape + (1,) * len(extra))
            union += extra
            place = sorted(range(len(spins_)), key=lambda a: union.index(spins_[a]))
            have = set(spins_)
            f = f.permute(place).reshape([q if s in have else 1 for s in union])
            product = f if product is None else product * f
        product = product.sum(0)
        scale = product.detach().abs().max()
        log_z = log_z + torch.log(scale)
        product = product / scale
        if len(union) == 1:
            log_z = log_z + torch.log(product)
        else:
            add(tuple(union[1:]), product)
    return log_z


def _from_log(log_z):
    """(mantissa, exponent of two) of exp(log_z)."""
    k = math.floor(log_z.real / math.log(2))
    # the real part's multiple of log 2 is taken off in exact arithmetic
    rest = float(Fraction(log_z.real) - k * _LOG2)
    return _split(cmath.exp(complex(rest, log_z.imag)), k)


_LOG2 = Fraction(math.log(2)) + Fraction(2.3190468138462996e-17)  # log 2 in two parts


def _jones(q, spins, writhe, tau, z):
    """(V, log2 |V|) = A Z, with the fractional powers of t from its principal fourth root."""
    t = _t(q)
    root = cmath.exp(cmath.log(t) / 4)
    base = -(root ** 2 + root ** -2)
    log2_a = -(spins + 1) * math.log2(abs(base)) + (3 * writhe + tau) * math.log2(abs(root))
    unit = (base / abs(base)) ** (-(spins + 1)) * (-1) ** writhe * (root / abs(root)) ** (3 * writhe + tau)
    log2_v = log2_a + math.log2(abs(z[0])) + z[1]
    return z[0] / abs(z[0]) * unit * 2.0 ** log2_v, log2_v


def exact(case, seed):
    pds, qs = _diagrams(case, seed)
    derivative = case["kind"] in ("gradient", "fit")
    graphs = [_tait(pd) for pd in pds]
    orders = [None] * len(pds)
    cost = 0.0
    for i, (q, g) in enumerate(zip(qs, graphs)):
        if q == 3 and case["couplings"] == "jones":
            continue
        orders[i] = _order(g[0], g[1])
        cost += (5 if derivative else 2) * (1e-2 * g[0] / 100 + 4e-8 * q ** orders[i][1])
    if cost > 15:
        return None
    zs, grads = [], []
    if case["couplings"] != "jones":
        J = _couplings(case, seed, [_Edges(g) for g in graphs], qs)
    at = 0
    for q, (spins, ends, eps, _), order in zip(qs, graphs, orders):
        if order is None:
            zs.append(_gauss_sum(spins, ends, eps))
            continue
        if case["couplings"] == "jones":
            x = torch.from_numpy(_jones_weights(q, eps))
            zs.append(_from_log(complex(_log_z(spins, ends, x, q, order[0]))))
            continue
        j = torch.from_numpy(J[at:at + len(eps)]).requires_grad_(derivative)
        at += len(eps)
        log_z = _log_z(spins, ends, torch.exp(j), q, order[0])
        zs.append(_from_log(complex(log_z.detach())))
        if derivative:
            log_z.real.backward()
            grads.append(j.grad)
    if case["kind"] in ("values", "pipeline"):
        v = [_jones(q, g[0], g[3], int(g[2].sum()), z) for q, g, z in zip(qs, graphs, zs)]
        return {"v": np.array([a for a, _ in v]), "log2": np.array([b for _, b in v])}
    if case["kind"] == "fit":
        m, e = zs[0]
        return {"log_z": torch.tensor(cmath.log(m) + e * math.log(2), dtype=torch.complex128),
                "grad": grads[0]}
    out = {"mantissa": np.array([[m.real, m.imag] for m, _ in zs]),
           "exp2": np.array([e for _, e in zs], np.int64)}
    if case["kind"] == "gradient":
        # autograd gives a real loss's gradient conjugated
        out["grad"] = torch.view_as_real(torch.cat(grads).conj().resolve_conj())
    return out


class _Edges:
    """A Tait graph's signs under the name that _couplings reads them by."""

    def __init__(self, graph):
        self.graph = graph

    def edges(self):
        return self.graph[1], self.graph[2]
