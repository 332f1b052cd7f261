"""Every way the engine computes a step, on plans that are known to take it: the
way is read off the device program and asserted on the CPU, the values are
compared on the GPU.

Couplings are positive, so that Z and its derivatives are sums of positive
terms and no error is magnified: a value is off by about u sqrt(n) with n, the
roundings along its chain of steps and contracted entries, below 10^4.  That
is 6e-6 in complex64 (bound: the suite's 1e-5) and 1e-14 in complex128 (bound
1e-12).  A derivative is a ratio of two such values: twice the bounds."""

from __future__ import annotations

import functools
from collections import Counter

import numpy as np
import pytest

from oracle import potts
from paper_1807_02119_amd import gen, kn
from tests import image_model as im
from tests.oracle_helpers import TOL32, rel_err

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: TOL32}
SERIAL = dict(big_step_macs_log2=24, big_step_outs_log2=24)


# ------------------------------------------------------------------ knots and values


@functools.lru_cache(maxsize=None)
def _knot(source):
    kind, *args = source
    if kind == "lattice":
        return gen.lattice_knot((45, args[0]), args[1], 2 * args[1])
    return gen.config_knots("q3_200_600", args[0], count=args[1] + 1)[args[1]][0]


@functools.lru_cache(maxsize=None)
def _network(source):
    """Tait graph and couplings."""
    t = kn.Tait(_knot(source).pd)
    uv, _ = t.edges()
    edges = [tuple(int(x) for x in e) for e in uv]
    return t, edges, np.random.default_rng(len(edges)).uniform(0.0, 0.5, len(edges))


@functools.lru_cache(maxsize=None)
def _z(source, q):
    t, edges, J = _network(source)
    return potts.partition_function(t.n_vertices, edges, np.exp(J), q)


def _plan(source, q, precision=0, **kw):
    return kn.Plan(_network(source)[0], q, precision=precision, jones_only=False, **kw)


def _check_z(source, q, precision, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, _, J = _network(source)
    mo, eo = _z(source, q)
    z = kn.contract(_plan(source, q, precision, **kw),
                    torch.from_numpy(J.astype(np.complex128)).to("cuda"))
    torch.cuda.synchronize()
    (m, e), = kn.scalars_from_device(z)
    err = rel_err(m * 2.0 ** (e - eo), mo)
    print(f"{source} q={q} precision={precision} {kw}: {err:.1e}", flush=True)
    assert err <= TOL[precision], err


# ------------------------------------------------------------------ the way of each step


def _ways(plan):
    """Counter of the ways the steps of a plan's image are computed."""
    img, out = im.Image(plan.image()), Counter()
    for t in img.tasks:
        if int(t["kind"]) == 0:
            _serial_ways(img, t, out)
    for s in img.steps:
        nb, nm, nn, nk, mode, tile, n_ks, kseg = (
            int(s[f]) for f in ("nb", "nm", "nn", "nk", "mode", "tile", "n_ks", "kseg"))
        split = "split" if n_ks > 1 else "whole"
        if mode == 1:
            outs = min(tile, nb * nm * nn)
            if outs == 1 and kseg >= 1024:
                out["tile", "all wavefronts", split] += 1
            elif outs >= 512 and kseg <= 64:
                out["tile", "B in LDS" if nb * nk * nn <= outs else "B in memory", split] += 1
            else:
                out["tile", "lanes share" if kseg > 64 or outs < 512 else "long", split] += 1
        elif mode >= 2:
            for take in _regions(mode == 3, int(s["n_mb"]), int(s["n_nb"]), nb, tile):
                chunk = 8 if mode == 3 and take == 4 else 16
                out["block", 64 if mode == 3 else 32, take, split,
                    "reuse" if kseg > 2 * chunk else "short"] += 1
    return out


def _regions(wide, n_mb, n_nb, nb, per):
    """Blocks joined in each region of a step's tasks."""
    paired, total = (n_mb & ~1) * n_nb, nb * n_mb * n_nb
    for start in range(0, total, per):
        blk, end = start, min(total, start + per)
        while blk < end:
            r, take = blk % (n_mb * n_nb), 1
            if r < paired and r % (2 * n_nb) % 2 == 0:
                col = r % (2 * n_nb) >> 1
                four = col + 1 < n_nb if wide or n_nb > 1 else r + 4 <= paired
                take = 4 if four and blk + 4 <= end else 2 if blk + 2 <= end else 1
            yield take
            blk += take


def _serial_ways(img, task, out):
    q = int(img.knots[int(task["knot"])]["q"])
    lo, made = int(task["state_lo"]), int(task["state_len"])

    def in_lds(t):
        return not lo + 768 <= t < lo + made

    first = int(task["first"])
    steps = img.steps[first:first + int(task["count"])]
    i = 0
    while i < len(steps):  # chunks of at most 64 steps and 1536 digits
        j = digits = 0
        while i + j < len(steps) and j < 64:
            digits += sum((int(steps[i + j]["ranks"]) >> b) & 255 for b in (0, 8, 16, 24))
            if digits > 1536:
                break
            j += 1
        chunk, i = steps[i:i + j], i + j
        flat = Counter()
        for s in chunk:
            outs, nk = int(s["nb"]) * int(s["nm"]) * int(s["nn"]), int(s["nk"])
            rk = (int(s["ranks"]) >> 16) & 255
            lds = all(in_lds(int(s[x])) for x in "abc")
            if lds and outs <= 1 << 15 and (rk <= 2 or (rk == 3 and outs >= 512)):
                flat[int(s["lvl"])] += outs
            else:
                out["unit"] += 1
                out["unit", "states in memory"] += not lds
        for n in flat.values():
            out["level", "tiles" if n > 512 else "outputs"] += 1


# ------------------------------------------------------------------ serial levels

LEVELS = [(2, 400), (3, 200), (4, 120), (5, 60), (6, 40), (7, 50), (8, 20)]


@pytest.mark.parametrize("q, lo", LEVELS)
def test_plans_have_levels_of_tiles(q, lo):
    ways = _ways(_plan(("lattice", q, lo), q, **SERIAL))
    assert ways["level", "tiles"] and ways["level", "outputs"], ways


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lds_bytes", [256, 131072])
@pytest.mark.parametrize("q, lo", LEVELS)
def test_levels(q, lo, lds_bytes, precision):
    _check_z(("lattice", q, lo), q, precision, lds_bytes=lds_bytes, **SERIAL)


# more tensors than a task has states for in LDS
MANY = dict(SERIAL, fork_serial_log2=40)


def test_plan_has_states_in_memory():
    ways = _ways(_plan(("lattice", 2, 700), 2, **MANY))
    assert ways["unit", "states in memory"] >= 100, ways


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lds_bytes", [256, 98304])
def test_states_in_memory(lds_bytes, precision):
    _check_z(("lattice", 2, 700), 2, precision, lds_bytes=lds_bytes, **MANY)


# ------------------------------------------------------------------ tile tasks

TILES = [
    (("work", 0, 11), dict(big_step_macs_log2=1, tile_outputs=1, split_min_log2=30),
     ("tile", "all wavefronts", "whole")),
    (("work", 0, 71), dict(big_step_macs_log2=1, tile_outputs=1, split_min_log2=10),
     ("tile", "all wavefronts", "split")),
    (("work", 0, 11), dict(big_step_macs_log2=1, tile_outputs=1, split_min_log2=5),
     ("tile", "lanes share", "split")),
    (("work", 0, 20), dict(big_step_macs_log2=1, tile_outputs=27, split_min_log2=8),
     ("tile", "lanes share", "split")),
    (("work", 0, 20), dict(big_step_macs_log2=1, tile_outputs=27, split_min_log2=30),
     ("tile", "lanes share", "whole")),
    (("work", 0, 5), dict(big_step_macs_log2=1, tile_outputs=2048), ("tile", "B in LDS", "whole")),
    (("work", 0, 5), dict(big_step_macs_log2=1, tile_outputs=512),
     ("tile", "B in memory", "whole")),
]


@pytest.mark.parametrize("source, kw, way", TILES)
def test_plans_have_tiles(source, kw, way):
    ways = _ways(_plan(source, 3, **kw))
    assert ways[way], ways


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("source, kw, way", TILES)
def test_tiles(source, kw, way, precision):
    _check_z(source, 3, precision, **kw)


# ------------------------------------------------------------------ output blocks

BLOCKS = [
    # 128 x 128, 128 x 64 and 64 x 64 regions of many chunks
    (("work", 2, 29), dict(big_step_macs_log2=6, gemm64_pct=100000, gemm_tasks_log2=1),
     [("block", 64, 4, "whole", "reuse"), ("block", 64, 2, "whole", "reuse")]),
    (("work", 2, 29), dict(big_step_macs_log2=6, gemm64_pct=100000, gemm_tasks_log2=30),
     [("block", 64, 1, "whole", "reuse")]),
    # 64 x 64 or 128 x 32, 64 x 32 and 32 x 32 regions of many chunks
    (("work", 2, 24), dict(big_step_macs_log2=6, gemm64_pct=1, gemm_tasks_log2=1),
     [("block", 32, 4, "whole", "reuse"), ("block", 32, 2, "whole", "reuse"),
      ("block", 32, 1, "whole", "reuse")]),
    # split contracted indices
    (("work", 0, 16), dict(big_step_macs_log2=6, gemm64_pct=100000, gemm_tasks_log2=1,
                           split_min_log2=7),
     [("block", 64, 4, "split", "reuse"), ("block", 64, 2, "split", "reuse")]),
    (("work", 0, 16), dict(big_step_macs_log2=6, gemm64_pct=100000, gemm_tasks_log2=30,
                           split_min_log2=7), [("block", 64, 1, "split", "reuse")]),
    (("work", 0, 85), dict(big_step_macs_log2=6, gemm64_pct=1, gemm_tasks_log2=1,
                           split_min_log2=7), [("block", 32, 4, "split", "reuse")]),
]


@pytest.mark.parametrize("source, kw, want", BLOCKS)
def test_plans_have_blocks(source, kw, want):
    ways = _ways(_plan(source, 3, **kw))
    assert all(ways[w] for w in want), ways


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("source, kw, want", BLOCKS)
def test_blocks(source, kw, want, precision):
    _check_z(source, 3, precision, **kw)


# ------------------------------------------------------------------ gradients


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lds_bytes", [256, 98304])
@pytest.mark.parametrize("q, lo", [(2, 100), (3, 100), (5, 50), (3, 500)])
def test_gradient(q, lo, lds_bytes, precision):
    """Intermediates in LDS or in global memory; the last knot's tasks have more
    tensors than states in LDS."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    source = ("lattice", q, lo)
    t, edges, J = _network(source)
    mo, eo = _z(source, q)
    p = _plan(source, q, precision, gradient=True, lds_bytes=lds_bytes)
    if lo == 500:
        assert max(int(x["state_len"]) for x in im.Image(p.image()).tasks) > 768
    z, g = kn.contract_backward(p, torch.from_numpy(J.astype(np.complex128)).to("cuda"))
    torch.cuda.synchronize()
    (m, e), = kn.scalars_from_device(z)
    g = g.cpu().numpy()
    err = rel_err(m * 2.0 ** (e - eo), mo)
    assert err <= TOL[precision], err
    worst = 0.0
    for k in range(3, len(edges), len(edges) // 7):
        if edges[k][0] == edges[k][1]:
            want = 1.0
        else:
            alg = potts.ComplexAlgebra(q)
            f, const = potts.edge_factors(alg, edges, np.exp(J), replace=k)
            mk, ek = potts.eliminate(alg, t.n_vertices, f, const, edges=edges)
            want = (mk / mo) * 2.0 ** (ek - eo)
        worst = max(worst, rel_err(complex(*g[k]), want))
    print(f"{source} q={q} precision={precision} lds={lds_bytes}: Z {err:.1e}, d {worst:.1e}",
          flush=True)
    assert worst <= 2 * TOL[precision], worst
