"""Plans near a memory limit: a layout with the default step thresholds that
misses the limit gives way to the tighter one that meets it."""

from __future__ import annotations

import functools

import numpy as np
import pytest

from paper_1807_02119_amd import gen, kn
from tests.oracle_helpers import TOL64, oracle_z, rel_err

NOALLOC_MAX_BYTES = 64 << 20  # KN_NOALLOC_MAX_BYTES in include/kn.h
TIGHT = dict(big_step_outs_log2=12, tile_outs_log2=10)


@functools.lru_cache(maxsize=None)
def _knot():
    """263 crossings: at q = 6 a workspace of 67.7 MB with thresholds of 2^13 and
    2^11 outputs, of 66.9 MB with 2^12 and 2^10."""
    return gen.lattice_knot((99, 18, 34), 168, 264)


def test_plan_fits_the_library_workspace():
    t = kn.Tait(_knot().pd)
    wide = kn.Plan(t, 6, big_step_outs_log2=13, tile_outs_log2=11)
    tight = kn.Plan(t, 6, **TIGHT)
    assert tight.workspace_bytes <= NOALLOC_MAX_BYTES < wide.workspace_bytes
    p = kn.Plan(t, 6)
    assert p.workspace_bytes == tight.workspace_bytes and p.image() == tight.image()
    _, (many,) = kn.plan_many([np.ascontiguousarray(_knot().pd, dtype=np.int32)], [6])
    assert many.workspace_bytes == tight.workspace_bytes
    # a caller's own thresholds are taken as they are
    assert wide.stats["workspace_bytes"] > NOALLOC_MAX_BYTES


def test_plan_fits_the_budget():
    """The smallest budget that the tight thresholds meet is met by default."""
    found = 0
    for d, q in gen.config_knots("q3_200_600", 0, count=24):
        t = kn.Tait(d.pd)
        w, tight = kn.Plan(t, q), kn.Plan(t, q, **TIGHT)
        if tight.workspace_bytes >= w.workspace_bytes:
            continue
        found += 1
        p = kn.Plan(t, q, mem_budget_bytes=tight.workspace_bytes)
        assert p.workspace_bytes == tight.workspace_bytes
        with pytest.raises(kn.KnError):
            kn.Plan(t, q, mem_budget_bytes=tight.workspace_bytes - 1)
    assert found >= 2, found


@pytest.mark.gpu
def test_library_workspace_holds_the_plan():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = kn.Plan(kn.Tait(_knot().pd), 6)
    z = kn.contract_noalloc(p, z=kn.alloc_scalars(1))
    torch.cuda.synchronize()
    (m, e), = kn.scalars_from_device(z)
    _, mo, eo = oracle_z(_knot(), 6)
    assert rel_err(m * 2.0 ** (e - eo), mo) <= TOL64
