"""Steps whose last wavefronts are partly filled: units that share a contracted
index out to a power of two of lanes which does not divide it, and tiles whose
outputs do not fill their last wavefront.  Lanes past the end take part in
reading the strides held in other lanes' registers and add nothing."""

from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")

from paper_1807_02119_amd import gen, kn
from tests import image_model as im
from tests.oracle_helpers import TOL32, TOL64, oracle_z, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kn.lib()
    yield
    torch.cuda.synchronize()


def _check(d, q, precision, **kw):
    p = kn.Plan(kn.Tait(d.pd), q, precision=precision, **kw)
    z = kn.contract(p)
    torch.cuda.synchronize()
    (m, e), = kn.scalars_from_device(z)
    _, mo, eo = oracle_z(d, q)
    err = rel_err(m * 2.0 ** (e - eo), mo)
    print(f"n={d.n} q={q} precision={precision} {kw}: {err:.1e}", flush=True)
    assert err <= (TOL32 if precision else TOL64), err
    return im.Image(p.image()).steps


def _lanes(outs, nk, q):
    """Lanes per output of a unit."""
    n = 1
    while n < 64 and 2 * n <= nk // q and outs * n < (512 if nk // n >= 16 else 64):
        n *= 2
    return n


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q, lo", [(3, 200), (5, 60), (6, 40)])
def test_units(q, lo, precision):
    steps = _check(gen.lattice_knot((45, q), lo, 2 * lo), q, precision, big_step_macs_log2=24,
                   big_step_outs_log2=24)
    ragged = 0
    for s in steps:
        outs, nk = int(s["nb"]) * int(s["nm"]) * int(s["nn"]), int(s["nk"])
        if nk > q ** 3 or (nk == q ** 3 and outs < 512):
            ragged += (nk // q) % _lanes(outs, nk, q) != 0
    assert ragged > 0


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("outs", [65, 1000, 2047])
@pytest.mark.parametrize("q, lo, hi", [(3, 200, 300), (5, 90, 160)])
def test_tiles(q, lo, hi, outs, precision):
    steps = _check(gen.lattice_knot((46, q), lo, hi), q, precision, big_step_macs_log2=1,
                   tile_outputs=outs)
    # (a tile of fewer than 512 outputs has several lanes per output)
    rows = [(min(int(s["tile"]), int(s["nb"]) * int(s["nm"]) * int(s["nn"])), int(s["nk"]))
            for s in steps if int(s["mode"]) == 1]
    assert any((n < 512) == (outs < 512) and n % 64 and 1 < nk <= 64 for n, nk in rows)
