"""The paths a contraction step can take on the device, at the sizes where they
meet: regions of output blocks (joined in fours, in pairs or alone, with ragged
edges), levels of serial steps computed in output tiles, one output per lane or
as units of several lanes per output, tile tasks with operand B in LDS or in
global memory, and gradient plans whose intermediates live in LDS.

Tolerances: a sum over N steps of products of contracted extent K, each rounded
in unit u, is off by a few times sqrt(N K) u of its terms' size.  N K is below
10^6 here, so 10^3 u times a cancellation of up to 10^2 against the largest
term: 1e-10 in complex128 (u = 1.1e-16), 1e-2 in complex64 (u = 6e-8)."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1807_02119_amd import gen, kn
from tests import image_model as im
from tests.oracle_helpers import oracle_z, rel_err

pytestmark = pytest.mark.gpu

TOL = {0: 1e-10, 1: 1e-2}
_Z = {}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kn.lib()
    yield
    torch.cuda.synchronize()


def _check(d, q, precision=0, **kw):
    p = kn.Plan(kn.Tait(d.pd), q, precision=precision, **kw)
    z = kn.contract(p, workspace=kn.alloc_workspace(p.workspace_bytes))
    torch.cuda.synchronize()
    (m, e), = kn.scalars_from_device(z)
    key = (q, np.asarray(d.pd).tobytes())
    if key not in _Z:
        _Z[key] = oracle_z(d, q)[1:]
    mo, eo = _Z[key]
    err = rel_err(m * 2.0 ** (e - eo), mo)
    modes = sorted({int(s["mode"]) for s in im.Image(p.image()).steps})
    print(f"n={d.n} q={q} precision={precision} {kw} modes {modes}: {err:.1e}", flush=True)
    assert err <= TOL[precision], err
    return modes


# blocks per task 1 (single blocks), 2, 4 and more (regions), 32- and 64-blocks
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("gemm_tasks_log2", [1, 2, 3, 30])
@pytest.mark.parametrize("gemm64_pct", [1, 100000])
def test_block_regions(gemm64_pct, gemm_tasks_log2, precision):
    d, q = gen.config_knots("q3_200_600", 0, count=12)[5]
    modes = _check(d, q, precision, big_step_macs_log2=6, gemm64_pct=gemm64_pct,
                   gemm_tasks_log2=gemm_tasks_log2)
    assert (3 if gemm64_pct > 1 else 2) in modes, modes


# everything in serial runs: single outputs, 2 x 2 and 3 x 3 tiles with and
# without a remainder (q = 2 .. 8), operands in LDS, in global memory and both
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lds_bytes", [256, 4096, 131072])
@pytest.mark.parametrize("q", [2, 3, 4, 5, 6, 7, 8])
def test_serial_levels(q, lds_bytes, precision):
    lo = 200 if q <= 3 else 60 if q <= 5 else 20
    d = gen.lattice_knot((45, q), lo, 2 * lo)
    modes = _check(d, q, precision, big_step_macs_log2=24, big_step_outs_log2=24,
                   lds_bytes=lds_bytes)
    assert modes == [0], modes


# every step a tile task: tiles smaller and larger than B (LDS or not), one
# output per task, and ranges of contracted entries
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("outs", [1, 7, 512, 513, 2049])
@pytest.mark.parametrize("q", [2, 3, 5])
def test_tile_tasks(q, outs, precision):
    d = gen.lattice_knot((46, q), 60, 110) if q == 5 else gen.lattice_knot((46, q), 200, 300)
    modes = _check(d, q, precision, big_step_macs_log2=1, tile_outputs=outs)
    assert 1 in modes, modes


@pytest.mark.parametrize("q", [2, 3, 5])
def test_gradient_homes(q):
    """The gradient with intermediates in LDS has the values it has with all of
    them in global memory."""
    d = gen.lattice_knot((47, q), 60, 100)
    tait = kn.Tait(d.pd)
    rng = np.random.default_rng(q)
    J = torch.tensor(rng.normal(scale=0.3, size=2 * tait.n_edges), dtype=torch.float64,
                     device="cuda")
    out = []
    for lds in (256, 98304):
        p = kn.Plan(tait, q, gradient=True, jones_only=False, lds_bytes=lds)
        z, g = kn.contract_backward(p, J)
        torch.cuda.synchronize()
        out.append((kn.scalars_from_device(z)[0], g.cpu().numpy()))
    (m0, e0), (m1, e1) = out[0][0], out[1][0]
    assert rel_err(m1 * 2.0 ** (e1 - e0), m0) <= TOL[0]
    assert np.abs(out[1][1] - out[0][1]).max() <= TOL[0] * max(1.0, np.abs(out[0][1]).max())
