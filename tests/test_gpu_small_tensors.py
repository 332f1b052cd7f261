"""Tensors whose entries are all subnormal: their shift is that of the least
normal number, so that the step after brings them back to full precision
(without a shift the products keep the few bits a subnormal number has).

The knots are connected sums of a trefoil, whose Tait graph is a triangle here,
and a small lattice knot.  With q = 2 and the triangle's weights x = 2^e, every
spin configuration has at least one equal pair in the triangle, so Z = x Z_1 +
x^3 Z_3, and Z_1 comes from a sum over all configurations with x = 2^-100."""

from __future__ import annotations

import itertools

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1807_02119_amd import gen, kn
from tests.oracle_helpers import TOL32, TOL64, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kn.lib()
    yield
    torch.cuda.synchronize()


def _connected_sum(a, b):
    """Arc 0 of each diagram is cut and its ends joined to the other's."""
    ma, mb = 2 * len(a), 2 * len(b)

    def relabel(pd, shift, after):
        rows = []
        for r in pd.tolist():
            positive = (r[1] - r[3]) % (2 * len(pd)) == 1
            incoming = (True, not positive, False, positive)
            rows.append([x + shift if x else (shift if i else after) for x, i in zip(r, incoming)])
        return rows

    return np.array(relabel(a, 0, ma) + relabel(b, ma, 0), np.int32)


TREFOIL = np.array([[2, 5, 3, 0], [0, 3, 1, 4], [4, 1, 5, 2]])


@pytest.mark.parametrize("opts", [{}, dict(big_step_macs_log2=1)], ids=["serial", "tiles"])
@pytest.mark.parametrize("precision, e", [(0, -1050), (0, -1030), (0, -1023), (1, -140), (1, -130)])
@pytest.mark.parametrize("seed, scale", [(4, 10), (1, 20), (4, 20)])
def test_subnormal_tensors(seed, scale, precision, e, opts):
    pd = np.asarray(gen.lattice_knot((78, seed), 6, 16).pd)
    t = kn.Tait(_connected_sum(TREFOIL, pd - pd.min()))
    ends, _ = t.edges()
    ends = np.asarray(ends)
    assert len({tuple(sorted(x)) for x in ends[:3].tolist()}) == 3  # the triangle
    rng = np.random.default_rng(seed)
    J = scale * rng.random(t.n_edges) + 1j * rng.uniform(-1, 1, t.n_edges) * 0.3
    spins = np.array(list(itertools.product(range(2), repeat=int(ends.max()) + 1)))
    w = np.ones(len(spins), np.complex128)
    for j, (u, v) in enumerate(ends):
        w *= np.where(spins[:, u] == spins[:, v], 2.0 ** -100 if j < 3 else np.exp(J[j]), 1)
    J[:3] = e * np.log(2)
    p = kn.Plan(t, 2, jones_only=False, precision=precision, **opts)
    z = kn.contract(p, torch.from_numpy(J).to("cuda"))
    torch.cuda.synchronize()
    (m, ez), = kn.scalars_from_device(z)
    err = rel_err(m * 2.0 ** (ez - e - 100), w.sum())
    print(f"n={t.n_edges} seed={seed} scale={scale} precision={precision} e={e} {opts}: {err:.1e}",
          flush=True)
    assert err <= (TOL32 if precision else TOL64), err
