"""A serial step's offsets are products of 24 bits: the image check refuses one
whose operands have more than 2^24 entries, however consistent it is otherwise."""

from __future__ import annotations

import numpy as np
import pytest

from paper_1807_02119_amd import gen, kn
from tests import image_model as im


def _image_with(rb, rm, rk, rn):
    """The image of a plan at q = 3 in which the first serial step has been given
    these ranks, and its tensors and the arena sizes to match."""
    p = kn.Plan(kn.Tait(gen.lattice_knot((45, 3), 100, 200).pd), 3)
    raw = bytearray(p.image())
    img = im.Image(bytes(raw))

    def view(dtype, off, n):
        return np.frombuffer(raw, dtype, int(n), int(img.h[off]))

    step = next(i for i, s in enumerate(img.steps) if int(s["mode"]) == 0)
    s = view(im.STEP, "o_steps", img.h["n_steps"])[step:step + 1]
    nb, nm, nk, nn = 3 ** rb, 3 ** rm, 3 ** rk, 3 ** rn
    s["ranks"] = rb | rm << 8 | rk << 16 | rn << 24
    s["nb"], s["nm"], s["nk"], s["nn"] = nb, nm, nk, nn
    s["home_a"] = s["home_b"] = s["home_c"] = 0
    tensors = view(im.TENSOR, "o_tensors", img.h["n_tensors"])
    for t, size in (("a", nb * nm * nk), ("b", nb * nk * nn), ("c", nb * nm * nn)):
        tensors[int(s[t][0])] = (0, size, -1)
    n = 2 * rb + rm + 2 * rk + rn
    view("<i4", "o_strides", img.h["n_strides"])[int(s["str"][0]):][:n] = 0
    h = np.frombuffer(raw, im.HDR, 1)
    h["arena_elems"] = 3 ** 17
    h["guard_off"] = int(h["arena_off"][0]) + 16 * 3 ** 17
    h["workspace_bytes"] = int(h["guard_off"][0]) + 4096
    return bytes(raw), step


# 2 nb + nm + 2 nk + nn is below 3072 in every case
@pytest.mark.parametrize("ranks, refused", [
    ((5, 6, 5, 0), True),    # A of 3^16 entries
    ((5, 0, 5, 6), True),    # B
    ((5, 5, 5, 0), False),   # 3^15 = 14.3 M < 2^24
    ((4, 0, 5, 6), False),
])
def test_serial_operands_beyond_24_bits_are_refused(ranks, refused):
    raw, step = _image_with(*ranks)
    r = kn.image_check(raw)
    # (the steps after it, whose operands it has changed, fail for other reasons)
    assert ((r["code"], r["step"]) == (6, step)) == refused and r["step"] >= step, r
    assert refused or r["step"] > step, r
