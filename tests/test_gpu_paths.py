"""Kernel forms that the library chooses between by size: each at the sizes
where its tiles end, against the direct sum or against another form."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lf():
    import paper_2211_00354_amd as lf
    torch.cuda.set_device(0)
    return lf


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("p", [4, 8, 12, 15, 17, 24, 30, 36])
def test_m2l_forms_agree_bit_for_bit(lf, p, precision):
    # 256^2 leaf boxes of rays (1024 tiles: the form for many tiles) against
    # bands of 18 rows of boxes (96 tiles: the form for few), ragged at their
    # ends.  Every form adds each output's MFMA products in the same order, so
    # the outputs are equal bits; p covers every K-step count.
    f = wl.random_field(3000, 30.0, seed=41, masses="powerlaw")
    g = lf.Grid(-32.0, -32.0, 0.125, 0.125, 512, 512)
    xy, m = dev(f.xy), dev(f.m)
    plan = lf.Plan(xy, m, grid=g, precision=precision, p=p, leaf_level=8)
    whole = lf.deflect(plan=plan, grid=g)
    for j0 in range(0, 512, 35):
        ny = min(35, 512 - j0)
        band = lf.Grid(g.x0, g.y0 + j0 * g.dy, g.dx, g.dy, g.nx, ny)
        part = lf.deflect(plan=plan, grid=band)
        assert torch.equal(part, whole[j0 * 512:(j0 + ny) * 512]), (p, precision, j0)
    plan.close()
    if precision == "fp64" and p >= 30:
        ref = lf.deflect(xy, m, grid=g, method="direct")
        # truncation: the interaction list's ratio is at most 0.55, 0.55^30 = 2e-8
        # of a box's field; sums cancel below that
        assert float((whole - ref).norm() / ref.norm()) < 1e-8
