"""Reported launch shapes are those of the float iterations (problems built on the host only)."""
import pytest

import lrh_workloads as W
from paper_2609_40336_amd import lrh


def shapes(P):
    return {s["De"]: s for s in P.shapes()}


@pytest.mark.parametrize("cplx,n,want", [(False, 10, 16), (False, 2048, 16), (False, 2049, 8), (False, 13000, 8),
                                         (False, 13001, 1), (True, 2048, 16), (True, 24576, 8), (True, 24577, 1)])
def test_reported_shape_is_the_iterations(cplx, n, want):
    d = (W.random_chain(n + 2, seed=1, top_len=3, subintervals=True) if cplx else
         W.with_tops(W.heisenberg_chain(n + 2, field_x=0.4), [tuple(range(i, i + 3)) for i in range(n)],
                     subintervals=True))
    P = lrh.Problem(d, -1)
    assert shapes(P)[8]["n"] == n and shapes(P)[8]["W"] == want
    P.force_shape(8, 64, f32=True)
    assert shapes(P)[8]["W"] == 64


def test_reported_block_is_the_one_launched():
    """Bonds and sites share a launch in the bonds' block; with 8 x 8 clusters in lanes, blocks of 64."""
    P = lrh.Problem(W.heisenberg_square(4), -1)
    P.force_shape(2, 1, block=256)
    assert shapes(P)[2]["block"] == 64
    P.force_shape(4, 1, block=128)
    assert shapes(P)[4]["block"] == shapes(P)[2]["block"] == 128
    P = lrh.Problem(W.xxz_triangular(4, 0.5, seed=1), -1)
    P.force_shape(4, 1, block=128)
    assert shapes(P)[4]["block"] == shapes(P)[2]["block"] == 64
    P.force_shape(8, 1, block=256)
    assert [shapes(P)[k]["block"] for k in (2, 4, 8)] == [128, 128, 256]
