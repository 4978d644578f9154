"""Kernel variants at the sizes where they can go wrong (edges of tiles and
blocks, remainders, smallest sizes), against the float64 oracle.

Tolerance: the library's float64 bar, 1e-9 relative (2-norm of a vector, |.| of
the log marginal likelihood); the problems are conditioned at most about 1e4, so
float64 rounding leaves four orders of margin."""
import numpy as np
import pytest

import synth
from oracle import lma as olma

pytestmark = pytest.mark.gpu

BAR = 1e-9


@pytest.fixture(scope="module")
def lib():
    import paper_1411_4510_amd as lma
    lma.load()
    return lma


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


def check_fit(lib, p, bar=BAR, precision="fp64"):
    ref = olma.fit_predict(p)
    st = lib.fit_problem(p, precision=precision)
    mean, var = st.predict(p.U, p.u_block_ptr)
    lml = st.lml()
    st.free()
    assert rel(mean.cpu().numpy(), ref["mean"]) < bar
    assert rel(var.cpu().numpy(), ref["var"]) < bar
    assert abs(lml - ref["lml"]) < bar * abs(ref["lml"])


# one window of n points: its last diagonal tile has n mod 128 real rows
@pytest.mark.parametrize("n,s", [(16, 1), (17, 15), (31, 16), (33, 17), (112, 5), (113, 127), (127, 128), (129, 129),
                                 (255, 40), (257, 143)])
def test_diagonal_tile_block_edges(lib, n, s):
    s = min(s, n)
    p = synth.make_random(seed=100 + n, n=n, d=2, M=1, s=s, n_u=9, B=0, uneven=(n, n), sn2=0.05)
    check_fit(lib, p)


# windows from one to a dozen tiles in one launch of the vector solves, some with an
# empty separator; forward and backward (the mixed path runs both; its bar is 1e-4)
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("B", [0, 1, 4])
def test_vector_solves_of_unequal_windows(lib, B, precision, bar):
    p = synth.make_random(seed=61, n=1500, d=3, M=5, s=70, n_u=60, B=B, uneven=(20, 700), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)


# launches of few tiles run in pieces of 64 x 64 and 32 x 32: windows of 1 to 16 tiles
# (16 and fewer tiles per launch, up to 128, more), pieces of padding only (blocks of
# 130 and 33 points), test tiles of a few rows
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("n,M,B,s,n_u", [(33, 1, 0, 7, 3), (130, 1, 0, 33, 200), (520, 4, 3, 130, 70),
                                         (1600, 8, 2, 260, 333), (4200, 25, 4, 97, 31)])
def test_pieces_of_tiles(lib, n, M, B, s, n_u, precision, bar):
    p = synth.make_random(seed=n, n=n, d=4, M=M, s=s, n_u=n_u, B=B, uneven=(max(1, n // M - 15), n // M + 15), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)
