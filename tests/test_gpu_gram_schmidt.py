"""Dot products and updates over many and over long Krylov vectors.

Long vectors are read in a different order than short ones when there are
few of them, in single solves only: at either side of the two lengths where
that changes (2^21 entries for the update, 2^22 for the dot products) a cell
solved alone equals the same cell in a batch bit for bit, whole and folded
vectors, at every count up to nine.

More than 32 vectors: the iterate after k steps of one long cycle against the
oracle's.  Tolerance 1e-7: the preconditioner agrees with the oracle's to 1e-10
and the Hessenberg systems have condition numbers below 1e3 (a change of b
of 1e-10 moves these iterates by less than 1e-9)."""
import numpy as np
import pytest

import oracle as O
import p4d_inputs as pi
from tests.gpu_util import rel, say, solver_for, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [32, 33, 41, 63])
def test_cycles_of_more_than_32_vectors(steps):
    p = pi.make_custom(20, 18, 61, (5, 6), seed=104, sigma_log=2.5, corr_cells=3.0)
    kw = dict(pc=O.PC_BJ, cheb_degree=1, restart=63, maxit=steps, rtol=1e-15)
    xo, io = O.Oracle(p).setup(cgs2=True, **kw).solve(p.b)
    x, info = solver_for(p, restart=63).setup(cgs2=1, **kw).solve(to_dev(p.b))
    say(f"{steps} steps: residual {info.relres_true:.3e} / {io.relres_true:.3e}")
    assert info.iters == io.iters == steps
    assert rel(to_np(x), xo) <= 1e-7


def in_a_batch_and_alone(p, **opts):
    from paper_2602_07225_amd import P4DBatch
    B = P4DBatch([p], pc_prec=0, restart=opts["restart"])
    B.setup(rtol=1e-15, **opts)
    (xb,), (ib,) = B.solve([p.b])
    x1, i1 = B.solve_cell(0, to_dev(p.b))
    assert ib.iters == i1.iters == opts["maxit"] and ib.relres_est == i1.relres_est
    assert np.any(to_np(x1)) and np.array_equal(to_np(xb), to_np(x1))
    B.close()


# restart 64 is the longest cycle
@pytest.mark.parametrize("pc", [O.PC_SCHUR, O.PC_BJ])
@pytest.mark.parametrize("cgs2", [0, 1])
def test_longest_cycle_in_a_batch_and_alone(pc, cgs2):
    p = pi.make_custom(20, 18, 61, (5, 6), seed=104, sigma_log=2.5, corr_cells=3.0)
    in_a_batch_and_alone(p, pc=pc, cgs2=cgs2, cheb_degree=1, restart=64, maxit=64)


# entries of a vector: below 2^21, between, above 2^22
@pytest.mark.parametrize("dims,nr,pc,lo,hi", [((30, 30, 90), (16, 16), O.PC_BJ, 0, 2 ** 21),
                                              ((40, 40, 120), (16, 16), O.PC_BJ, 2 ** 21, 2 ** 22),
                                              ((48, 48, 144), (15, 17), O.PC_BJ, 2 ** 22, 2 ** 24),
                                              ((56, 56, 200), (3, 4), O.PC_SCHUR, 2 ** 21, 2 ** 22),
                                              ((71, 73, 240), (4, 3), O.PC_SCHUR, 2 ** 22, 2 ** 24)])
def test_long_vectors_in_a_batch_and_alone(dims, nr, pc, lo, hi):
    p = pi.make_custom(*dims, nr, seed=105)
    o = p.offsets
    n = p.N if pc == O.PC_BJ else int(o[3] + o[1])   # folded: electrode-level and surface rows
    say(f"{dims} pc {pc}: {n} entries")
    assert lo <= n < hi
    in_a_batch_and_alone(p, pc=pc, cgs2=1, cheb_degree=1, restart=9, maxit=9)
