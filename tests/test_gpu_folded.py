"""Solves whose Krylov vectors keep their particle rows as a multiple of the
cycle's first vector (all unknowns, SCHUR preconditioner, FP64 Z basis): the
iterate after k steps, through restarts, against the oracle, whose vectors are
whole.

Tolerance: the operator agrees with the oracle's to 1e-13 and the
preconditioner to 1e-10 (relative, the bounds of the parity tests); the
Hessenberg systems of these meshes have condition numbers below 1e3, so the
iterate of the same step agrees to 1e-7."""
import numpy as np
import pytest

import oracle as O
import p4d_inputs as pi
from tests.gpu_util import rel, say, solver_for, to_dev, to_np

pytestmark = pytest.mark.gpu

# meshes: the smallest cell, one with fewest / most radial points, odd extents
# with N_r one off the register classes, one thicker separator than electrodes
MESH = {"smallest": lambda: pi.make_custom(2, 2, 5, (3, 64), seed=61, na=2, ns=1),
        "odd": lambda: pi.make_custom(13, 9, 23, (13, 21), seed=62, sigma_log=0.5, corr_cells=3.0),
        "thick_separator": lambda: pi.make_custom(6, 7, 24, (3, 4), seed=63, na=2, ns=20)}


@pytest.mark.parametrize("mesh", sorted(MESH))
@pytest.mark.parametrize("restart,maxit,cgs2", [(30, 3, 0), (1, 3, 0), (2, 5, 1), (3, 7, 0)])
@pytest.mark.parametrize("transpose", [False, True])
def test_iterate_equals_the_oracles(mesh, restart, maxit, cgs2, transpose):
    p = MESH[mesh]()
    say(f"{mesh} N={p.N} restart {restart} maxit {maxit} cgs2 {cgs2} transpose {transpose}")
    kw = dict(rtol=1e-13, restart=restart, maxit=maxit)
    orc = O.Oracle(p).setup(cgs2=bool(cgs2), **kw)
    xo, io = orc.solve(p.b, transpose=transpose)
    s = solver_for(p).setup(cgs2=cgs2, **kw)
    x, info = (s.solve_adjoint if transpose else s.solve)(to_dev(p.b))
    assert info.iters == io.iters
    assert rel(to_np(x), xo) <= 1e-7


@pytest.mark.parametrize("particles", ["zero", "only"])
def test_particle_part_of_the_right_hand_side(particles):
    """b without a particle part (alpha multiplies nothing) and with nothing
    else: the solution against the oracle's."""
    p = MESH["odd"]()
    b = p.b.copy()
    if particles == "zero":
        b[p.offsets[3]:] = 0.0
    else:
        b[:p.offsets[3]] = 0.0
    xo, io = O.Oracle(p).setup(rtol=1e-9).solve(b)
    x, info = solver_for(p).setup(rtol=1e-9).solve(to_dev(b))
    assert info.status == 0 and abs(info.iters - io.iters) <= 1
    assert info.relres_true <= 1e-9
    assert rel(to_np(x), xo) <= 1e-7
    assert np.all(np.isfinite(to_np(x)))
