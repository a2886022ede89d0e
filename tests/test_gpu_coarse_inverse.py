"""The dense inverse of the coarsest grid at sizes around its block width and
its kernels' limits, and the factored z-lines, through the preconditioner
against the oracle's.

Tolerance: 1e-9.  The coarsest systems have condition numbers up to ~1e6, so
two FP64 inversions differ by up to ~1e-10 in what they return, and the finer
levels' sums add as much (the parity tests' bound, 1e-10)."""
import numpy as np
import pytest

import oracle as O
import p4d_inputs as pi
from tests.gpu_util import field_errors, say, solver_for, to_dev, to_np

pytestmark = pytest.mark.gpu

# coarsest grids of (anode, cathode, whole cell) nodes: one workgroup up to 64
# and 80 unknowns, blocks of 32 (exact multiples, remainders, most blocks) above
MESH = [(4, 4, 13, 60),      # below the finest level only
        (5, 5, 16, 1024),    # 150 / 175 / 400: the whole grid dense
        (4, 4, 24, 400),     # 144 / 160 / 384
        (4, 8, 30, 1024),    # 960: most blocks
        (3, 3, 27, 256),     # 90 / 99 / 243
        (4, 4, 15, 272),     # 80 / 96 / 240: boxes on either side of the limit
        (4, 4, 17, 272)]     # 96 / 112 / 272


@pytest.mark.parametrize("nx,ny,nz,coarse_max", MESH)
def test_preconditioner_with_large_coarsest_grids(nx, ny, nz, coarse_max):
    p = pi.make_custom(nx, ny, nz, (4, 5), seed=81, sigma_log=0.5, corr_cells=3.0)
    r = np.random.default_rng(9).standard_normal(p.N)
    orc = O.Oracle(p).setup(coarse_max=coarse_max)
    s = solver_for(p, coarse_max=coarse_max).setup(coarse_max=coarse_max)
    errs = field_errors(p, to_np(s.apply_pc(to_dev(r))), orc.apply_pc(r))
    say(f"{nx}x{ny}x{nz} coarse_max {coarse_max}", {k: f"{v:.1e}" for k, v in errs.items()})
    assert max(errs.values()) <= 1e-9


# z extents around the factoring's groups of eight rows, line counts around
# the tile widths
@pytest.mark.parametrize("nx,ny,nz", [(9, 5, 13), (34, 2, 25), (5, 4, 37), (17, 9, 61), (2, 2, 13)])
@pytest.mark.parametrize("degree", [1, 2])
def test_zline_preconditioner(nx, ny, nz, degree):
    p = pi.make_case3_like(nx=nx, ny=ny, nz=nz, nr=(4, 5), seed=82)
    r = np.random.default_rng(10).standard_normal(p.N)
    kw = dict(smoother=O.SMOOTH_ZLINE, cheb_degree=degree)
    orc = O.Oracle(p).setup(**kw)
    s = solver_for(p, smoother=O.SMOOTH_ZLINE).setup(**kw)
    errs = field_errors(p, to_np(s.apply_pc(to_dev(r))), orc.apply_pc(r))
    say(f"{nx}x{ny}x{nz} degree {degree}", {k: f"{v:.1e}" for k, v in errs.items()})
    assert max(errs.values()) <= 1e-9


# lines around 32 rows per run of the substitutions: one, two and three rows a
# lane, the last lanes' runs short or empty
@pytest.mark.parametrize("nz", [31, 32, 33, 64, 65, 90])
def test_zline_substitutions_around_their_runs(nz):
    p = pi.make_custom(7, 3, nz, (4, 5), seed=83, sigma_log=0.5, corr_cells=3.0)
    r = np.random.default_rng(11).standard_normal(p.N)
    orc = O.Oracle(p).setup(smoother=O.SMOOTH_ZLINE)
    s = solver_for(p, smoother=O.SMOOTH_ZLINE).setup(smoother=O.SMOOTH_ZLINE)
    errs = field_errors(p, to_np(s.apply_pc(to_dev(r))), orc.apply_pc(r))
    say(f"7x3x{nz}", {k: f"{v:.1e}" for k, v in errs.items()})
    assert max(errs.values()) <= 1e-9
