"""The end of the V-cycle in one workgroup per box (one or two smoothed levels
above the dense solve) against the same stages one launch after another, as
the batched solve runs them: the arithmetic is the same, so the solutions are
equal bit for bit.  Meshes on either side of the kernel's limits: 512 nodes of
the lower level, 512 and 1024 of the upper one, boxes that enter it at
different levels."""
import numpy as np
import pytest

import p4d_inputs as pi
from tests.gpu_util import say, to_dev, to_np

pytestmark = pytest.mark.gpu

# (nx, ny, nz): level sizes of the whole-cell boxes below the finest
MESH = [(9, 9, 21),      # 275, 54: one smoothed level in the kernel
        (14, 14, 41),    # 1344 (its own launches), 250, 63
        (12, 12, 39),    # 980 = two nodes per thread, 176, 54
        (13, 13, 39),    # 980, with odd extents
        (11, 13, 21),    # 462: one node per thread, two levels
        (2, 2, 300),     # 604, 304, 156: long in z, two-point axes kept
        (25, 20, 23)]    # 1716, 294, 48: the electrodes enter at another level


@pytest.mark.parametrize("dims", MESH)
@pytest.mark.parametrize("degree,pc_prec", [(1, 0), (2, 0), (3, 0), (4, 0), (2, 1)])
def test_equals_the_stages_one_by_one(dims, degree, pc_prec):
    from paper_2602_07225_amd import P4DBatch
    p = pi.make_custom(*dims, (5, 6), seed=71, sigma_log=0.5, corr_cells=3.0)
    B = P4DBatch([p], pc_prec=pc_prec)
    B.setup(rtol=1e-8, cheb_degree=degree, maxit=40)
    (xb,), (ib,) = B.solve([p.b])
    x1, i1 = B.solve_cell(0, to_dev(p.b))
    say(f"{dims} degree {degree} prec {pc_prec}: {ib.iters} / {i1.iters} iterations")
    assert ib.iters == i1.iters and ib.status == i1.status
    assert np.any(to_np(x1)) and np.array_equal(to_np(xb[:]), to_np(x1))
    B.close()


# levels between the finest and the tail: the correction and the first
# post-smoothing step in one launch, tiles of 8 x 8 x 4 nodes with remainders
# of one node, of all but one, and none; a two-point axis
@pytest.mark.parametrize("dims", [(33, 17, 66), (30, 31, 47), (2, 70, 90)])
@pytest.mark.parametrize("degree,pc_prec", [(1, 0), (2, 0), (3, 1)])
def test_corrected_and_smoothed_at_once_equals_the_stages(dims, degree, pc_prec):
    test_equals_the_stages_one_by_one(dims, degree, pc_prec)
