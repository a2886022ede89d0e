"""One batch solved with whole and with folded Krylov vectors in turn (FP32 and
FP64 Z basis, one recording of its stages serves both): each solve equals the
single cells', bit for bit, in every mode of applying the preconditioner."""
import numpy as np
import pytest

import p4d_inputs as pi
from tests.gpu_util import say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("pc_prec", [0, 1])
def test_z_precisions_in_turn(mode, pc_prec):
    from paper_2602_07225_amd import P4DBatch
    # radial classes 8, 12, 32 and 64, the largest cell in the middle
    cells = [pi.make_custom(*d, nr, seed=95 + i, sigma_log=0.5, corr_cells=3.0)
             for i, (d, nr) in enumerate([((7, 8, 21), (3, 8)), ((9, 7, 25), (9, 12)), ((14, 13, 38), (30, 6)),
                                          ((6, 6, 19), (64, 40))])]
    B = P4DBatch(cells, pc_prec=pc_prec)
    B.setup(rtol=1e-7, maxit=40)
    B.set_pc_mode(mode)
    for z_fp32 in (0, 1, 0, 1):
        xs, infos = B.solve([p.b for p in cells], z_fp32=z_fp32)
        for i, p in enumerate(cells):
            x1, i1 = B.solve_cell(i, to_dev(p.b), z_fp32=z_fp32)
            say(f"mode {mode} prec {pc_prec} z_fp32 {z_fp32} cell {i}: {infos[i].iters} / {i1.iters}")
            assert infos[i].iters == i1.iters and np.array_equal(to_np(xs[i]), to_np(x1))
    B.close()
