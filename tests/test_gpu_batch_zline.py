"""Batches whose cells are smoothed along z-lines: every cell as it is solved
alone, whichever way the batch is told to apply its preconditioner, and the
oracle's solution.

Tolerance against the oracle: both stop at a residual of 1e-9 ||b||, and the
systems of these cells carry a residual to the solution with at most a factor
of some hundreds, so the solutions agree to 1e-6."""
import numpy as np
import pytest
import torch

import oracle as O
import p4d_inputs as pi
from tests.gpu_util import rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def zline_batch(cells):
    from paper_2602_07225_amd import P4DBatch, _lib as L

    class ZLineBatch(P4DBatch):
        # the workspace is laid out for z-line smoothing
        def __init__(self, probs):
            self.device, self.n = torch.device("cuda"), len(probs)
            self.batch = L.p4d_batch_create([L.desc_from(p) for p in probs])
            self.cells = [L.p4d_batch_cell(self.batch, i) for i in range(self.n)]
            sizes = [L.p4d_vector_size(c) for c in self.cells]
            self.N, self.n_elem, self.n_e = ([s[q] for s in sizes] for q in (0, 2, 3))
            self.ws_opts = L.default_opts(coarse_max=64, smoother=O.SMOOTH_ZLINE)
            nbytes = L.p4d_batch_workspace_size(self.batch, self.ws_opts)
            self.ws = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
            L.p4d_batch_set_workspace(self.batch, self.ws.data_ptr(), nbytes, self.ws_opts)
            for i, p in enumerate(probs):
                self.upload(i, p.sigma, p.kappa, p.g, p.s, p.e)

    return ZLineBatch(cells)


@pytest.mark.parametrize("pc", [O.PC_SCHUR, O.PC_BJ])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_zline_cells_in_a_batch(pc, mode):
    cells = [pi.make_custom(8, 8, 24, (8, 8), seed=91, sigma_log=0.5, corr_cells=3.0),
             pi.make_custom(12, 9, 31, (5, 9), seed=92, sigma_log=0.5, corr_cells=3.0)]
    B = zline_batch(cells)
    opts = dict(rtol=1e-9, maxit=200, pc=pc, cheb_degree=1, cgs2=int(pc == O.PC_BJ))
    B.setup(smoother=O.SMOOTH_ZLINE, **opts)
    B.set_pc_mode(mode)
    xs, infos = B.solve([p.b for p in cells])
    for i, p in enumerate(cells):
        x1, i1 = B.solve_cell(i, to_dev(p.b))
        xo, io = O.Oracle(p).setup(smoother=O.SMOOTH_ZLINE, **opts).solve(p.b)
        say(f"cell {i} pc {pc} mode {mode}: {infos[i].iters} / {i1.iters} / {io.iters} iterations")
        assert infos[i].status == 0 and infos[i].iters == i1.iters and abs(i1.iters - io.iters) <= 2
        assert np.array_equal(to_np(xs[i]), to_np(x1))
        assert rel(to_np(xs[i]), xo) <= 1e-6
    B.close()
