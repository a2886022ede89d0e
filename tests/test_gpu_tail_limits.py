"""Which levels the end of the V-cycle takes into one workgroup per box, and
which take the correction and the first smoothing step in one launch: level
sizes worked out here from the coarsening rule, with each mesh on the side of a
limit that it stands for, solved alone and stage by stage (in a batch) with
equal solutions, bit for bit.

Limits: 1024 nodes of the upper level (512: one per thread), 152 KB of LDS (with
coarse inverses of more than about 100 unknowns), a box with two smoothed levels
left enters only if every box does, 512 tiles for the fused correction.  (The
512 nodes of the lower level are out of reach: the coarsest level below it would
not fit the LDS.)"""
import numpy as np
import pytest

import p4d_inputs as pi
from tests.gpu_util import say, to_dev, to_np


def vol(d):
    return d[0] * d[1] * d[2]


def levels(dims, coarse_max):
    out = [dims]
    while vol(out[-1]) > coarse_max:
        c = tuple(n if n <= 2 else n // 2 + 1 for n in out[-1])
        if c == out[-1] or len(out) == 16:
            break
        out.append(c)
    return out


def lds_bytes(top, sub, coarse):
    with_halo = sum(vol(tuple(n + 2 for n in d)) for d in (top, sub) if d)
    nodes = sum(vol(d) for d in (top, sub) if d)
    return 8 * (with_halo + nodes + 6 * vol(coarse) + vol(coarse) ** 2)


def route(dims, coarse_max):
    """Per box (anode, cathode, whole cell): (level it leaves at, upper, lower,
    coarsest level); tiles of every level that still has launches."""
    nx, ny, nz = dims
    na, ns, _ = pi.layer_split(nz)
    box = [levels((nx, ny, z), coarse_max) for z in (na - 1, nz - na - ns, nz)]
    left, tiles, act, l = {}, {}, [0, 1, 2], 1
    while act := [b for b in act if len(box[b]) - 1 > l]:
        def tail(b):
            if len(box[b]) - 2 - l > 1:
                return None
            t = (box[b][l], box[b][l + 1] if len(box[b]) - 2 - l == 1 else None, box[b][-1])
            return t if vol(t[0]) <= 1024 and lds_bytes(*t) <= 152 * 1024 else None
        every = all(tail(b) for b in act)
        for b in act:
            if tail(b) and (every or tail(b)[1] is None):
                left[b] = (l, *tail(b))
        act = [b for b in act if b not in left]
        if act:   # (the whole cell's box stands for phi_e and c_e)
            tiles[l] = sum((2 if b == 2 else 1) * -(-box[b][l][0] // 8) * -(-box[b][l][1] // 8) * -(-box[b][l][2] // 4)
                           for b in act)
        l += 1
    return left, tiles


def top(r, b):
    return vol(r[0][b][1])


# mesh, coarse_max, what it stands for
CASES = [((6, 14, 62), 64, lambda r: top(r, 2) == 1024 and r[0][2][2] and not r[1]),
         ((5, 20, 60), 64, lambda r: r[1] and r[0][2][0] == 2),            # 1023 nodes with two levels below
         ((6, 6, 62), 64, lambda r: top(r, 2) == 512 and r[0][2][2]),
         ((5, 16, 36), 64, lambda r: top(r, 2) == 513 and r[0][2][2] and r[0][0][2] is None),
         ((5, 16, 36), 100, lambda r: top(r, 2) == 513 and r[0][2][2] is None),
         ((14, 14, 14), 138, lambda r: top(r, 2) == 512 and r[0][2][2] is None),
         ((5, 12, 60), 138, lambda r: 150 * 1024 < lds_bytes(*r[0][2][1:]) <= 152 * 1024),
         ((5, 14, 46), 138, lambda r: 2 not in r[0] and 0 in r[0]),        # whole cell: over the LDS
         ((7, 21, 60), 64, lambda r: r[0][0][0] == 2 and vol(levels((7, 21, 24), 64)[1]) == 572),   # electrodes wait
         ((21, 14, 41), 64, lambda r: r[0][2][0] == 2 and r[0][2][2] and r[0][0][2] is None)]
TILES = [((48, 50, 81), lambda r: r[1][1] == 512), ((32, 50, 114), lambda r: r[1][1] == 516)]


def solved_both_ways(dims, coarse_max, degree, pc_prec):
    from paper_2602_07225_amd import P4DBatch
    p = pi.make_custom(*dims, (4, 5), seed=72, sigma_log=0.5, corr_cells=3.0)
    B = P4DBatch([p], pc_prec=pc_prec, coarse_max=coarse_max)
    B.setup(rtol=1e-8, cheb_degree=degree, maxit=40)
    (xb,), (ib,) = B.solve([p.b])
    x1, i1 = B.solve_cell(0, to_dev(p.b))
    say(f"{dims} coarse_max {coarse_max} degree {degree} prec {pc_prec}: {ib.iters} / {i1.iters} iterations")
    assert ib.iters == i1.iters and ib.status == i1.status
    assert np.any(to_np(x1)) and np.array_equal(to_np(xb), to_np(x1))
    B.close()


@pytest.mark.parametrize("dims,coarse_max,side", CASES)
def test_meshes_lie_where_they_should(dims, coarse_max, side):
    assert side(route(dims, coarse_max))


@pytest.mark.gpu
@pytest.mark.parametrize("dims,coarse_max,side", CASES)
@pytest.mark.parametrize("degree,pc_prec", [(1, 0), (2, 0), (3, 1)])
def test_levels_in_one_workgroup(dims, coarse_max, side, degree, pc_prec):
    assert side(route(dims, coarse_max))
    solved_both_ways(dims, coarse_max, degree, pc_prec)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,side", TILES)
def test_correction_and_step_around_the_tile_limit(dims, side):
    assert side(route(dims, 64))
    solved_both_ways(dims, 64, 2, 0)
