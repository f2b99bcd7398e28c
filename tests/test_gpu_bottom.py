"""GPU parity of the bottom CG that keeps runs of cells in a lane (levels of
more than 1024 cells): single-level solves, so that CG alone produces the
result, against the oracle's and on both sides of the layout's limits."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import lib, rel_l2

# (extents, cut along x or None, periodic): run lengths 2 to 5 along each axis,
# idle lanes and short last runs, rows that wrap, a level past the run layout
CASES = [
    ((15, 11, 7), None, (False, False, False)),    # 1155 cells: runs of 2
    ((13, 9, 13), None, (True, False, False)),     # runs of 2, odd periodic x
    ((11, 17, 15), 5, (False, True, False)),       # runs of 3, two boxes
    ((15, 11, 19), None, (False, False, True)),    # runs of 4
    ((23, 12, 16), 11, (False, False, False)),     # runs of 5, x in LDS, two boxes
    ((16, 15, 20), None, (True, True, True)),      # runs of 5, singular
    ((17, 19, 17), None, (False, False, False)),   # 5491 cells: no runs
]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ext,cut,per", CASES)
def test_bottom_cg_runs_vs_oracle(ext, cut, per, precision):
    print(f"[bottom] {ext} cut {cut} periodic {per} precision {precision}", flush=True)
    P = lib()
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes = [dom] if cut is None else [((0, 0, 0), (cut - 1, ext[1] - 1, ext[2] - 1)),
                                       ((cut, 0, 0), dom[1])]
    rng = np.random.default_rng(11)
    alpha = 0.0 if all(per) else 1.0
    bf = W.harmonic_faces(np.exp(0.5 * rng.standard_normal(ext)), per)
    f = rng.uniform(-1.0, 1.0, ext)
    if all(per):
        f -= f.mean()
    fb = W.scatter_cells(f, boxes)
    b = [W.scatter_faces(bf[d], boxes, d) for d in range(3)]
    s = P.MLMG(boxes, dom, per, alpha, 1.0,
               b=[P.MultiFab.from_numpy(boxes, b[d], 0,
                                        ixtype=tuple(int(e == d) for e in range(3)))
                  for d in range(3)],
               opts=dict(tune=0, precision=precision, bottom_rel_tol=1e-6, min_bottom_edge=64))
    phi = s.cell_mf(1, fill=0.0)
    info = s.solve(phi, P.MultiFab.from_numpy(boxes, fb, 0), 1e-10)
    torch.cuda.synchronize()
    assert info["nlevels"] == 1 and info["converged"]
    lev = O.make_level(boxes, dom, per, alpha, 1.0, None, b)
    ophi = O.new_cell_data(lev)
    O.solve(lev, ophi, fb, 1e-11, opts=O.Opts(bottom_tol=1e-12, min_bottom_edge=64))
    got = W.gather_cells(phi.valid_numpy(), boxes, ext)
    ref = W.gather_cells(ophi, boxes, ext, ng=1)
    # the residual is at most 1e-10 of max|f|, and the largest element of A^-1
    # over the diagonal's inverse is below 1e2 on these grids
    assert rel_l2(got, ref) <= 1e-8
    s.close()
