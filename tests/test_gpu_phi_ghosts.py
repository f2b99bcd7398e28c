"""After a solve phi's face ghosts hold the solution of the neighbouring boxes
and periodic images, with the levels stored as one grid and as boxes."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import lib

CASES = [
    # extents, boxes along x and y, periodic, opts
    ((32, 32, 16), (2, 2), (False, False, False), {}),
    ((32, 16, 24), (2, 1), (True, False, True), dict(precision=1)),
    ((48, 32, 16), (3, 2), (False, True, False), dict(krylov=1)),
    ((32, 32, 32), (1, 1), (True, True, True), {}),
    ((32, 16, 16), (2, 1), (True, False, False), dict(max_iter=2)),  # not converged
    ((32, 16, 16), (2, 1), (True, False, False), dict(nu2=0)),       # levels as boxes
    ((32, 16, 16), (2, 1), (True, True, True), dict(nu2=0)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("ext,nb,per,opts", CASES)
def test_face_ghosts_after_a_solve(ext, nb, per, opts):
    print(f"[phi ghosts] {ext} {nb} {per} {opts}", flush=True)
    P = lib()
    rng = np.random.default_rng(4)
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    w, h = ext[0] // nb[0], ext[1] // nb[1]
    boxes = [((i * w, j * h, 0), ((i + 1) * w - 1, (j + 1) * h - 1, ext[2] - 1))
             for j in range(nb[1]) for i in range(nb[0])]
    f = rng.uniform(-1.0, 1.0, ext)
    f -= f.mean()
    s = P.MLMG(boxes, dom, per, 0.0 if all(per) else 0.5, 1.0, opts=dict(tune=0, **opts))
    phi = s.cell_mf(1, fill=7.0)
    s.solve(phi, P.MultiFab.from_numpy(boxes, W.scatter_cells(f, boxes), 0), 1e-9,
            raise_on_fail=False)
    torch.cuda.synchronize()
    got = phi.to_numpy()
    s.close()
    G = W.gather_cells(phi.valid_numpy(), boxes, ext, ng=0)
    for b, (lo, hi) in enumerate(boxes):
        for d in range(3):
            for side, at in ((0, lo[d] - 1), (-1, hi[d] + 1)):
                if not per[d] and not 0 <= at < ext[d]:
                    continue
                sl = [slice(1, -1)] * 3
                sl[d] = side
                src = [slice(l, u + 1) for l, u in zip(lo, hi)]
                src[d] = at % ext[d]
                assert np.array_equal(got[b][tuple(sl)], G[tuple(src)]), (b, d, side)
