"""A solve that ends in a non-finite value leaves its handle as good as a new
one: the same handle then gives the bits of a handle that never failed, on the
same right-hand side and after its coefficients have been replaced.  Grids whose
rows carry padding, with walls, with periodic directions and singular; a bottom
with coarsenings of its own."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import lib

GRIDS = [
    # extents, periodic, alpha, opts
    ((36, 24, 20), (False, False, False), 0.7, {}),
    ((40, 24, 24), (True, False, True), 0.7, {}),
    ((32, 32, 24), (True, True, True), 0.0, {}),
    ((72, 72, 72), (False, False, False), 0.7, dict(min_bottom_edge=18)),
]

FAILS = [
    # precision, krylov, scale of b, scale of the right-hand side
    (0, 1, 1.0, 1e160),  # r.z overflows
    (1, 1, 1.0, 1e-60),  # r rounds to 0 in FP32: 0 / 0
    (1, 1, 1e39, 1.0),   # FP32 coefficients overflow
    (1, 0, 1e39, 1.0),
    (0, 0, 1e306, 1.0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("precision,krylov,bscale,fscale", FAILS)
@pytest.mark.parametrize("ext,per,alpha,opts", GRIDS)
def test_solve_after_a_failed_one(ext, per, alpha, opts, precision, krylov, bscale, fscale):
    print(f"[recover] {ext} {per} precision {precision} krylov {krylov} b x {bscale} f x {fscale}",
          flush=True)
    P = lib()
    rng = np.random.default_rng(5)
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes = [dom]
    bf = W.harmonic_faces(np.exp(0.5 * rng.standard_normal(ext)), per)
    f = rng.uniform(-1.0, 1.0, ext)
    if alpha == 0.0:
        f -= f.mean()

    def faces(scale):
        return [P.MultiFab.from_numpy(boxes, W.scatter_faces(scale * bf[d], boxes, d), 0,
                                      ixtype=tuple(int(e == d) for e in range(3)))
                for d in range(3)]

    def rhs(scale):
        return P.MultiFab.from_numpy(boxes, W.scatter_cells(scale * f, boxes), 0)

    def solver():
        return P.MLMG(boxes, dom, per, alpha, 1.0, b=faces(1.0),
                      opts=dict(tune=0, precision=precision, krylov=krylov, **opts))

    def solution(s):
        phi = s.cell_mf(1, fill=0.0)
        info = s.solve(phi, rhs(1.0), 1e-9, history=True)
        torch.cuda.synchronize()
        assert info["converged"]
        return phi.valid_numpy()[0], info["history"]

    fresh = solver()
    ref, hist = solution(fresh)
    fresh.close()
    s = solver()
    if bscale != 1.0:
        s.set_coefficients(b=faces(bscale))
    bad = s.cell_mf(1, fill=0.0)
    info = s.solve(bad, rhs(fscale), 1e-9, raise_on_fail=False)
    assert info["status"] == P._lib.MG_ERR_NAN and not info["converged"]
    s.set_coefficients(b=faces(1.0))
    for _ in range(2):
        got, h = solution(s)
        assert np.array_equal(got, ref)
        assert h == hist
    s.close()
