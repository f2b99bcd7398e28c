"""Boxes that hold different coefficients for the face they share (or for the two
ends of a periodic direction): every box's cells use their own, as the operator
and the oracle do.  The same handle then goes back to coefficients that agree
and gives the bits of a handle that never had others."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import lib

CASES = [
    # extents, boxes along x and z, periodic, direction of the differing faces, a, opts
    ((32, 16, 32), (2, 2), (False, False, False), 0, False, {}),
    ((32, 16, 32), (2, 2), (False, True, False), 2, True, dict(use_graph=0)),
    ((32, 32, 16), (2, 1), (True, False, False), 0, False, {}),
    ((16, 32, 16), (1, 1), (False, True, False), 1, False, {}),  # one box, periodic ends
    ((32, 16, 32), (2, 2), (False, False, True), 2, False, dict(precision=1)),
    ((64, 32, 32), (2, 1), (False, False, False), 0, False, dict(precision=1)),
]


def problem(ext, nb, per, d, with_a):
    rng = np.random.default_rng(8)
    w, t = ext[0] // nb[0], ext[2] // nb[1]
    boxes = [((i * w, 0, k * t), ((i + 1) * w - 1, ext[1] - 1, (k + 1) * t - 1))
             for k in range(nb[1]) for i in range(nb[0])]
    bf = W.harmonic_faces(np.exp(0.5 * rng.standard_normal(ext)), per)
    good = [W.scatter_faces(bf[e], boxes, e) for e in range(3)]
    own = [[x.copy() for x in g] for g in good]
    for x in own[d]:  # every box's last face along d, a fifth larger
        sl = [slice(None)] * 3
        sl[d] = -1
        x[tuple(sl)] *= 1.2
    f = W.scatter_cells(rng.uniform(-1.0, 1.0, ext), boxes)
    a = W.scatter_cells(rng.uniform(0.5, 2.0, ext), boxes) if with_a else None
    return boxes, good, own, f, a


@pytest.mark.gpu
@pytest.mark.parametrize("ext,nb,per,d,with_a,opts", CASES)
def test_each_boxes_own_faces(ext, nb, per, d, with_a, opts):
    print(f"[shared faces] {ext} {nb} {per} along {d} {opts}", flush=True)
    P = lib()
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes, good, own, f, a = problem(ext, nb, per, d, with_a)
    plen = tuple(n / max(ext) for n in ext)
    f32 = opts.get("precision", 0) == 1

    def faces(v):
        return [P.MultiFab.from_numpy(boxes, v[e], 0, ixtype=tuple(int(e == q) for q in range(3)))
                for e in range(3)]

    amf = P.MultiFab.from_numpy(boxes, a, 0) if with_a else None
    rhs = P.MultiFab.from_numpy(boxes, f, 0)

    def solver(v):
        return P.MLMG(boxes, dom, per, 0.8, 1.0, a=amf, b=faces(v),
                      opts=dict(tune=0, bottom_rel_tol=1e-12, **opts), prob_hi=plen)

    def solution(s):
        phi = s.cell_mf(1, fill=0.0)
        info = s.solve(phi, rhs, 1e-10, history=True)
        torch.cuda.synchronize()
        return W.gather_cells(phi.valid_numpy(), boxes, ext, ng=0), info

    lev = O.make_level(boxes, dom, per, 0.8, 1.0, a, own, prob_len=plen)
    ophi = O.new_cell_data(lev)
    o = O.solve(lev, ophi, f, 1e-10, opts=O.Opts(bottom_tol=1e-12))
    ref = W.gather_cells(ophi, boxes, ext, ng=1)
    fresh = solver(good)
    gref, ginfo = solution(fresh)
    fresh.close()
    s = solver(own)
    for turn in range(2):
        got, info = solution(s)
        assert info["converged"]
        # residual histories to rounding (FP32 V-cycles: to theirs), and the
        # solution within twice the residual tolerance over alpha * min a
        if not f32:
            assert info["iters"] == o["iters"]
            for x, y in zip(info["history"], o["history"]):
                assert abs(x - y) <= 1e-6 * y + 1e-12 * o["normf"]
        bound = 2e-10 * max(np.max(np.abs(x)) for x in f) / (0.8 * (0.5 if with_a else 1.0))
        assert np.max(np.abs(got - ref)) <= bound
        s.set_coefficients(a=amf, b=faces(good))
        for _ in range(2):
            x, xinfo = solution(s)
            assert np.array_equal(x, gref)
            assert xinfo["history"] == ginfo["history"]
        s.set_coefficients(a=amf, b=faces(own))
    s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("ulps,boxes_used", [(1, False), (8, True)])
def test_rounding_is_no_difference(ulps, boxes_used):
    """Boxes whose shared faces differ by rounding keep the fast storage, where
    nothing is exchanged; the solution is the oracle's either way."""
    print(f"[shared faces] {ulps} units in the last place", flush=True)
    P = lib()
    ext, per, d = (32, 16, 32), (False, False, True), 0
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes, good, _, f, _ = problem(ext, (2, 2), per, d, False)
    own = [[x.copy() for x in g] for g in good]
    for x in own[d]:
        x[-1] *= 1.0 + ulps * 2.0 ** -52
    lev = O.make_level(boxes, dom, per, 0.8, 1.0, None, own)
    ophi = O.new_cell_data(lev)
    O.solve(lev, ophi, f, 1e-10, opts=O.Opts(bottom_tol=1e-12))
    s = P.MLMG(boxes, dom, per, 0.8, 1.0,
               b=[P.MultiFab.from_numpy(boxes, own[e], 0,
                                        ixtype=tuple(int(e == q) for q in range(3)))
                  for e in range(3)],
               opts=dict(tune=0, bottom_rel_tol=1e-12, ghost_write=0))
    phi = s.cell_mf(1, fill=0.0)
    s.profile(True)
    s.solve(phi, P.MultiFab.from_numpy(boxes, f, 0), 1e-10)
    torch.cuda.synchronize()
    assert (s.kernel_stats(P._lib.FAM_EXCHANGE)[1] > 0) == boxes_used
    got = W.gather_cells(phi.valid_numpy(), boxes, ext, ng=0)
    ref = W.gather_cells(ophi, boxes, ext, ng=1)
    assert np.max(np.abs(got - ref)) <= 2e-10 * max(np.max(np.abs(x)) for x in f) / 0.8
    s.close()
