"""GPU parity of the V-cycle on the split-colour layout where its kernels
change form: rows whose pairs do not fill the last wide load, periodic rows that
rule wide loads out, rows shorter than a cache line, levels smoothed in blocks, domains with low corners
away from zero, cell coefficients, the tail in LDS and in memory, and levels
large enough for wide loads and for whole sweeps per pass.  Two V-cycles against the oracle, cell by cell."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import lib

CASES = [
    # extents, low corner, periodic, boxes along x, a, opts
    ((24, 16, 40), (0, 0, 0), (False, False, False), 1, False, {}),
    ((20, 12, 12), (8, -8, 16), (True, False, True), 1, True, {}),
    ((48, 24, 16), (-16, 32, 0), (False, True, False), 2, True, {}),
    ((64, 32, 32), (0, 0, 0), (True, True, True), 2, False, dict(coarse_tail=4096)),
    ((64, 32, 32), (0, 0, 0), (False, False, True), 2, True, dict(coarse_tail=8192)),
    # two sweeps to a launch: FP64 blocks of 4 pairs with ragged ends above, FP32
    # blocks of 8 pairs
    ((56, 52, 60), (0, 0, 0), (False, False, True), 1, True, {}),
    ((64, 64, 48), (0, 0, 0), (True, False, False), 2, False, dict(use_graph=0)),
    # two FP64 pairs per lane: rows that fill, leave a remainder, wrap
    ((132, 96, 96), (0, 0, 0), (False, False, False), 1, True, {}),
    ((136, 96, 88), (0, 0, 0), (True, False, True), 1, False, {}),
    ((132, 96, 96), (0, 0, 0), (True, False, False), 1, False, {}),
    # four FP32 pairs per lane
    ((132, 128, 128), (0, 0, 0), (False, False, False), 1, False, {}),
    ((136, 128, 128), (0, 0, 0), (True, False, False), 1, True, {}),
    # whole sweeps per pass (levels above 256 MiB): two tiles along x with a
    # remainder, ragged rows and planes; FP64 alone at 7.5 M cells
    ((260, 200, 148), (0, 0, 0), (False, True, False), 1, False, dict(only64=1)),
    ((132, 244, 236), (0, 0, 0), (True, False, True), 1, True, dict(only64=1, nu1=1, nu2=1)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("krylov", [0, 1])
@pytest.mark.parametrize("ext,lo,per,nx,with_a,opts", CASES)
def test_two_cycles_vs_oracle(ext, lo, per, nx, with_a, opts, krylov):
    opts = dict(opts)
    only64 = opts.pop("only64", 0)
    nu = dict(nu1=opts.get("nu1", 2), nu2=opts.get("nu2", 2))
    print(f"[flat] {ext} at {lo} periodic {per} krylov {krylov} {opts}", flush=True)
    P = lib()
    rng = np.random.default_rng(3)
    dom = (lo, tuple(a + n - 1 for a, n in zip(lo, ext)))
    w = ext[0] // nx
    boxes = [((lo[0] + i * w, lo[1], lo[2]), (lo[0] + (i + 1) * w - 1, dom[1][1], dom[1][2]))
             for i in range(nx)]
    alpha = 0.0 if all(per) and not with_a else 0.7
    plen = tuple(n / max(ext) for n in ext)
    bf = W.harmonic_faces(np.exp(0.7 * rng.standard_normal(ext)), per)
    f = rng.uniform(-1.0, 1.0, ext)
    if alpha == 0.0:
        f -= f.mean()
    guess = rng.uniform(-1.0, 1.0, ext) * 1e-3
    a = rng.uniform(0.5, 2.0, ext) if with_a else None
    fb = W.scatter_cells(f, boxes, dlo=lo)
    b = [W.scatter_faces(bf[d], boxes, d, dlo=lo) for d in range(3)]
    ab = W.scatter_cells(a, boxes, dlo=lo) if with_a else None

    def mf(v, **kw):
        return P.MultiFab.from_numpy(boxes, v, **kw)

    bmf = [mf(b[d], ixtype=tuple(int(e == d) for e in range(3))) for d in range(3)]
    lev = O.make_level(boxes, dom, per, alpha, 1.0, ab, b, prob_len=plen)
    # few bottom iterations, the same on both sides: large bottoms stay cheap
    oopts = O.Opts(max_iter=2, bottom_tol=0.0, bottom_max_iter=6, symmetric=bool(krylov),
                   **nu)
    ophi = W.scatter_cells(guess, boxes, ng=1, dlo=lo)
    if krylov:
        oinfo = O.pcg_solve(lev, ophi, fb, 1e-30, opts=oopts)
    else:
        oinfo = O.solve(lev, ophi, fb, 1e-30, opts=oopts)
    ref = W.gather_cells(ophi, boxes, ext, ng=1, dlo=lo)
    for precision in (0,) if only64 else (0, 1):
        s = P.MLMG(boxes, dom, per, alpha, 1.0, a=mf(ab) if with_a else None, b=bmf,
                   opts=dict(tune=0, max_iter=2, bottom_rel_tol=0.0, bottom_max_iter=6,
                             precision=precision, krylov=krylov, **opts), prob_hi=plen)
        phi = mf(W.scatter_cells(guess, boxes, ng=1, dlo=lo), ngrow=1)
        info = s.solve(phi, mf(fb), 1e-30, raise_on_fail=False, history=True)
        torch.cuda.synchronize()
        got = W.gather_cells(phi.valid_numpy(), boxes, ext, ng=0, dlo=lo)
        err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
        # FP64: rounding of two cycles; FP32 V-cycles: their rounding (6e-8 each
        # operation, some hundred operations deep)
        assert err <= (1e-11 if precision == 0 else 2e-5), (precision, err)
        h = np.array(info["history"]) / oinfo["history"][0]
        o = np.array(oinfo["history"]) / oinfo["history"][0]
        assert info["iters"] == 2
        assert np.all(np.abs(h - o) <= (1e-9 if precision == 0 else 1e-4)), (h, o)
        s.close()
