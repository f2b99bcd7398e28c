"""The solver with its levels kept as boxes: the tests of the solve, of its
options that change nothing but the launches (bit for bit) and of MG-PCG again,
on handles in the least workspace, which holds no other storage.  With the
default workspace those tests run on levels stored as one grid, where the
options marked [boxes] in amrmg.h change nothing."""

import functools

import pytest
import torch

import test_gpu_pcg as K
import test_gpu_solve as S
import workloads as W
from gpu_util import gpu_solver, lib

AGAIN = [
    S.test_lognormal_dirichlet_64,
    S.test_aggregated_hierarchy,
    S.test_mixed_bc_with_cell_coefficient,
    S.test_one_cycle_elementwise,
    S.test_uneven_boxes,
    S.test_float32_refinement_vs_fp64_oracle,
    S.test_tile_shapes_and_graph_bitwise_identical,
    S.test_tuned_shapes_bitwise_identical,
    S.test_class_tile_shapes_bitwise_identical,
    S.test_fused_sweeps_bitwise_equal_half_sweeps,
    S.test_ghost_write_through_bitwise_equal_exchanges,
    S.test_stop_fold_bitwise_equal_plain_loop,
    S.test_quad_smoother_bitwise_fp32_256,
    S.test_quad_smoother_bitwise_fp32_uneven_boxes,
    S.test_coarse_tail_bitwise_equal_launches,
    S.test_c1_bench_configuration,
    K.test_pcg_matches_oracle,
    K.test_pcg_and_vcycles_reach_the_same_solution,
    K.test_pcg_float32_preconditioner_vs_oracle,
]


def _again(test):
    @functools.wraps(test)  # with its parameters and marks
    def run(*args, **kw):
        return test(*args, **kw)
    return run


for _t in AGAIN:
    globals()[_t.__name__.replace("test_", "test_boxes_", 1)] = _again(_t)


@pytest.fixture(autouse=True)
def least_workspace(monkeypatch):
    P = lib()
    full = P.MLMG

    def least(*args, **kw):
        s = full(*args, **kw, least_workspace=True)
        room = P.workspace_bytes(s.boxes, s.domain, s.periodic, s.opts, s.has_a)
        # no room for a grid per level (with nu2 = 0 there is never one)
        assert s.opts.nu2 == 0 or s.workspace.numel() < 0.85 * room
        return s

    monkeypatch.setattr(P, "MLMG", least)
    yield full


@pytest.mark.gpu
def test_which_storage_a_handle_solves_on(least_workspace, monkeypatch):
    """With an exchange before every half-sweep, solves over boxes exchange and
    the others have nothing to exchange."""
    print("[boxes] storage by workspace", flush=True)
    P = lib()
    cfg = W.config_lognormal(32, 16)
    boxes = cfg["boxes"]
    rhs = P.MultiFab.from_numpy(boxes, W.scatter_cells(cfg["rhs"], boxes), 0)
    seen = []
    for full in (False, True):
        if full:
            monkeypatch.setattr(P, "MLMG", least_workspace)
        s = gpu_solver(cfg, opts=dict(tune=0, ghost_write=0, max_iter=2))
        s.profile(True)
        s.solve(s.cell_mf(1, fill=0.0), rhs, 1e-10, raise_on_fail=False)
        torch.cuda.synchronize()
        seen.append(s.kernel_stats(P._lib.FAM_EXCHANGE)[1])
        s.close()
    assert seen[0] > 0 and seen[1] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_mg_solve_on_a_composite_handle(precision):
    """mg_solve on a composite handle solves its coarse level alone, over boxes:
    the bits of a handle without the fine level, before and after a composite
    solve."""
    import ctypes as C
    print(f"[boxes] mg_solve on a composite handle precision {precision}", flush=True)
    P = lib()
    cfg = W.config_lognormal(32, 16)
    boxes, opts = cfg["boxes"], dict(tune=0, precision=precision, stop_fold=0)
    rhs = P.MultiFab.from_numpy(boxes, W.scatter_cells(cfg["rhs"], boxes), 0)
    one = P.MLMG(boxes, W.domain_box(32), (False,) * 3, cfg["alpha"], cfg["beta"], opts=opts)
    ref = one.cell_mf(1, fill=0.0)
    one.solve(ref, rhs, 1e-10)
    fine = [((8, 8, 8), (23, 23, 23))]
    s = P.CompositeMLMG(boxes, fine, W.domain_box(32), cfg["alpha"], cfg["beta"], opts=opts)
    for _ in range(2):
        phi = P.MultiFab(boxes, 1, fill=0.0)
        pm, rm, info = phi.c_struct(), rhs.c_struct(), P._lib.MgInfo()
        P._lib.check(P._lib.lib.mg_solve(s.handle, C.byref(pm), C.byref(rm), 1e-10, 0.0,
                                         C.byref(info), None), "mg_solve")
        torch.cuda.synchronize()
        assert info.converged
        for x, y in zip(phi.valid_numpy(), ref.valid_numpy()):
            assert (x == y).all()
        pc, pf = P.MultiFab(boxes, 1, fill=0.0), P.MultiFab(fine, 1, fill=0.0)
        assert s.solve(pc, pf, rhs, P.MultiFab(fine, 0, fill=1.0), 1e-8)["converged"]
    one.close()
    s.close()
