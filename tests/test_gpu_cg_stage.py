"""CG stages run as one launch: grids around a workgroup's part (1024 unknowns) and its halo, the
largest such grids, and the first ones past them, against the residual test in FP64; handles on
several threads, whose launches wait for workgroups of their own."""
import threading

import numpy as np
import pytest
import torch

import workloads as W
from oracle import operators
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi

# one unknown, one group, less than a group more; 1023 .. 1026; parts that end inside a row; a slab
# that is the whole grid and one that is not; 127 and 128 parts; past the last part, past the slab
SHAPES = [(1, 1, 1), (4, 1, 1), (7, 1, 1), (11, 31, 3), (16, 16, 4), (25, 41, 1), (19, 27, 2), (9, 12, 19),
          (13, 13, 13), (37, 5, 12), (23, 23, 23), (40, 40, 41), (50, 51, 51), (64, 32, 64), (64, 33, 64),
          (64, 50, 20)]


def _solve(shape, bc, storage, block, seed=3):
    st = M.Stepper(shape, bc, W.HEAT, 1.5, (0.0, 0.0, 0.0), A.FMT_STENCIL, 'SDIRK3',
                   M.precisions(storage, 'cg', precond='bj' if block else 'none', block=block or 8), 2e-3)
    rhs = np.random.default_rng(seed).standard_normal(st.N)
    x, info = st.solve(0, torch.from_numpy(rhs).cuda())
    Mx = operators.stage_matrix(operators.operator(shape, bc, W.HEAT, 1.5, (0.0, 0.0, 0.0)),
                                st.dt * st.tab.a_lo[0])
    got = x.cpu().numpy()
    res = np.linalg.norm(rhs - Mx @ got)
    # the device's own residual test, and rounding: of 9 FP64 operations a row on both sides
    lim = st.prec.outer_tol * np.linalg.norm(rhs) + 32 * 2.0 ** -53 * np.linalg.norm(abs(Mx) @ np.abs(got))
    st.close()
    return info, res, lim


@pytest.mark.parametrize("storage", ['fp64', 'fp32'])
@pytest.mark.parametrize("bc", [W.DIRICHLET, W.PERIODIC])
@pytest.mark.parametrize("shape", SHAPES)
def test_stage_meets_its_residual_test(shape, bc, storage):
    for block in (8, 2, 0):
        log_case('cg_stage', shape=shape, bc=bc, storage=storage, block=block)
        info, res, lim = _solve(shape, bc, storage, block)
        assert info['converged'] == 1, info
        assert res <= lim, (block, res, lim)


def test_handles_on_several_threads():
    log_case('cg_stage_threads')
    out = {}

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            st = M.Stepper((40, 40, 60), W.DIRICHLET, W.HEAT, 1.0, (0.0, 0.0, 0.0), A.FMT_STENCIL, 'SDIRK3',
                           M.precisions('fp32', 'cg'), 2e-3)
            u = torch.from_numpy(np.random.default_rng(1).standard_normal(st.N)).cuda()
            st.set_u(u)
            for _ in range(4):
                st.step(2)
            out[k] = st.get_u()
            st.close()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert len(out) == 4
    for k in range(1, 4):  # fixed-order sums: the same bits whatever else runs
        assert np.array_equal(out[0], out[k])
