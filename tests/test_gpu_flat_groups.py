"""Grids whose x-rows are no whole number of value groups (the groups then straddle rows), and
the table of distinct block-Jacobi inverses of the matrix-free operator: the operators, the
preconditioner and a stage solve against the FP64 oracle at the sizes where a row end, a plane
edge, the partial last group or the short last block can go wrong."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import krylov, operators
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi

U = {A.FP64: 2.0 ** -53, A.FP32: 2.0 ** -24, A.FP16: 2.0 ** -11}
NP = {A.FP64: np.float64, A.FP32: np.float32, A.FP16: np.float16}
# rows shorter than, as long as and one longer than a group (4 or 8 values) and a block; one and
# two rows or planes; last groups and last blocks of every length
SHAPES = [(1, 5, 3), (2, 3, 7), (3, 4, 5), (5, 1, 9), (5, 2, 2), (7, 3, 3), (8, 3, 5), (9, 1, 1), (9, 2, 3),
          (9, 5, 4), (10, 3, 3), (11, 6, 1), (12, 3, 5), (13, 4, 6), (15, 3, 3), (17, 9, 5), (20, 5, 3),
          (33, 4, 3)]
OPS = [(W.DIRICHLET, W.HEAT, 1.5, (0.0, 0.0, 0.0)), (W.PERIODIC, W.ADVDIFF, 0.3, (-1.0, 0.5, -0.25))]


@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("shape", SHAPES)
def test_operators_and_preconditioner(shape, op, storage):
    bc, kind, diff, b = op
    log_case('flat_apply', shape=shape, bc=bc, storage=storage)
    K = operators.operator(shape, bc, kind, diff, b)
    N = int(np.prod(shape))
    rng = np.random.default_rng(5)
    for block in (8, 4, 2, 1):
        prec = M.precisions(storage, 'gmres', block=block)
        st = M.Stepper(shape, bc, kind, diff, b, A.FMT_STENCIL, 'SDIRK3', prec, 2e-3)
        sd = st.prec.storage
        u_c = U[A.FP64] if sd == A.FP64 else U[A.FP32]
        tiny = {A.FP64: 0.0, A.FP32: 2.0 ** -150, A.FP16: 2.0 ** -25}[sd]
        Mx = operators.stage_matrix(K, st.dt * st.tab.a_lo[0])
        x = rng.standard_normal(N).astype(NP[sd])
        xf = x.astype(np.float64)
        dev = torch.from_numpy(x).cuda()
        z = st.apply(A.APPLY_BJ_LP, dev, 0).cpu().numpy().astype(np.float64)
        inv = krylov.block_jacobi_inverses(Mx, block)
        ref = krylov.block_jacobi_apply(inv, xf, block)
        absd = krylov.block_jacobi_apply([np.abs(d) for d in inv], np.abs(xf), block)
        bound = 2 * U[sd] * np.abs(ref) + (16 * u_c + 2 * U[sd]) * absd + tiny
        assert np.all(np.abs(z - ref) <= bound + 1e-300), block
        if block == 8:
            y = st.apply(A.APPLY_M_LP, dev, 0).cpu().numpy().astype(np.float64)
            ref = Mx @ xf
            bound = 2 * U[sd] * np.abs(ref) + 18 * u_c * (abs(Mx) @ np.abs(xf)) + tiny
            assert np.all(np.abs(y - ref) <= bound + 1e-300)
            k = st.apply(A.APPLY_K64, torch.from_numpy(xf).cuda()).cpu().numpy()
            assert np.all(np.abs(k - K @ xf) <= 16 * U[A.FP64] * (abs(K) @ np.abs(xf)) + 1e-300)
        st.close()


@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("krylov_name", ['cg', 'gmres'])
@pytest.mark.parametrize("shape", [(5, 7, 3), (9, 5, 4), (13, 6, 5), (17, 9, 7), (37, 11, 6)])
def test_stage_solve_on_misaligned_caller_vectors(shape, krylov_name, storage):
    # the caller's vectors start 8 bytes past a 16-byte boundary and end at their last value; the
    # values around the result are not written
    bc, kind, diff, b = OPS[0] if krylov_name == 'cg' else OPS[1]
    log_case('flat_solve', shape=shape, krylov=krylov_name, storage=storage)
    st = M.Stepper(shape, bc, kind, diff, b, A.FMT_STENCIL, 'SDIRK3', M.precisions(storage, krylov_name), 2e-3)
    N = st.N
    rng = np.random.default_rng(6)
    rhs = torch.zeros(N + 2, dtype=torch.float64, device='cuda')
    rhs[1:N + 1] = torch.from_numpy(rng.standard_normal(N)).cuda()
    x = torch.full((N + 2,), 7.0, dtype=torch.float64, device='cuda')
    rc, info = A.mprk_solve(st.h, 0, rhs[1:].data_ptr(), x[1:].data_ptr())
    assert rc == A.OK and info['converged'] == 1, info
    Mx = operators.stage_matrix(operators.operator(shape, bc, kind, diff, b), st.dt * st.tab.a_lo[0])
    import scipy.sparse.linalg as spla
    ref = spla.spsolve(Mx.tocsc(), rhs[1:N + 1].cpu().numpy())
    got = x.cpu().numpy()
    st.close()
    assert got[0] == 7.0 and got[-1] == 7.0
    # the residual test: ||M (x - ref)|| <= outer_tol ||rhs|| and ||M^-1|| <= 1
    tol = st.prec.outer_tol * np.linalg.norm(rhs.cpu().numpy())
    assert np.linalg.norm(got[1:N + 1] - ref) <= 1.01 * tol + 1e-13 * np.linalg.norm(ref)


@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("shape", [(66, 67, 65), (90, 66, 66), (74, 73, 73), (89, 81, 73), (7, 9, 5)])
def test_cg_steps_on_both_sides_of_the_one_value_line(shape, storage):
    # CG with one value per thread and with groups of values: past the one-launch stages, on both
    # sides of 3 2^17 (FP64, FP32) and 2^19 (FP16) unknowns; the stage system's residual test
    bc, kind, diff, b = OPS[0]
    log_case('flat_cg_line', shape=shape, storage=storage)
    st = M.Stepper(shape, bc, kind, diff, b, A.FMT_STENCIL, 'SDIRK3', M.precisions(storage, 'cg'), 2e-3)
    rhs = np.random.default_rng(8).standard_normal(st.N)
    x, info = st.solve(0, torch.from_numpy(rhs).cuda())
    Mx = operators.stage_matrix(operators.operator(shape, bc, kind, diff, b), st.dt * st.tab.a_lo[0])
    got = x.cpu().numpy()
    lim = st.prec.outer_tol * np.linalg.norm(rhs) + 32 * U[A.FP64] * np.linalg.norm(abs(Mx) @ np.abs(got))
    st.close()
    assert info['converged'] == 1, info
    assert np.linalg.norm(rhs - Mx @ got) <= lim
