"""GMRES and its operators on odd grids on both sides of the sizes where a thread takes one value and
where it takes a group of four or eight, rows shorter than a group among them, against the FP64
oracle."""
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
# FP64 and FP32: up to 2^14 unknowns one value, up to 2^16 groups of four (rows of 3, 5, 7 and 9 among
# them), one value again up to 2^18 (FP32) and 5 2^16 (FP64); FP16 groups of eight past 2^19
SHAPES = [((27, 25, 24), ''), ((27, 25, 25), ''), ((3, 73, 77), ''), ((5, 61, 60), ''), ((7, 49, 50), ''),
          ((9, 43, 44), ''), ((41, 40, 39), ''), ((41, 40, 41), ''), ((63, 65, 64), 'fp32'), ((65, 65, 65), 'fp32'),
          ((69, 69, 68), 'fp64'), ((69, 69, 69), 'fp64'), ((81, 81, 79), 'fp16'), ((81, 81, 81), 'fp16'),
          ((9, 241, 243), 'fp16'), ((5, 331, 331), 'fp16')]
CASES = [(s, st) for s, only in SHAPES for st in ('fp64', 'fp32', 'fp16') if only in ('', st)]


@pytest.mark.parametrize("shape,storage", CASES)
def test_operators_and_a_stage_solve(shape, storage):
    log_case('flat_lines', shape=shape, storage=storage)
    bc, kind, diff, b = W.PERIODIC, W.ADVDIFF, 0.3, (-1.0, 0.5, -0.25)
    K = operators.operator(shape, bc, kind, diff, b)
    N = int(np.prod(shape))
    rng = np.random.default_rng(5)
    for block in (8, 2):
        st = M.Stepper(shape, bc, kind, diff, b, A.FMT_STENCIL, 'SDIRK3', M.precisions(storage, 'gmres', block=block), 2e-4)
        sd = st.prec.storage
        u_c = U[A.FP64] if sd == A.FP64 else U[A.FP32]
        tiny = {A.FP64: 0.0, A.FP32: 2.0 ** -150, A.FP16: 2.0 ** -25}[sd]  # half the smallest spacing
        Mx = operators.stage_matrix(K, st.dt * st.tab.a_lo[0])
        x = rng.standard_normal(N).astype(NP[sd])
        xf = x.astype(np.float64)
        dev = torch.from_numpy(x).cuda()
        z = st.apply(A.APPLY_BJ_LP, dev, 0).cpu().numpy().astype(np.float64)
        inv = krylov.block_jacobi_inverses(Mx, block)
        ref = krylov.block_jacobi_apply(inv, xf, block)
        absd = krylov.block_jacobi_apply([np.abs(d) for d in inv], np.abs(xf), block)
        ones = krylov.block_jacobi_apply([np.ones_like(d) for d in inv], np.abs(xf), block)
        bound = 2 * U[sd] * np.abs(ref) + (16 * u_c + 2 * U[sd]) * absd + tiny * (1.0 + ones)  # (stored entries too)
        assert np.all(np.abs(z - ref) <= bound + 1e-300)
        y = st.apply(A.APPLY_M_LP, dev, 0).cpu().numpy().astype(np.float64)
        ref = Mx @ xf
        assert np.all(np.abs(y - ref) <= 2 * U[sd] * np.abs(ref) + 18 * u_c * (abs(Mx) @ np.abs(xf)) + tiny + 1e-300)
        rhs = rng.standard_normal(N)
        got, info = st.solve(0, torch.from_numpy(rhs).cuda())
        got = got.cpu().numpy()
        lim = st.prec.outer_tol * np.linalg.norm(rhs) + 32 * U[A.FP64] * np.linalg.norm(abs(Mx) @ np.abs(got))
        st.close()
        assert info['converged'] == 1 and np.linalg.norm(rhs - Mx @ got) <= lim, info


@pytest.mark.parametrize("krylov_name", ['cg', 'gmres'])
@pytest.mark.parametrize("over", [dict(precond='bj', block=8), dict(precond='bj', block=2), dict(precond='none')])
@pytest.mark.parametrize("fmt", [A.FMT_STENCIL, A.FMT_CSR])
def test_fp64_arithmetic_over_fp16_storage(krylov_name, over, fmt):
    # past 2^19 unknowns, where FP16 takes groups of eight elsewhere; the stage system's residual test
    shape = (83, 81, 79)
    log_case('flat_lines_cb16', krylov=krylov_name, fmt=fmt, **over)
    bc, kind, diff, b = ((W.DIRICHLET, W.HEAT, 1.5, (0.0, 0.0, 0.0)) if krylov_name == 'cg'
                         else (W.PERIODIC, W.ADVDIFF, 0.3, (-1.0, 0.5, -0.25)))
    st = M.Stepper(shape, bc, kind, diff, b, fmt, 'SDIRK3',
                   M.precisions('fp16', krylov_name, compute=A.FP64, **over), 2e-4)
    rhs = np.random.default_rng(8).standard_normal(st.N)
    x, info = st.solve(0, torch.from_numpy(rhs).cuda())
    Mx = operators.stage_matrix(operators.operator(shape, bc, kind, diff, b), st.dt * st.tab.a_lo[0])
    got = x.cpu().numpy()
    lim = st.prec.outer_tol * np.linalg.norm(rhs) + 32 * U[A.FP64] * np.linalg.norm(abs(Mx) @ np.abs(got))
    st.close()
    assert info['converged'] == 1 and np.linalg.norm(rhs - Mx @ got) <= lim, info


@pytest.mark.parametrize("shape", [(91, 89, 89), (91, 91, 89)])
@pytest.mark.parametrize("krylov_name,over", [('cg', {}), ('cg', {'bj_adapt_tol': 1e-5}),
                                              ('gmres', {'bj_adapt_tol': 1e-5})])
def test_fp16_lines_of_cg_and_adaptive_inverses(shape, krylov_name, over):
    # 11 2^16 unknowns: one value up to there, groups of eight past it; the residual test
    log_case('flat_lines_fp16', shape=shape, krylov=krylov_name, **over)
    bc, kind, diff, b = ((W.DIRICHLET, W.HEAT, 1.5, (0.0, 0.0, 0.0)) if krylov_name == 'cg'
                         else (W.PERIODIC, W.ADVDIFF, 0.3, (-1.0, 0.5, -0.25)))
    st = M.Stepper(shape, bc, kind, diff, b, A.FMT_STENCIL, 'SDIRK3', M.precisions('fp16', krylov_name, **over), 2e-4)
    rhs = np.random.default_rng(8).standard_normal(st.N)
    x, info = st.solve(0, torch.from_numpy(rhs).cuda())
    Mx = operators.stage_matrix(operators.operator(shape, bc, kind, diff, b), st.dt * st.tab.a_lo[0])
    got = x.cpu().numpy()
    lim = st.prec.outer_tol * np.linalg.norm(rhs) + 32 * U[A.FP64] * np.linalg.norm(abs(Mx) @ np.abs(got))
    st.close()
    assert info['converged'] == 1 and np.linalg.norm(rhs - Mx @ got) <= lim, info
