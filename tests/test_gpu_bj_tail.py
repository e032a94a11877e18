"""Block-Jacobi on grids whose last group of values reaches past the last block: stored inverses and
their indexes are read inside what the bind wrote, whatever the workspace held before."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operators
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi


class Filled:
    """A handle on a workspace filled with 0xFF bytes (NaN in every type, -1 as an index)."""

    def __init__(self, shape, storage, krylov, fmt, **over):
        self.shape, self.N = shape, int(np.prod(shape))
        self.bc = W.DIRICHLET if krylov == 'cg' else W.PERIODIC
        self.kind, self.diff, self.vel = ((W.HEAT, 1.0, (0.0, 0.0, 0.0)) if krylov == 'cg'
                                          else (W.ADVDIFF, 1e-2, (1.0, 0.5, 0.25)))
        self.prec, self.dt = M.precisions(storage, krylov, **over), 5e-4 if krylov == 'cg' else 2e-3
        self.tab = M.tableau('SDIRK3')
        op = A.mprk_operator(self.kind, fmt, self.diff, (A.C.c_double * 3)(*self.vel))
        self.h = A.mprk_create(A.mprk_grid(*shape, self.bc), op, self.tab, self.prec, self.dt,
                               torch.cuda.current_stream().cuda_stream)
        n = A.mprk_workspace_bytes(self.h)
        self.u = torch.zeros(self.N, dtype=torch.float64, device='cuda')
        self.ws = torch.full((n,), 255, dtype=torch.uint8, device='cuda')
        A.mprk_bind(self.h, self.u.data_ptr(), self.ws.data_ptr(), n)

    def solve(self, seed=4):
        rhs = np.random.default_rng(seed).standard_normal(self.N)
        r = torch.from_numpy(rhs).cuda()
        x = torch.zeros_like(r)
        rc, info = A.mprk_solve(self.h, 0, r.data_ptr(), x.data_ptr())
        assert rc == A.OK, (rc, info)
        return rhs, x.cpu().numpy(), info

    def residual_test(self, rhs, x):
        """(||rhs - M x||, the outer tolerance and the rounding of 9 FP64 operations a row)."""
        Mx = operators.stage_matrix(operators.operator(self.shape, self.bc, self.kind, self.diff, self.vel),
                                    self.dt * self.tab.a_lo[0])
        lim = self.prec.outer_tol * np.linalg.norm(rhs) + 32 * 2.0 ** -53 * np.linalg.norm(abs(Mx) @ np.abs(x))
        return np.linalg.norm(rhs - Mx @ x), lim

    def close(self):
        A.mprk_destroy(self.h)


# N % 4 = 1, 2, 3 and N % 8 = 1: the last group holds one to seven unknowns of its four or eight
@pytest.mark.parametrize("shape", [(37, 37, 37), (9, 5, 5), (9, 10, 3), (11, 5, 1), (1, 1, 1)])
@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("block", [1, 2, 4])
def test_shared_inverses_by_index(shape, storage, block):
    # the index of every block is in bounds, and the inverses are those stored per block
    log_case('bj_tail_index', shape=shape, storage=storage, block=block)
    a = Filled(shape, storage, 'gmres', A.FMT_CSR, block=block, bj_shared=1)
    rhs, x, info = a.solve()
    res, lim = a.residual_test(rhs, x)
    b = Filled(shape, storage, 'gmres', A.FMT_CSR, block=block, bj_shared=0)
    _, y, jnfo = b.solve()
    a.close()
    b.close()
    assert info['converged'] == 1 and res <= lim, (info, res, lim)
    assert info['iters'] == jnfo['iters'] and np.array_equal(x, y)


# odd grids on which CG takes groups of values (past 3 2^17 and, in FP16, 11 2^16 unknowns) and, in
# FP16, smaller ones
@pytest.mark.parametrize("shape,storage,block", [((77, 73, 71), 'fp32', 2), ((77, 73, 71), 'fp32', 1),
                                                 ((77, 73, 71), 'fp64', 2), ((83, 81, 79), 'fp16', 4),
                                                 ((83, 81, 79), 'fp16', 2), ((83, 81, 79), 'fp16', 1),
                                                 ((91, 91, 89), 'fp16', 4), ((91, 91, 89), 'fp16', 2),
                                                 ((91, 91, 89), 'fp16', 1)])
@pytest.mark.parametrize("fmt,over", [(A.FMT_CSR, {}), (A.FMT_CSR, {'bj_adapt_tol': 1e-1}),
                                      (A.FMT_STENCIL, {'bj_adapt_tol': 1e-1})])
def test_cg_sums_of_the_last_group(shape, storage, block, fmt, over):
    log_case('bj_tail_cg', shape=shape, storage=storage, block=block, fmt=fmt, **over)
    a = Filled(shape, storage, 'cg', fmt, block=block, **over)
    rhs, x, info = a.solve()
    res, lim = a.residual_test(rhs, x)
    a.close()
    assert info['converged'] == 1 and res <= lim, (info, res, lim)
