"""The batched form on grids whose x-rows are shorter than a block-Jacobi block and do not divide it:
every block has an inverse of its own, and the solves take the iterations of the single-problem form."""
import numpy as np
import pytest

import workloads as W
from oracle import krylov, operators
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi


# last blocks and last groups of four, whole and partial
@pytest.mark.parametrize("shape", [(3, 8, 11), (3, 7, 5), (1, 9, 13), (1, 16, 8), (3, 20, 20), (5, 6, 7)])
@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("block", [2, 4, 8])
def test_iterations_of_the_single_problem_form(shape, storage, block):
    log_case('batch_short_rows', shape=shape, storage=storage, block=block)
    # a stiff x axis, so that the blocks (and a wrong block's inverse) matter
    dt, N = 5e-2, int(np.prod(shape))
    u0 = np.random.default_rng(9).standard_normal(N)
    over = dict(precond='bj', block=block, stage_start=A.START_RHS, inner_stop=A.STOP_RTOL)
    b = M.Batch([{'shape': shape, 'diff': 1.0, 'dt': dt}], 'SDIRK2', M.precisions(storage, 'cg', **over))
    b.set_u(0, u0)
    b.step(1)
    sb, ub = b.stats(0), b.get_u(0).ravel()
    b.close()
    s = M.Stepper(shape, W.DIRICHLET, W.HEAT, 1.0, (0.0, 0.0, 0.0), A.FMT_CSR, 'SDIRK2',
                  M.precisions(storage, 'cg', **over), dt)
    s.set_u(u0)
    ss, us = s.step(1), s.get_u().ravel()
    s.close()
    print(sb['iters'], ss['iters'], sb['passes'], ss['passes'])
    assert sb['passes'][:2] == ss['passes'][:2] and all(ss['converged'])
    # one iteration a pass of room: the two forms add their sums in other orders
    for i, j, p in zip(sb['iters'], ss['iters'], ss['passes']):
        assert abs(i - j) <= p, (sb, ss)
    assert np.linalg.norm(ub - us) <= {'fp64': 1e-10, 'fp32': 1e-5, 'fp16': 1e-3}[storage] * np.linalg.norm(u0)
