"""Inner products of the FDM-preconditioned CG on flat groups: every product is added in FP64, so the
norm that opens an inner solve is the FP64 sum of its FP32 squares."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operators
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi


@pytest.mark.parametrize("storage,shape,seed", [('fp32', (77, 72, 72), 4), ('fp16', (83, 80, 80), 5),
                                                ('fp16', (91, 90, 90), 5)])
def test_norm_is_an_fp64_sum(storage, shape, seed):
    # an absolute tolerance 1.5e-11 above and below the norm decides whether the first solve iterates;
    # the FP64 sums of the device and of numpy agree to about 1e-13, groups added in FP32 are 7e-11 and more off
    log_case('fdm_sums', storage=storage, shape=shape)
    dt, N = 2e-3, int(np.prod(shape))
    rhs = np.random.default_rng(seed).standard_normal(N) + 2.0 * (np.arange(N) // (shape[0] * shape[1]) % 2)
    K = operators.operator(shape, W.PERIODIC, W.HEAT, 1.0, (0.0, 0.0, 0.0))
    iters = {}
    for side in (1, -1):
        prec = M.precisions(storage, 'cg', precond='fdm', rtol=0.0, refine_max=1, inner_stop=A.STOP_RTOL,
                            stage_start=A.START_RHS, outer_tol=0.0)
        tab = M.tableau('SDIRK3')
        res = dt * tab.a_lo[0] * (K @ rhs)  # the residual of the start value x = rhs
        scale = np.linalg.norm(res) / np.sqrt(N)
        r = (res / scale).astype(np.float16 if storage == 'fp16' else np.float32).astype(np.float32)
        sq = r * r
        exact = np.sqrt(np.sum(sq.astype(np.float64)))
        vec = 8 if storage == 'fp16' else 4
        groups = sq[:N // vec * vec].reshape(-1, vec)
        coarse = groups[:, 0].copy()
        for k in range(1, vec):
            coarse += groups[:, k]
        off = np.sqrt(np.sum(coarse.astype(np.float64)) + np.sum(sq[N // vec * vec:], dtype=np.float64)) / exact - 1.0
        assert abs(off) > 6e-11, off  # (the input tells the two sums apart)
        prec.atol = scale * exact * (1.0 + side * 1.5e-11)
        st = M.Stepper(shape, W.PERIODIC, W.HEAT, 1.0, (0.0, 0.0, 0.0), A.FMT_STENCIL, tab, prec, dt)
        _, info = st.solve(0, torch.from_numpy(rhs).cuda())
        iters[side] = info['iters']
        st.close()
    assert iters[1] == 0 and iters[-1] >= 1, iters
