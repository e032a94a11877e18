"""The folded y and z contractions of the complex fast-diagonalisation preconditioner at the axis
lengths where the fold or its tiles can go wrong: axes of one to four values (all their own mirrors
but some), n/2 + 1 around a chunk of 16 and a tile of 64, odd and even, against FFTs in FP64."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import closed_form
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi

U = {'fp64': 2.0 ** -53, 'fp32': 2.0 ** -24, 'fp16': 2.0 ** -11}
DT = {'fp64': torch.float64, 'fp32': torch.float32, 'fp16': torch.float16}
SHAPES = [(8, 1, 2), (8, 3, 4), (6, 2, 1), (7, 4, 3), (12, 30, 31), (13, 32, 33), (2, 29, 34), (8, 126, 127),
          (9, 128, 129), (16, 125, 6)]


@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("shape", SHAPES)
def test_folded_contractions(shape, storage):
    log_case('fdm_fold', shape=shape, storage=storage)
    b = (1.0, 0.5, -0.25)
    st = M.Stepper(shape, W.PERIODIC, W.ADVDIFF, 1e-2, b, A.FMT_STENCIL, 'SDIRK3',
                   M.precisions(storage, 'gmres', precond='fdm'), 2e-3)
    sigma = st.dt * (st.tab.a_hi[0] + st.tab.a_lo[0])
    xd = torch.from_numpy(np.random.default_rng(21).standard_normal(st.N)).to('cuda', DT[storage])
    y = st.apply(A.APPLY_FDM_LP, xd, stage=0).double().cpu().numpy()
    st.close()
    x = xd.double().cpu().numpy()
    lam = closed_form.periodic_eigenvalues(shape, 1e-2, b, central=False)
    ref = np.real(np.fft.ifftn(np.fft.fftn(x.reshape(shape[::-1])) / (1.0 - sigma * lam))).ravel()
    # six unitary contractions of at most max(shape) terms and the fold's sum in the compute type,
    # relative to ||x|| (|1 / P_D| <= 1); the result rounded to the storage type
    u_c = U['fp64' if storage == 'fp64' else 'fp32']
    lim = 6 * (max(shape) + 8) * u_c * np.linalg.norm(x) + U[storage] * np.linalg.norm(ref)
    lim += 2.0 ** -25 * np.sqrt(x.size) if storage == 'fp16' else 0.0
    assert np.linalg.norm(y - ref) <= lim
