"""Batches of as many problems, and schedules of as many workgroups, as the device has held at once:
four or five per compute unit in FP32, two to four in FP64."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_util import log_case, reference_solution, rel_l2_floor

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')

# storage, block (0: no preconditioner), workgroups per compute unit
HELD = [('fp32', 0, 5), ('fp32', 1, 5), ('fp32', 2, 5), ('fp32', 4, 4), ('fp32', 8, 4), ('fp64', 0, 4),
        ('fp64', 1, 4), ('fp64', 2, 3), ('fp64', 4, 3), ('fp64', 8, 2), ('fp16', 0, 5), ('fp16', 8, 4)]
TOL = {'fp64': 1e-11, 'fp32': 1e-6, 'fp16': 1e-3}


def _check(b, probs, idx, storage):
    for i in idx:
        assert b.stats(i)['steps'] == 1
        assert rel_l2_floor(b.get_u(i), reference_solution(probs[i]), probs[i].u0) <= TOL[storage]


@pytest.mark.parametrize("storage,block,per_cu", HELD)
def test_problems_and_workgroups_held_at_once(storage, block, per_cu):
    log_case('batch_capacity', storage=storage, block=block, per_cu=per_cu)
    most = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    prec = M.precisions(storage, 'cg', precond='bj' if block else 'none', block=block or 8)
    kinds = [W.heat_modes(n=n, seed=n, nsteps=1) for n in (3, 4, 5, 6)]
    probs = [kinds[i % 4] for i in range(most)]
    b = M.Batch([{'shape': p.n, 'diff': p.diff, 'dt': p.dt} for p in probs], 'SDIRK3', prec)
    assert min(b.schedule) >= 1 and sum(b.schedule) <= most
    for i, p in enumerate(probs):
        b.u[i].copy_(torch.from_numpy(np.ravel(p.u0)))
    b.step(1)
    _check(b, probs, (0, 1, 2, 3, most - 1), storage)
    b.close()
    # the same number of workgroups on few problems
    big = W.heat_modes(n=24, seed=5, nsteps=1)
    each = [128] * (most // 128) + ([most % 128] if most % 128 else [])
    b = M.Batch([{'shape': big.n, 'diff': big.diff, 'dt': big.dt} for _ in each], 'SDIRK3', prec, schedule=each)
    for i in range(len(each)):
        b.set_u(i, big.u0)
    b.step(1)
    _check(b, [big] * len(each), (0, len(each) - 1), storage)
    b.close()
