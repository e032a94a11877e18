"""The batched stage kernel on grids whose rows, chunks and last groups are no multiple of a
thread's group of unknowns, and with schedules of one workgroup up to one per 64 rows, against the
FP64 oracle's closed form."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import log_case, reference_solution, rel_l2_floor

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')

TOL = {'fp64': 1e-11, 'fp32': 1e-6, 'fp16': 1e-3}


@pytest.mark.parametrize("storage", ['fp64', 'fp32', 'fp16'])
@pytest.mark.parametrize("block", [8, 4, 1])
@pytest.mark.parametrize("wide", [False, True])
def test_ragged_sizes(storage, block, wide):
    log_case('batch_groups', storage=storage, block=block, wide=wide)
    probs = [W.heat_modes(n=n, seed=n, nsteps=2) for n in (5, 8, 9, 13, 16, 17, 21, 30)]
    # wide: one workgroup per 64 rows where the device holds that many
    sched = [min(120, max(1, (p.N + 63) // 64)) for p in probs] if wide else None
    b = M.Batch([{'shape': p.n, 'diff': p.diff, 'dt': p.dt} for p in probs], 'SDIRK3',
                M.precisions(storage, 'cg', block=block), schedule=sched)
    for i, p in enumerate(probs):
        b.set_u(i, p.u0)
    b.step(2)
    for i, p in enumerate(probs):
        assert b.stats(i)['steps'] == 2
        err = rel_l2_floor(b.get_u(i), reference_solution(p), p.u0)
        assert err <= TOL[storage], (p.n, err)
    b.close()
