"""Records of the most recent step when a small CG problem's stages run as one launch each: stages that a
strict miss skipped report nothing of an earlier step, and steered steps leave the step graph the
histories that it needs."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import log_case

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi


@pytest.mark.parametrize("n", [8, 24])  # one workgroup, several
@pytest.mark.parametrize("storage", ['fp64', 'fp32'])
@pytest.mark.parametrize("graph", [False, True])
def test_skipped_stages_report_nothing(n, storage, graph):
    log_case('strict_records', n=n, storage=storage, graph=graph)
    p = W.heat_modes(n=n, nsteps=1)
    p.precision, p.precond = storage, 'none'
    smooth = W.sine_mode((n, n, n), (1, 1, 1))
    # one CG iteration a pass, two passes: exact for the sine mode, far from the tolerance otherwise
    st = M.from_problem(p, strict=1, maxit=1, refine_max=2, stage_start=A.START_RHS,
                        outer_tol=1e-6 if storage == 'fp32' else 1e-10)
    st.set_step_graph(graph)
    st.set_u(smooth)
    st.step(2)
    ok = st.step(1)
    assert all(ok['converged'][:3]) and min(ok['iters'][:3]) >= 1
    st.set_u(W.random_field(n, 11))
    rc, one = st.step(1, check=False)
    assert rc == A.ENOTCONV
    rc, three = st.step(3, check=False)  # the last step of this call is skipped as a whole
    st.close()
    assert rc == A.ENOTCONV
    assert one['converged'][0] == 0 and one['passes'][0] == 2 and one['resid'][0] > 0.0
    for s, skipped in ((one, (1, 2)), (three, (0, 1, 2))):
        for i in skipped:
            assert (s['iters'][i], s['passes'][i], s['resid'][i], s['converged'][i]) == (0, 0, 0.0, 0), s


@pytest.mark.parametrize("n", [8, 24])
@pytest.mark.parametrize("storage", ['fp64', 'fp32'])
def test_graph_enabled_after_steered_steps_replays(n, storage):
    log_case('graph_after_steps', n=n, storage=storage)
    p = W.heat_modes(n=n, nsteps=1)
    p.precision = storage
    a, b = M.from_problem(p), M.from_problem(p)
    a.step(1)
    a.set_step_graph(True)
    s = a.step(3)
    t = b.step(4)
    ua, ub = a.get_u(), b.get_u()
    a.close()
    b.close()
    assert s['graph_steps'] == 3
    assert s['iters'] == t['iters'] and np.array_equal(ua, ub)
