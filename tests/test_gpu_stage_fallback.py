"""One-launch stages of small CG problems where their workgroups may not wait for each other: a stage
that has timed out is run again on the per-kernel path, and a stream that reaches a part of the device
takes that path from the start."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_util import log_case, reference_solution, rel_l2

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')
A = M._abi

TOL = {'fp64': 1e-11, 'fp32': 1e-6}
ERROR = 104  # byte offset in the control record of the flag that a bounded wait sets


class Handle:
    """A handle on a workspace whose control record is known: all of it is zero after the bind, and the
    rest was filled with 0xFF before."""

    def __init__(self, p):
        grid = A.mprk_grid(p.n, p.n, p.n, p.bc)
        op = A.mprk_operator(p.kind, A.FMT_STENCIL, p.diff, (A.C.c_double * 3)(*p.b))
        prec = M.precisions(p.precision, p.krylov, precond=p.precond)
        self.h = A.mprk_create(grid, op, M.tableau(p.tableau), prec, p.dt, torch.cuda.current_stream().cuda_stream)
        n = A.mprk_workspace_bytes(self.h)
        self.u = torch.zeros(p.n ** 3, dtype=torch.float64, device='cuda')
        self.ws = torch.full((n,), 255, dtype=torch.uint8, device='cuda')
        A.mprk_bind(self.h, self.u.data_ptr(), self.ws.data_ptr(), n)
        self.u.copy_(torch.from_numpy(np.ravel(p.u0)))
        nz = np.flatnonzero(np.concatenate(([1], self.ws.cpu().numpy(), [1])))
        run = int(np.argmax(np.diff(nz)))
        assert nz[run + 1] - nz[run] > 2048  # (the longest run of zeros is the record)
        self.ctl = (int(nz[run]) + 255) // 256 * 256

    def time_out(self):
        self.ws[self.ctl + ERROR:self.ctl + ERROR + 4].view(torch.int32)[0] = 1
        torch.cuda.synchronize()

    def step(self, n):
        rc, s = A.mprk_step(self.h, n)
        assert rc == A.OK, (rc, s)
        return s

    def close(self):
        A.mprk_destroy(self.h)


@pytest.mark.parametrize("storage", ['fp64', 'fp32'])
@pytest.mark.parametrize("graph", [False, True])
def test_steps_after_a_time_out(storage, graph):
    log_case('stage_time_out', storage=storage, graph=graph)
    p = W.heat_modes(n=24, nsteps=6)
    p.precision = storage
    a, b = Handle(p), M.from_problem(p)
    A.mprk_set_step_graph(a.h, graph)
    a.step(2)
    b.step(2)
    a.time_out()
    s = a.step(3)             # run on the per-kernel path, as under profiling
    A.mprk_profile(b.h, 1)
    t = b.step(3)
    assert s['steps'] == 5 and all(s['converged'][:3]) and s['iters'] == t['iters'] and s['graph_steps'] == 0
    assert np.array_equal(a.u.cpu().numpy(), b.get_u().ravel())
    assert a.step(1)['steps'] == 6  # and stays usable
    assert rel_l2(a.u.cpu().numpy(), reference_solution(p)) <= TOL[storage]
    a.close()
    b.close()


@pytest.mark.parametrize("storage", ['fp64', 'fp32'])
def test_solve_after_a_time_out(storage):
    log_case('stage_time_out_solve', storage=storage)
    p = W.heat_modes(n=24, nsteps=1)
    p.precision = storage
    a, b = Handle(p), M.from_problem(p)
    rhs = torch.from_numpy(np.random.default_rng(3).standard_normal(p.N)).cuda()
    a.time_out()
    x = rhs.clone()  # solved in place
    rc, info = A.mprk_solve(a.h, 0, x.data_ptr(), x.data_ptr())
    assert rc == A.OK and info['converged'] == 1, (rc, info)
    A.mprk_profile(b.h, 1)
    y, jnfo = b.solve(0, rhs)
    assert info == jnfo and torch.equal(x, y)
    a.close()
    b.close()


def test_stream_that_reaches_a_part_of_the_device():
    log_case('stage_cu_mask')
    hip = ctypes.CDLL('libamdhip64.so')
    s = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 1)(0xffff)  # 16 compute units
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(s), ctypes.c_uint32(1), mask) == 0
    p = W.heat_modes(n=50, nsteps=2)
    a = M.from_problem(p)
    A.mprk_profile(a.h, 1)  # the per-kernel path
    a.step(2)
    with torch.cuda.stream(torch.cuda.ExternalStream(s.value)):
        b = M.from_problem(p)
        b.step(2)
        ub = b.get_u()
        b.close()
    ua = a.get_u()
    a.close()
    hip.hipStreamDestroy(s)
    assert np.array_equal(ua, ub)
