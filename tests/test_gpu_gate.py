"""Small CG problems (stages of one launch each) and batches stepped at the same time on several streams:
same results as alone, whatever runs beside them, and calls that return."""
import threading
import time

import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_util import log_case, reference_solution, rel_l2_floor

pytestmark = pytest.mark.gpu

M = pytest.importorskip('paper_2412_16638_amd')


def _run(fns):
    """Every function on a thread and a stream of its own."""
    out, errs = {}, []

    def go(k, fn):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                out[k] = fn()
        except Exception as e:  # noqa: BLE001
            errs.append((k, e))

    ts = [threading.Thread(target=go, args=(k, fn)) for k, fn in enumerate(fns)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs, errs
    return out


def _single(n, storage, steps, graph=False):
    def fn():
        p = W.heat_modes(n=n, seed=n, nsteps=steps)
        p.precision = storage
        st = M.from_problem(p)
        st.set_step_graph(graph)
        st.step(2)
        st.step(steps - 2)
        u = st.get_u()
        st.close()
        return u
    return fn


def _batch(probs, storage, steps, schedule=None):
    def fn():
        b = M.Batch([{'shape': p.n, 'diff': p.diff, 'dt': p.dt} for p in probs], 'SDIRK3',
                    M.precisions(storage, 'cg'), schedule=schedule)
        for i, p in enumerate(probs):
            b.u[i].copy_(torch.from_numpy(np.ravel(p.u0)))
        b.stream.synchronize()
        for _ in range(steps):
            b.step(1)
        for i in range(len(probs)):
            assert b.stats(i)['steps'] == steps
        us = [u.cpu().numpy() for u in b.u]
        b.close()
        return us
    return fn


@pytest.mark.parametrize("storage", ['fp32', 'fp64'])
def test_more_calls_than_the_device_holds(storage):
    # eight problems of 98 to 128 workgroups; long calls, so that they take turns
    log_case('gate_calls', storage=storage)
    fns = [_single(n, storage, 60, graph) for n, graph in ((48, False), (50, True), (46, False), (50, False)) * 2]
    together = _run(fns)
    for k in range(4):
        alone = _run([fns[k]])[0]
        assert np.array_equal(together[k], alone) and np.array_equal(together[k + 4], alone)


@pytest.mark.parametrize("wide", [False, True])
def test_batches_beside_calls(wide):
    # two FP32 batches that fit beside each other or not, an FP16 batch that fills the device
    log_case('gate_batches', wide=wide)
    probs = [W.heat_modes(n=n, seed=n, nsteps=12) for n in (17, 24, 30, 33, 40)]
    sched = [min(150, (p.N + 63) // 64) for p in probs] if wide else None
    fns = [_batch(probs, 'fp32', 12, sched), _batch(probs, 'fp32', 12, sched), _batch(probs[:3], 'fp16', 12),
           _single(50, 'fp32', 12), _single(24, 'fp64', 12, True), _single(44, 'fp64', 12)]
    together = _run(fns)
    for k, fn in enumerate(fns):
        alone = _run([fn])[0]
        if k < 3:
            assert all(np.array_equal(a, b) for a, b in zip(together[k], alone))
            for p, u in zip(probs, together[k]):
                err = rel_l2_floor(u, reference_solution(p), p.u0)
                assert err <= (1e-3 if k == 2 else 1e-6), (k, p.n, err)
        else:
            assert np.array_equal(together[k], alone)


def test_batch_step_returns_while_calls_run():
    # a call of many steps holds the device; a batch that does not fit beside it is still only enqueued
    log_case('gate_async')
    p = W.heat_modes(n=50, nsteps=1)
    probs = [W.heat_modes(n=n, seed=n, nsteps=1) for n in (17, 24, 30)]
    b = M.Batch([{'shape': q.n, 'diff': q.diff, 'dt': q.dt} for q in probs], 'SDIRK3', M.precisions('fp16', 'cg'))
    for i, q in enumerate(probs):
        b.set_u(i, q.u0)
    b.step(1)
    torch.cuda.synchronize()
    done = threading.Event()
    began = threading.Event()

    def call():
        with torch.cuda.stream(torch.cuda.Stream()):
            st = M.from_problem(p)
            st.step(1)
            began.set()
            for _ in range(4):
                st.step(400)  # about 0.3 s each
            done.set()
            st.close()

    t = threading.Thread(target=call)
    t.start()
    began.wait()
    time.sleep(0.05)
    t0 = time.perf_counter()
    b.step(2)
    took = time.perf_counter() - t0
    running = not done.is_set()
    t.join()
    assert b.stats(0)['steps'] == 3
    b.close()
    assert running and took < 0.1, (running, took)
