"""Small 1D meshes (whole runs in one workgroup) and non-physical averages: a run to an end
time tests for them after 2 steps and then after at most 64 more at a time, as on larger
meshes, a run of a number of steps at its end; state, clock and step count are those of
the steps it took.  Long runs are split over several launches.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]
OK, NONPHYSICAL = 0, -4


def _run(fam, U, t_final, max_steps, dt_fixed=0.0):
    """(status, steps, time) of fam_run."""
    from paper_2609_26194_amd import load_library
    n, t = ctypes.c_int(-1), ctypes.c_double(-1.0)
    fam.stream.wait_stream(torch.cuda.current_stream())
    r = load_library().fam_run(fam.h, ctypes.c_void_p(U.data_ptr()), float(t_final), int(max_steps), float(dt_fixed),
                               ctypes.byref(n), ctypes.byref(t))
    torch.cuda.synchronize()
    return r, n.value, t.value


def _same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan())).all())


def _euler(n, u):
    x = (np.arange(n) + 0.5) / n
    v = np.where(x < 0.5, -u, u) * np.ones(n)
    U = np.zeros((3, 2, n))
    U[0, 0], U[1, 0], U[2, 0] = 1.0, v, 1.0 + 0.5 * v * v
    return U


def _fam(n, **kw):
    from paper_2609_26194_amd import Fam, FamConfig
    return Fam(FamConfig(dim=1, nx=n, k=5, system="euler", bc_x="transmissive", oe="type2", cfl=0.2, **kw))


@pytest.mark.parametrize("n", [120, 510, 511])
def test_a_cell_of_negative_pressure_ends_the_run_after_two_steps(n):
    U0 = _euler(n, 0.0)
    U0[2, 0, n // 2] = -0.01
    fam = _fam(n)
    U, V = to_dev(U0), to_dev(U0)
    r, steps, t = _run(fam, U, 1.0, 0)
    log(f"n={n}: status {r} after {steps} steps, t = {t:.3e}")
    assert r == NONPHYSICAL and steps == 2
    fam.set_time(0.0)
    for _ in range(2):
        fam.step(V)
    torch.cuda.synchronize()
    assert _same(U, V)
    # the flag of an earlier call that nobody checked
    assert _run(fam, to_dev(_euler(n, 0.0)), t + 1.0, 0)[:2] == (NONPHYSICAL, 2)
    # a run of a number of steps is tested at its end
    fam.set_time(0.0)
    assert _run(fam, to_dev(U0), 0.0, 1500)[:2] == (NONPHYSICAL, 1500)
    fam.close()


@pytest.mark.parametrize("n", [120, 510, 511])
def test_a_vacuum_is_noticed_after_the_second_chunk(n):
    """Two streams that part faster than the gas can follow; chunks of 2 and 64 steps."""
    U0 = to_dev(_euler(n, 4.0))
    fam = _fam(n)
    V, first = U0.clone(), 0
    for k in range(1, 200):
        fam.step(V)
        try:
            fam.check()
        except Exception:
            first = k
            break
    assert first > 0
    fam.set_time(0.0)
    U = U0.clone()
    r, steps, t = _run(fam, U, 1.0, 0)
    log(f"n={n}: non-physical in step {first}, noticed after {steps}")
    assert r == NONPHYSICAL and first <= steps == 66
    fam.set_time(0.0)
    W = U0.clone()
    for _ in range(steps):
        fam.step(W)
    torch.cuda.synchronize()
    assert _same(U, W)
    fam.close()


@pytest.mark.parametrize("limit", [0, 2500, 2501, 1024, 1025])
def test_runs_longer_than_a_launch(limit):
    """Some 2700 steps to the end time, or a step count short of it; the same steps by single calls."""
    from paper_2609_26194_amd import Fam, FamConfig
    n = 63
    fam = Fam(FamConfig(dim=1, nx=n, k=5, system="burgers", oe="type2", cfl=0.1))
    x = (np.arange(n) + 0.5) / n
    U0 = np.zeros((1, 2, n))
    U0[0, 0] = 1.0 + 0.5 * np.sin(2.0 * np.pi * x)
    t_end, dt = 1.0, 1.0 / 2700.5
    U, V = to_dev(U0), to_dev(U0)
    r, steps, t = _run(fam, U, t_end, limit, dt)
    log(f"limit {limit}: {steps} steps, t = {t}")
    assert r == OK and steps == (limit or 2701)
    fam.set_time(0.0)
    for k in range(steps):
        fam.step(V, dt if k < 2700 else t_end - _clock(dt, 2700))
    torch.cuda.synchronize()
    assert t == (t_end if limit == 0 else _clock(dt, limit))
    assert torch.equal(U, V)
    fam.close()


def _clock(dt, steps):
    t = 0.0
    for _ in range(steps):
        t += dt
    return t
