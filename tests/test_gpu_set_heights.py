"""Strip-tile heights that a caller sets or the autotuner picks are the ones launched, on
meshes so small that the default height is a row or two too.

The shape of a launch shows in its time only: a wave's march over H rows is bound by the
rows' latency where every tile has a SIMD to itself, so a launch with tiles of 64 rows
takes many times as long as one with tiles of a few (the test asks for twice).
"""
import pytest
import torch

import fam_inputs as fi
from gpu_util import both_configs, log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


def _launch_us(fam, U, dt, reps=20):
    """(stage, OE) microseconds a launch, the least of five rounds."""
    from paper_2609_26194_amd.fam import fam_oe, fam_stage
    V, W = torch.empty_like(U), torch.empty_like(U)
    best = [1e30, 1e30]
    for _ in range(5):
        for which in (0, 1):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            fam.stream.synchronize()
            a.record(fam.stream)
            for _ in range(reps):
                fam_stage(fam.h, 0, U, U, V, dt) if which == 0 else fam_oe(fam.h, U, W, dt)
            b.record(fam.stream)
            b.synchronize()
            best[which] = min(best[which], 1e3 * a.elapsed_time(b) / reps)
    return best


@pytest.mark.parametrize("system,k", [("euler", 5), ("euler", 6), ("burgers", 4)])
def test_two_set_heights_are_two_launch_shapes(system, k):
    from paper_2609_26194_amd import Fam
    n = 256
    _, cfg = both_configs(dim=2, nx=n, ny=n, k=k, system=system, oe="type2", cfl=0.2)
    U = to_dev(fi.random_euler_state_2d(n, n, 3, amp=0.1))
    U = U if system == "euler" else U[:1].contiguous()
    fam = Fam(cfg)
    dt = fam.dt(U)
    base = _launch_us(fam, U, dt)
    fam.set_tiling(64, 64)
    tall = _launch_us(fam, U, dt)
    fam.set_tiling(8, 8)
    least = _launch_us(fam, U, dt)
    fam.close()
    log(f"{system} k={k}: default {base}, 64 rows {tall}, least height {least} us")
    for q in (0, 1):
        assert tall[q] > 2.0 * base[q]
        assert least[q] < 1.5 * base[q]   # 8 stands for the default of a mesh this small


def test_autotuner_compares_shapes_that_differ():
    """On small meshes the least height wins by far, so a tuner that times what it names reports it."""
    from paper_2609_26194_amd import Fam, FamConfig
    kw = dict(dim=2, k=5, system="euler", bc_x="transmissive", bc_y="transmissive", oe="type2", cfl=0.2)
    n = 128
    U = to_dev(fi.batch_instance(0, n))
    fam = Fam(FamConfig(nx=n, ny=n, **kw))
    hs, ho = fam.autotune(U, reps=5)
    fam.close()
    bat = Fam(None, batch=[FamConfig(nx=n, ny=n, **kw)] * 4)
    hb, _ = bat.autotune(torch.cat([U.reshape(-1)] * 4), reps=5)
    bat.close()
    log(f"autotuned {n}x{n}: stage {hs}, OE {ho}; batch of four: {hb}")
    assert (hs, ho, hb) == (8, 8, 8)
