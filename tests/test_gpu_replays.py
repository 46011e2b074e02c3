"""Runs long enough for fam_run to replay its graph of 8 steps (chunks of 40 and more): 47
steps are five replays, three pairs of launches and an odd step.  Each equals, bit for bit,
the same steps in calls too short for a graph, of a context whose launch shapes may differ.
"""
import pytest
import torch

import fam_inputs as fi
from gpu_util import log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]
LONG, SHORT = 47, (24, 23)


def _quadrant(nx, ny, k=5, **kw):
    from paper_2609_26194_amd import FamConfig
    return (FamConfig(dim=2, nx=nx, ny=ny, k=k, system="euler", bc_x="transmissive", bc_y="transmissive", oe="type2",
                      cfl=0.2, pp=True, **kw), fi.four_quadrant(nx, 3, ny=ny))


def _case(name):
    """(config, state, stage and OE heights or None)"""
    from paper_2609_26194_amd import FamConfig
    if name == "segment_list":
        return (*_quadrant(130, 100), (0, 24))
    if name == "ordered_tiles":   # 17 strips of 90 tiles: more than the wave slots of k = 6
        return (*_quadrant(1000, 900, k=6), (10, 10))
    if name in ("double_mach", "double_mach_list"):
        return (FamConfig(dim=2, nx=96, ny=32, x1=3.0, y1=1.0, k=5, system="euler", oe="type2", cfl=0.2, pp=True,
                          dmr=True), fi.double_mach(96, 32), (0, 8) if name == "double_mach_list" else None)
    if name == "type1":
        return (FamConfig(dim=2, nx=70, ny=61, k=4, system="euler", oe="type1", cfl=0.2),
                fi.density_waves(70, ny=61), None)
    assert name == "1d_tiles"
    return (FamConfig(dim=1, nx=600, x0=-5.0, x1=5.0, k=5, system="euler", bc_x="transmissive", oe="type2", cfl=0.2),
            fi.shu_osher(600), None)


@pytest.mark.parametrize("name", ["segment_list", "ordered_tiles", "double_mach", "double_mach_list", "type1",
                                  "1d_tiles"])
def test_long_run_equals_short_calls(name):
    from paper_2609_26194_amd import Fam
    cfg, U0h, tiling = _case(name)
    U0 = to_dev(U0h)
    ref = Fam(cfg)
    V = U0.clone()
    for n in SHORT:
        ref.run(V, 0.0, n)
    t_ref = ref.run(V.clone(), 1e-300, 0)[1]   # the clock: a run to a time behind it does nothing
    ref.close()
    fam = Fam(cfg)
    if tiling is not None:
        fam.set_tiling(*tiling)
    U = U0.clone()
    n, t = fam.run(U, 0.0, LONG)
    log(f"{name}: {n} steps to t = {t:.6e}")
    assert n == LONG and t == t_ref and torch.equal(U, V)
    # again on the same buffer, with other work between: the kept graph
    junk = torch.randn(4096, device="cuda").cumsum(0)
    torch.cuda.synchronize()
    del junk
    fam.set_time(0.0)
    U.copy_(U0)
    assert fam.run(U, 0.0, LONG) == (LONG, t_ref)
    assert torch.equal(U, V)
    fam.close()


@pytest.mark.parametrize("tune", [False, True])
def test_long_run_of_a_limiter_batch(tune):
    from paper_2609_26194_amd import Fam
    sizes = [64, 96, 130, 62, 200, 75]
    cfgs = [_quadrant(n, n)[0] for n in sizes]
    U0 = torch.cat([to_dev(fi.batch_instance(i, n)).reshape(-1) for i, n in enumerate(sizes)])
    ref, bat = Fam(None, batch=cfgs), Fam(None, batch=cfgs)
    V, U = U0.clone(), U0.clone()
    for n in SHORT:
        ref.run(V, 0.0, n)
    if tune:
        log(f"tuned batch: {bat.autotune(U0, reps=2)}")
    for _ in range(2):
        U.copy_(U0)
        n, _t = bat.run(U, 0.0, LONG)
        assert n == LONG and torch.equal(U, V)
    ref.close()
    bat.close()


def test_shape_changes_drop_the_graph():
    """Long runs on one buffer with the tiling changed, and tuned, between them."""
    from paper_2609_26194_amd import Fam
    cfg, U0h = _quadrant(130, 100)
    U0 = to_dev(U0h)
    ref, fam = Fam(cfg), Fam(cfg)
    V, U = U0.clone(), U0.clone()
    for shape in (None, (0, 24), (16, 33), "tuned", (8, 8)):
        for n in SHORT:
            ref.run(V, 0.0, n)
        if shape == "tuned":
            fam.autotune(U, reps=2)
        elif shape is not None:
            fam.set_tiling(*shape)
        n, t = fam.run(U, 0.0, LONG)
        log(f"shape {shape}: t = {t:.6e}")
        assert n == LONG and torch.equal(U, V), shape
    ref.close()
    fam.close()


def test_long_runs_to_an_end_time():
    """Chunks of 2, then up to 64 steps: graphs and their remainders, in a batch and on one mesh."""
    from paper_2609_26194_amd import Fam
    cfg, U0h = _quadrant(64, 62)
    U0 = to_dev(U0h)
    one = Fam(cfg)
    V = U0.clone()
    dt = 1.0 / 4096.0
    steps, t = one.run(V, 150.5 * dt, 0, dt)
    assert steps == 151 and t == 150.5 * dt
    W = U0.clone()
    for k in range(151):
        one.step(W, dt if k < 150 else 0.5 * dt)
    torch.cuda.synchronize()
    assert torch.equal(V, W)
    bat = Fam(None, batch=[cfg, cfg])
    Ub = torch.cat([U0.reshape(-1)] * 2)
    assert bat.run(Ub, 150.5 * dt, 0, dt) == (151, 150.5 * dt)
    assert torch.equal(Ub.view(2, -1), V.reshape(1, -1).expand(2, -1))
    one.close()
    bat.close()
