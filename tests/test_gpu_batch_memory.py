"""What a batch of many small meshes allocates beside its two stage states, and that its
time steps, from one pair of wave-speed maxima per instance, are those of single meshes.
"""
import numpy as np
import pytest
import torch

import fam_inputs as fi
from gpu_util import log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


def test_a_small_instance_costs_little_beside_its_states():
    """16x16 Euler meshes (24 KB a state): tables, work list and step books take under 4 KB each."""
    from paper_2609_26194_amd import Fam, FamConfig
    n, size = 4000, 16
    cfgs = [FamConfig(dim=2, nx=size, ny=size, k=5, system="euler", oe="type2")] * n
    Fam(None, batch=cfgs[:2]).close()   # the library's own first-use memory
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    bat = Fam(None, batch=cfgs)
    used = before - torch.cuda.mem_get_info()[0]
    extra = (used - 2 * 8 * bat.len) / n
    log(f"{n} meshes of {size}^2: {used / 2**20:.1f} MiB, {extra:.0f} bytes an instance beside the stage states")
    bat.close()
    assert extra < 4096


@pytest.mark.parametrize("system,k", [("euler", 5), ("burgers", 3)])
def test_many_instances_take_the_time_steps_of_single_meshes(system, k):
    """Meshes below, at and above the blocks of the wave-speed reduction (256 cells each, 256 a
    mesh at most), more of them than a wave of the bookkeeping has lanes."""
    from paper_2609_26194_amd import Fam, FamConfig
    sizes = [(16, 16), (17, 16), (3, 5), (300, 257), (64, 64)] * 14
    kw = dict(dim=2, k=k, system=system, oe="type2", cfl=0.2)
    cfgs = [FamConfig(nx=a, ny=b, **kw) for a, b in sizes]
    states = []
    for i, (a, b) in enumerate(sizes):
        U = fi.random_euler_state_2d(a, b, i, amp=0.1 + 0.002 * i)
        states.append(to_dev(U if system == "euler" else U[:1]))
    bat = Fam(None, batch=cfgs)
    Ub = torch.cat([s.reshape(-1) for s in states])
    dts = bat.dt(Ub)
    used = torch.zeros(len(sizes), dtype=torch.float64, device="cuda")
    got = []
    for _ in range(2):
        bat.step(Ub, 0.0, used)
        got.append(used.clone())
    bat.check()
    for i, (cfg, U) in enumerate(zip(cfgs[:10], states)):
        fam = Fam(cfg)
        assert fam.dt(U)[0] == dts[i]
        one = torch.zeros(1, dtype=torch.float64, device="cuda")
        for g in got:
            fam.step(U, 0.0, one)
            assert one[0] == g[i]
        o = bat.offsets()[i]
        assert torch.equal(Ub[o:o + U.numel()], U.reshape(-1))
        fam.close()
    bat.close()
