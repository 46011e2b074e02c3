"""Launch shapes of small and mid-size meshes: strip tiles of one row up to a few dozen,
widths that leave every kind of last strip, and states whose rows start on any 8-byte
boundary (rows are loaded 16 bytes a lane where their addresses allow it).

A periodic state of a small period stays periodic under the scheme, so every cell of the
large mesh must equal its image in the small one (bitwise: the arithmetic does not depend
on the tiling), and the small result is the oracle's within 1e-12.
"""
import numpy as np
import pytest
import torch

import fam_inputs as fi
import oracle.scheme as S
from gpu_util import both_configs, log, needs_gpu, rel_linf, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]
H = 1.0 / 1024.0   # cell size: the same floating-point number on either mesh

# period (px, py) and its repeats: 120x80 (1 row a tile), 403x297, 420x300, 122x1100,
# 516x510, 720x700 (2 to 10 rows), 1201x900, 1024x1040 (10 rows and more)
MESHES = [(12, 10, 10, 8), (13, 27, 31, 11), (14, 10, 30, 30), (61, 11, 2, 100), (12, 10, 43, 51),
          (12, 14, 60, 50), (1201, 9, 1, 100), (16, 10, 64, 104)]


@pytest.mark.parametrize("px,py,mx,my", MESHES)
@pytest.mark.parametrize("k,pp", [(3, False), (4, True), (5, False), (5, True), (6, False), (6, True)])
def test_every_tile_height_and_width(px, py, mx, my, k, pp):
    nx, ny, nsteps = px * mx, py * my, 2
    log(f"{nx}x{ny} from {px}x{py}, k={k}, limiter {pp}")
    kw = dict(dim=2, k=k, system="euler", bc_x="periodic", bc_y="periodic", oe="type2", cfl=0.2, pp=pp)
    ora, small_cfg = both_configs(nx=px, ny=py, x1=px * H, y1=py * H, **kw)
    _, big_cfg = both_configs(nx=nx, ny=ny, x1=nx * H, y1=ny * H, **kw)
    U0 = fi.random_euler_state_2d(px, py, 31 + k, amp=0.4 if pp else 0.1)
    ref, _, _ = S.run(torch.tensor(U0), ora, nsteps=nsteps)
    from paper_2609_26194_amd import Fam
    small = Fam(small_cfg)
    Us = to_dev(U0)
    small.run(Us, 0.0, nsteps)
    small.check()
    assert rel_linf(Us, ref) <= 1e-12
    tiled = to_dev(U0).repeat(1, 1, my, mx)
    for shift in (0, 1):   # the state at a 16-byte boundary and 8 bytes after one
        store = torch.empty(tiled.numel() + 1, dtype=torch.float64, device="cuda")
        Ub = store[shift:shift + tiled.numel()].view(tiled.shape)
        Ub.copy_(tiled)
        big = Fam(big_cfg)
        big.run(Ub, 0.0, nsteps)
        big.check()
        big.close()
        view = Ub.view(4, 3, my, py, mx, px)
        assert torch.equal(view, Us.view(4, 3, 1, py, 1, px).expand_as(view)), f"shift {shift}"


@pytest.mark.parametrize("system,k", [("advection", 3), ("burgers", 4), ("burgers", 6)])
@pytest.mark.parametrize("px,py,mx,my", [MESHES[0], MESHES[1], MESHES[4], MESHES[6]])
def test_scalar_equations(px, py, mx, my, system, k):
    nx, ny = px * mx, py * my
    log(f"{system} {nx}x{ny} from {px}x{py}, k={k}")
    kw = dict(dim=2, k=k, system=system, bc_x="periodic", bc_y="periodic", oe="type2", cfl=0.2)
    ora, small_cfg = both_configs(nx=px, ny=py, x1=px * H, y1=py * H, **kw)
    _, big_cfg = both_configs(nx=nx, ny=ny, x1=nx * H, y1=ny * H, **kw)
    rng = np.random.default_rng(7)
    U0 = 0.05 * rng.standard_normal((1, 3, py, px))
    U0[0, 0] += 1.0
    ref, _, _ = S.run(torch.tensor(U0), ora, nsteps=2)
    from paper_2609_26194_amd import Fam
    small, big = Fam(small_cfg), Fam(big_cfg)
    Us, Ub = to_dev(U0), to_dev(U0).repeat(1, 1, my, mx).contiguous()
    small.run(Us, 0.0, 2)
    big.run(Ub, 0.0, 2)
    assert rel_linf(Us, ref) <= 1e-12
    view = Ub.view(1, 3, my, py, mx, px)
    assert torch.equal(view, Us.view(1, 3, 1, py, 1, px).expand_as(view))
