"""Tiles of many rows against tiles of one or two, bit for bit, for every boundary, order and
variant whose rows are loaded or reconstructed differently: ghost rows built inside the row
loop (double Mach reflection), mapped ones, characteristic variables, the jump table of
k = 6, Type I; and the work lists of batches, whose default tiles have 16 rows from some
two million cells on.  Meshes this small run with the least heights by default, and those
are compared with the oracle in the tests of parity.
"""
import pytest
import torch

import fam_inputs as fi
from gpu_util import log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]
HEIGHTS = [(9, 12), (16, 9), (40, 33), (0, 16)]


def _same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan())).all())


def _steps(cfg, U0, tiling, steps=3):
    from paper_2609_26194_amd import Fam
    fam = Fam(cfg)
    if tiling is not None:
        fam.set_tiling(*tiling)
    U = U0.clone()
    for _ in range(steps):
        fam.step(U)
    torch.cuda.synchronize()
    fam.close()
    return U


def _compare(cfg, U0):
    ref = _steps(cfg, U0, None)
    assert not _same(ref, U0)
    for tiling in HEIGHTS:
        if tiling[0] == 0 and not cfg.pp:
            continue
        assert _same(_steps(cfg, U0, tiling), ref), tiling


@pytest.mark.parametrize("k,char", [(3, False), (4, False), (5, False), (6, False), (5, True)])
@pytest.mark.parametrize("pp", [True, False])
@pytest.mark.parametrize("oe", ["type2", "off"])
def test_double_mach_rows(k, char, pp, oe):
    from paper_2609_26194_amd import FamConfig
    nx, ny = 187, 61
    log(f"double Mach reflection {nx}x{ny} k={k} char={char} limiter={pp} oe={oe}")
    cfg = FamConfig(dim=2, nx=nx, ny=ny, x1=3.0, y1=1.0, k=k, system="euler", oe=oe, cfl=0.2, pp=pp, dmr=True,
                    char_vars=char)
    _compare(cfg, to_dev(fi.double_mach(nx, ny)))


@pytest.mark.parametrize("nx,ny", [(187, 61), (122, 90)])
@pytest.mark.parametrize("bc_x,bc_y", [("transmissive", "transmissive"), ("periodic", "transmissive"),
                                       ("transmissive", "periodic")])
@pytest.mark.parametrize("system,k,opts", [
    ("euler", 3, dict(pp=True)), ("euler", 4, dict(pp=True)), ("euler", 5, dict(pp=True)), ("euler", 6, dict(pp=True)),
    ("euler", 3, {}), ("euler", 4, dict(oe="type1")), ("euler", 5, dict(oe="off")),
    ("euler", 6, dict(k6_jump_from_table=True)), ("euler", 5, dict(char_vars=True, pp=True)),
    ("euler", 5, dict(char_vars=True)), ("advection", 3, dict(a=(0.8, -0.5))), ("burgers", 4, dict(oe="type1")),
    ("burgers", 5, {}), ("burgers", 6, dict(k6_jump_from_table=True))])
def test_mapped_ghost_rows(nx, ny, bc_x, bc_y, system, k, opts):
    from paper_2609_26194_amd import FamConfig
    log(f"{system} {nx}x{ny} k={k} {bc_x}/{bc_y} {opts}")
    cfg = FamConfig(**{**dict(dim=2, nx=nx, ny=ny, k=k, system=system, bc_x=bc_x, bc_y=bc_y, oe="type2", cfl=0.2),
                       **opts})
    U = fi.random_euler_state_2d(nx, ny, 17 + k, amp=0.5 if cfg.pp else 0.2)
    _compare(cfg, to_dev(U if system == "euler" else U[:1]))


@pytest.mark.parametrize("system,k,opts", [
    ("euler", 3, dict(pp=True)), ("euler", 4, dict(pp=True)), ("euler", 5, dict(pp=True)), ("euler", 6, dict(pp=True)),
    ("euler", 3, dict(oe="off")), ("euler", 4, {}), ("euler", 5, {}), ("euler", 6, dict(k6_jump_from_table=True)),
    ("advection", 3, dict(a=(0.8, -0.5))), ("advection", 4, {}), ("burgers", 5, {}), ("burgers", 6, {})])
@pytest.mark.parametrize("bc_x,bc_y", [("transmissive", "periodic"), ("periodic", "transmissive")])
def test_batches_of_sixteen_row_tiles(system, k, opts, bc_x, bc_y):
    from paper_2609_26194_amd import Fam, FamConfig
    sizes = [(250, 233), (130, 301), (61, 170)]
    reps, steps = 20, 2
    log(f"batch of {reps} x {sizes}: {system} k={k} {bc_x}/{bc_y} {opts}")
    kw = {**dict(dim=2, k=k, system=system, bc_x=bc_x, bc_y=bc_y, oe="type2", cfl=0.2), **opts}
    cfgs = [FamConfig(nx=a, ny=b, **kw) for a, b in sizes]
    states = []
    for i, (a, b) in enumerate(sizes):
        U = fi.random_euler_state_2d(a, b, 40 + i, amp=0.5 if "pp" in opts else 0.2)
        states.append(to_dev(U if system == "euler" else U[:1]))
    bat = Fam(None, batch=cfgs * reps)
    Ub = torch.cat([s.reshape(-1) for s in states] * reps)
    for _ in range(steps):
        bat.step(Ub)
    torch.cuda.synchronize()
    bat.close()
    want = torch.cat([_steps(c, s, None, steps).reshape(-1) for c, s in zip(cfgs, states)])
    assert _same(Ub.view(reps, -1), want.expand(reps, -1))
