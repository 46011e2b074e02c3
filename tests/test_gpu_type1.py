"""Type I statistics over meshes of one block of cells, a few, and more cells than the
reduction has threads, against the oracle (relative L-infinity 1e-12 as in the other
parity tests: the mean enters through D = max |u - mean|, whose rounding is 1e-16)."""
import numpy as np
import pytest
import torch

import fam_inputs as fi
import oracle.scheme as S
from gpu_util import both_configs, log, needs_gpu, rel_linf, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("dim,nx,ny", [(1, 3, 1), (1, 256, 1), (1, 257, 1), (2, 9, 7), (2, 16, 16), (2, 61, 40),
                                       (2, 320, 219)])
@pytest.mark.parametrize("system", ["burgers", "euler"])
def test_statistics(dim, nx, ny, system):
    log(f"Type I {system} {nx}x{ny}")
    kw = dict(dim=dim, nx=nx, k=4, system=system, bc_x="periodic", oe="type1", cfl=0.2)
    if dim == 2:
        kw.update(ny=ny, bc_y="periodic")
    ora, cfg = both_configs(**kw)
    rng = np.random.default_rng(5)
    if system == "burgers":
        U0 = 0.1 * rng.standard_normal((1, dim + 1) + ((ny, nx) if dim == 2 else (nx,)))
        U0[0, 0] += 0.5
    else:
        U0 = fi.random_euler_state_2d(nx, ny, 3, amp=0.1) if dim == 2 else fi.smooth_euler_1d(nx)
    ref, _, _ = S.run(torch.tensor(U0), ora, nsteps=2)
    from paper_2609_26194_amd import Fam
    fam = Fam(cfg)
    U = to_dev(U0)
    fam.run(U, 0.0, 2)
    fam.check()
    err = rel_linf(U, ref)
    log(f"  rel Linf {err:.3e}")
    assert err <= 1e-12
