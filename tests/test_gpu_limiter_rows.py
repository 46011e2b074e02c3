"""The positivity limiter where a discontinuity runs along a row: every cell of the rows beside
it fails the cheap test, some of them are limited.  Rows of fewer cells than take the point
test, of just as many, a full strip and more than one, against the oracle at 1e-12; and the
limiter has to act (the run without it differs)."""
import pytest
import torch

import fam_inputs as fi
import oracle.scheme as S
from gpu_util import both_configs, log, needs_gpu, rel_linf, to_dev
from oracle.physics import NonPhysicalState

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("nx", [3, 5, 6, 7, 60, 61, 124])
@pytest.mark.parametrize("k", [3, 4, 5, 6])
def test_discontinuity_along_a_row(nx, k):
    ny = 14
    kw = dict(dim=2, nx=nx, ny=ny, x1=nx / 16.0, y1=ny / 16.0, k=k, system="euler", bc_x="periodic",
              bc_y="transmissive", oe="type2", cfl=0.05)
    ora, cfg = both_configs(pp=True, **kw)
    U0 = fi.random_euler_state_2d(nx, ny, 9 + nx, amp=0.1)
    U0[:, :, ny // 2:] *= 0.02
    ref, _, _ = S.run(torch.tensor(U0), ora, nsteps=2)
    from paper_2609_26194_amd import Fam
    fam = Fam(cfg)
    U = to_dev(U0)
    fam.run(U, 0.0, 2)
    fam.check()
    err = rel_linf(U, ref)
    on, _, _ = S.run(torch.tensor(U0), ora, nsteps=1)
    try:
        off, _, _ = S.run(torch.tensor(U0), both_configs(pp=False, **kw)[0], nsteps=1)
        acts = rel_linf(on, off)
    except NonPhysicalState:
        acts = 1.0
    log(f"{nx}x{ny} k={k}: rel Linf {err:.2e}, with against without the limiter {acts:.1e}")
    assert err <= 1e-12
    assert acts > 1e-6
