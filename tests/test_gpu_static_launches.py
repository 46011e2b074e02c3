"""fam_step_static enqueues nothing that its step does not read: the limiter, which works
inside the stage launches, adds no launch on meshes whose tiles all start at once.  On a
flat wide mesh with more tiles than wave slots, which orders them, the step stays fam_step's.
"""
import ctypes

import pytest
import torch

import fam_inputs as fi
from gpu_util import log, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


def _nodes(cfg, U):
    """Nodes of the graph that a captured fam_step_static call makes."""
    from paper_2609_26194_amd.fam import fam_step_static
    hip = ctypes.CDLL("libamdhip64.so")
    s = torch.cuda.Stream()
    h, g, n = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
    fam_step_static(cfg, s.cuda_stream, U)   # looks the scratch array up
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(h, 2) == 0   # relaxed
    fam_step_static(cfg, s.cuda_stream, U)
    assert hip.hipStreamEndCapture(h, ctypes.byref(g)) == 0
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(g) == 0
    return n.value


@pytest.mark.parametrize("nx,ny,k", [(96, 80, 5), (203, 131, 6), (512, 480, 4)])
def test_the_limiter_adds_no_launch(nx, ny, k):
    from paper_2609_26194_amd import FamConfig
    U = to_dev(fi.random_euler_state_2d(nx, ny, 1, amp=0.1))
    kw = dict(dim=2, nx=nx, ny=ny, k=k, system="euler", oe="type2", cfl=0.2)
    off, on = _nodes(FamConfig(**kw), U), _nodes(FamConfig(pp=True, **kw), U)
    log(f"{nx}x{ny} k={k}: {off} launches without the limiter, {on} with it")
    assert on == off


def test_flat_mesh_with_ordered_tiles():
    from paper_2609_26194_amd import Fam, FamConfig
    from paper_2609_26194_amd.fam import fam_step_static
    nx, ny = 22000, 15   # 367 strips of five tiles
    cfg = FamConfig(dim=2, nx=nx, ny=ny, k=6, system="euler", oe="type2", cfl=0.2, pp=True, bc_x="transmissive",
                    bc_y="transmissive")
    U0 = to_dev(fi.random_euler_state_2d(nx, ny, 5, amp=0.6))
    fam = Fam(cfg)
    Ue, Us = U0.clone(), U0.clone()
    for _ in range(2):
        fam.step(Ue)
        torch.cuda.synchronize()
        fam_step_static(cfg, torch.cuda.current_stream().cuda_stream, Us)
    torch.cuda.synchronize()
    assert torch.equal(Ue, Us) and not torch.equal(Ue, U0)
    fam.close()
