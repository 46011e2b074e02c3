"""1D meshes on either side of the sizes where the path changes: one lane per cell in one
workgroup (scalar equations up to 1022 cells, Euler up to 510) against tiles of 62 cells,
and within the workgroup the edges of a wave (62 and 63 cells) and the smallest mesh.
Oracle parity at 1e-12; the run to an end time takes the oracle's number of steps.
"""
import numpy as np
import pytest
import torch

import fam_inputs as fi
import oracle.scheme as S
from gpu_util import both_configs, log, needs_gpu, rel_linf, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]


def _state(system, n, seed):
    rng = np.random.default_rng(seed)
    if system != "euler":
        U = 0.05 * rng.standard_normal((1, 2, n))
        U[0, 0] += 1.0
        return U
    U = 0.02 * rng.standard_normal((3, 2, n))
    U[0, 0] += 1.0
    U[1, 0] += 0.3
    U[2, 0] += 2.5
    return U


@pytest.mark.parametrize("system,sizes", [("burgers", (3, 62, 63, 500, 1022, 1023)), ("advection", (4, 190, 1022)),
                                          ("euler", (3, 5, 62, 63, 510, 511))])
@pytest.mark.parametrize("oe", ["type1", "type2", "off"])
@pytest.mark.parametrize("k,bc,char", [(3, "periodic", False), (4, "transmissive", False), (5, "periodic", False),
                                       (5, "transmissive", True), (6, "transmissive", False)])
def test_run_and_step(system, sizes, oe, k, bc, char):
    if char and system != "euler":
        pytest.skip("characteristic variables: Euler")
    from paper_2609_26194_amd import Fam
    for n in sizes:
        kw = dict(dim=1, nx=n, k=k, system=system, bc_x=bc, oe=oe, cfl=0.2, char_vars=char)
        ora, cfg = both_configs(**kw)
        U0 = _state(system, n, n + k)
        ref, t_ref, _ = S.run(torch.tensor(U0), ora, nsteps=3)
        fam = Fam(cfg)
        U = to_dev(U0)
        steps, t = fam.run(U, 0.0, 3)
        fam.check()
        err = rel_linf(U, ref)
        log(f"{system} n={n} k={k} {bc} {oe} char={char}: rel Linf {err:.2e}")
        assert steps == 3 and abs(t - t_ref) <= 1e-14 * t_ref and err <= 1e-12
        # the same three steps by single calls, and by a run that ends inside its fourth step
        V = to_dev(U0)
        for _ in range(3):
            fam.step(V)
        fam.check()
        assert torch.equal(V, U)
        t_end = 1.2 * t_ref
        ref, _, n_ref = S.run(torch.tensor(U0), ora, t_final=t_end)
        fam.set_time(0.0)
        W = to_dev(U0)
        steps, t = fam.run(W, t_end, 0)
        fam.check()
        assert steps == n_ref and t == t_end and rel_linf(W, ref) <= 1e-12
        fam.close()
