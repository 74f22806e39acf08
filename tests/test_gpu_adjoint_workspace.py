"""The adjoint's workspace: what one call leaves in it must not reach the next.

A planar dJ/dU after a non-planar one on the same tape, and on a new tape whose blocks were the
old one's, with workspaces of fewer and of more fields than one clearing launch takes (3 adjoint
states and 2 per step of a segment; 16 a launch), must give the bits of the first call."""
import numpy as np
import pytest
import torch

from test_gpu_two_lane import field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('every', [1, 6, 7, 15])
@pytest.mark.parametrize('integrator', ['ssprk2', 'fe'])
def test_adjoint_calls_do_not_see_each_other(gpu_lib, every, integrator):
    nx, ny, n = 37, 22, 15
    W = np.ascontiguousarray(field('planar', nx, ny))
    g = np.random.default_rng(3)
    dJ = g.standard_normal((14, ny, nx))
    flat = dJ.copy()
    flat[[3, 6, 8, 12]] = 0.0
    s = gpu_lib.MaxEntSolver(system=14, dim=2, nx=nx, ny=ny, order=2, integrator=integrator, cfl=0.3,
                             bc=('periodic',) * 4)

    def run():
        s.init_state(W)
        s.record(every, n)
        s.step(n, tau_ref=0.05)

    def adjoint(d):
        dU, grads = s.adjoint(torch.tensor(d).cuda())
        return dU.clone(), list(grads)

    run()
    first, g1 = adjoint(flat)
    full, g2 = adjoint(dJ)
    assert not torch.equal(first, full)
    again, g3 = adjoint(flat)
    assert torch.equal(first, again) and g1 == g3
    run()
    again, g3 = adjoint(flat)
    assert torch.equal(first, again) and g1 == g3
    again, g3 = adjoint(dJ)
    assert torch.equal(full, again) and g2 == g3
    s.close()
