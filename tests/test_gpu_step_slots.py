"""The time step's hand-over from one step to the next: fixed and CFL steps in turn, steps after the
end time, and one step per call must give what one uninterrupted run gives, bit for bit, on grids
of one tile and of many (the CFL rate is kept in parts), in one and two dimensions."""
import numpy as np
import pytest
import torch

from test_gpu_two_lane import field

pytestmark = pytest.mark.gpu


def solver(S, kind, nx, ny, **kw):
    s = S.MaxEntSolver(system=5 if kind == 'five' else 14, dim=1 if ny == 1 else 2, nx=nx, ny=ny, order=2, cfl=0.3,
                       bc=('periodic',) * 4, **kw)
    s.init_state(np.ascontiguousarray(field(kind, nx, ny)))
    return s


@pytest.mark.parametrize('integrator', ['fe', 'ssprk2'])
@pytest.mark.parametrize('kind, nx, ny', [('five', 31, 1), ('axial', 1000, 1), ('full', 70000, 1), ('planar', 16, 15),
                                          ('planar', 131, 77), ('planar', 400, 400), ('full', 290, 250)])
def test_split_runs_equal_one_run(gpu_lib, kind, nx, ny, integrator):
    one = solver(gpu_lib, kind, nx, ny, integrator=integrator)
    a = one.step(7, tau_ref=0.05)
    dt, ref = a['dt_last'], one.get('conserved').clone()
    one.close()
    # one step per call, then an end time that the run has reached (idle steps), then on
    s = solver(gpu_lib, kind, nx, ny, integrator=integrator)
    for _ in range(4):
        i = s.step(1, tau_ref=0.05)
    i2 = s.step(5, tau_ref=0.05, t_end=i['t'])
    assert i2['steps'] == 4 and i2['t'] == i['t']
    b = s.step(3, tau_ref=0.05)
    assert (b['t'], b['steps'], b['dt_last']) == (a['t'], 7, dt)
    assert torch.equal(s.get('conserved'), ref)
    # a fixed step, and CFL steps from its state: the rate is that of the state loaded afresh
    s.step(2, dt=0.5 * dt, tau_ref=0.05)
    mid = s.get('conserved').clone()
    c = s.step(2, tau_ref=0.05)
    end = s.get('conserved').clone()
    s.init_state(mid, repr='conserved')
    d = s.step(2, tau_ref=0.05)
    assert c['dt_last'] == d['dt_last']
    assert torch.equal(s.get('conserved'), end)
    s.close()


@pytest.mark.parametrize('integrator', ['fe', 'ssprk2'])
@pytest.mark.parametrize('kind, nx, ny', [('planar', 40, 33), ('axial', 130, 1)])
@pytest.mark.parametrize('n', [1, 2, 3])
def test_a_symmetric_state_after_a_full_one(gpu_lib, kind, nx, ny, integrator, n):
    """The planes a reduced kernel does not write are zero in the state it hands back, whichever
    kernels ran in the solver before."""
    s = solver(gpu_lib, kind, nx, ny, integrator=integrator)
    s.step(n, tau_ref=0.05)
    ref = s.get('conserved').clone()
    s.init_state(np.ascontiguousarray(field('full', nx, ny)))
    s.step(3, tau_ref=0.05)
    s.init_state(np.ascontiguousarray(field(kind, nx, ny)))
    info = s.step(n, tau_ref=0.05)
    assert info['reduced'] > 0
    assert torch.equal(s.get('conserved'), ref)
    # the full kernels on the same state, then the reduced ones from where they ended
    s.set_reduced(False)
    s.init_state(np.ascontiguousarray(field(kind, nx, ny)))
    s.step(3, tau_ref=0.05)
    s.set_reduced(True)
    s.step(n, tau_ref=0.05)
    odd = s.get('conserved')[[3, 6, 8, 12] + ([2, 5, 11] if kind == 'axial' else [])]
    assert int((odd != 0).sum()) == 0
    s.close()
