"""Loading and reading a field in place (device buffers of the solver's device) and through the
staging buffer (host buffers): the same state, first time step, symmetry and checks, at sizes with
and without row padding, of less than one workgroup and of several cells per thread, and from
buffers that start at any multiple of eight bytes."""
import numpy as np
import pytest
import torch

from test_gpu_two_lane import field

pytestmark = pytest.mark.gpu


def solver(S, kind, nx, ny):
    return S.MaxEntSolver(system=5 if kind == 'five' else 14, dim=1 if ny == 1 else 2, nx=nx, ny=ny, order=2, cfl=0.3,
                          bc=('periodic',) * 4)


@pytest.mark.parametrize('kind, nx, ny', [('five', 4, 1), ('five', 600001, 1), ('axial', 257, 1), ('full', 5, 1),
                                          ('planar', 4, 4), ('planar', 1103, 701), ('full', 33, 65), ('full', 64, 16)])
def test_device_and_host_buffers_give_the_same(gpu_lib, kind, nx, ny):
    W = field(kind, nx, ny)
    got = []
    for where in ('host', 'device', 'odd device'):
        s = solver(gpu_lib, kind, nx, ny)
        if where == 'host':
            src = np.ascontiguousarray(W)
        elif where == 'device':
            src = torch.tensor(W).cuda()
        else:
            store = torch.zeros(W.size + 1, dtype=torch.float64, device='cuda')
            src = store[1:].view(W.shape)
            src.copy_(torch.tensor(W))
        s.init_state(src)
        prim, cons = s.get('primitive').clone(), s.get('conserved').clone()
        s.init_state(cons, repr='conserved')
        assert torch.equal(s.get('conserved'), cons)
        info = s.step(1, tau_ref=0.05)
        got.append((prim, cons, s.get('sigma').clone(), s.get('closing').clone(), info['dt_last'], info['reduced']))
        s.close()
    scale = np.abs(W).reshape(W.shape[0], -1).max(1)
    err = np.abs(got[0][0].cpu().numpy().reshape(W.shape[0], -1) - W.reshape(W.shape[0], -1)).max(1)
    # primitives -> conserved -> primitives: a few roundings of sums of at most ten products
    assert (err <= 64 * 2.0 ** -53 * 20 * max(scale.max(), 1.0)).all()
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0][:4], other[:4])) and got[0][4:] == other[4:]


@pytest.mark.parametrize('nx, ny', [(7, 5), (1103, 701)])
@pytest.mark.parametrize('where', ['first', 'middle', 'last'])
def test_one_cell_decides_symmetry_and_checks(gpu_lib, nx, ny, where):
    W = field('planar', nx, ny)
    j, i = dict(first=(0, 0), middle=(ny // 2, nx // 3), last=(ny - 1, nx - 1))[where]
    s = solver(gpu_lib, 'planar', nx, ny)
    s.init_state(torch.tensor(W).cuda())
    assert s.info()['reduced'] == 1
    odd = W.copy()
    odd[12, j, i] = 1e-300
    s.init_state(torch.tensor(odd).cuda())
    assert s.info()['reduced'] == 0
    for bad, code in ((np.nan, 'NONFINITE'), (-1.0, 'UNREALIZABLE')):
        V = W.copy()
        V[4, j, i] = bad
        with pytest.raises(gpu_lib.MaxentError, match=code):
            s.init_state(torch.tensor(V).cuda())
    s.init_state(torch.tensor(W).cuda())
    assert s.info()['reduced'] == 1
    s.close()
