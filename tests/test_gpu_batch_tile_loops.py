"""The batch's tile loop where test_gpu_batch_ranges does not take it: the 14-moment kernel (a flow with
transverse moments, and symmetric tubes with the reduced mode off), the midpoint update, periodic
ends (a tile's halo wraps, also of a tube that one workgroup walks in several tiles), and the
shapes with several cells per thread.  Every tube is the tube run alone, bit for bit."""
import numpy as np
import pytest

from paper_2401_15233_amd import inputs as I

pytestmark = pytest.mark.gpu

N = [4, 5, 59, 60, 61, 124, 125, 252, 253, 3000] + [int(k) for k in np.exp(np.random.default_rng(3).uniform(1.5, 8.0, 60))]


def field(n, seed, transverse):
    """Smooth along the tube and periodic: two beams of nearly equal weight, with or without
    transverse parts of velocity and separation."""
    g = np.random.default_rng(seed)
    x = (np.arange(n) + 0.5) / n

    def wave(base, amp):
        return base + amp * np.sin(2 * np.pi * (g.integers(1, 4) * x + g.random()))
    rho, T, skew = wave(1.0, 0.3), wave(0.8, 0.1), wave(0.0, 0.1)
    u = np.stack([wave(0.2, 0.4)] + [wave(0.0, 0.3) if transverse else 0.0 * x for _ in range(2)])
    d = np.stack([wave(0.8, 0.1)] + [wave(0.4, 0.2) if transverse else 0.0 * x for _ in range(2)])
    w = 0.5 * rho * np.stack([1.0 + skew, 1.0 - skew])
    m = np.stack([u + d, u - d])                        # [beam][3][n]
    um = (w[:, None] * m).sum(0) / rho
    c = m - um
    cc = (c * c).sum(1)
    P = [(w * (c[:, i] * c[:, j] + (T if i == j else 0.0))).sum(0)
         for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]
    q = [(w * c[:, i] * (cc + 5.0 * T)).sum(0) for i in range(3)]
    R = (w * (cc * cc + 10.0 * T * cc + 15.0 * T * T)).sum(0)
    return np.stack([rho, *um, *P, *q, R])[:, None, :]


@pytest.mark.parametrize('launch', [(64, 1, 1), (64, 4, 1), (128, 2, 1), (256, 1, 1)])
@pytest.mark.parametrize('kernel,integrator,bc,precision', [
    ('transverse', 'ssprk2', 'periodic', 'fp64'),
    ('transverse', 'midpoint', 'reflective', 'fp64'),
    ('transverse', 'ssprk2', 'transmissive', 'mixed'),
    ('full', 'midpoint', 'periodic', 'fp64'),
    ('axial', 'midpoint', 'periodic', 'fp64'),
    ('axial', 'midpoint', 'periodic', 'mixed'),
])
def test_tile_loops(gpu_lib, launch, kernel, integrator, bc, precision):
    num = dict(order=2, integrator=integrator, limiter='minmod', flux='hll', cfl=0.5, precision=precision,
               bc=(bc,) * 2 + ('transmissive',) * 2)
    insts = [dict(n=n, tau_ref=I.kn_to_tau_ref(0.1), t_end=1.0) for n in N]
    W = [field(n, k, kernel == 'transverse') for k, n in enumerate(N)]
    b = gpu_lib.MaxEntBatch(insts, **num)
    b.set_reduced(kernel != 'full')
    b.init_state(np.concatenate(W, -1))
    b.set_launch(*launch)
    info = b.step(3, chunk=3)
    parts = b.split(b.get('conserved').cpu().numpy())
    b.close()
    for k in list(range(10)) + list(range(10, len(N), 11)):
        s = gpu_lib.MaxEntSolver(system=14, dim=1, nx=N[k], **num)
        # (a tube of this batch runs the kernel that the whole batch's state takes)
        s.set_reduced(kernel != 'full')
        s.init_state(W[k])
        si = s.step(3, tau_ref=insts[k]['tau_ref'], t_end=1.0)
        U = s.get('conserved').cpu().numpy()[:, 0, :]
        assert si['reduced'] == (2 if kernel == 'axial' else 0)
        s.close()
        pi = info['instances'][k]
        assert pi['steps'] == si['steps'] and pi['t'] == si['t'], N[k]
        assert np.array_equal(parts[k], U), (N[k], np.abs(parts[k] - U).max())
