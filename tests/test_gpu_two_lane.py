"""Faces shared by two lanes (small grids) against faces of one lane (large grids).

A periodic field repeated side by side has the solution of the single field, repeated.  The
single field has at most as many tiles as the two-lane launch takes, the repeated one has more,
so the two runs go through the two kernels.  Both evaluate every face in the same operations,
so the results are the same bits, whatever the sizes are to the tiles (60 cells in 1D, 16 x 15 in
2D); the smaller run is held to the oracle by the parity tests."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def field(kind, nx, ny):
    """Independent states from cell to cell, near a Maxwellian and on its realizable side (R below
    15 p^2 / rho; above it the closure is singular, and the oracle too fails)."""
    g = np.random.default_rng(7)

    def r(scale, base=0.0):
        return base + scale * g.uniform(-1, 1, (ny, nx))

    rho, p = r(0.3, 1.0), r(0.2, 1.0)
    z = 0.0 * rho
    even_z = kind == 'planar'
    ux, uy, uz = r(0.5), r(0.5), z if even_z else r(0.5)
    R = 15.0 * p * p / rho * r(0.05, 0.85)
    if kind == 'five':
        return np.stack([rho, ux, p, r(0.1), R / 5.0]).reshape(5, nx)
    if kind == 'axial':
        d = r(0.1)
        return np.stack([rho, ux, z, z, p + 2 * d, z, z, p - d, z, p - d, r(0.1), z, z, R]).reshape(14, nx)
    d, e = r(0.1), r(0.1)
    W = np.stack([rho, ux, uy, uz, p + d, r(0.1), z if even_z else r(0.1), p + e, z if even_z else r(0.1),
                  p - d - e, r(0.1), r(0.1), z if even_z else r(0.1), R])
    return W if ny > 1 else W.reshape(14, nx)


@pytest.mark.parametrize('kind, nx, ny, rx, ry, opt', [
    ('planar', 256, 480, 1, 2, dict()),                                       # 512 tiles, the last with two lanes
    ('planar', 256, 481, 1, 2, dict(limiter='vanalbada', flux='rusanov')),    # 528, one lane on both sides
    ('planar', 137, 211, 2, 3, dict(integrator='midpoint')),
    ('planar', 7, 4, 50, 90, dict(order=1)),
    ('full', 256, 240, 2, 1, dict()),                                         # 256 tiles
    ('full', 33, 16, 9, 13, dict(flux='rusanov')),
    ('full', 61440, 1, 2, 1, dict()),                                         # 1024 tiles
    ('full', 61, 1, 1100, 1, dict(order=1)),
    ('axial', 122880, 1, 2, 1, dict()),                                       # 2048 tiles
    ('axial', 59, 1, 4400, 1, dict(limiter='vanalbada')),
    ('five', 122880, 1, 2, 1, dict(order=1)),
    ('five', 121, 1, 2200, 1, dict(integrator='midpoint')),
])
def test_repeated_field_gives_repeated_solution(gpu_lib, kind, nx, ny, rx, ry, opt):
    W = field(kind, nx, ny)
    dim = 1 if ny == 1 else 2
    got = []
    for ax, ay in ((1, 1), (rx, ry)):
        kw = dict(system=5 if kind == 'five' else 14, dim=dim, nx=nx * ax, ny=ny * ay, cfl=0.3, order=2,
                  x1=float(ax), y1=float(ay), bc=('periodic',) * 4)
        kw.update(opt)
        s = gpu_lib.MaxEntSolver(**kw)
        s.init_state(np.ascontiguousarray(np.tile(W, (1, ay, ax) if dim == 2 else (1, ax))))
        info = s.step(2, dt=0.02 / max(nx, ny), tau_ref=0.05)
        got.append(s.get('conserved').clone())
        s.close()
        assert info['fail_code'] == 0 and info['steps'] == 2 and info['reduced'] == dict(planar=1, axial=2).get(kind, 0)
    small, large = got
    reps = (1, ry, rx) if dim == 2 else (1, rx)
    assert torch.equal(large.reshape(large.shape[0], -1), small.reshape(W.shape).repeat(reps).reshape(W.shape[0], -1))
