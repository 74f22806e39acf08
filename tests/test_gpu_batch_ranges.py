"""Batched tubes where a workgroup walks several tiles and several tubes.

One workgroup per CU and many tubes of 4 to 3000 cells: the ranges hold up to a dozen tiles,
end inside tubes and run over whole tubes of a few cells, so tiles of one and of different tubes
follow each other in a workgroup (the next tile's cells are loaded while the last one is worked
on, and CFL rates are reduced per tube of a range).  Every tube must be the tube run alone, bit
for bit, in state, time and number of steps."""
import numpy as np
import pytest

from paper_2401_15233_amd import inputs as I
from test_gpu_batch import NUM

pytestmark = pytest.mark.gpu


def tubes():
    g = np.random.default_rng(11)
    n = [4, 5, 59, 60, 61, 123, 124, 125, 251, 252, 253, 3000] + [int(k) for k in np.exp(g.uniform(1.5, 8.0, 150))]
    out = []
    for k in n:
        d = dict(n=k, p_ratio=float(g.uniform(2, 20)), rho_ratio=float(g.uniform(2, 10)),
                 kn=float(np.exp(g.uniform(-5, 2))), t_end=1.0)
        d['tau_ref'] = I.kn_to_tau_ref(d['kn'])
        out.append(d)
    return out


@pytest.mark.parametrize('precision', ['fp64', 'mixed'])
@pytest.mark.parametrize('launch', [(64, 1, 1), (128, 1, 1), (256, 1, 1), (64, 2, 1)])
@pytest.mark.parametrize('bc', ['transmissive', 'reflective'])
def test_ranges_of_several_tiles_and_tubes(gpu_lib, precision, launch, bc):
    num = dict(NUM, bc=(bc,) * 2 + ('transmissive',) * 2)
    insts = tubes()
    b = gpu_lib.MaxEntBatch(insts, precision=precision, **num)
    b.init_state(I.batch_sod_prims(insts))
    b.set_launch(*launch)
    info = b.step(3, chunk=3)
    parts = b.split(b.get('conserved').cpu().numpy())
    b.close()
    for k in list(range(12)) + list(range(20, len(insts), 19)):
        d = insts[k]
        s = gpu_lib.MaxEntSolver(system=14, dim=1, nx=d['n'], precision=precision, **num)
        s.init_state(I.batch_sod_prims([d]))
        si = s.step(3, tau_ref=d['tau_ref'], t_end=d['t_end'])
        U = s.get('conserved').cpu().numpy()[:, 0, :]
        s.close()
        pi = info['instances'][k]
        assert pi['steps'] == si['steps'] and pi['t'] == si['t'], d
        assert np.array_equal(parts[k], U), d
