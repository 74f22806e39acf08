"""A batch solver that is loaded again: the steps take the kernels of the present state's symmetry and
of the present mode (maxent_set_reduced), whatever an earlier call of the same chunk length
captured.  Bit for bit the results of a new solver."""
import numpy as np
import pytest

from paper_2401_15233_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [300, 64, 129]
INST = [dict(n=n, tau_ref=I.kn_to_tau_ref(kn), t_end=0.2) for n, kn in zip(SIZES, (0.01, 0.1, 1.0))]


def axial():
    return np.concatenate([I.sod_prims(14, n) for n in SIZES], axis=-1).reshape(14, 1, -1)


def transverse():
    """The same tubes with a transverse flow (u_y, u_z) that changes along them."""
    W = axial()
    x = np.arange(W.shape[-1])
    W[2] += 0.3 * np.sin(0.1 * x)
    W[3] += 0.2 * np.cos(0.07 * x)
    return W


def run(gpu_lib, calls):
    s = gpu_lib.MaxEntBatch(INST, precision='fp64', order=2, integrator='ssprk2', cfl=0.5)
    s.set_launch(64, 1, 4)
    out = []
    for W, reduced in calls:
        s.set_reduced(reduced)
        s.init_state(W)
        info = s.step(10, chunk=5)
        out.append((s.get('conserved').cpu().numpy(), [i['t'] for i in info['instances']]))
    s.close()
    return out


@pytest.mark.parametrize('calls', [
    [('axial', True), ('transverse', True)],
    [('transverse', True), ('axial', True), ('transverse', True)],
    [('axial', True), ('axial', False), ('axial', True)],
    [('transverse', False), ('axial', False), ('transverse', True), ('axial', True)],
])
def test_reloaded_batch_equals_a_new_one(gpu_lib, calls):
    fields = {'axial': axial(), 'transverse': transverse()}
    calls = [(fields[f], r) for f, r in calls]
    for k, (U, t) in enumerate(run(gpu_lib, calls)):
        U1, t1 = run(gpu_lib, [calls[k]])[0]
        assert t == t1, k
        assert np.array_equal(U, U1), (k, np.abs(U - U1).max())


def test_mode_changed_between_steps(gpu_lib):
    """Without a new load: the steps after maxent_set_reduced run the other kernels."""
    def go(modes):
        s = gpu_lib.MaxEntBatch(INST, precision='fp64', order=2, integrator='ssprk2', cfl=0.5)
        s.set_launch(64, 1, 4)
        s.init_state(axial())
        got = []
        for m in modes:
            s.set_reduced(m)
            s.step(5, chunk=5)
            got.append(s.get('conserved').cpu().numpy())
        s.close()
        return got
    a, b = go([True, True]), go([False, False])
    assert not np.array_equal(a[0], b[0])      # the two kernels differ by rounding
    c, d = go([True, False]), go([False, True])
    assert np.array_equal(c[0], a[0]) and not np.array_equal(c[1], a[1])
    assert np.array_equal(d[0], b[0]) and not np.array_equal(d[1], b[1])
