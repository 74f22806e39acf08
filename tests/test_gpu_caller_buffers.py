"""Device buffers of the caller that the kernels may not use in place: one that ends before the field
does is refused (DEVICE), as a copy from or to it is, and one that is not aligned as doubles are
gives the same values as an aligned one."""
import ctypes

import numpy as np
import pytest

from paper_2401_15233_amd import inputs as I

pytestmark = pytest.mark.gpu

NX, NY = 64, 40
KW = dict(system=14, dim=2, nx=NX, ny=NY, bc=('transmissive',) * 4)
FIELD = 14 * NX * NY * 8
DEVICE = -3


@pytest.fixture()
def short_buffer():
    """Half a field, from the runtime itself (torch's allocator rounds its blocks up)."""
    import torch
    torch.zeros(1, device='cuda')
    path = next(l.split()[-1] for l in open('/proc/self/maps') if 'libamdhip64.so' in l)
    hip = ctypes.CDLL(path)
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(FIELD // 2)) == 0
    yield p
    assert hip.hipFree(p) == 0


def test_short_buffers_are_refused(gpu_lib, short_buffer):
    s = gpu_lib.MaxEntSolver(**KW)
    L = s._lib
    assert L.maxent_init_state(s._h, 0, short_buffer, 1, 0.0) == DEVICE
    s.init_state(I.crossed_jets_developed(NX, NY, seed=1))
    before = s.get('conserved').clone()
    for repr in (0, 1, 3):
        assert L.maxent_get_moments(s._h, repr, short_buffer, 1) == DEVICE
    # half a field holds one component of it
    assert L.maxent_get_moments(s._h, 2, short_buffer, 1) == 0
    s.record(2, 2)
    s.step(2, tau_ref=0.01)
    g = (ctypes.c_double * 3)()
    w = np.random.default_rng(1).standard_normal(s.shape)
    wp = w.ctypes.data_as(ctypes.c_void_p)
    assert L.maxent_step_adjoint(s._h, short_buffer, 1, None, 0, g) == DEVICE
    assert L.maxent_step_adjoint(s._h, wp, 0, short_buffer, 1, g) == DEVICE
    out, _ = s.adjoint(w)                  # the calls after a refused one work
    assert np.isfinite(out.cpu().numpy()).all()
    s.init_state(before, repr='conserved')
    assert (s.get('conserved') == before).all()
    s.close()


def test_unaligned_buffers(gpu_lib):
    import torch
    W0 = I.crossed_jets_developed(NX, NY, seed=2)
    raw = torch.zeros(FIELD + 16, dtype=torch.uint8, device='cuda')
    assert raw.data_ptr() % 8 == 0
    raw[4:4 + FIELD] = torch.from_numpy(np.ascontiguousarray(W0)).cuda().reshape(-1).view(torch.uint8)
    a, b = gpu_lib.MaxEntSolver(**KW), gpu_lib.MaxEntSolver(**KW)
    a.init_state(W0)
    torch.cuda.synchronize()
    assert b._lib.maxent_init_state(b._h, 0, ctypes.c_void_p(raw.data_ptr() + 4), 1, 0.0) == 0
    U = a.get('conserved')
    assert (U == b.get('conserved')).all()
    assert b._lib.maxent_get_moments(b._h, 1, ctypes.c_void_p(raw.data_ptr() + 4), 1) == 0
    assert torch.equal(raw[4:4 + FIELD].clone().view(torch.float64), U.reshape(-1))
    a.close()
    b.close()
