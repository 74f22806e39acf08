"""MaxEntSteps with an inflow that the solver refuses: the call raises and the solver's state is as it
was, with an earlier tape's steps held or not; a valid call afterwards works."""
import pytest

from oracle import moments as mo
from paper_2401_15233_amd import inputs as I

pytestmark = pytest.mark.gpu

KW = dict(system=14, dim=2, nx=16, ny=16, order=2, integrator='ssprk2', cfl=0.4,
          bc=('jet', 'transmissive', 'transmissive', 'transmissive'),
          jets=[(0.35, 0.1, 30.0), (0.65, 0.1, -30.0)])


@pytest.mark.parametrize('taped', [False, True])
@pytest.mark.parametrize('bad', [(-1.0, 1.0), (3.0, 0.0), (float('nan'), 1.0), (3.0, float('inf'))])
def test_refused_inflow_leaves_the_state(gpu_lib, bad, taped):
    import torch
    from paper_2401_15233_amd.autograd import MaxEntSteps

    def field(seed):
        return torch.tensor(mo.prim_to_cons14(I.crossed_jets_developed(16, 16, seed=seed)), device='cuda')

    def params(mach, rho):
        return torch.tensor([mach, rho, I.kn_to_tau_ref(0.1, L_ref=0.1)], dtype=torch.float64)

    s = gpu_lib.MaxEntSolver(**KW)
    if taped:
        MaxEntSteps.apply(field(1), params(3.0, 1.0), s, 2)
    else:
        s.init_state(field(1), repr='conserved')
    before = s.get('conserved').clone()
    with pytest.raises(gpu_lib.MaxentError) as e:
        MaxEntSteps.apply(field(2), params(*bad), s, 2)
    assert e.value.status == 'INVAL'
    assert torch.equal(s.get('conserved'), before)
    assert (s.problem.jet_mach, s.problem.jet_rho) == (3.0, 1.0)
    U = MaxEntSteps.apply(field(2), params(2.5, 1.1), s, 2)
    t = gpu_lib.MaxEntSolver(**KW)
    assert torch.equal(U, MaxEntSteps.apply(field(2), params(2.5, 1.1), t, 2))
    s.close()
    t.close()
