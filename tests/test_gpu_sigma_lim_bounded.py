"""Every run of the sigma_lim study (5-moment Sod tube, first order, forward Euler) reaches its end
time within a bounded number of steps: where the CFL step follows near-Junk cells it can
collapse under another rounding, and such a run must fail here, with its count and step, instead
of stepping on without end."""
import pytest

from paper_2401_15233_amd import inputs as I

pytestmark = pytest.mark.gpu

T_END = 0.2
BOUND = 200000      # the longest run (sigma_lim = 1e-5, Kn = 1) takes 79231


@pytest.mark.parametrize('sigma_lim', [1e-2, 1e-3, 1e-4, 1e-5])
def test_study_runs_end(gpu_lib, sigma_lim):
    for kn in (1e-3, 1e-2, 0.1, 1.0, 0.0):
        s = gpu_lib.MaxEntSolver(system=5, dim=1, nx=1000, order=1, integrator='fe', flux='hll', cfl=0.5,
                                 bc=('transmissive',) * 4, sigma_lim=sigma_lim)
        s.init_state(I.sod_prims(5, 1000))
        tau = I.kn_to_tau_ref(kn) if kn > 0 else 0.0
        info = {'t': 0.0, 'steps': 0}
        while info['t'] < T_END * (1.0 - 1e-12) and info['steps'] < BOUND:
            info = s.step(5000, tau_ref=tau, t_end=T_END)
        s.close()
        print(f'sigma_lim {sigma_lim:g} Kn {kn:g}: {info["steps"]} steps', flush=True)
        assert info['t'] >= T_END * (1.0 - 1e-12), (sigma_lim, kn, info['steps'], info['dt_last'])
