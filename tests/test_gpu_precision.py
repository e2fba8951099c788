"""What a step of vanishing length leaves as it is.  At dt = 1e-300 every change of a field is far below its last place,
and what remains is the forming of the momenta and the velocities from them: with values of few bits the momenta, their
sums and the quotients are exact, so any quantity that is not handed on as formed shows in the last place."""
import numpy as np
import pytest

from paper_1602_02359_amd import workloads as W
from gpu_common import gpu_solver, owned

pytestmark = pytest.mark.gpu


def _few_bits(prob, seed):
    rng = np.random.default_rng(seed)
    f = prob.fields
    f["rho"][:] = 2 * rng.integers(1, 500, prob.shape) + 1
    for k in ("vx", "vy", "vz"):
        if f.get(k) is not None:
            f[k][:] = rng.integers(1, 4096, prob.shape) / 64.0 * rng.choice((-1.0, 1.0), prob.shape)
    return prob


@pytest.mark.parametrize("geo", ["cart", "cyl"])
@pytest.mark.parametrize("eos", ["iso", "adi"])
@pytest.mark.parametrize("nx,ny,nz", [(53, 5, 9), (161, 4, 70), (7, 3, 3), (130, 9, 1)])
def test_conserved_quantities_are_handed_on(geo, eos, nx, ny, nz):
    """Density, energy, v_y and v_z after the step, bit for bit, through the Y sweep, the Z/X (or ring) pass and 12d; the
    planes in one chunk and in several."""
    print("handed on", geo, eos, nx, ny, nz, flush=True)
    prob = W.random_problem(geo, nx=nx, ny=ny, nz=nz, eos=eos, seed=nx, fargo=geo == "cyl",
                            bc=("reflect",) * 4 if geo == "cyl" else ("periodic",) * 4)
    s = gpu_solver(_few_bits(prob, nx))
    before = {k: None if v is None else v.clone() for k, v in s.state.items()}
    s.fargo_step(1e-300)
    s.fargo_check()
    for k in ("rho", "e", "vy", "vz"):
        if before[k] is not None:
            sl = owned(prob, k)[:2] + (slice(0, nx),)
            assert (s.state[k][sl] == before[k][sl]).all(), k
