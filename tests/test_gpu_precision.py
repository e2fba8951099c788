"""The last place of a step.  At dt = 1e-300 every change of a field is far below its last place, and what remains is the
forming of the momenta and the velocities from them: with values of few bits the momenta, their sums and the quotients
are exact, so any quantity that is not handed on as formed shows in the last place, and so does the rounding of a ring's
1/R.  Mass that flows into an all but empty row is the product of the flux and 1/V, and shows the rounding of 1/V."""
import math

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


def _spherical(nx, ny, nz, eos="iso"):
    prob = W.random_problem("sph", nx=nx, ny=ny, nz=nz, eos=eos, seed=nx, fargo=True, bc=("fixed",) * 4)
    prob.params["omega"] = 0.0
    return prob


@pytest.mark.parametrize("eos", ["iso", "adi"])
@pytest.mark.parametrize("nx,ny,nz", [(53, 16, 12), (7, 40, 30)])
def test_spherical_radius_is_divided_by_once(eos, nx, ny, nz):
    """v_x of a uniform density on a spherical mesh is (R v) (1/R), R and 1/R rounded once, in every ring."""
    print("spherical radius", eos, nx, ny, nz, flush=True)
    prob = _spherical(nx, ny, nz, eos)
    prob.fields["rho"][:] = 1.0
    s = gpu_solver(prob)
    v = s.download()["vx"]
    s.fargo_step(1e-300)
    s.fargo_check()
    sin = np.array([math.sin(z) for z in W.centres(prob.params["zmin"])])
    R = W.centres(prob.params["ymin"])[None, :, None] * sin[:, None, None]
    sl = owned(prob, "vx")
    assert np.array_equal(s.download()["vx"][sl], ((R * v) * (1.0 / R))[sl])


@pytest.mark.parametrize("geo,nz", [("cart", 7), ("cyl", 7), ("sph", 7), ("cyl", 1), ("cart", 1)])
def test_volume_is_divided_by_once(geo, nz):
    """Rows of unit density moving at unit speed into rows of density 1e-200: what arrives is the flux, S dt, times 1/V,
    the quotient of Tab. "geom" rounded once, row by row of the boundary between the two, bit for bit."""
    nx, ny = 9, 24
    dt = 1.7e-100
    for row in range(1, ny, 3):
        print("volume", geo, nz, "row", row, flush=True)
        prob = W.random_problem(geo, nx=nx, ny=ny, nz=nz, eos="iso", seed=5, fargo=False, bc=("fixed",) * 4)
        p, f = prob.params, prob.fields
        p["omega"] = 0.0
        if nz == 1:
            p["zmin"] = np.array([0.0, 0.7])
        for k in ("vx", "vz", "pot"):
            if f.get(k) is not None:
                f[k][:] = 0.0
        f["vy"][:], f["cs"][:], f["rho"][:] = 1.0, 1e-150, 1.0
        f["rho"][:, W.NGH + row:] = 1e-200
        s = gpu_solver(prob)
        s.fargo_step(dt)
        s.fargo_check()
        a, b = p["ymin"][W.NGH + row], p["ymin"][W.NGH + row + 1]
        dx = (p["xmax"] - p["xmin"]) / nx
        got = s.download()["rho"]
        for k in range(W.NGH if nz > 1 else 0, (W.NGH if nz > 1 else 0) + nz):
            c, d = p["zmin"][k], p["zmin"][k + 1]
            if geo == "cart":
                iv, sy, syk = 1.0 / (b - a), 1.0, dx * (d - c)
            elif geo == "cyl":
                iv, sy, syk = 2.0 / ((b * b - a * a) * dx), a * dx, d - c
            else:
                iv, sy, syk = 3.0 / ((b * b * b - a * a * a) * dx), a * a * dx, math.cos(c) - math.cos(d)
            assert (got[k, W.NGH + row] == (iv / syk) * ((sy * syk) * dt)).all(), (k, row)
