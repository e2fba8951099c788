"""Small and medium meshes, where the marching kernels (Y and Z sweeps, the fused Z/X pass, the source step) take more
and shorter chunks to fill the chip: one step against the oracle at the oracle's time step, at chunk counts that divide
the zones and ones that leave a ragged last chunk, down to chunks of a single zone, across periodic, reflecting and
fixed sides.  FP64 on random states within the 1e-12 of one step that every parity test holds; FP32 on disks within
2e-6 of the oracle on the stored state, the bar of one FP32 step."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1602_02359_amd import workloads as W
from gpu_common import errors, gpu_solver

pytestmark = pytest.mark.gpu

SIDES = {"periodic": ("periodic",) * 4, "reflect": ("reflect",) * 4}
MESHES = [("cart", 64, 3, 3, "adi", "periodic"), ("cart", 65, 16, 4, "iso", "periodic"),
          ("cart", 40, 13, 17, "adi", "reflect"), ("cyl", 130, 12, 9, "iso", "reflect"),
          ("cyl", 193, 33, 33, "iso", "reflect"), ("sph", 70, 24, 13, "adi", "reflect"),
          ("cyl", 300, 129, 1, "iso", "reflect"), ("cyl", 64, 1000, 1, "adi", "reflect"),
          ("cyl", 20, 400, 5, "adi", "reflect")]
DISKS = [("sph", 70, 24, 13), ("sph", 136, 9, 4), ("sph", 260, 40, 37), ("cyl", 150, 23, 17), ("cyl", 64, 5, 3),
         ("2d", 300, 129, 1), ("2d", 64, 1000, 1)]


def _step(prob):
    s = gpu_solver(prob)
    ref = {k: None if v is None else np.ascontiguousarray(v) for k, v in s.download().items()}
    dt = O.step(prob.params, ref)
    s.fargo_step(dt)
    s.fargo_check()
    err = errors(prob, s.download(), ref)
    print("  ", err, flush=True)
    return max(err.values())


@pytest.mark.parametrize("geo,nx,ny,nz,eos,side", MESHES)
def test_chunked_step_fp64(geo, nx, ny, nz, eos, side):
    print("chunked step", geo, nx, ny, nz, eos, side, flush=True)
    prob = W.random_problem(geo, nx=nx, ny=ny, nz=nz, eos=eos, seed=100 + nx + nz, fargo=geo != "cart", bc=SIDES[side])
    assert _step(prob) <= 1e-12


@pytest.mark.parametrize("geo,nx,ny,nz", DISKS)
def test_chunked_step_fp32(geo, nx, ny, nz):
    print("chunked step fp32", geo, nx, ny, nz, flush=True)
    make = {"sph": W.disk3d_sph, "cyl": W.disk3d_cyl_planet, "2d": W.disk2d_cyl}[geo]
    prob = make(nx=nx, ny=ny, noise=1e-2, **({} if nz == 1 else {"nz": nz}))
    prob.params["precision"] = "fp32"
    assert _step(prob) <= 2e-6
