"""The transport's FP32 passes at the edges of their segments, windows and groups: one step on disks against the oracle on
the stored state, at its time step, within the 2e-6 of one FP32 step.  The frame is turned at any rate (v_x less R times
what the frame's rotation gains: the same motion), so that a ring's circular shift goes either way, far and not at all,
and its residual has either sign."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1602_02359_amd import workloads as W
from gpu_common import errors, gpu_solver

pytestmark = pytest.mark.gpu


def _turned_step(prob, turn):
    p = prob.params
    R = W.centres(p["ymin"])[None, :, None]
    if p["geometry"] == "sph":
        R = R * np.sin(W.centres(p["zmin"]))[:, None, None]
    p["omega"] += turn
    prob.fields["vx"] = prob.fields["vx"] - turn * R
    p["precision"] = "fp32"
    s = gpu_solver(prob)
    ref = {k: None if v is None else np.ascontiguousarray(v) for k, v in s.download().items()}
    shift = O.ring_split(p, ref["vx"], O.cfl_dt(p, {k: None if v is None else v.copy() for k, v in ref.items()}))
    dt = O.step(p, ref)
    s.fargo_step(dt)
    s.fargo_check()
    err = errors(prob, s.download(), ref)
    print("  shifts %d .. %d, residuals %.2f .. %.2f, errors" % (shift[1].min(), shift[1].max(), shift[2].min(),
                                                              shift[2].max()), err, flush=True)
    return max(err.values())


@pytest.mark.parametrize("nx,turn", [(1, 0.5), (5, -1.5), (115, 1.0), (116, 4.0), (117, -4.0), (127, 0.6), (128, 1.4),
                                     (129, -40.0), (239, 2.0), (240, -2.0), (241, 3.0), (255, -60.0), (256, 70.0),
                                     (257, 1.01), (480, -7.0), (481, 0.99)])
def test_ring_segments_and_windows_fp32(nx, turn):
    print("ring segments fp32", nx, turn, flush=True)
    assert _turned_step(W.disk2d_cyl(nx=nx, ny=12, noise=1e-2), turn) <= 2e-6


@pytest.mark.parametrize("nx,ny,turn", [(130, 4, 0.0), (233, 7, 2.0), (2000, 300, 0.0), (2000, 301, 3.0), (3100, 285, -1.0),
                                        (3100, 286, 0.5)])
def test_ring_groups_fp32(nx, ny, turn):
    """v_y across the workgroups of 3, 7 and 15 rings."""
    print("ring groups fp32", nx, ny, turn, flush=True)
    assert _turned_step(W.disk2d_cyl(nx=nx, ny=ny, noise=1e-2), turn) <= 2e-6


@pytest.mark.parametrize("geo", ["cyl", "sph"])
@pytest.mark.parametrize("nx,turn", [(1, 0.5), (3, -1.5), (115, 3.0), (116, -3.0), (117, 1.0), (127, 0.6), (128, 20.0),
                                     (129, -20.0), (231, 1.4), (232, -1.0), (233, 2.0)])
def test_fused_z_x_pass_fp32(geo, nx, turn):
    """Rings one zone around a wave's 116 zones, two such segments and its window of 128."""
    print("fused z/x pass fp32", geo, nx, turn, flush=True)
    make = W.disk3d_sph if geo == "sph" else W.disk3d_cyl_planet
    assert _turned_step(make(nx=nx, ny=7, nz=9, noise=1e-2), turn) <= 2e-6
