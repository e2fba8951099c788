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

SIDES = {"periodic": ("periodic",) * 4, "reflect": ("reflect",) * 4, "fixed": ("fixed",) * 4,
         "mixed": ("reflect", "outflow", "outflow", "reflect"), "outflow": ("outflow",) * 4,
         "half": ("fixed", "outflow", "reflect", "fixed")}
MESHES = [("cart", 64, 3, 3, "adi", "periodic"), ("cart", 65, 16, 4, "iso", "periodic"),
          ("cart", 40, 13, 17, "adi", "reflect"), ("cyl", 130, 12, 9, "iso", "reflect"),
          ("cyl", 193, 33, 33, "iso", "reflect"), ("sph", 70, 24, 13, "adi", "reflect"),
          ("cyl", 300, 129, 1, "iso", "reflect"), ("cyl", 64, 1000, 1, "adi", "reflect"),
          ("cyl", 20, 400, 5, "adi", "reflect"),
          # three zones between the sides: every ghost mirrors a zone next to the other side
          ("cyl", 33, 3, 3, "adi", "mixed"), ("cart", 64, 3, 3, "adi", "outflow"), ("sph", 40, 3, 3, "iso", "reflect"),
          # caller-fixed sides in both directions, tiles that hold one side, both, or none
          ("cart", 70, 5, 4, "iso", "fixed"), ("cyl", 130, 40, 9, "adi", "half"), ("cart", 70, 33, 1, "adi", "half"),
          ("cyl", 64, 200, 1, "iso", "fixed")]
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


@pytest.mark.parametrize("nx,ny", [(2, 9), (61, 33), (62, 64), (63, 31), (125, 5), (187, 100), (640, 40)])
@pytest.mark.parametrize("side", ["fixed", "reflect", "outflow"])
def test_viscous_pass_at_segment_edges(nx, ny, side):
    """Box 7d where a ring is shorter than a wave's 62 columns, fills them exactly and spills over by one, with chunks of
    one row and of many, against the oracle."""
    print("viscous pass", nx, ny, side, flush=True)
    prob = W.disk2d_visc(nx=nx, ny=ny, alpha=0.05, noise=0.2, seed=nx + ny)
    prob.params["bc"] = SIDES[side]
    rng = np.random.default_rng(nx)
    for k in ("vx", "vy"):
        prob.fields[k] += 0.02 * rng.standard_normal(prob.shape)
    assert _step(prob) <= 1e-12


@pytest.mark.parametrize("nx,turn", [(115, 0.0), (116, -3.0), (117, 3.0), (127, 0.4), (128, -0.4), (129, 50.0),
                                     (239, -1.0), (240, 2.0), (241, -2.0), (255, 70.0), (256, -70.0), (257, 1.0),
                                     (480, 7.0), (481, -0.01)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_ring_segments_and_windows(nx, turn, precision):
    """Rings one zone around a wave's segment (116 zones), two of them, its window (128) and two of those, the frame
    turned so that the circular shift goes either way, far and not at all, against the oracle."""
    print("ring segments", nx, turn, precision, flush=True)
    if precision == "fp64":
        prob = W.random_problem("cyl", nx=nx, ny=6, nz=1, eos="adi", seed=nx, fargo=True, bc=SIDES["reflect"])
        prob.fields["vx"] += turn
    else:
        prob = W.disk2d_cyl(nx=nx, ny=12, noise=1e-2)
        prob.params["precision"] = "fp32"
    assert _step(prob) <= (1e-12 if precision == "fp64" else 2e-6)


@pytest.mark.parametrize("geo,nx,ny,eos,side", [("cyl", 40, 3, "iso", "reflect"), ("cyl", 130, 4, "adi", "fixed"),
                                                ("cart", 150, 3, "iso", "periodic"), ("cart", 233, 7, "adi", "periodic"),
                                                ("cyl", 2000, 300, "iso", "half"), ("cart", 1900, 301, "adi", "periodic"),
                                                ("cyl", 3100, 286, "adi", "outflow"), ("cart", 3100, 285, "iso", "periodic")])
def test_ring_groups(geo, nx, ny, eos, side):
    """v_y across the workgroups of the 2D ring pass (3, 7 or 15 rings each) and over a periodic side, one ring more than
    a whole number of workgroups and exactly that, against the oracle."""
    print("ring groups", geo, nx, ny, eos, side, flush=True)
    prob = W.random_problem(geo, nx=nx, ny=ny, nz=1, eos=eos, seed=nx + ny, fargo=geo != "cart", bc=SIDES[side])
    assert _step(prob) <= 1e-12


@pytest.mark.parametrize("geo,eos", [("cyl", "iso"), ("sph", "adi"), ("cart", "adi")])
@pytest.mark.parametrize("nx,turn", [(5, 0.3), (52, -3.0), (53, 3.0), (54, 0.0), (63, -0.4), (64, 20.0), (65, -20.0),
                                     (106, 1.0), (107, -1.0)])
def test_fused_z_x_pass_fp64(geo, eos, nx, turn):
    """The fused Z/X pass where a ring is one zone around a wave's 53 zones, two such segments and its window of 64."""
    print("fused z/x pass", geo, eos, nx, turn, flush=True)
    prob = W.random_problem(geo, nx=nx, ny=5, nz=7, eos=eos, seed=nx, fargo=geo != "cart",
                            bc=SIDES["periodic" if geo == "cart" else "reflect"])
    if geo != "cart":
        prob.fields["vx"] += turn
    assert _step(prob) <= 1e-12


@pytest.mark.parametrize("nx,ny", [(1, 5), (2, 4), (3, 3), (58, 33), (60, 70), (61, 32), (62, 9), (120, 40), (123, 31)])
@pytest.mark.parametrize("geo,eos", [("cyl", "iso"), ("cyl", "adi"), ("cart", "iso"), ("cart", "adi")])
@pytest.mark.parametrize("side", ["periodic", "fixed", "half"])
def test_source_march_on_2d_meshes(nx, ny, geo, eos, side):
    """Rings one zone around the 61 columns of a wave (60 with an energy) and two such segments, a wave's window longer
    than the ring, few rows and several chunks, against the oracle."""
    if geo == "cyl" and side == "periodic":
        side = "outflow"
    print("source march", nx, ny, geo, eos, side, flush=True)
    prob = W.random_problem(geo, nx=nx, ny=ny, nz=1, eos=eos, seed=nx + ny, fargo=geo != "cart", bc=SIDES[side])
    assert _step(prob) <= 1e-12


@pytest.mark.parametrize("nx,ny", [(60, 70), (61, 32), (62, 9), (122, 33)])
def test_source_march_on_2d_meshes_fp32(nx, ny):
    print("source march fp32", nx, ny, flush=True)
    prob = W.disk2d_cyl(nx=nx, ny=ny, noise=1e-2)
    prob.params["precision"] = "fp32"
    assert _step(prob) <= 2e-6


@pytest.mark.parametrize("nx,ny,nz,eos,v0", [(1, 2100, 1, "adi", "minmax"), (2, 700, 3, "iso", "minmax"),
                                              (127, 2048, 1, "iso", "mean"), (129, 300, 7, "adi", "minmax"),
                                              (641, 1100, 2 + 1, "iso", "mean"), (1281, 12, 1, "adi", "mean"),
                                              (2561, 700, 3, "iso", "minmax"), (4095, 5, 3, "adi", "mean")])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_time_step_pass_by_ring_count(nx, ny, nz, eos, v0, precision):
    """dt of Eq. cfl2 (within the two codes' bound) and every ring's v0 where a wave, and where a workgroup, takes a
    ring: few and many rings, odd lengths, rings shorter than a wave, one zone more than a chunk, the longest."""
    import torch
    from gpu_common import dt_close
    print("time-step pass", nx, ny, nz, eos, v0, precision, flush=True)
    prob = W.random_problem("cyl", nx=nx, ny=ny, nz=nz, eos=eos, seed=nx, fargo=True, bc=("fixed", "fixed", "reflect", "reflect"))
    prob.params.update(v0_mode=v0, precision=precision)
    s = gpu_solver(prob)
    st = {k: None if v is None else np.ascontiguousarray(v) for k, v in s.download().items()}
    want = O.cfl_dt(prob.params, st)
    assert dt_close(s.fargo_cfl_dt(), want)
    g0, gN, _ = s.fargo_ring_split(s.state["vx"], want)
    torch.cuda.synchronize()
    o0, oN, _ = O.ring_split(prob.params, st["vx"], want)
    if v0 == "minmax":
        assert np.array_equal(g0.cpu().numpy(), o0.ravel())
    else:  # the order of the sum differs: a few units of n u
        assert np.allclose(g0.cpu().numpy(), o0.ravel(), rtol=4096 * 2.0 ** -53, atol=4096 * 2.0 ** -53)
    assert np.array_equal(gN.cpu().numpy(), oN.ravel())


@pytest.mark.parametrize("field,value", [("vx", np.inf), ("vx", -np.inf), ("vx", np.nan), ("rho", 0.0), ("cs", np.inf)])
def test_non_finite_state_is_reported(field, value):
    """One bad zone is reported, and an infinite velocity or sound speed leaves no time step to advance by."""
    from paper_1602_02359_amd import fargo as F
    prob = W.disk2d_cyl(nx=130, ny=20, noise=1e-2)
    prob.fields[field][0, 9, 129] = value
    s = gpu_solver(prob)
    before = s.state["rho"].clone()
    s.fargo_step(0.0)
    dt = s.fargo_get_dt()
    with pytest.raises(F.FargoError) as e:
        s.fargo_check()
    assert e.value.code == -4  # FARGO_ENONFINITE
    if np.isinf(value):
        assert dt == 0.0
        ok = np.ones(before.shape, dtype=bool)
        ok[0, 8:11] = False
        assert np.array_equal(s.state["rho"].cpu().numpy()[ok], before.cpu().numpy()[ok])
