"""The forms that calls too small to fill the chip take, against the forms of larger calls,
bit for bit (they share the arithmetic of every voxel and pixel): the cone backprojection of
volumes of up to 64 blocks, with 8 and 4 threads per column segment, against 16-row blocks,
which never split; the detector backprojection of up to 128 tiles, in four workgroups per
tile, against a call with more.  View counts around the 64 views set out at a time."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(P, orbit, nx, ny, nz, det, V, n_theta=24):
    g = synth.Grid(nu=det, nv=det, du=1.0, dv=1.0, n_theta=n_theta, n_s=synth.radon_bins(det, det), ds=1.0, nx=nx,
                   ny=ny, nz=nz, vx=1.0, vy=1.0, vz=1.0)
    views = synth.circle_orbit(V, 750.0, 1200.0) if orbit == "circle" else synth.sinusoid_orbit(V, 750.0, 1200.0)
    return P.Plan(g, views)


# orbit, volume, detector side, views
VOLUMES = [("circle", (1, 1, 1), 24, 1), ("sinusoid", (17, 5, 9), 40, 2), ("circle", (16, 32, 8), 64, 3),
           ("sinusoid", (32, 32, 32), 72, 64), ("circle", (33, 31, 30), 72, 65), ("sinusoid", (48, 40, 41), 96, 131),
           ("circle", (64, 64, 64), 120, 67), ("sinusoid", (64, 62, 57), 120, 66)]


@pytest.mark.parametrize("case", VOLUMES, ids=str)
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_small_volumes_match_the_unsplit_blocks(case, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    orbit, (nx, ny, nz), det, V = case
    plan = _plan(P, orbit, nx, ny, nz, det, V)
    print("\n[gpu small volume]", case, dtype, flush=True)
    torch.manual_seed(3)
    gF = torch.randn(V, det, det, device="cuda").to(getattr(torch, dtype))
    got, want = (torch.full((nz, ny, nx), float("nan"), device="cuda") for _ in range(2))
    P.dc_cone_bp(plan, gF, got)
    got_relu = got.clone()
    P.dc_cone_bp(plan, gF, got_relu, accumulate=True, relu=True, v0=V // 3, nv=V - V // 3)
    plan.set_knobs(bp_block_y=16)
    P.dc_cone_bp(plan, gF, want)
    assert torch.equal(got, want)
    P.dc_cone_bp(plan, gF, want, accumulate=True, relu=True, v0=V // 3, nv=V - V // 3)
    assert torch.equal(got_relu, want)
    plan.close()


@pytest.mark.parametrize("det", [33, 64, 130])
@pytest.mark.parametrize("dtype", ["float32", "float16"])
def test_few_tiles_match_many(det, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    V = 130
    plan = _plan(P, "sinusoid", 4, 4, 4, det, V, n_theta=70)
    print("\n[gpu few tiles]", det, dtype, flush=True)
    torch.manual_seed(4)
    H = torch.randn((V,) + tuple(plan.sino_shape), device="cuda").to(getattr(torch, dtype))
    many = torch.full((V, det, det), float("nan"), device="cuda", dtype=H.dtype)
    P.dc_detector_bp(plan, H, many)
    Gg = torch.full((V, det, det), float("nan"), device="cuda")
    P.dc_weight_radon_adjoint(plan, H, Gg)
    for v0, nv in ((0, 1), (5, 14), (V - 3, 3)):
        few = torch.full_like(many, 7.0)
        P.dc_detector_bp(plan, H, few, v0=v0, nv=nv)
        assert torch.equal(few[v0:v0 + nv], many[v0:v0 + nv]) and int((few != 7.0).sum()) <= nv * det * det
        few = torch.full_like(Gg, 7.0)
        P.dc_weight_radon_adjoint(plan, H, few, v0=v0, nv=nv)
        assert torch.equal(few[v0:v0 + nv], Gg[v0:v0 + nv])
    plan.close()
